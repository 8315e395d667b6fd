"""The MLP's backward kernel at the row counts where its loops change (GPU):
one row, around the 32 rows that are summed at a time and the 128 rows held in
LDS, and several rounds of them, against the FP64 oracle.  A gradient is a sum
of at most 300 FP32 products of factors with errors of a few ulp: 1e-4 of the
larger of its size and 1% of the largest gradient."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 31, 32, 127, 128, 129, 170, 300])
def test_backward_rows_match_oracle(B):
    import torch

    from oracle import mlp as omlp
    from paper_2607_18991_amd import learned, nz

    rng = np.random.default_rng(900 + B)
    bits = learned.to_bf16_bits(rng.normal(0, 0.25, size=nz.NZ_MLP_NPARAM).astype(np.float32))
    p64 = omlp.bf16_to_f64(bits)
    x = np.concatenate([rng.integers(0, 2, size=(B, 7)), rng.normal(size=(B, 1))], axis=1).astype(np.float32)
    dy = rng.normal(size=(B, 2)).astype(np.float32)
    pb, xd = torch.from_numpy(bits.view(np.int16)).cuda(), torch.from_numpy(x).cuda()
    y = torch.empty((B, 2), dtype=torch.float32, device="cuda")
    act = torch.empty((B, nz.NZ_MLP_NACT), dtype=torch.float32, device="cuda")
    g = torch.full((nz.NZ_MLP_NPARAM,), float("nan"), dtype=torch.float32, device="cuda")
    nz.nz_mlp_forward(pb, xd, y, act)
    nz.nz_mlp_backward(pb, xd, act, torch.from_numpy(dy).cuda(), g)
    torch.cuda.synchronize()
    _, cache = omlp.forward(p64, x.astype(np.float64))
    want = omlp.backward(p64, x.astype(np.float64), cache, dy.astype(np.float64))
    err = np.abs(g.cpu().numpy() - want)
    assert (err <= 1e-4 * np.maximum(np.abs(want), 1e-2 * np.abs(want).max())).all(), np.nanmax(err)

"""Host threads whose lattices differ share a sweep kernel (GPU): each launch asks
for its own amount of LDS, and neither may lose by the other's.  Against the
oracle; integers, so the bar is equality."""
import threading

import pytest

from gpu_util import assert_same, oracle_batch, run_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ls", [(14, 16), (11, 13)])
def test_threads_with_unlike_lattices(Ls):
    import torch

    # (more samples than CUs at L = 11 and 13: the form with two workgroups per CU)
    count = 8 if Ls[0] > 13 else 280
    jobs = [[dict(L=L, zone_mask=0x1F, seed=0x7EAD + L, nsamples=count)] for L in Ls]
    out = [[], []]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(6):
                out[k].append(run_batch(jobs[k]))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        want = oracle_batch(jobs[k])
        assert len(out[k]) == 6
        for gn, gm, _, _ in out[k]:
            assert_same(jobs[k], gn, gm, *want)

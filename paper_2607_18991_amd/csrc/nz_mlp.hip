// nz_mlp.hip -- the small MLP of the learned prefill: (7 zone-mask bits,
// standardised size variable L^(-1/nu)) -> 64 -> 64 -> (u, v), tanh after the
// hidden layers; u, v
// estimate ln mean and ln std of n*/N.  Weights are stored as bfloat16 and
// widened exactly to float; every product and sum is FP32.  The network is
// about 5k parameters and is evaluated for a few hundred rows, so the kernels
// are latency-bound single-pass loops rather than matrix-core tiles.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/nz.h"

#define NZ_API extern "C" __attribute__((visibility("default")))

namespace nzmlp {

constexpr int IN = 8, H = 64, OUT = 2;
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + IN * H;
constexpr int OFF_W2 = OFF_B1 + H;
constexpr int OFF_B2 = OFF_W2 + H * H;
constexpr int OFF_W3 = OFF_B2 + H;
constexpr int OFF_B3 = OFF_W3 + H * OUT;
constexpr int NPARAM = OFF_B3 + OUT;
static_assert(NPARAM == NZ_MLP_NPARAM, "parameter layout");
static_assert(NZ_MLP_NACT == 2 * H, "activation cache layout");

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// Round to nearest, ties to even (NaN kept quiet).
__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return static_cast<uint16_t>((u >> 16) | 0x40u);
    const uint32_t lsb = (u >> 16) & 1u;
    return static_cast<uint16_t>((u + 0x7FFFu + lsb) >> 16);
}

// One workgroup of 64 threads per row; thread j owns hidden unit j.
__global__ __launch_bounds__(64) void mlp_forward_kernel(const uint16_t *__restrict__ p, const float *__restrict__ x,
                                                         float *__restrict__ y, float *__restrict__ act, int32_t B)
{
    __shared__ float h1[H], h2[H], xin[IN];
    const int b = blockIdx.x;
    if (b >= B) return;
    const int j = threadIdx.x;
    if (j < IN) xin[j] = x[b * IN + j];
    __syncthreads();
    float a = bf16_to_f32(p[OFF_B1 + j]);
    for (int i = 0; i < IN; ++i) a = fmaf(xin[i], bf16_to_f32(p[OFF_W1 + i * H + j]), a);
    h1[j] = tanhf(a);
    __syncthreads();
    a = bf16_to_f32(p[OFF_B2 + j]);
    for (int k = 0; k < H; ++k) a = fmaf(h1[k], bf16_to_f32(p[OFF_W2 + k * H + j]), a);
    h2[j] = tanhf(a);
    act[b * NZ_MLP_NACT + j] = h1[j];
    act[b * NZ_MLP_NACT + H + j] = h2[j];
    __syncthreads();
    if (j < OUT) {
        a = bf16_to_f32(p[OFF_B3 + j]);
        for (int k = 0; k < H; ++k) a = fmaf(h2[k], bf16_to_f32(p[OFF_W3 + k * OUT + j]), a);
        y[b * OUT + j] = a;
    }
}

// Backward: every workgroup owns a slice of the parameters and goes over all
// rows, ROWS at a time, so nothing is shared between workgroups and no atomics
// are needed.  It forms the pre-activation gradients its slice needs in LDS
// (those of the second layer are two multiply-adds each, so every workgroup
// forms its own), then every thread adds the rows' contributions to its
// parameter: sums of TILE rows, added up in row order.  The order is fixed, so
// results are deterministic, and the same for any ROWS.
//
// Bound by latency: 170 rows took 105 us in one workgroup of 256 threads; the
// 25 workgroups here leave the whole training step (four launches) at 30 us, down
// from 121, so they cost about as much as their launch.
constexpr int BT = 256;
constexpr int TILE = 32;    // rows summed before they are added to the total
constexpr int ROWS = 128;   // rows in LDS at a time
constexpr int LD = H + 1;   // padded: a column's rows lie in different banks
constexpr int W2_WGS = H * H / BT;     // slices of W2: 4 of its rows each
constexpr int W1_K = 8;                // hidden units per slice of W1, b1
constexpr int W1_WGS = H / W1_K;
constexpr int BACKWARD_WGS = W2_WGS + W1_WGS + 1;   // the last one: b2, W3, b3
static_assert(ROWS % TILE == 0 && H % W1_K == 0 && BT % H == 0, "whole tiles and slices");

// dz2 = (dy W3^T) * (1 - h2^2) of rows r0 .. r0 + rows - 1, zero behind them.
__device__ __forceinline__ void backward_dz2(const uint16_t *__restrict__ p, const float *__restrict__ act,
                                             const float *__restrict__ dy, int r0, int rows, float (*dz2)[LD])
{
    const int k = threadIdx.x % H;   // (the same in every step: BT is a multiple of H)
    float w3[OUT];
    for (int o = 0; o < OUT; ++o) w3[o] = bf16_to_f32(p[OFF_W3 + k * OUT + o]);
#pragma unroll 8
    for (int r = threadIdx.x / H; r < ROWS; r += BT / H) {
        const int row = r0 + min(r, rows - 1);
        const float h2 = act[row * NZ_MLP_NACT + H + k];
        float g = 0.0f;
        for (int o = 0; o < OUT; ++o) g = fmaf(dy[row * OUT + o], w3[o], g);
        const float v = g * (1.0f - h2 * h2);
        dz2[r][k] = r < rows ? v : 0.0f;
    }
}

// acc += sums of TILE rows of term(r, g), r < rows; term adds row r to g.
template <typename F>
__device__ __forceinline__ void add_tiles(float &acc, int rows, F &&term)
{
    int t0 = 0;
    for (; t0 + TILE <= rows; t0 += TILE) {
        float g = 0.0f;
#pragma unroll
        for (int r = 0; r < TILE; ++r) g = term(t0 + r, g);   // (unrolled: the LDS reads run ahead)
        acc += g;
    }
    if (t0 < rows) {
        float g = 0.0f;
        for (int r = t0; r < rows; ++r) g = term(r, g);
        acc += g;
    }
}

__global__ __launch_bounds__(BT) void mlp_backward_kernel(const uint16_t *__restrict__ p, const float *__restrict__ x,
                                                          const float *__restrict__ act, const float *__restrict__ dy,
                                                          float *__restrict__ grad, int32_t B)
{
    __shared__ float dz2[ROWS][LD];
    __shared__ float side[ROWS][W1_K + 1];   // h1 of the slice's units, then dz1 of them
    __shared__ float xin[ROWS][IN];
    __shared__ float w2[W1_K][LD];
    const int t = threadIdx.x, wg = blockIdx.x;
    float acc = 0.0f;

    if (wg < W2_WGS) {
        // grad W2[k][j] = sum_r h1[r][k] dz2[r][j]: thread t owns k = 4 wg + t / H, j = t % H
        constexpr int KS = BT / H;
        const int kk = t / H, j = t % H, k0 = KS * wg;
        for (int r0 = 0; r0 < B; r0 += ROWS) {
            const int rows = min(ROWS, B - r0);
            backward_dz2(p, act, dy, r0, rows, dz2);
            for (int e = t; e < rows * KS; e += BT) side[e / KS][e % KS] = act[(r0 + e / KS) * NZ_MLP_NACT + k0 + e % KS];
            __syncthreads();
            add_tiles(acc, rows, [&](int r, float g) { return fmaf(side[r][kk], dz2[r][j], g); });
            __syncthreads();
        }
        grad[OFF_W2 + (k0 + kk) * H + j] = acc;
        return;
    }
    if (wg < W2_WGS + W1_WGS) {
        // grad W1[i][k] = sum_r x[r][i] dz1[r][k] and b1[k] = sum_r dz1[r][k], with
        // dz1 = (dz2 W2^T) * (1 - h1^2), for the slice's W1_K units k
        const int k0 = W1_K * (wg - W2_WGS);
        for (int e = t; e < W1_K * H; e += BT) w2[e / H][e % H] = bf16_to_f32(p[OFF_W2 + (k0 + e / H) * H + e % H]);
        const int i = t / W1_K, kk = t % W1_K;   // threads of i < IN own W1, those of i == IN b1
        for (int r0 = 0; r0 < B; r0 += ROWS) {
            const int rows = min(ROWS, B - r0);
            backward_dz2(p, act, dy, r0, rows, dz2);
            for (int e = t; e < rows * IN; e += BT) xin[e / IN][e % IN] = x[(r0 + e / IN) * IN + e % IN];
            __syncthreads();
            for (int e = t; e < rows * W1_K; e += BT) {
                const int r = e / W1_K, c = e % W1_K;
                const float h1 = act[(r0 + r) * NZ_MLP_NACT + k0 + c];
                float g = 0.0f;
#pragma unroll 16
                for (int j = 0; j < H; ++j) g = fmaf(dz2[r][j], w2[c][j], g);
                side[r][c] = g * (1.0f - h1 * h1);
            }
            __syncthreads();
            if (i < IN) add_tiles(acc, rows, [&](int r, float g) { return fmaf(xin[r][i], side[r][kk], g); });
            else if (i == IN) add_tiles(acc, rows, [&](int r, float g) { return g + side[r][kk]; });
            __syncthreads();
        }
        if (i < IN) grad[OFF_W1 + i * H + k0 + kk] = acc;
        else if (i == IN) grad[OFF_B1 + k0 + kk] = acc;
        return;
    }
    // b2[j] = sum_r dz2[r][j] (threads 0 .. 63), W3[k][o] = sum_r h2[r][k] dy[r][o]
    // (64 .. 191), b3[o] = sum_r dy[r][o] (192, 193)
    for (int r0 = 0; r0 < B; r0 += ROWS) {
        const int rows = min(ROWS, B - r0);
        backward_dz2(p, act, dy, r0, rows, dz2);
        __syncthreads();
        if (t < H) add_tiles(acc, rows, [&](int r, float g) { return g + dz2[r][t]; });
        __syncthreads();
        for (int e = t; e < rows * H; e += BT) dz2[e / H][e % H] = act[(r0 + e / H) * NZ_MLP_NACT + H + e % H];   // h2
        for (int e = t; e < rows * OUT; e += BT) xin[e / OUT][e % OUT] = dy[(r0 + e / OUT) * OUT + e % OUT];
        __syncthreads();
        const int q = t - H;
        if (q >= 0 && q < H * OUT) add_tiles(acc, rows, [&](int r, float g) { return fmaf(dz2[r][q / OUT], xin[r][q % OUT], g); });
        else if (q >= H * OUT && q < H * OUT + OUT) add_tiles(acc, rows, [&](int r, float g) { return g + xin[r][q - H * OUT]; });
        __syncthreads();
    }
    if (t < H) grad[OFF_B2 + t] = acc;
    else if (t < H + H * OUT) grad[OFF_W3 + t - H] = acc;
    else if (t < H + H * OUT + OUT) grad[OFF_B3 + t - H - H * OUT] = acc;
}

// Adam with decoupled weight decay; FP32 master weights, BF16 copy rewritten.
__global__ __launch_bounds__(256) void mlp_adam_kernel(float *__restrict__ w, uint16_t *__restrict__ wb,
                                                       const float *__restrict__ g, float *__restrict__ m,
                                                       float *__restrict__ v, float lr, float b1, float b2, float eps,
                                                       float wd, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPARAM) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1;
    const float vh = vi / c2;
    const float wi = w[i] - lr * (mh / (sqrtf(vh) + eps) + wd * w[i]);
    w[i] = wi;
    wb[i] = f32_to_bf16(wi);
}

// Weighted squared error and its gradient; one workgroup, fixed summation order.
__global__ __launch_bounds__(256) void mlp_loss_kernel(const float *__restrict__ y, const float *__restrict__ t,
                                                       const float *__restrict__ w, float *__restrict__ dy,
                                                       float *__restrict__ loss, int32_t B)
{
    __shared__ float red[256];
    float sw = 0.0f;
    for (int b = threadIdx.x; b < B; b += 256) sw += w[b];
    red[threadIdx.x] = sw;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    const float inv = 1.0f / red[0];
    __syncthreads();
    float acc = 0.0f;
    for (int b = threadIdx.x; b < B; b += 256) {
        const float wn = w[b] * inv;
        for (int o = 0; o < OUT; ++o) {
            const float r = y[b * OUT + o] - t[b * OUT + o];
            acc = fmaf(wn * r, r, acc);
            dy[b * OUT + o] = 2.0f * wn * r;
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = red[0];
}

}  // namespace nzmlp

namespace nz {
int set_error(int code, const char *msg);
}

namespace {
int mlp_fail(hipError_t e)
{
    return e == hipSuccess ? NZ_OK : nz::set_error(NZ_EDEVICE, hipGetErrorString(e));
}
}  // namespace

NZ_API int nz_mlp_forward(const uint16_t *params_bf16, const float *x, float *y, float *act, int32_t B, void *stream)
{
    if (!params_bf16 || !x || !y || !act || B < 1) return nz::set_error(NZ_EINVAL, "nz_mlp_forward: NULL pointer or B < 1");
    hipLaunchKernelGGL(nzmlp::mlp_forward_kernel, dim3(B), dim3(64), 0, static_cast<hipStream_t>(stream), params_bf16,
                       x, y, act, B);
    return mlp_fail(hipGetLastError());
}

NZ_API int nz_mlp_backward(const uint16_t *params_bf16, const float *x, const float *act, const float *dy, float *grad,
                           int32_t B, void *stream)
{
    if (!params_bf16 || !x || !act || !dy || !grad || B < 1) return nz::set_error(NZ_EINVAL, "nz_mlp_backward: NULL pointer or B < 1");
    hipLaunchKernelGGL(nzmlp::mlp_backward_kernel, dim3(nzmlp::BACKWARD_WGS), dim3(nzmlp::BT), 0, static_cast<hipStream_t>(stream),
                       params_bf16, x, act, dy, grad, B);
    return mlp_fail(hipGetLastError());
}

NZ_API int nz_mlp_adam(float *params_fp32, uint16_t *params_bf16, const float *grad, float *adam_m, float *adam_v,
                       const float hyper[5], int32_t step, void *stream)
{
    if (!params_fp32 || !params_bf16 || !grad || !adam_m || !adam_v || !hyper || step < 1)
        return nz::set_error(NZ_EINVAL, "nz_mlp_adam: NULL pointer or step < 1");
    const float lr = hyper[0], b1 = hyper[1], b2 = hyper[2], eps = hyper[3], wd = hyper[4];
    if (!(lr >= 0.0f) || !(b1 >= 0.0f && b1 < 1.0f) || !(b2 >= 0.0f && b2 < 1.0f) || !(eps > 0.0f) || !(wd >= 0.0f))
        return nz::set_error(NZ_EINVAL, "nz_mlp_adam: hyper-parameters out of range");
    const float c1 = 1.0f - powf(b1, static_cast<float>(step));
    const float c2 = 1.0f - powf(b2, static_cast<float>(step));
    hipLaunchKernelGGL(nzmlp::mlp_adam_kernel, dim3((nzmlp::NPARAM + 255) / 256), dim3(256), 0,
                       static_cast<hipStream_t>(stream), params_fp32, params_bf16, grad, adam_m, adam_v, lr, b1, b2,
                       eps, wd, c1, c2);
    return mlp_fail(hipGetLastError());
}

NZ_API int nz_mlp_loss(const float *y, const float *target, const float *weight, float *dy, float *loss, int32_t B,
                       void *stream)
{
    if (!y || !target || !weight || !dy || !loss || B < 1)
        return nz::set_error(NZ_EINVAL, "nz_mlp_loss: NULL pointer or B < 1");
    hipLaunchKernelGGL(nzmlp::mlp_loss_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream), y, target,
                       weight, dy, loss, B);
    return mlp_fail(hipGetLastError());
}

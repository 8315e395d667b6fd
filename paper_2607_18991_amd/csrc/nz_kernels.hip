// nz_kernels.hip -- CDNA4 (gfx950) kernels of the Newman-Ziff first-spanning
// sweep on sc(5) (Malarz & Woloszyn, Sec. II.B; neighbourhoods of Sec. II.A.2).
//
// Pipeline per chunk of samples (all launched on one stream):
//   nz_expand_kernel   a descriptor per sample from the host's runs of samples;
//   nz_clear_kernel    zero the bucket counters and bitset summaries;
//   nz_keys_kernel     Philox4x32-10 key of every site (integer VALU bound);
//                      sites below the prefill threshold T0 are occupied at once
//                      (bitset word per 32 sites, site list, a list entry that is
//                      its own parent); sites in the key band [T0, T0 + nb <<
//                      shift) are appended to the bucket of their key;
//   nz_hook, compress, bulk connected components of the prefilled sites on their
//   accum kernels      list positions (hooking with CAS links, then every entry
//                      points at its root and border sites add their flags to the
//                      root's word; sizes in largest-cluster runs only); a state
//                      that already spans is flagged for backoff;
//   nz_sweep_kernel    persistent: every workgroup pops a sample (longest first)
//                      and adds whole buckets of its band at a time, merging a
//                      block's sites and the clusters they touch in LDS; the
//                      root words' two border flags (or a winding loop) decide
//                      spanning, and n* is found within the block in which it happens.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "nz_internal.h"

namespace nz {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11): per round, counter words
// 0 and 2 are multiplied by two fixed odd constants; the high halves, xor-ed
// with words 1/3 and the round key, and the low halves form the next counter.
// The key advances by the Weyl increments between rounds.

constexpr uint32_t kPhiloxMulA = 0xD2511F53u;
constexpr uint32_t kPhiloxMulB = 0xCD9E8D57u;
constexpr uint32_t kWeylA = 0x9E3779B9u;
constexpr uint32_t kWeylB = 0xBB67AE85u;

// 32x32 -> 64-bit product as one v_mad_u64_u32 (left to itself the compiler
// forms the last round's products with separate v_mul_hi_u32 / v_mul_lo_u32,
// two more quarter-rate instructions per Philox block).
__device__ __forceinline__ uint64_t mul_wide(uint32_t x, uint32_t m)
{
    uint64_t r, carry;
    asm("v_mad_u64_u32 %0, %1, %2, %3, 0" : "=v"(r), "=&s"(carry) : "v"(x), "s"(m));
    (void)carry;
    return r;
}

// Three-input XOR in one gfx950 instruction (v_bitop3_b32, truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Keys of sites 2j and 2j + 1: both come from the block of counter j (word 3:
// domain tag 0); the even site takes words (1, 0), the odd site words (3, 2).
// Each round's two 32x32 products are formed as full 64-bit products (one
// v_mad_u64_u32 each) and each of its two three-way XORs is one instruction.
__device__ __forceinline__ void site_key_pair(uint32_t seed_lo, uint32_t seed_hi, uint32_t smp_lo, uint32_t smp_hi,
                                              uint32_t j, uint64_t &k_even, uint64_t &k_odd)
{
    uint32_t c0 = j, c1 = smp_lo, c2 = smp_hi, c3 = 0u;
    uint32_t k0 = seed_lo, k1 = seed_hi;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t a = mul_wide(c0, kPhiloxMulA);
        // round 0's c2 is the sample's high word, the same in every lane
        const uint64_t b = r == 0 ? static_cast<uint64_t>(kPhiloxMulB) * c2 : mul_wide(c2, kPhiloxMulB);
        c0 = xor3(static_cast<uint32_t>(b >> 32), c1, k0);
        c1 = static_cast<uint32_t>(b);
        c2 = xor3(static_cast<uint32_t>(a >> 32), c3, k1);
        c3 = static_cast<uint32_t>(a);
        k0 += kWeylA;
        k1 += kWeylB;
    }
    k_even = (static_cast<uint64_t>(c1) << 32) | c0;
    k_odd = (static_cast<uint64_t>(c3) << 32) | c2;
}

// floor(n / L) for n < 2^32 with magic = ceil(2^64 / L) (0 for L = 1).
__device__ __forceinline__ uint32_t div_by_L(uint32_t n, uint64_t magic)
{
    return static_cast<uint32_t>(__umul64hi(static_cast<uint64_t>(n), magic));
}

// Packed coordinates x0 | x1 << 6 | ... | x4 << 24.  Packed values order like
// site indices (x4 most significant), so (key, packed) sorts like (key, site).
__device__ __forceinline__ uint32_t pack_coords(uint32_t i, uint32_t L, uint64_t magic)
{
    uint32_t pc = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t q = div_by_L(i, magic);
        pc |= (i - q * L) << (6 * j);
        i = q;
    }
    return pc | (i << 24);
}

// Bits (5j + d + 2) for the d in [-2, 2] that keep x + d inside [0, L).
__device__ __forceinline__ uint32_t allowed_axis(int32_t x, int32_t L)
{
    const int32_t lo = max(0, 2 - x);
    const int32_t hi = min(4, L + 1 - x);
    return hi >= lo ? ((2u << hi) - (1u << lo)) : 0u;
}

// Periodic boundaries: the index correction of an offset whose steps leave
// the lattice on the axes of `out` (the offset's code bits outside the allowed
// set): +L^(j+1) for a negative step that left through 0, -L^(j+1) for a
// positive one past L-1 (one wrap suffices for L >= 5).
__device__ __forceinline__ int32_t wrap_fix(uint32_t out, int32_t L)
{
    int32_t fix = 0, p = L;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const uint32_t b = (out >> (5 * j)) & 31u;
        fix += (b & 0x03u) ? p : 0;
        fix -= (b & 0x18u) ? p : 0;
        p *= L;
    }
    return fix;
}

// The steps every axis allows from the site with packed coordinates pc.
__device__ __forceinline__ uint32_t allowed_of(uint32_t pc, int32_t L)
{
    return allowed_axis(pc & 63, L) | (allowed_axis((pc >> 6) & 63, L) << 5) | (allowed_axis((pc >> 12) & 63, L) << 10) |
           (allowed_axis((pc >> 18) & 63, L) << 15) | (allowed_axis(pc >> 24, L) << 20);
}

// The bits of a row's code that belong to axes 1..4.
constexpr uint32_t kRowAxes = 0x1FFFFE0u;

// Relaxed wavefront-scope accesses: ordinary cached loads and stores that the
// compiler neither merges nor elides.  They serve state private to one wave and
// the cache-tolerant walks of the bulk connected components; links and counts
// shared by all workgroups use agent-scope atomics.
template <typename T>
__device__ __forceinline__ T ld_w(T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); }
template <typename T>
__device__ __forceinline__ void st_w(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); }

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

template <typename T>
__device__ __forceinline__ T bcast(T v, int lane)
{
    return static_cast<T>(__builtin_amdgcn_readlane(static_cast<int>(v), lane));
}

// ---------------------------------------------------------------------------
// The samples of a chunk from its runs (the host plans runs of samples, so that
// a batch of thousands costs it a few dozen records).

__global__ __launch_bounds__(256) void nz_expand_kernel(const NzRun *__restrict__ runs, NzSample *__restrict__ desc,
                                                        NzState *__restrict__ state, int32_t *__restrict__ queue,
                                                        int32_t *__restrict__ out_index, int32_t *__restrict__ list,
                                                        int32_t *__restrict__ qhead)
{
    const NzRun &r = runs[blockIdx.y];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *qhead = 0;
    for (int32_t k = static_cast<int32_t>(blockIdx.x) * 256 + static_cast<int32_t>(threadIdx.x); k < r.count;
         k += static_cast<int32_t>(gridDim.x) * 256) {
        const int32_t di = r.desc0 + k;
        const uint64_t off = static_cast<uint64_t>(k) * r.stride;
        NzSample d = r.first;
        d.sample += static_cast<uint64_t>(k);
        d.off_par += off;
        d.off_occ += off;
        d.off_sites += off;
        d.off_counts += off;
        d.off_prefix += off;
        d.off_parc += off;
        d.off_wrec += off;
        d.off_sum += off;
        d.off_win += off;
        desc[di] = d;
        NzState s;
        s.status = NZ_ST_PENDING;
        s.nstar = 0;
        s.mass = 0;
        s.n0 = 0;
        s.smax = 0;
        state[di] = s;
        queue[r.queue0 + k] = di;
        out_index[di] = r.out0 + k;
        if (r.list0 >= 0) list[r.list0 + k] = di;
    }
}

// ---------------------------------------------------------------------------
// Clearing: bucket counters and summaries; samples that back off also take
// their next threshold and start over.

__global__ __launch_bounds__(256) void nz_clear_kernel(NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                       int32_t nsamp, int32_t level, uint8_t *__restrict__ ws,
                                                       NzState *__restrict__ state)
{
    if (static_cast<int32_t>(blockIdx.x) >= nsamp) return;
    const int sid = list ? list[blockIdx.x] : static_cast<int>(blockIdx.x);
    NzSample &d = desc[sid];
    const int32_t nb = list ? d.nbb[level] : d.nb;
    uint32_t *counts = reinterpret_cast<uint32_t *>(ws + d.off_counts);
    for (int b = threadIdx.x; b < nb; b += blockDim.x) counts[b] = 0u;
    uint32_t *sum = reinterpret_cast<uint32_t *>(ws + d.off_sum);
    for (int w = threadIdx.x; w < d.sum_words; w += blockDim.x) sum[w] = 0u;
    if (list && threadIdx.x == 0) {
        d.T0 = d.T0b[level];
        d.nb = nb;
        state[sid].status = NZ_ST_PENDING;
        state[sid].n0 = 0;
        state[sid].smax = 0;
    }
}

// ---------------------------------------------------------------------------
// Keys, prefill occupancy and band bucketing.  A block covers
// KEYS_THREADS * 2 * KEYS_ITERS consecutive sites of one sample, wave w the
// KEYS_WAVE_SITES sites from w * KEYS_WAVE_SITES; per iteration a wave takes
// 128 consecutive sites, lane l the pair (2l, 2l + 1) that shares one Philox
// block, so two ballots yield four bitset words.  Lane `it` keeps iteration
// it's ballots; after the loop lane l builds word l & 3 of iteration 16 g +
// l / 4 for every group g of 16 iterations, so the bit interleave runs once for
// all of a wave's words.  A wave's fixed costs (its sample's descriptor, the
// list atomic, the scans) are paid once per KEYS_WAVE_SITES sites: with 1024,
// 2048, 4096 and 8192 sites per wave the kernel alone took 2.99, 1.97, 1.77
// and 1.71 ms for 2000 samples of L = 16, zones 1-7, and 6.72, 4.58, 3.43 and
// 2.88 ms for zone 1.

constexpr int KEYS_THREADS = 256;
constexpr int KEYS_LOCAL_THREADS = 1024;   // at most
#ifndef NZ_KEYS_ITERS
#define NZ_KEYS_ITERS 64
#endif
constexpr int KEYS_ITERS = NZ_KEYS_ITERS;
constexpr int KEYS_WAVE_SITES = 128 * KEYS_ITERS;
constexpr int KEYS_GROUPS = KEYS_ITERS / 16;   // groups of 64 bitset words in a wave's range
constexpr int KEYS_SITES_PER_BLOCK = KEYS_THREADS * 2 * KEYS_ITERS;
static_assert(KEYS_ITERS % 16 == 0 && KEYS_ITERS <= 64, "whole 64-word groups; lane it keeps iteration it");
static_assert(KEYS_SITES_PER_BLOCK == (KEYS_THREADS / 64) * KEYS_WAVE_SITES, "waves tile the block");

// by_xcd: the workgroups of one sample share blockIdx mod 8, so that they are
// dispatched to one XCD: the sample's band buckets and their counters, which
// every workgroup of the sample appends to, then stay in one L2 and a bucket's
// lines fill there.  Measured alone (1000 samples, L = 16): zone 1 plain, 16% of
// the sites in the band, 11.1 -> 7.5 ms (L = 24, 200 samples: 19.5 -> 10.9);
// with 4% or less in the band the spread over all XCDs is faster (zones 1-2
// plain 1.50 against 1.88 ms, zone 1 prefilled 1.38 against 1.87), and few
// samples would leave XCDs idle; the planner draws the line at 8%.

// Predicate code of an unsigned less-than for the lane-mask compare builtins.
constexpr int kIcmpUlt = 36;

// The 16 bits of x moved to the even bit positions of a 32-bit word.
__device__ __forceinline__ uint32_t spread_even(uint32_t x)
{
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    x = (x | (x << 1)) & 0x55555555u;
    return x;
}

struct KeysCtx {
    uint64_t T0;
    int32_t shift;
    uint64_t nb;
    uint32_t cap;
    uint32_t L;
    uint64_t magic;
    int32_t *par;
    uint32_t *sites;
    uint32_t *counts;
};

// Dynamic LDS of the local kernel: the bucket counters, then the waves' queues.
extern __shared__ __attribute__((aligned(16))) uint32_t keys_lds[];

// Band sites of a wave are queued in LDS and bucketed 64 at a time, one per
// lane, so the bucketing work runs on full waves although only a few percent of
// the sites fall into the band.
constexpr uint32_t KEYS_BQ = 192;   // queue entries per wave (< 64 left + 128 new)

template <bool LOCAL>
__device__ __forceinline__ void keys_bucket(const KeysCtx &c, uint64_t K, uint32_t i)
{
    const uint64_t b = (K - c.T0) >> c.shift;
    uint32_t slot;
    if constexpr (LOCAL) slot = atomicAdd(&keys_lds[b], 1u);
    else slot = atomicAdd(&c.counts[b], 1u);
    if (slot < c.cap) c.sites[b * c.cap + slot] = pack_coords(i, c.L, c.magic);
}

// The iterations of one wave over a block: keys, the prefill and band masks,
// the prefill ballots (lane it keeps iteration it's) and the band queue.
// FULL: the block lies wholly inside the lattice (no site needs a range test);
// BALL: the band reaches 2^64 (every key at or above T0 is in it); HI: T0 and
// the band's end are multiples of 2^32, so comparing high words decides.
struct KeysIter {
    const KeysCtx &c;
    uint64_t *qk;
    uint32_t *qs;
    uint32_t N;
    uint32_t wave_base;
    uint32_t lane;
    uint64_t band_end;
    uint32_t seed_lo, seed_hi, smp_lo, smp_hi;
};

template <bool LOCAL, bool FULL, bool BALL, bool HI>
__device__ __forceinline__ void keys_iters(const KeysIter &k, uint32_t &be_lo, uint32_t &be_hi, uint32_t &bo_lo,
                                           uint32_t &bo_hi, int &its, uint32_t &nq)
{
    const KeysCtx &c = k.c;
    uint64_t *qk = k.qk;
    uint32_t *qs = k.qs;
    const uint32_t lane = k.lane, lane2 = 2u * k.lane;
    for (int it = 0; it < KEYS_ITERS; ++it) {
        const uint32_t wbase = k.wave_base + static_cast<uint32_t>(it) * 128u;   // (scalar)
        if (wbase >= k.N) break;
        its = it + 1;
        uint64_t K0, K1;
        site_key_pair(k.seed_lo, k.seed_hi, k.smp_lo, k.smp_hi, (wbase >> 1) + lane, K0, K1);
        // lane masks of the compares (prefilled: key < T0; band: T0 <= key <
        // band_end), combined on the scalar unit
        const uint64_t vm0 = FULL ? ~0ull : __builtin_amdgcn_uicmp(wbase + lane2, k.N, kIcmpUlt);
        const uint64_t vm1 = FULL ? ~0ull : __builtin_amdgcn_uicmp(wbase + lane2 + 1u, k.N, kIcmpUlt);
        uint64_t be, bo, qe, qo;
        if constexpr (HI) {
            // T0 and band_end are multiples of 2^32: the keys' high words decide
            const uint32_t h0 = static_cast<uint32_t>(K0 >> 32), h1 = static_cast<uint32_t>(K1 >> 32);
            const uint32_t t0 = static_cast<uint32_t>(c.T0 >> 32), te = static_cast<uint32_t>(k.band_end >> 32);
            be = vm0 & __builtin_amdgcn_uicmp(h0, t0, kIcmpUlt);
            bo = vm1 & __builtin_amdgcn_uicmp(h1, t0, kIcmpUlt);
            qe = (vm0 & ~be) & (BALL ? ~0ull : __builtin_amdgcn_uicmp(h0, te, kIcmpUlt));
            qo = (vm1 & ~bo) & (BALL ? ~0ull : __builtin_amdgcn_uicmp(h1, te, kIcmpUlt));
        } else {
            be = vm0 & __builtin_amdgcn_uicmpl(K0, c.T0, kIcmpUlt);
            bo = vm1 & __builtin_amdgcn_uicmpl(K1, c.T0, kIcmpUlt);
            qe = (vm0 & ~be) & (BALL ? ~0ull : __builtin_amdgcn_uicmpl(K0, k.band_end, kIcmpUlt));
            qo = (vm1 & ~bo) & (BALL ? ~0ull : __builtin_amdgcn_uicmpl(K1, k.band_end, kIcmpUlt));
        }
        if (lane == static_cast<uint32_t>(it)) {
            be_lo = static_cast<uint32_t>(be);
            be_hi = static_cast<uint32_t>(be >> 32);
            bo_lo = static_cast<uint32_t>(bo);
            bo_hi = static_cast<uint32_t>(bo >> 32);
        }
        // band: queued, then bucketed in full waves
        const uint32_t nqe = static_cast<uint32_t>(__popcll(qe));
        if (qe) {
            if (__builtin_amdgcn_inverse_ballot_w64(qe)) {
                const uint32_t e = nq + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(qe >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(qe), 0u));
                qk[e] = K0;
                qs[e] = wbase + lane2;
            }
        }
        if (qo) {
            if (__builtin_amdgcn_inverse_ballot_w64(qo)) {
                const uint32_t e = nq + nqe + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(qo >> 32),
                                                                        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(qo), 0u));
                qk[e] = K1;
                qs[e] = wbase + lane2 + 1u;
            }
        }
        nq = __builtin_amdgcn_readfirstlane(nq + nqe + static_cast<uint32_t>(__popcll(qo)));
        __builtin_amdgcn_wave_barrier();
        if (nq >= 64u) {
            uint32_t base = 0;
            for (; base + 64u <= nq; base += 64u) keys_bucket<LOCAL>(c, qk[base + lane], qs[base + lane]);
            // move the remainder (< 64 entries) to the front
            const uint32_t rest = nq - base;
            uint64_t rk = 0;
            uint32_t rs = 0;
            if (lane < rest) {
                rk = qk[base + lane];
                rs = qs[base + lane];
            }
            __builtin_amdgcn_wave_barrier();
            if (lane < rest) {
                qk[lane] = rk;
                qs[lane] = rs;
            }
            __builtin_amdgcn_wave_barrier();
            nq = __builtin_amdgcn_readfirstlane(rest);
        }
    }
}

// One wave's KEYS_WAVE_SITES consecutive sites from wave_base (a multiple of
// 2048, so that its bitset words start on a 64-word boundary) of sample sid,
// queue qk / qs.  Waves work alone: no workgroup barrier, so a wave that waits
// for its list atomic or its sample's descriptor leaves the SIMD to the others.
// The wave's prefilled sites are appended to the sample's list in site order
// with one atomic on *n0, and every bitset word's list position is stored, so
// that a site's list position is that of its word plus the set bits below it.
template <bool LOCAL>
__device__ __forceinline__ void keys_wave(const NzSample &d, uint32_t N, uint32_t wave_base, uint64_t *qk, uint32_t *qs,
                                          uint8_t *__restrict__ ws, uint32_t *n0)
{
    const uint32_t lane = lane_id();
    const uint32_t seed_lo = static_cast<uint32_t>(d.seed), seed_hi = static_cast<uint32_t>(d.seed >> 32);
    const uint32_t smp_lo = static_cast<uint32_t>(d.sample), smp_hi = static_cast<uint32_t>(d.sample >> 32);
    const uint32_t occ_words = ((N + 63u) >> 6) << 1;   // padded to whole 64-site words

    KeysCtx c;
    c.T0 = d.T0;
    c.shift = d.shift;
    c.nb = static_cast<uint64_t>(d.nb);
    c.cap = static_cast<uint32_t>(d.cap);
    c.L = static_cast<uint32_t>(d.L);
    c.magic = d.magic;
    c.par = reinterpret_cast<int32_t *>(ws + d.off_par);
    c.sites = reinterpret_cast<uint32_t *>(ws + d.off_sites);
    c.counts = reinterpret_cast<uint32_t *>(ws + d.off_counts);
    uint32_t *occ = reinterpret_cast<uint32_t *>(ws + d.off_occ);
    uint32_t *prefix = reinterpret_cast<uint32_t *>(ws + d.off_prefix);
    // keys in [T0, band_end) fall into the band (band_end saturates at 2^64)
    const uint64_t span = c.nb << c.shift;
    const bool band_all = c.shift >= 64 || (span >> c.shift) != c.nb || c.T0 + span < c.T0;
    const uint64_t band_end = c.T0 + span;

    uint32_t nq = 0;        // wave-uniform
    // wave-uniform choices held in scalar registers: whether the wave's range
    // lies wholly inside the lattice (then no site needs a range test) and
    // whether the band reaches 2^64
    const bool full = __builtin_amdgcn_readfirstlane(wave_base + KEYS_WAVE_SITES <= N ? 1u : 0u) != 0u;
    const bool ball = __builtin_amdgcn_readfirstlane(band_all ? 1u : 0u) != 0u;
    // thresholds on 2^32 boundaries (the planner's choice): 32-bit compares
    const bool hi = __builtin_amdgcn_readfirstlane(
                        ((c.T0 | (band_all ? 0ull : band_end)) & 0xFFFFFFFFull) == 0ull ? 1u : 0u) != 0u;
    // even / odd prefill ballots of iteration it, held by lane it
    uint32_t be_lo = 0, be_hi = 0, bo_lo = 0, bo_hi = 0;
    int its = 0;            // iterations this wave ran (wave-uniform)
    // the loop is compiled for each combination of the two wave-uniform
    // choices, so that no iteration tests them
    KeysIter ki{c, qk, qs, N, wave_base, lane, band_end, seed_lo, seed_hi, smp_lo, smp_hi};
    if (hi) {
        if (full) {
            if (ball) keys_iters<LOCAL, true, true, true>(ki, be_lo, be_hi, bo_lo, bo_hi, its, nq);
            else keys_iters<LOCAL, true, false, true>(ki, be_lo, be_hi, bo_lo, bo_hi, its, nq);
        } else {
            if (ball) keys_iters<LOCAL, false, true, true>(ki, be_lo, be_hi, bo_lo, bo_hi, its, nq);
            else keys_iters<LOCAL, false, false, true>(ki, be_lo, be_hi, bo_lo, bo_hi, its, nq);
        }
    } else if (full) {
        if (ball) keys_iters<LOCAL, true, true, false>(ki, be_lo, be_hi, bo_lo, bo_hi, its, nq);
        else keys_iters<LOCAL, true, false, false>(ki, be_lo, be_hi, bo_lo, bo_hi, its, nq);
    } else {
        if (ball) keys_iters<LOCAL, false, true, false>(ki, be_lo, be_hi, bo_lo, bo_hi, its, nq);
        else keys_iters<LOCAL, false, false, false>(ki, be_lo, be_hi, bo_lo, bo_hi, its, nq);
    }
    if (lane < nq) keys_bucket<LOCAL>(c, qk[lane], qs[lane]);

    // Word q of iteration it (sites wave_base + 128 it .. + 127) interleaves
    // bits 16q .. 16q + 15 of the even and odd ballots.  The range's words come
    // in groups of 64, one word per lane: lane l of group g builds word 64 g + l,
    // that of iteration 16 g + l / 4.  Words of iterations that did not run are
    // zero; words past the padded bitset are not stored.
    const uint32_t q = lane & 3u;
    const uint32_t w0 = wave_base >> 5;
    uint32_t word[KEYS_GROUPS];
    bool mine[KEYS_GROUPS];
#pragma unroll
    for (int g = 0; g < KEYS_GROUPS; ++g) {
        const int src = 16 * g + static_cast<int>(lane >> 2);
        const uint32_t elo = static_cast<uint32_t>(__shfl(static_cast<int>(be_lo), src));
        const uint32_t ehi = static_cast<uint32_t>(__shfl(static_cast<int>(be_hi), src));
        const uint32_t olo = static_cast<uint32_t>(__shfl(static_cast<int>(bo_lo), src));
        const uint32_t ohi = static_cast<uint32_t>(__shfl(static_cast<int>(bo_hi), src));
        const uint32_t sh = 16u * (q & 1u);
        const uint32_t e16 = ((q < 2u ? elo : ehi) >> sh) & 0xFFFFu;
        const uint32_t o16 = ((q < 2u ? olo : ohi) >> sh) & 0xFFFFu;
        mine[g] = src < its;
        word[g] = mine[g] ? (spread_even(e16) | (spread_even(o16) << 1)) : 0u;
        const uint32_t w = w0 + 64u * static_cast<uint32_t>(g) + lane;
        if (mine[g] && w < occ_words) occ[w] = word[g];
    }
    if (d.T0 == 0) return;   // plain sample: nothing prefilled (uniform over the grid)

    // summary bits of the range's non-empty words, and the exclusive scan of
    // the word counts of every group
    uint32_t *sum = reinterpret_cast<uint32_t *>(ws + d.off_sum);
    const uint32_t gs = static_cast<uint32_t>(d.sum_shift);
    uint32_t wc[KEYS_GROUPS], excl[KEYS_GROUPS], cnt[KEYS_GROUPS];
    uint32_t total = 0;
#pragma unroll
    for (int g = 0; g < KEYS_GROUPS; ++g) {
        wc[g] = static_cast<uint32_t>(__popc(word[g]));
        const uint32_t wg0 = w0 + 64u * static_cast<uint32_t>(g);   // a multiple of 64
        if (d.sum_words > 0) {
            const uint64_t nzw = __ballot(wc[g] != 0u);
            if (gs == 0u) {
                // one bit per word: the group's bits fill two whole words
                const uint32_t half = lane < 2u ? static_cast<uint32_t>(nzw >> (32u * lane)) : 0u;
                if (half) atomicOr(&sum[(wg0 >> 5) + lane], half);
            } else if (lane == 0u && nzw) {
                // bit j of v: any of the 2^gs words j << gs .. of the group (1 <=
                // gs <= 4); k is a multiple of 64 >> gs, so v fits in one word
                const uint32_t span_bits = 64u >> gs;
                const uint64_t grp = (1ull << (1u << gs)) - 1ull;
                uint32_t v = 0u;
                for (uint32_t j = 0; j < span_bits; ++j)
                    if ((nzw >> (j << gs)) & grp) v |= 1u << j;
                const uint32_t k = wg0 >> gs;
                atomicOr(&sum[k >> 5], v << (k & 31u));
            }
        }
        uint32_t incl = wc[g];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = static_cast<uint32_t>(__shfl_up(static_cast<int>(incl), o));
            if (lane >= static_cast<uint32_t>(o)) incl += v;
        }
        excl[g] = incl - wc[g];
        cnt[g] = __builtin_amdgcn_readlane(incl, 63);
        total += cnt[g];
    }
    uint2 *wrec = reinterpret_cast<uint2 *>(ws + d.off_wrec);
    if (total == 0u) {   // wave-uniform: nothing prefilled in the range
        if (!d.wrap)
#pragma unroll
            for (int g = 0; g < KEYS_GROUPS; ++g) {
                const uint32_t w = w0 + 64u * static_cast<uint32_t>(g) + lane;
                if (mine[g] && w < occ_words) wrec[w] = make_uint2(0u, 0u);
            }
        return;
    }
    uint32_t got = 0u;
    if (lane == 0u) got = atomicAdd(n0, total);
    uint32_t base = __builtin_amdgcn_readlane(got, 0);
    const uint32_t cap = static_cast<uint32_t>(d.prefix_cap);
    int32_t *parc = reinterpret_cast<int32_t *>(ws + d.off_parc);
#pragma unroll
    for (int g = 0; g < KEYS_GROUPS; ++g) {
        const uint32_t w = w0 + 64u * static_cast<uint32_t>(g) + lane;
        uint32_t pos = base + excl[g];
        if (!d.wrap && mine[g] && w < occ_words) wrec[w] = make_uint2(pos, word[g]);
        // the word's sites in bit order, one lane per word
        uint32_t bits = word[g];
        const uint32_t site0 = w << 5;
        while (bits) {
            const uint32_t sidx = site0 + static_cast<uint32_t>(__builtin_ctz(bits));
            bits &= bits - 1u;
            if (pos < cap) {
                prefix[pos] = sidx;
                // parent = itself (periodic first-wrap: lattice entry, displacement 0)
                if (d.wrap) reinterpret_cast<uint64_t *>(c.par)[sidx] = sidx;
                else parc[pos] = static_cast<int32_t>(pos);
            }
            ++pos;
        }
        base += cnt[g];
    }
}

// A workgroup per KEYS_SITES_PER_BLOCK sites.
__global__ __launch_bounds__(KEYS_THREADS) void nz_keys_kernel(const NzSample *__restrict__ desc,
                                                               const int32_t *__restrict__ list, int32_t first, int32_t count,
                                                               bool by_xcd, int32_t blocks_per_sample,
                                                               uint8_t *__restrict__ ws, NzState *__restrict__ state)
{
    __shared__ uint64_t bq_key[KEYS_THREADS / 64][KEYS_BQ];
    __shared__ uint32_t bq_site[KEYS_THREADS / 64][KEYS_BQ];
    const uint32_t wave = threadIdx.x >> 6;
    const int32_t vb = static_cast<int32_t>(blockIdx.x);
    int which = vb / blocks_per_sample;
    int blk = vb % blocks_per_sample;
    if (by_xcd) {
        const int k = vb >> 3;
        which = (k / blocks_per_sample) * 8 + (vb & 7);
        blk = k % blocks_per_sample;
        if (which >= count) return;   // (uniform over the workgroup)
    }
    const int sid = list ? list[first + which] : first + which;
    const NzSample &d = desc[sid];
    const uint32_t N = static_cast<uint32_t>(d.N);
    const uint32_t wave_base =
        __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(blk) * KEYS_SITES_PER_BLOCK + KEYS_WAVE_SITES * wave);
    if (wave_base >= N) return;   // wave-uniform
    keys_wave<false>(d, N, wave_base, bq_key[wave], bq_site[wave], ws, reinterpret_cast<uint32_t *>(&state[sid].n0));
}

// One workgroup per sample, for samples whose band holds more than 3% of the
// sites.  With several workgroups per sample every band site costs a returning
// atomic on its bucket's counter in the L2, and the chip does 29 G of those a
// second wherever the counters lie, an eighth of the rate of the stores they
// order; here the counters and the length of the prefill list are
// in LDS, and the counters are written out once.  Keys, several workgroups per
// sample / one: L = 16 zone 1 plain (16% of the sites in the band) 7.6 / 1.7 ms
// for 1000 samples, 0.93 / 0.36 for 125, L = 24 10.7 / 3.6 for 200; zones 1-2
// plain (4.4%) 1.43 / 1.05 ms for 1000, L = 24 3.2 / 2.3 for 200; zone 1 prefilled,
// L = 16 (3.2%) 1.70 / 1.17 for 1000.  With less in the band the atomics are few
// and the finer spread over the chip wins: zone 1 prefilled, L = 24 (2.2%), 2.3 / 2.7 for
// 200, zones 1-6 prefilled, L = 16, 0.81 / 0.88 for 1000.  max_nb: words of the
// counters (an even number; every sample of the launch has at most so many
// buckets).
__global__ __launch_bounds__(KEYS_LOCAL_THREADS, 8) void nz_keys_kernel_local(const NzSample *__restrict__ desc, int32_t first,
                                                                              int32_t max_nb, uint8_t *__restrict__ ws,
                                                                              NzState *__restrict__ state)
{
    __shared__ uint32_t n0;
    const int sid = first + static_cast<int>(blockIdx.x);
    const NzSample &d = desc[sid];
    const uint32_t N = static_cast<uint32_t>(d.N);
    const int32_t nb = min(d.nb, max_nb);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    for (int32_t b = static_cast<int32_t>(threadIdx.x); b < nb; b += static_cast<int32_t>(blockDim.x)) keys_lds[b] = 0u;
    if (threadIdx.x == 0) n0 = 0u;
    __syncthreads();
    uint64_t *qk = reinterpret_cast<uint64_t *>(keys_lds + max_nb) + wave * KEYS_BQ;
    uint32_t *qs = keys_lds + max_nb + 2 * waves * KEYS_BQ + wave * KEYS_BQ;
    for (uint32_t base = wave * KEYS_WAVE_SITES; base < N; base += waves * KEYS_WAVE_SITES)
        keys_wave<true>(d, N, base, qk, qs, ws, &n0);
    __syncthreads();
    uint32_t *counts = reinterpret_cast<uint32_t *>(ws + d.off_counts);
    for (int32_t b = static_cast<int32_t>(threadIdx.x); b < nb; b += static_cast<int32_t>(blockDim.x)) counts[b] = keys_lds[b];
    if (threadIdx.x == 0) state[sid].n0 = static_cast<int32_t>(n0);
}

// ---------------------------------------------------------------------------
// Bulk connected components of the prefilled sites (hook, then label).
// During this phase par[i] is a plain parent index and a root points to
// itself.  Every link goes from a larger index to a smaller one, and only an
// agent-scope CAS that finds par[u] == u links u, so along every path indices
// decrease and no cycle can form.  The walks therefore read through the caches
// (wavefront-scope accesses): a stale entry is still an ancestor (or a former
// root), which can only make a CAS fail and retry from the value it returns,
// one true step further up; path-halving writes store an ancestor.

// Workgroup l of a prefill launch covers block x of sample slot y.  The
// workgroups of one sample share l mod 8, so they are dispatched to the same
// XCD and the sample's bitset and parents stay in that XCD's L2.
__device__ __forceinline__ bool xcd_slot(int32_t nlist, int32_t bx, int32_t &y, int32_t &x)
{
    const uint32_t l = blockIdx.x;
    const uint32_t k = l >> 3;
    y = static_cast<int32_t>((k / static_cast<uint32_t>(bx)) * 8u + (l & 7u));
    x = static_cast<int32_t>(k % static_cast<uint32_t>(bx));
    return y < nlist;
}

// The bulk labelling runs on the prefilled sites' list positions, not on
// lattice indices: parc[i] is the parent of list entry i, so the whole forest
// of a sample is 4 bytes per prefilled site and stays in the L2 of the XCD that
// holds the sample.  The list position of an occupied neighbour t is the
// position of its bitset word plus the set bits below t in that word; both are
// read as one 8-byte record per word.
// The forest stays what it is through the sweep: prefilled sites have no lattice
// entries, their roots keep their root words in it, and band sites link to its
// nodes.

// A union-find node id: a lattice site s (< 2^29) or LIST_NODE | i, list entry
// i of the sample's prefilled sites.  Parent entries hold node ids or root
// words (bit 31 set).
constexpr int32_t LIST_NODE = 0x20000000;

// Hook: one lane per prefilled site and its forward half of the offset table
// (one row of each +-d pair), six rows loaded at a time.  The edges a
// wave finds (site, occupied neighbour) are not linked where they are found:
// each offset slot has only a few lanes with an occupied neighbour, so linking
// slot by slot would run one round of dependent finds per slot with most lanes
// idle.  They are appended to a per-wave edge buffer in LDS instead, and the
// buffer is linked 64 edges at a time, every lane with an edge of its own.
constexpr int HOOK_UNROLL = 6;   // rows checked together
constexpr int HOOKW_UNROLL = 8;  // half as many rows (each has an entry per side)
// edges buffered per wave: one offset slot adds at most 64, and the buffer is
// emptied whenever it holds 64 or more (a small buffer leaves LDS for more
// resident workgroups: this kernel is bound by the latency of its dependent
// loads and atomics)
constexpr int HOOK_EBUF = 128;
constexpr int HOOK_ROWS = 150;   // one row of every +- pair of the widest neighbourhood (149)

// Summary words a hook workgroup stages in LDS (the host sizes summaries to at
// most 1025 words).
constexpr int32_t HOOK_SUM_MAX = 1025;

// Words of the occupation map outside the lattice: one before, two behind.
constexpr uint32_t MAP_PAD = 3;

// The map's shift for a lattice of N sites when map_words words are there.
__host__ __device__ __forceinline__ uint32_t map_shift(uint32_t N, uint32_t map_words)
{
    uint32_t ms = 0;
    while ((((N - 1u) >> ms) >> 5) + 1u + MAP_PAD > map_words) ++ms;
    return ms;
}

// Links list positions a and b: CAS links go from the larger root to the
// smaller, only onto an entry that is still a root, retried from the parent the
// CAS returns.
__device__ __forceinline__ void cc_link(int32_t *par, int32_t a, int32_t b)
{
    // A root may point at any smaller member of another tree (links go from larger
    // to smaller positions, so every entry's root is at or below it): where the
    // larger end is still its own root, one CAS without finds does (zone 1, L = 16,
    // 1000 samples: hook 3.08 -> 2.94 ms).
    const int32_t top = max(a, b), low = min(a, b);
    int32_t seen = ld_w(&par[top]);
    if (seen == top && __hip_atomic_compare_exchange_strong(&par[top], &seen, low, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT))
        return;
    a = seen;
    b = low;
    for (;;) {
        // both finds in step, so that their loads overlap; path splitting: every
        // entry on the way skips to its grandparent
        int32_t u = a, v = b;
        int32_t pu = ld_w(&par[u]), pv = ld_w(&par[v]);
        while (pu != u || pv != v) {
            const int32_t gu = ld_w(&par[pu]), gv = ld_w(&par[pv]);
            if (gu != pu) st_w(&par[u], gu);
            if (gv != pv) st_w(&par[v], gv);
            u = pu;
            v = pv;
            pu = gu;
            pv = gv;
        }
        if (u == v) return;
        const int32_t hi = max(u, v), lo = min(u, v);
        int32_t expected = hi;
        if (__hip_atomic_compare_exchange_strong(&par[hi], &expected, lo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return;
        // hi is no longer a root: go on from the parent the CAS returned
        a = expected;
        b = lo;
    }
}

// The buffered edges 0 .. ne-1 of one wave, 64 at a time.
__device__ __forceinline__ void hook_flush(int32_t *par, const int32_t *ei, const int32_t *ej, int32_t ne, uint32_t lane)
{
    for (int32_t e0 = 0; e0 < ne; e0 += 64) {
        const int32_t e = e0 + static_cast<int32_t>(lane);
        if (e < ne) cc_link(par, ld_w(&ei[e]), ld_w(&ej[e]));
    }
}

// PER: periodic coordinates (compiled apart, so that the free-boundary hook
// carries no wrap correction).
template <bool PER>
__global__ __launch_bounds__(256) void nz_hook_kernel(const NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                      int32_t nlist, int32_t bx, const NzOffset *__restrict__ tabs,
                                                      uint8_t *__restrict__ ws, NzState *__restrict__ state)
{
    __shared__ uint32_t hsum[HOOK_SUM_MAX];
    __shared__ int32_t ebuf_i[4][HOOK_EBUF];
    __shared__ int32_t ebuf_j[4][HOOK_EBUF];
    int32_t y, x;
    if (!xcd_slot(nlist, bx, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    const int32_t n0 = state[sid].n0;
    if (n0 > d.prefix_cap || d.wrap || x * 256 >= n0) return;   // (uniform over the workgroup)
    // A sparse prefill (under one site in 32) leaves most bitset words empty:
    // the workgroup stages the bitset summary in LDS and skips the loads of
    // empty words.
    const bool use_sum = d.sum_words > 0 && d.sum_words <= HOOK_SUM_MAX && static_cast<int64_t>(n0) * 32 < d.N;
    if (use_sum) {
        const uint32_t *sum_g = reinterpret_cast<const uint32_t *>(ws + d.off_sum);
        for (int32_t w = static_cast<int32_t>(threadIdx.x); w < d.sum_words; w += 256) hsum[w] = sum_g[w];
    }
    __syncthreads();
    const uint32_t gs = static_cast<uint32_t>(d.sum_shift);
    const int32_t L = d.L;
    const int32_t rh = d.rows >> 1;   // one row of every +- pair
    const uint64_t magic = d.magic;
    int32_t *par = reinterpret_cast<int32_t *>(ws + d.off_parc);
    const uint32_t *occ = reinterpret_cast<const uint32_t *>(ws + d.off_occ);
    const uint2 *wrec = reinterpret_cast<const uint2 *>(ws + d.off_wrec);
    const uint32_t *prefix = reinterpret_cast<const uint32_t *>(ws + d.off_prefix);
    const NzOffset *tab = tabs + d.tab;
    const uint32_t lane = lane_id();
    const uint32_t wave = threadIdx.x >> 6;
    int32_t *ei = ebuf_i[wave];
    int32_t *ej = ebuf_j[wave];
    int32_t ne = 0;   // edges in the buffer (wave-uniform), carried from pass to pass
    // the wave's 64 sites per pass (wave-uniform loop; lanes past n0 idle)
    for (int32_t ib = x * 256 + static_cast<int32_t>(wave) * 64; ib < n0; ib += bx * 256) {
        const int32_t i = ib + static_cast<int32_t>(lane);
        const bool act = i < n0;
        const int32_t s = act ? static_cast<int32_t>(prefix[i]) : 0;
        const uint32_t pc = pack_coords(static_cast<uint32_t>(s), static_cast<uint32_t>(L), magic);
        const uint32_t A = act ? allowed_of(pc, L) : 0u;
        int32_t below = -1;   // the first neighbour found with a smaller list position
        // appends the lanes' edges (i, j) and links the buffer when it is full
        auto push = [&](bool edge, int32_t j) {
            const uint64_t mk = __ballot(edge);
            if (edge) {
                const int32_t e = ne + static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(
                                           static_cast<uint32_t>(mk >> 32),
                                           __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mk), 0u)));
                st_w(&ei[e], i);
                st_w(&ej[e], j);
            }
            ne += static_cast<int32_t>(__popcll(mk));
            if (ne >= 64) {
                // link the last 64; the rest stays for a later round
                __builtin_amdgcn_wave_barrier();
                ne -= 64;
                hook_flush(par, ei + ne, ej + ne, 64, lane);
                __builtin_amdgcn_wave_barrier();
            }
        };
        const int32_t x0 = static_cast<int32_t>(pc & 63);
        for (int32_t k0 = 0; k0 < rh; k0 += HOOK_UNROLL) {
            // side 1 (periodic only): the steps that leave along axis 0, on the
            // other side of the row
            for (int side = 0; side < (PER ? 2 : 1); ++side) {
                int32_t b[HOOK_UNROLL];
                uint32_t v[HOOK_UNROLL];
#pragma unroll
                for (int q = 0; q < HOOK_UNROLL; ++q) {
                    NzOffset o;
                    o.stride = 0;
                    o.code = 0u;
                    if (k0 + q < rh) o = tab[k0 + q];
                    const uint32_t out = o.code & ~A & kRowAxes;
                    uint32_t dm;   // the row's sites to look at, from b on
                    if constexpr (PER) {
                        b[q] = s + o.stride - 2 + (out ? wrap_fix(out, L) : 0);
                        dm = act ? o.code & (side ? ~A : A) & 31u : 0u;
                        if (side) b[q] += x0 < 2 ? L : -L;
                    } else {
                        b[q] = s + o.stride - 2;
                        dm = act && out == 0u ? o.code & A & 31u : 0u;
                    }
                    const int32_t c = __builtin_ctz(dm | 32u);
                    const uint32_t p0 = dm ? static_cast<uint32_t>(b[q] + c) : 0u;
                    const uint32_t wi = p0 >> 5;
                    const bool maybe = !use_sum || ((hsum[(wi >> gs) >> 5] >> ((wi >> gs) & 31)) & 1u);
                    const uint32_t w0 = dm && maybe ? occ[wi] : 0u;
                    uint32_t w1 = 0u;
                    if (o.code & 31u & ((o.code & 31u) - 1u)) {   // (uniform) more than one site in the row
                        const uint32_t p1 = static_cast<uint32_t>(b[q] + 31 - __builtin_clz(dm | 1u));
                        if (dm && (p1 >> 5) != wi) w1 = occ[wi + 1u];
                    }
                    v[q] = (__builtin_amdgcn_alignbit(w1, w0, p0 & 31u) << c) & dm;
                }
                // list positions of the occupied neighbours, from their words' records
                // (loaded together for the first site of every row)
                uint2 rec[HOOK_UNROLL];
#pragma unroll
                for (int q = 0; q < HOOK_UNROLL; ++q)
                    rec[q] = v[q] ? wrec[static_cast<uint32_t>(b[q] + __builtin_ctz(v[q])) >> 5] : make_uint2(0u, 0u);
#pragma unroll
                for (int q = 0; q < HOOK_UNROLL; ++q) {
                    bool first = true;
                    while (__ballot(v[q] != 0u)) {
                        bool edge = false;
                        int32_t j = 0;
                        if (v[q]) {
                            const int c = __builtin_ctz(v[q]);
                            v[q] &= v[q] - 1u;
                            const uint32_t p = static_cast<uint32_t>(b[q] + c);
                            if (!first) rec[q] = wrec[p >> 5];
                            j = static_cast<int32_t>(rec[q].x + static_cast<uint32_t>(__popc(rec[q].y & ((1u << (p & 31)) - 1u))));
                            // the first neighbour below is linked without finds (at the end)
                            edge = below >= 0 || j > i;
                            if (!edge) below = j;
                        }
                        push(edge, j);
                        first = false;
                    }
                }
            }
        }
        // Links go from larger to smaller positions, so every entry's root is at
        // or below it: i may point at any smaller member of a neighbour's tree
        // as long as it is a root itself.  One CAS, no finds; an entry that
        // another wave has already linked takes the ordinary way.
        bool left = false;
        if (below >= 0) {
            int32_t expected = i;
            left = !__hip_atomic_compare_exchange_strong(&par[i], &expected, below, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
        }
        push(left, below);
    }
    __builtin_amdgcn_wave_barrier();
    hook_flush(par, ei, ej, ne, lane);
}

// The pairs a wave has found: list position of a site, lattice index of an
// occupied neighbour.
struct HookEdges {
    int32_t *par;
    const uint2 *wrec;
    int32_t *ei, *ep;   // LDS, HOOK_EBUF each
    int32_t ne;         // pairs in the buffer (wave-uniform), carried from pass to pass
    uint32_t lane;

    // links the pairs e0 .. e0 + n - 1 (n <= 64): neighbours' list positions from
    // their words' records
    __device__ __forceinline__ void link(int32_t e0, int32_t n)
    {
        __builtin_amdgcn_wave_barrier();
        if (static_cast<int32_t>(lane) < n) {
            const int32_t p = ld_w(&ep[e0 + static_cast<int32_t>(lane)]);
            const uint2 rec = wrec[p >> 5];
            const int32_t i = ld_w(&ei[e0 + static_cast<int32_t>(lane)]);
            const int32_t j = static_cast<int32_t>(rec.x + static_cast<uint32_t>(__popc(rec.y & ((1u << (p & 31)) - 1u))));
            cc_link(par, i, j);
        }
        __builtin_amdgcn_wave_barrier();
    }
    // appends the lanes' occupied neighbours: bit 5q + c of mask is the site c of
    // row k0 + q of site s, entry i; links the buffer when it is full
    template <bool PER>
    __device__ __forceinline__ void push(uint32_t mask, const NzOffset *rows, int32_t k0, int32_t i, int32_t s, uint32_t A, int32_t L)
    {
        uint64_t mk;
        while ((mk = __ballot(mask != 0u)) != 0ull) {
            if (mask) {
                const int bit = __builtin_ctz(mask);
                mask &= mask - 1u;
                const int q = (bit * 13) >> 6, c = bit - 5 * q;   // bit / 5 for bit < 30
                const NzOffset o = rows[k0 + q];
                int32_t p = s + o.stride - 2 + c;
                if constexpr (PER) {
                    const uint32_t out = o.code & ~A & (kRowAxes | (1u << c));
                    if (out) p += wrap_fix(out, L);
                }
                const int32_t e = ne + static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(
                                           static_cast<uint32_t>(mk >> 32),
                                           __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mk), 0u)));
                st_w(&ei[e], i);
                st_w(&ep[e], p);
            }
            ne += static_cast<int32_t>(__popcll(mk));
            if (ne >= 64) {
                ne -= 64;   // the last 64; the rest stays for a later round
                link(ne, 64);
            }
        }
    }
};

// The sites ib + lane, ib + bx * blockDim + lane, .. of one wave.  EXACT: the map
// is the occupation; else a bit stands for 1 << ms sites, and a set one sends the
// check to the bitset.
template <bool PER, bool EXACT>
__device__ __forceinline__ void hook_map_sites(HookEdges &ed, const uint32_t *map, uint32_t ms, const NzOffset *rows, int32_t rh,
                                               const NzOffset *__restrict__ tab, const uint32_t *__restrict__ occ,
                                               const uint32_t *__restrict__ prefix, int32_t ib, int32_t step, int32_t n0, int32_t L,
                                               uint64_t magic, uint32_t words)
{
    for (; ib < n0; ib += step) {
        const int32_t i = ib + static_cast<int32_t>(ed.lane);
        const bool act = i < n0;
        const int32_t s = act ? static_cast<int32_t>(prefix[i]) : 0;
        const uint32_t pc = pack_coords(static_cast<uint32_t>(s), static_cast<uint32_t>(L), magic);
        const uint32_t A = act ? allowed_of(pc, L) : 0u;
        const int32_t x0 = static_cast<int32_t>(pc & 63);
        for (int32_t k0 = 0; k0 < rh; k0 += HOOK_UNROLL) {
            // side 1 (periodic only): the steps that leave along axis 0, on the
            // other side of the row
            for (int side = 0; side < (PER ? 2 : 1); ++side) {
                int32_t b[HOOK_UNROLL];   // the row's sites start here
                uint32_t want[HOOK_UNROLL], w0[HOOK_UNROLL], w1[HOOK_UNROLL];
#pragma unroll
                for (int q = 0; q < HOOK_UNROLL; ++q) {
                    NzOffset o;
                    o.stride = 0;
                    o.code = 0u;
                    if (k0 + q < rh) o = tab[k0 + q];   // (uniform: scalar registers)
                    const uint32_t out = o.code & ~A & kRowAxes;
                    if constexpr (PER) {
                        want[q] = act ? o.code & (side ? ~A : A) & 31u : 0u;
                        b[q] = want[q] ? s + o.stride - 2 + (out ? wrap_fix(out, L) : 0) + (side ? (x0 < 2 ? L : -L) : 0) : 0;
                    } else {
                        want[q] = out == 0u ? o.code & A & 31u : 0u;
                        b[q] = out == 0u ? s + o.stride - 2 : 0;
                    }
                    const int32_t w = (EXACT ? b[q] >> 5 : b[q] >> (ms + 5u)) + 1;
                    w0[q] = map[w];
                    w1[q] = map[w + 1];
                }
                uint32_t mask = 0u;   // of row q: bits 5q ..
                if constexpr (EXACT) {
#pragma unroll
                    for (int q = 0; q < HOOK_UNROLL; ++q)
                        mask |= (__builtin_amdgcn_alignbit(w1[q], w0[q], static_cast<uint32_t>(b[q]) & 31u) & want[q]) << (5 * q);
                } else {
#pragma unroll
                    for (int q = 0; q < HOOK_UNROLL; ++q) {
                        // the map bits of sites b .. b + 4 (at most three)
                        const int32_t k = b[q] >> ms, n = ((b[q] + 4) >> ms) - k;
                        const uint32_t any = __builtin_amdgcn_alignbit(w1[q], w0[q], static_cast<uint32_t>(k) & 31u) & ((2u << n) - 1u);
                        const bool need = any != 0u && want[q] != 0u;
                        const uint32_t first = static_cast<uint32_t>(max(b[q], 0)) >> 5;
                        const uint32_t last = static_cast<uint32_t>(max(b[q], 0) + 4) >> 5;
                        w0[q] = need ? occ[first] : 0u;
                        w1[q] = need && last != first && last < words ? occ[last] : 0u;
                    }
#pragma unroll
                    for (int q = 0; q < HOOK_UNROLL; ++q) {
                        const int32_t b0 = max(b[q], 0);
                        const uint32_t v = __builtin_amdgcn_alignbit(w1[q], w0[q], static_cast<uint32_t>(b0) & 31u) << (b0 - b[q]);
                        mask |= (v & want[q]) << (5 * q);
                    }
                }
                ed.push<PER>(mask, rows, k0, i, s, A, L);
            }
        }
    }
    ed.link(0, ed.ne);
}

// The hook of sparse lists: the workgroup holds a map of the occupation in LDS,
// as the block sweep does, and a row of offsets costs a dozen instructions and
// one two-word read of it.  The kernel above takes some 45 with its summary, its
// two conditional loads and its ballots, and is bound by them (at L = 16, zones
// 1-4, 88% of its cycles issue vector instructions).  bx workgroups per sample,
// blockDim sites of the list at a time.  The kernel above / this one, 1000 samples
// of L = 16: zones 1-3 0.80 / 0.60 ms, 1-4 0.64 / 0.43, 1-7 0.47 / 0.25; L = 24
// (200, eight sites to a bit, 2% of the bits set), zones 1-7 1.01 / 0.70.  With more
// bits set it loses: at L = 24 the reads behind them (zones 1-4, 6%, 1.08 / 1.15;
// zones 1-3, 10%, 1.23 / 1.49), at L = 16 the links, which want the waves that the
// map's LDS takes away (zones 1-2, 4%, 1.28 / 1.32; zone 1, 15%, 3.1 / 3.4); the
// line lies at one bit in 32.
template <bool PER>
__global__ __launch_bounds__(1024) void nz_hook_kernel_map(const NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                           int32_t nlist, int32_t bx, uint32_t map_words,
                                                           const NzOffset *__restrict__ tabs, uint8_t *__restrict__ ws,
                                                           NzState *__restrict__ state)
{
    extern __shared__ uint32_t hook_map[];
    __shared__ NzOffset rows[HOOK_ROWS];
    __shared__ int32_t ebuf_i[16][HOOK_EBUF];
    __shared__ int32_t ebuf_p[16][HOOK_EBUF];
    int32_t y, x;
    if (!xcd_slot(nlist, bx, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    const int32_t n0 = state[sid].n0;
    const int32_t t = static_cast<int32_t>(threadIdx.x), nt = static_cast<int32_t>(blockDim.x);
    if (n0 > d.prefix_cap || d.wrap || x * nt >= n0) return;   // (uniform over the workgroup)
    const int32_t L = d.L;
    const int32_t rh = d.rows >> 1;   // one row of every +- pair
    const uint32_t N = static_cast<uint32_t>(d.N);
    const uint32_t ms = map_shift(N, map_words);
    const int32_t mwords = static_cast<int32_t>((((N - 1u) >> ms) >> 5) + 1u + MAP_PAD);
    const uint32_t *occ = reinterpret_cast<const uint32_t *>(ws + d.off_occ);
    const uint32_t *prefix = reinterpret_cast<const uint32_t *>(ws + d.off_prefix);
    const NzOffset *tab = tabs + d.tab;
    for (int32_t w = t; w < mwords; w += nt) hook_map[w] = 0u;
    for (int32_t k = t; k < rh; k += nt) rows[k] = tab[k];
    __syncthreads();
    for (int32_t k = t; k < n0; k += nt) {
        const uint32_t b = prefix[k] >> ms;
        atomicOr(&hook_map[1 + (b >> 5)], 1u << (b & 31));
    }
    __syncthreads();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    HookEdges ed{reinterpret_cast<int32_t *>(ws + d.off_parc), reinterpret_cast<const uint2 *>(ws + d.off_wrec), ebuf_i[wave],
                 ebuf_p[wave], 0, lane_id()};
    const int32_t ib = x * nt + static_cast<int32_t>(wave) * 64;
    const uint32_t words = ((N + 63u) >> 6) << 1;
    if (ms == 0) hook_map_sites<PER, true>(ed, hook_map, 0u, rows, rh, tab, occ, prefix, ib, bx * nt, n0, L, d.magic, words);
    else hook_map_sites<PER, false>(ed, hook_map, ms, rows, rh, tab, occ, prefix, ib, bx * nt, n0, L, d.magic, words);
}

__device__ __forceinline__ uint32_t border_flags(uint32_t s, uint32_t L, uint64_t magic)
{
    const uint32_t x0 = s - div_by_L(s, magic) * L;
    return (x0 == 0 ? NZ_FLO : 0u) | (x0 == L - 1 ? NZ_FHI : 0u);
}

// Compress: every member points straight at its root's node, and every root
// takes its root word: its own border flags, and size 1 in largest-cluster runs.
// The other runs keep no sizes of prefilled clusters (size 0): the sweep counts
// the members of the one cluster whose mass is asked for.  Each thread writes only its
// own entry and walks the forest read-only: a halving write here could replace
// an entry another thread has already pointed at its root with a non-root
// ancestor.  Roots never change in this kernel, so a walk stops at an entry that
// points to itself or already holds a root word.
//
// What bounds it is the latency of the walks, so a thread has WALKS of them under
// way (1000 samples of L = 16, zone 1: one 0.91 ms, two 0.88, four 0.79, eight
// 0.83), and so in the flag pass below (0.77 without the read before the atomic; with it one
// at a time 0.66, four 0.57, eight 0.68).
constexpr int WALKS = 4;

__global__ __launch_bounds__(256) void nz_compress_kernel(const NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                          int32_t nlist, int32_t bx, uint8_t *__restrict__ ws,
                                                          NzState *__restrict__ state)
{
    int32_t y, x;
    if (!xcd_slot(nlist, bx, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    const int32_t n0 = state[sid].n0;
    if (n0 > d.prefix_cap || d.wrap) return;
    const uint32_t L = static_cast<uint32_t>(d.L);
    int32_t *par = reinterpret_cast<int32_t *>(ws + d.off_parc);
    const uint32_t *prefix = reinterpret_cast<const uint32_t *>(ws + d.off_prefix);
    const int32_t step = bx * 256;
    for (int32_t k0 = x * 256 + static_cast<int32_t>(threadIdx.x); k0 < n0; k0 += WALKS * step) {
        int32_t r[WALKS], p[WALKS];
#pragma unroll
        for (int q = 0; q < WALKS; ++q) {
            r[q] = min(k0 + q * step, n0 - 1);   // (past the end: the last entry, not stored)
            p[q] = ld_w(&par[r[q]]);
        }
        for (bool more = true; more;) {
            more = false;
#pragma unroll
            for (int q = 0; q < WALKS; ++q)
                if (p[q] >= 0 && (p[q] & (LIST_NODE - 1)) != r[q]) {
                    r[q] = p[q] & (LIST_NODE - 1);   // (an entry already pointed at its root is a node id)
                    p[q] = ld_w(&par[r[q]]);
                    more = true;
                }
        }
#pragma unroll
        for (int q = 0; q < WALKS; ++q) {
            const int32_t k = k0 + q * step;
            if (k >= n0) continue;
            if (r[q] == k) {
                const uint32_t fl = d.periodic ? 0u : border_flags(prefix[k], L, d.magic);
                st_w(&par[k], static_cast<int32_t>(NZ_ROOT | fl | (d.smax_mode ? 1u : 0u)));
                if (fl == NZ_FLAGS) state[sid].status = NZ_ST_BACKOFF;   // L = 1: one site spans
            } else {
                st_w(&par[k], LIST_NODE | r[q]);
            }
        }
    }
}

// Border flags of the prefilled clusters (and their sizes in largest-cluster
// runs): a site on a border adds its flag to its root's word in the list forest.
// The flag OR returns the previous word, so the site that completes a root's
// pair of flags sees it: the state already spans and the sample backs off (not
// in largest-cluster runs, which stop below the window instead).
//
// A size for every cluster would take an atomic per member, and lattice entries
// a scattered 4-byte write per site: for 1000 samples of L = 16, zone 1 this
// pass took 3.9 ms with both, 2.1 with the lattice entries alone, and takes 0.57
// with the flags alone.  The sweep finds a prefilled site's list entry from its
// bitset word instead, and counts the members of the spanning cluster.
__global__ __launch_bounds__(256) void nz_accum_kernel(const NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                       int32_t nlist, int32_t bx, uint8_t *__restrict__ ws,
                                                       NzState *__restrict__ state)
{
    int32_t y, x;
    if (!xcd_slot(nlist, bx, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    if (d.wrap) return;
    const int32_t n0 = state[sid].n0;
    if (n0 > d.prefix_cap) {
        if (x == 0 && threadIdx.x == 0) state[sid].status = NZ_ST_PREFIX;
        return;
    }
    const bool sizes = d.smax_mode != 0;
    if (d.periodic && !sizes) return;   // nothing to add (uniform)
    const uint32_t L = static_cast<uint32_t>(d.L);
    int32_t *parc = reinterpret_cast<int32_t *>(ws + d.off_parc);
    const uint32_t *prefix = reinterpret_cast<const uint32_t *>(ws + d.off_prefix);
    bool spans = false;
    const int32_t step = bx * 256;
    for (int32_t k0 = x * 256 + static_cast<int32_t>(threadIdx.x); k0 < n0; k0 += WALKS * step) {
        uint32_t fl[WALKS], had[WALKS];
        int32_t r[WALKS];   // (< 0: nothing to add, or a root, whose word holds its own flags and size)
#pragma unroll
        for (int q = 0; q < WALKS; ++q) {
            const int32_t k = min(k0 + q * step, n0 - 1);
            fl[q] = d.periodic ? 0u : border_flags(prefix[k], L, d.magic);
        }
#pragma unroll
        for (int q = 0; q < WALKS; ++q) r[q] = k0 + q * step < n0 && (fl[q] || sizes) ? parc[k0 + q * step] : -1;
        // (most roots have the flag already: a read costs less than an atomic, and a
        // stale one only costs the atomic)
#pragma unroll
        for (int q = 0; q < WALKS; ++q)
            had[q] = r[q] >= 0 && fl[q] ? static_cast<uint32_t>(ld_w(&parc[r[q] & (LIST_NODE - 1)])) : 0u;
#pragma unroll
        for (int q = 0; q < WALKS; ++q) {
            if (r[q] < 0) continue;
            uint32_t *root = reinterpret_cast<uint32_t *>(&parc[r[q] & (LIST_NODE - 1)]);
            if (sizes) atomicAdd(root, 1u);
            if (fl[q] & ~had[q]) {
                const uint32_t old = atomicOr(root, fl[q]);
                spans = spans || ((old | fl[q]) & NZ_FLAGS) == NZ_FLAGS;
            }
        }
    }
    if (spans && !sizes) state[sid].status = NZ_ST_BACKOFF;
}

// Largest cluster of the prefilled state (smax mode): every root word offers
// its size.
__global__ __launch_bounds__(256) void nz_rootmax_kernel(const NzSample *__restrict__ desc,
                                                         const int32_t *__restrict__ list, int32_t nlist, int32_t bx,
                                                         uint8_t *__restrict__ ws, NzState *__restrict__ state)
{
    int32_t y, x;
    if (!xcd_slot(nlist, bx, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    if (!d.smax_mode) return;
    const int32_t n0 = state[sid].n0;
    if (n0 > d.prefix_cap) return;
    const int32_t *par = reinterpret_cast<const int32_t *>(ws + d.off_parc);
    int32_t best = 0;
    for (int32_t k = x * 256 + static_cast<int32_t>(threadIdx.x); k < n0; k += bx * 256) {
        const int32_t v = par[k];
        if (v < 0) best = max(best, static_cast<int32_t>(static_cast<uint32_t>(v) & NZ_SIZE));
    }
    if (best > 0) atomicMax(&state[sid].smax, best);
}

// Largest-cluster samples with lists of up to SIZES_RANGES ranges: the sizes of
// the clusters whose roots lie in one range of the list, counted in LDS by one
// workgroup, and their maximum.  `lds_range`: entries of a range.  In place of one
// atomic per site in the L2 (29 G a second over the chip) a workgroup reads its
// sample's list once per range: 1000 samples of L = 12, zone 1, 29000 prefilled
// sites each took 0.88 ms, and 0.11 for the maximum, and take 0.10 together.
constexpr int32_t SIZES_RANGE = 36864, SIZES_RANGES = 8;
extern __shared__ uint32_t sizes_lds[];

__global__ __launch_bounds__(1024) void nz_sizes_kernel(const NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                        int32_t nlist, int32_t ranges, int32_t lds_range,
                                                        uint8_t *__restrict__ ws, NzState *__restrict__ state)
{
    int32_t y, x;
    if (!xcd_slot(nlist, ranges, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    const int32_t n0 = state[sid].n0;
    const int32_t t = static_cast<int32_t>(threadIdx.x), step = static_cast<int32_t>(blockDim.x);
    if (n0 > d.prefix_cap) {
        if (x == 0 && t == 0) state[sid].status = NZ_ST_PREFIX;
        return;
    }
    const int32_t base = x * lds_range, cnt = min(lds_range, n0 - base);
    if (cnt <= 0) return;   // (uniform)
    int32_t *parc = reinterpret_cast<int32_t *>(ws + d.off_parc);
    for (int32_t j = t; j < cnt; j += step) sizes_lds[j] = 0u;
    __syncthreads();
    for (int32_t k = t; k < n0; k += step) {
        const int32_t v = parc[k];
        const int32_t j = (v & (LIST_NODE - 1)) - base;
        if (v >= 0 && j >= 0 && j < cnt) atomicAdd(&sizes_lds[j], 1u);
    }
    __syncthreads();
    int32_t best = 0;
    for (int32_t j = t; j < cnt; j += step) {
        const int32_t v = parc[base + j];
        if (v >= 0) continue;
        const uint32_t w = static_cast<uint32_t>(v) + sizes_lds[j];   // (a root's word holds its own 1)
        if (sizes_lds[j]) parc[base + j] = static_cast<int32_t>(w);
        best = max(best, static_cast<int32_t>(w & NZ_SIZE));
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) best = max(best, __shfl_xor(best, o));
    if ((t & 63) == 0 && best > 0) atomicMax(&state[sid].smax, best);
}

// Sum over the finished samples of a chunk of their S_max(n) windows (all
// samples of an smax-mode batch share one window of w entries).  A workgroup
// takes 256 entries of every gridDim.y-th sample: with all the samples of an entry
// in one thread, the 15 workgroups of a window of 3800 entries took 0.61 ms for
// 1000 samples, with the samples spread over the chip 0.01 ms.
__global__ __launch_bounds__(256) void nz_winsum_kernel(const NzSample *__restrict__ desc,
                                                        const NzState *__restrict__ state, int32_t nsamp, int32_t w,
                                                        const uint8_t *__restrict__ ws, uint64_t *__restrict__ out)
{
    for (int32_t i = blockIdx.x * 256 + static_cast<int32_t>(threadIdx.x); i < w; i += gridDim.x * 256) {
        uint64_t sum = 0;
        for (int32_t k = static_cast<int32_t>(blockIdx.y); k < nsamp; k += static_cast<int32_t>(gridDim.y)) {
            if (state[k].status != NZ_ST_DONE) continue;
            sum += reinterpret_cast<const uint32_t *>(ws + desc[k].off_win)[i];
        }
        if (sum) atomicAdd(reinterpret_cast<unsigned long long *>(&out[i]), static_cast<unsigned long long>(sum));
    }
}

// ---------------------------------------------------------------------------
// Periodic boundaries: n* is the first addition after which a cluster wraps
// around axis 0 (Newman & Ziff 2001, Sec. III).
//
// Every site's entry is one 64-bit word: the low half is the parent word of the
// free-boundary sweep (a parent index, or a root word), the high half the x0
// displacement of the site from its parent in the unwrapped lattice (0 at a
// root).  A site's displacement from its root is the sum along its path.  Every
// write stores an (ancestor, displacement to it) pair in one 64-bit store, so
// any entry a lane or thread reads, however stale, is consistent.  An edge
// t = s + d inside one cluster closes a loop, and the loop winds around axis 0
// exactly when the displacements of s and t from their common root differ by
// anything but d0; the cluster then wraps and takes both border flags, the
// state the spanning test looks for.

__device__ __forceinline__ uint64_t wword(uint32_t par, int32_t dx)
{
    return (static_cast<uint64_t>(static_cast<uint32_t>(dx)) << 32) | par;
}
__device__ __forceinline__ int32_t wpar(uint64_t e) { return static_cast<int32_t>(static_cast<uint32_t>(e)); }
__device__ __forceinline__ int32_t wdx(uint64_t e) { return static_cast<int32_t>(e >> 32); }

// Prefill phase: a root points to itself with displacement 0.  Root of x and
// the displacement of x from it; path splitting (each entry on the way skips to
// its grandparent, displacements added).
__device__ __forceinline__ int32_t ccw_find(uint64_t *pw, int32_t x, int32_t &disp)
{
    uint64_t e = ld_w(&pw[x]);
    int32_t D = 0;
    while (wpar(e) != x) {
        const int32_t p = wpar(e);
        const uint64_t g = ld_w(&pw[p]);
        if (wpar(g) != p) st_w(&pw[x], wword(static_cast<uint32_t>(wpar(g)), wdx(e) + wdx(g)));
        D += wdx(e);
        x = p;
        e = g;
    }
    disp = D;
    return x;
}

// Hook with displacements: as the free-boundary hook (CAS links the larger root
// below the smaller), the hooked root taking its displacement from the smaller
// one through the edge.  An edge whose ends already share a root is checked
// instead; a winding loop means the prefilled state already wraps, and the
// sample backs off.
__global__ __launch_bounds__(256) void nz_hookw_kernel(const NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                       int32_t nlist, int32_t bx, const NzOffset *__restrict__ tabs,
                                                       uint8_t *__restrict__ ws, NzState *__restrict__ state)
{
    int32_t y, x;
    if (!xcd_slot(nlist, bx, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    const int32_t n0 = state[sid].n0;
    if (n0 > d.prefix_cap || !d.wrap) return;
    const int32_t L = d.L;
    const int32_t rh = d.rows >> 1;   // one row of every +- pair
    const uint64_t magic = d.magic;
    uint64_t *pw = reinterpret_cast<uint64_t *>(ws + d.off_par);
    const uint32_t *occ = reinterpret_cast<const uint32_t *>(ws + d.off_occ);
    const uint32_t *prefix = reinterpret_cast<const uint32_t *>(ws + d.off_prefix);
    const NzOffset *tab = tabs + d.tab;
    bool wraps = false;
    for (int32_t i = x * 256 + static_cast<int32_t>(threadIdx.x); i < n0; i += bx * 256) {
        const int32_t s = static_cast<int32_t>(prefix[i]);
        const uint32_t pc = pack_coords(static_cast<uint32_t>(s), static_cast<uint32_t>(L), magic);
        const uint32_t A = allowed_axis(pc & 63, L) | (allowed_axis((pc >> 6) & 63, L) << 5) |
                           (allowed_axis((pc >> 12) & 63, L) << 10) | (allowed_axis((pc >> 18) & 63, L) << 15) |
                           (allowed_axis(pc >> 24, L) << 20);
        int32_t u = -1, Du = 0;   // a root (or ancestor) of s and the displacement of s from it
        const int32_t x0 = static_cast<int32_t>(pc & 63);
        for (int32_t k0 = 0; k0 < 2 * rh; k0 += HOOKW_UNROLL) {
            // entry k: row k / 2; odd entries are the steps that leave along axis
            // 0, on the other side of the row
            int32_t b[HOOKW_UNROLL];
            uint32_t v[HOOKW_UNROLL];
#pragma unroll
            for (int q = 0; q < HOOKW_UNROLL; ++q) {
                NzOffset o;
                o.stride = 0;
                o.code = 0u;
                if (k0 + q < 2 * rh) o = tab[(k0 + q) >> 1];
                const int side = q & 1;
                const uint32_t out = o.code & ~A & kRowAxes;
                b[q] = s + o.stride - 2 + (out ? wrap_fix(out, L) : 0);
                if (side) b[q] += x0 < 2 ? L : -L;
                const uint32_t dm = o.code & (side ? ~A : A) & 31u;
                const int32_t c = __builtin_ctz(dm | 32u);
                const uint32_t p0 = static_cast<uint32_t>(b[q] + c), p1 = static_cast<uint32_t>(b[q] + 31 - __builtin_clz(dm | 1u));
                const uint32_t w0 = dm ? occ[p0 >> 5] : 0u;
                const uint32_t w1 = dm && (p1 >> 5) != (p0 >> 5) ? occ[p1 >> 5] : 0u;
                v[q] = (__builtin_amdgcn_alignbit(w1, w0, p0 & 31u) << c) & dm;
            }
#pragma unroll
            for (int q = 0; q < HOOKW_UNROLL; ++q) {
              while (v[q]) {
                const int j = __builtin_ctz(v[q]);
                v[q] &= v[q] - 1u;
                const int32_t tn = b[q] + j, d0 = j - 2;
                if (u < 0) u = ccw_find(pw, s, Du);
                int32_t Dv;
                int32_t vr = ccw_find(pw, tn, Dv);
                for (;;) {
                    if (u == vr) {
                        if (Du + d0 != Dv) wraps = true;
                        break;
                    }
                    const int32_t hi = max(u, vr), lo = min(u, vr);
                    // x0(u) = x0(s) - Du and x0(vr) = x0(s) + d0 - Dv
                    const int32_t dx = hi == u ? Dv - Du - d0 : Du + d0 - Dv;
                    uint64_t expected = wword(static_cast<uint32_t>(hi), 0);
                    if (__hip_atomic_compare_exchange_strong(&pw[hi], &expected, wword(static_cast<uint32_t>(lo), dx),
                                                             __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                        if (hi == u) {
                            u = lo;
                            Du += dx;
                        }
                        break;
                    }
                    // hi is no longer a root: go on from the entry the CAS returned
                    int32_t Dp;
                    if (u == hi) {
                        u = ccw_find(pw, wpar(expected), Dp);
                        Du += wdx(expected) + Dp;
                    } else {
                        u = ccw_find(pw, u, Dp);
                        Du += Dp;
                    }
                    if (vr == hi) {
                        vr = ccw_find(pw, wpar(expected), Dp);
                        Dv += wdx(expected) + Dp;
                    } else {
                        vr = ccw_find(pw, vr, Dp);
                        Dv += Dp;
                    }
                }
              }
            }
        }
    }
    if (wraps) state[sid].status = NZ_ST_BACKOFF;
}

// Compress with displacements: every member holds (root, displacement from the
// root), every root its root word (size 1, no border flags).  Walks are
// read-only and each thread writes only its own entry, as in the
// free-boundary compress.
__global__ __launch_bounds__(256) void nz_compressw_kernel(const NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                           int32_t nlist, int32_t bx, uint8_t *__restrict__ ws,
                                                           NzState *__restrict__ state)
{
    int32_t y, x;
    if (!xcd_slot(nlist, bx, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    const int32_t n0 = state[sid].n0;
    if (n0 > d.prefix_cap || !d.wrap) return;
    uint64_t *pw = reinterpret_cast<uint64_t *>(ws + d.off_par);
    const uint32_t *prefix = reinterpret_cast<const uint32_t *>(ws + d.off_prefix);
    for (int32_t k = x * 256 + static_cast<int32_t>(threadIdx.x); k < n0; k += bx * 256) {
        const int32_t s = static_cast<int32_t>(prefix[k]);
        int32_t r = s, D = 0;
        uint64_t e = ld_w(&pw[r]);
        while (wpar(e) >= 0 && wpar(e) != r) {
            D += wdx(e);
            r = wpar(e);
            e = ld_w(&pw[r]);
        }
        st_w(&pw[s], r == s ? wword(NZ_ROOT | 1u, 0) : wword(static_cast<uint32_t>(r), D));
    }
}

// Sizes of the prefilled clusters: members add themselves to the low half of
// their root's entry.
__global__ __launch_bounds__(256) void nz_accumw_kernel(const NzSample *__restrict__ desc, const int32_t *__restrict__ list,
                                                        int32_t nlist, int32_t bx, uint8_t *__restrict__ ws,
                                                        NzState *__restrict__ state)
{
    int32_t y, x;
    if (!xcd_slot(nlist, bx, y, x)) return;
    const int sid = list[y];
    const NzSample &d = desc[sid];
    if (!d.wrap) return;
    const int32_t n0 = state[sid].n0;
    if (n0 > d.prefix_cap) {
        if (x == 0 && threadIdx.x == 0) state[sid].status = NZ_ST_PREFIX;
        return;
    }
    uint64_t *pw = reinterpret_cast<uint64_t *>(ws + d.off_par);
    const uint32_t *prefix = reinterpret_cast<const uint32_t *>(ws + d.off_prefix);
    for (int32_t k = x * 256 + static_cast<int32_t>(threadIdx.x); k < n0; k += bx * 256) {
        const int32_t s = static_cast<int32_t>(prefix[k]);
        const int32_t r = wpar(pw[s]);
        if (r >= 0) atomicAdd(reinterpret_cast<uint32_t *>(&pw[r]), 1u);   // low half: the root word
    }
}

// ---------------------------------------------------------------------------
// The block sweep: one workgroup per sample, up to B sites of the order at a
// time.
//
// A block is whole buckets of the key band (buckets are in key order, their
// entries are not), so nothing is sorted on the way.  Its sites are marked
// occupied, every (site, row of offsets) pair is checked by some lane, and the
// unions run as a connected-components pass in LDS over a graph whose nodes are
// the block's sites and the earlier clusters they touch.  Spanning (or
// wrapping) is monotone in the occupation: clusters only grow and flags only
// accumulate, so when no cluster spans after all the sites of the block none
// spanned after any of them, and the block is committed as a whole.  In the
// block in which a cluster spans, the smallest T such that the block's first T
// sites in (key, site) order span is found on that small graph,
// without touching memory again: n* is the count before the block plus T, the
// mass the size of the cluster of the T-th site.  A block that does not fit
// the tables is undone, sorted, and added in halves (one site has at most 892
// neighbours and always fits).
//
// What bounds it: the latency of a block's chain of dependent accesses (parent
// words and root words of the occupied neighbours, some eight barriers) and,
// for wide neighbourhoods, the checks themselves.  The checks therefore read a
// map of the occupation held in LDS (below), one row of up to five offsets at
// a time, and blocks are as large as the tables allow beside the map.  Measured
// (L = 16, zone 1 x 1000, prefilled): a block of up to 512 sites takes 16 us --
// marks 0.7, checks 1.9, parents and roots 9.8, unions 1.4, sizes and flags 0.9,
// write-back 0.9 -- against 24 us for 64 sites by one wave in the sweep this one
// replaced; ranks 7 and the smallest T 8 us once per sample.  With separate tables
// for a block's sites (marked in memory) and for the earlier roots the kernel
// took 2.39 ms for this batch and takes 2.13, at L = 24 6.59 and 5.29.  37
// samples of L = 13, z = 380 took 1.56 ms and take 0.11 ms, the periodic L = 12
// batch of 700 samples 26 ms and 0.5 ms.
//
// A block's sites have no entry in memory before it is committed: neighbours
// among them are found in the node table.

enum { BLK_SPAN = 0, BLK_WRAP = 1, BLK_SMAX = 2 };

struct SweepOut {
    int32_t *nstar;
    int32_t *mass;
    const int32_t *out_index; // per sample: position in the caller's output arrays
};

constexpr int BLK_EDGES = 1536;          // recorded (site, occupied neighbour) pairs per block
constexpr int BLK_CHUNK = 6;             // rows checked together (five bits each: one 32-bit mask)
constexpr int BLK_MAXROWS = 300;         // rows of the widest neighbourhood (298), in whole chunks
constexpr int BLK_CURVES = 4;            // clusters of a block that may raise the maximum at once
constexpr uint32_t BLK_EMPTY = 0xFFFFFFFFu;
constexpr int32_t NZ_NONE = static_cast<int32_t>(0x80000000u);   // (a root word of no cluster)
// Node ids: band sites, BAND_NODE | k; list nodes, LIST_NODE | index (both below
// 2^29; a block's own sites go by their lattice index until it is known to
// fit).  Entries with both bits are list nodes that the sweep wrote.
constexpr int32_t BAND_NODE = 0x40000000, BLK_LINKED = 0x40000000;
__device__ __forceinline__ int32_t node_id(int32_t v) { return (v & LIST_NODE) ? v & ~BLK_LINKED : v; }
constexpr uint32_t BLK_SMALL_MAP = 4096;  // words of the largest map that leaves room for several workgroups per CU
static_assert(BLK_MAXROWS % BLK_CHUNK == 0, "whole chunks");
static_assert(BLK_EDGES >= 892, "a block of one site always fits");

__device__ __forceinline__ int32_t site_of(uint32_t pc, int32_t L)
{
    return static_cast<int32_t>(pc & 63) +
           L * (static_cast<int32_t>((pc >> 6) & 63) +
                L * (static_cast<int32_t>((pc >> 12) & 63) +
                     L * (static_cast<int32_t>((pc >> 18) & 63) + L * static_cast<int32_t>(pc >> 24))));
}

// Accesses shared by the waves of one workgroup.
template <typename T>
__device__ __forceinline__ T ld_g(T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
template <typename T>
__device__ __forceinline__ void st_g(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

// Node words of the LDS forest: a root word (bit 31: cluster size and border
// flags before the block's unions) or the parent node, and for the wrap sweep
// the x0 displacement from it in the high half (one 64-bit word, so that every
// read is a consistent pair).
template <bool WRAP>
struct BlkWord {
    using type = uint32_t;
    static __device__ __forceinline__ uint32_t make(uint32_t lo, int32_t) { return lo; }
    static __device__ __forceinline__ uint32_t lo(uint32_t e) { return e; }
    static __device__ __forceinline__ int32_t dx(uint32_t) { return 0; }
};
template <>
struct BlkWord<true> {
    using type = uint64_t;
    static __device__ __forceinline__ uint64_t make(uint32_t lo, int32_t d)
    {
        return (static_cast<uint64_t>(static_cast<uint32_t>(d)) << 32) | lo;
    }
    static __device__ __forceinline__ uint32_t lo(uint64_t e) { return static_cast<uint32_t>(e); }
    static __device__ __forceinline__ int32_t dx(uint64_t e) { return static_cast<int32_t>(e >> 32); }
};

// One workgroup of NT threads, blocks of up to B sites.  The block's nodes -- its
// sites and the earlier roots it touches -- are slots of one open-addressing
// table keyed by node id, so a neighbour that belongs to the block, or is itself
// an earlier root already there, is found without leaving LDS.
template <int MODE_, bool PER_, int NT_, int B_>
struct BlkCfg {
    static constexpr int MODE = MODE_, NT = NT_, B = B_;
    static constexpr bool PER = PER_;
    // slots: a full block, the roots of one site's 892 neighbours
    static constexpr uint32_t RS = B > 256 ? 2048 : 1024;
    static constexpr uint32_t SHIFT = B > 256 ? 21 : 22;
    // the ranks and times within a block go where the map was, if that is large enough
    // (wrapping: where the node ids were, which a block that wraps needs no more)
    static constexpr bool OWN_SCRATCH = NT == 256 && MODE != 1;
    static constexpr bool ID_SCRATCH = NT == 256 && MODE == 1;
    // words: keys of the sites, 16-bit ranks of the slots, spanning: joining times of
    // the slots; largest cluster: these alone
    static constexpr uint32_t SCRATCH = MODE == 2 ? RS : B + RS / 2 + (MODE == 0 ? RS : 0);
    static_assert(B <= NT, "thread t loads entry t of a block");
    static_assert(RS % NT == 0 && RS >= B + 512 && RS >= 893 && RS <= 2048, "whole slots per thread; node numbers of 11 bits");
    static_assert(MODE != BLK_WRAP || PER, "wrapping needs periodic coordinates");
    static_assert(!ID_SCRATCH || SCRATCH <= RS, "the ids' space is large enough");
    static_assert(MODE != BLK_SMAX || OWN_SCRATCH, "the map stays in use");
};

template <typename C>
struct BlkLds {
    using W = BlkWord<C::MODE == BLK_WRAP>;
    typename W::type f[C::RS];         // the forest
    uint32_t rkey[C::RS];              // node ids (BLK_EMPTY: free)
    uint32_t et[BLK_EDGES];            // pair e: block position, row and step; then the two nodes, 16 bits each
    uint32_t pcs[C::B];                // packed coordinates of the block's sites
    NzOffset rows[BLK_MAXROWS];        // the sample's rows, padded with empty ones to whole chunks
    uint16_t spos[C::B];               // the sites' nodes
    // x0(first node) - x0(second node) of pair e: up to two steps for every site of the
    // lattice, since a cluster that does not wrap around axis 0 may wind around the others
    int32_t eq[C::MODE == BLK_WRAP ? BLK_EDGES : 1];
    uint32_t scratch[C::OWN_SCRATCH ? C::SCRATCH : 1];
    // largest-cluster sweep: the block position of every node (0xFFFF: an earlier
    // root), the clusters that can raise the maximum (`next`: which of them a root
    // is), their largest members and their growth at every position; one by one:
    // the pairs of every position as a linked list, and the running maximum after
    // every position
    uint16_t pos[C::MODE == BLK_SMAX ? C::RS : 1];
    uint16_t next[C::MODE == BLK_SMAX ? BLK_EDGES : 1];
    uint32_t first[C::MODE == BLK_SMAX ? C::B : 1];
    uint32_t smax[C::MODE == BLK_SMAX ? BLK_CURVES * C::B : 1];
    uint64_t member[C::MODE == BLK_SMAX ? BLK_CURVES : 1];   // size before the block << 32 | node
    uint32_t ends[C::MODE == BLK_SMAX ? BLK_CURVES : 1];
    uint32_t wsum[C::MODE == BLK_SMAX ? BLK_CURVES * (C::NT / 64) : 1];
    int32_t nbig;
    int32_t ecnt, nroots, flag, bad, claim;
    uint32_t total;                    // spanning: the size of the cluster of the T-th site
    uint32_t croot;                    //           and its root node
};

template <typename C>
__device__ __forceinline__ uint32_t blk_hash(uint32_t id) { return (id * 0x9E3779B1u) >> C::SHIFT; }

// The node of id, entered if it is not there yet (fresh); C::RS if the table is
// full.
template <typename C>
__device__ __forceinline__ uint32_t blk_enter(BlkLds<C> &S, uint32_t id, bool &fresh)
{
    uint32_t h = blk_hash<C>(id);
    fresh = false;
    for (uint32_t k = 0; k < C::RS; ++k) {
        uint32_t expected = BLK_EMPTY;
        if (__hip_atomic_compare_exchange_strong(&S.rkey[h], &expected, id, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP)) {
            fresh = true;
            return h;
        }
        if (expected == id) return h;
        h = (h + 1) & (C::RS - 1);
    }
    return C::RS;
}

// The node of id, C::RS if it is not (yet) there.
template <typename C>
__device__ __forceinline__ uint32_t blk_lookup(BlkLds<C> &S, uint32_t id)
{
    uint32_t h = blk_hash<C>(id);
    for (uint32_t k = 0; k < C::RS; ++k) {
        const uint32_t key = ld_g(&S.rkey[h]);
        if (key == id) return h;
        if (key == BLK_EMPTY) break;
        h = (h + 1) & (C::RS - 1);
    }
    return C::RS;
}

// Root of node x in the LDS forest with path halving, its root word, and the
// displacement D of x from it.  Only non-roots are rewritten (to an ancestor)
// and links only change roots, so concurrent finds and links keep the forest
// acyclic.
template <typename C>
__device__ __forceinline__ uint32_t blk_find(BlkLds<C> &S, uint32_t x, uint32_t &word, int32_t &D)
{
    using W = typename BlkLds<C>::W;
    D = 0;
    auto e = ld_g(&S.f[x]);
    while (!(W::lo(e) & NZ_ROOT)) {
        const uint32_t p = W::lo(e);
        const auto g = ld_g(&S.f[p]);
        if (W::lo(g) & NZ_ROOT) {
            D += W::dx(e);
            x = p;
            e = g;
            break;
        }
        const auto h = W::make(W::lo(g), W::dx(e) + W::dx(g));
        st_g(&S.f[x], h);
        D += W::dx(h);
        x = W::lo(g);
        e = ld_g(&S.f[x]);
    }
    word = W::lo(e);
    return x;
}

// The lattice side of one sample: occupancy bits, their map in LDS and the
// union-find entries.  Wrap sweep: 64-bit parent / root words with displacements,
// one per lattice site.  Else nodes are those of the labelling's list forest
// (LIST_NODE | i) and of the band sites (BAND_NODE | k).  A plain sample's band
// nodes are its lattice entries, k the site.  A prefilled sample's are a dense
// array, k the position in the band's order, with a node only for the sites that
// were roots when their block was committed; a lattice entry then names a node.
// The array lies where the band's buckets were: position k is at most the slot of
// its own entry, and the slots of a block have been read before it is committed.
// So of the reads that follow one another from a neighbour to its root only the
// first goes to the lattice array (32 samples of 4 MB per XCD at L = 16): the
// batches of 7 compact neighbourhoods take 20.3 ms instead of 20.9 at L = 16 and
// 33.0 instead of 34.2 at L = 24.  A plain sample starts from single sites, whose
// lattice entry is their root word itself: there the dense array costs a read more
// than it saves (zone 1, L = 16, 1000 samples: 17.5 ms against 16.6).
// An entry written by the sweep carries BLK_LINKED, which tells former roots
// (and members whose path was cut short) from the members that still point at
// their root of the labelling.
//
// The map: bit k of the map (k counted from word 1; words 0 and the last two
// are zero) is clear only if sites k << mshift .. are all empty.  Up to L = 16
// mshift is 0: the map is the occupation itself and nothing else is read.
// Larger lattices take the smallest mshift that fits, and a set bit sends the
// check to the bitset in memory.
template <int MODE>
struct BlkMem {
    uint32_t *occ;
    int32_t *par;
    int32_t *parc;
    int32_t *band;
    bool flat;                // the band nodes are the lattice entries
    uint64_t *pw;
    const uint2 *wrec;        // per bitset word: list position of its first prefilled site, prefilled bits
    int32_t n0;               // prefilled sites
    uint32_t *map;      // LDS
    uint32_t mshift;
    uint32_t occ_words;

    __device__ __forceinline__ void occ_set(uint32_t s) const
    {
        const uint32_t k = s >> mshift;
        __hip_atomic_fetch_or(&map[1 + (k >> 5)], 1u << (k & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (mshift)
            __hip_atomic_fetch_or(&occ[s >> 5], 1u << (s & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // (map bits that stand for several sites stay set: that only costs a load)
    __device__ __forceinline__ void occ_clear(uint32_t s) const
    {
        if (mshift)
            __hip_atomic_fetch_and(&occ[s >> 5], ~(1u << (s & 31)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            __hip_atomic_fetch_and(&map[1 + (s >> 5)], ~(1u << (s & 31)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ int32_t *entry(int32_t id) const
    {
        return &((id & LIST_NODE) ? parc : band)[id & (LIST_NODE - 1)];
    }
    // Root, root word and displacement from the root of an occupied site t that
    // is no site of the block.  What the sweep waits for here is the fabric: every
    // 4-byte read moves a line, and a CU gets some 300 lines a microsecond, so
    // only what is needed is read (a prefilled site has no lattice entry).  Paths
    // are split: every entry on the way skips to its grandparent.
    __device__ __forceinline__ void resolve(int32_t t, int32_t &root, uint32_t &word, int32_t &disp) const
    {
        disp = 0;
        if constexpr (MODE == BLK_WRAP) {
            int32_t x = t;
            uint64_t e = ld_g(&pw[t]);
            while (wpar(e) >= 0) {
                const int32_t p = wpar(e);
                const uint64_t g = ld_g(&pw[p]);
                if (wpar(g) < 0) {
                    disp += wdx(e);
                    x = p;
                    e = g;
                    break;
                }
                const uint64_t h = wword(static_cast<uint32_t>(wpar(g)), wdx(e) + wdx(g));
                st_g(&pw[x], h);
                disp += wdx(h);
                x = wpar(g);
                e = ld_g(&pw[x]);
            }
            root = x;
            word = static_cast<uint32_t>(wpar(e));
        } else {
            int32_t x = BAND_NODE | t;   // (a root only if flat)
            int32_t *at = &par[t];
            if (n0 > 0) {
                const uint2 rec = wrec[static_cast<uint32_t>(t) >> 5];
                const uint32_t bit = static_cast<uint32_t>(t) & 31u;
                if ((rec.y >> bit) & 1u) {
                    x = LIST_NODE | static_cast<int32_t>(rec.x + static_cast<uint32_t>(__popc(rec.y & ((1u << bit) - 1u))));
                    at = entry(x);
                }
            }
            int32_t v = ld_g(at);
            while (v >= 0) {
                x = node_id(v);
                int32_t *up = entry(x);
                const int32_t g = ld_g(up);
                if (g >= 0) st_g(at, g | BLK_LINKED);
                at = up;
                v = g;
            }
            root = x;
            word = static_cast<uint32_t>(v);
        }
    }
    // node's final entry: a root word, or (parent, displacement)
    __device__ __forceinline__ void commit(int32_t node, bool is_root, uint32_t word, int32_t parent, int32_t disp) const
    {
        if constexpr (MODE == BLK_WRAP) st_g(&pw[node], is_root ? wword(word, 0) : wword(static_cast<uint32_t>(parent), disp));
        else st_g(entry(node), is_root ? static_cast<int32_t>(word) : parent | BLK_LINKED);
    }
};

// Records the occupied neighbours of the block's sites as pairs.  Items of 64
// sites x BLK_CHUNK rows are dealt to the waves; a row (read from LDS, the same
// for all lanes) costs a lane about a dozen instructions and one two-word read
// of the map; 3.4 offsets of the widest neighbourhood share a row.
// EXACT: the map is the occupation (mshift == 0); else a set map bit sends the
// check to the bitset.  The reads of an item's rows are issued together.
// More pairs than the list holds end the scan: a block of a small dense lattice
// has ten times as many, and finding them all is most of its time (12000 samples
// of L = 3, zones 1-7: 2.41 ms to the end, 0.78 so; L = 5 periodic 4.17, 2.03).
template <bool EXACT, typename C>
__device__ __forceinline__ void blk_scan(BlkLds<C> &S, const BlkMem<C::MODE> &m, int nrows, int32_t L, int lo, int len)
{
    constexpr bool PER = C::PER;
    constexpr int NW = C::NT / 64;
    const uint32_t lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int groups = (len + 63) >> 6, chunks = (nrows + BLK_CHUNK - 1) / BLK_CHUNK;
    int g = wave, c = 0, have = -1;
    while (g >= groups) {
        g -= groups;
        ++c;
    }
    int32_t s = 0, x0 = 0;
    uint32_t A = 0;
    int i = 0;
    bool in = false;
    while (c < chunks) {
        if (g != have) {
            have = g;
            i = g * 64 + static_cast<int>(lane);
            in = i < len;
            const uint32_t pc = in ? S.pcs[lo + i] : 0u;
            x0 = static_cast<int32_t>(pc & 63);
            s = site_of(pc, L);
            A = in ? allowed_of(pc, L) : 0u;
        }
        // side 1 (periodic only): the steps that leave along axis 0, on the
        // other side of the row
        for (int side = 0; side < (PER ? 2 : 1); ++side) {
            const int32_t off0 = (PER && side) ? (x0 < 2 ? L : -L) : 0;
            int32_t bq[BLK_CHUNK];
            uint32_t want[BLK_CHUNK], w0[BLK_CHUNK], w1[BLK_CHUNK];
#pragma unroll
            for (int q = 0; q < BLK_CHUNK; ++q) {
                const NzOffset o = S.rows[c * BLK_CHUNK + q];   // (padding rows have no site)
                const uint32_t out = o.code & ~A & kRowAxes;
                if constexpr (PER) {
                    want[q] = in ? o.code & (side ? ~A : A) & 31u : 0u;
                    bq[q] = want[q] ? s + o.stride - 2 + (out ? wrap_fix(out, L) : 0) + off0 : 0;
                } else {
                    want[q] = out == 0u ? o.code & A & 31u : 0u;
                    bq[q] = out == 0u ? s + o.stride - 2 : 0;
                }
                if constexpr (EXACT) {
                    const int32_t w = (bq[q] >> 5) + 1;
                    w0[q] = m.map[w];
                    w1[q] = m.map[w + 1];
                } else {
                    const int32_t w = (bq[q] >> (m.mshift + 5u)) + 1;
                    w0[q] = m.map[w];
                    w1[q] = m.map[w + 1];
                }
            }
            if constexpr (!EXACT) {
#pragma unroll
                for (int q = 0; q < BLK_CHUNK; ++q) {
                    // the map bits of sites b .. b + 4 (at most three)
                    const int32_t k0 = bq[q] >> m.mshift, n = ((bq[q] + 4) >> m.mshift) - k0;
                    const uint32_t any = __builtin_amdgcn_alignbit(w1[q], w0[q], static_cast<uint32_t>(k0) & 31u) & ((2u << n) - 1u);
                    const bool need = any != 0u && want[q] != 0u;
                    const uint32_t first = static_cast<uint32_t>(max(bq[q], 0)) >> 5;
                    const uint32_t last = static_cast<uint32_t>(max(bq[q], 0) + 4) >> 5;
                    w0[q] = need ? ld_g(&m.occ[first]) : 0u;
                    w1[q] = need && last != first && last < m.occ_words ? ld_g(&m.occ[last]) : 0u;
                }
            }
            uint32_t mask = 0u;
#pragma unroll
            for (int q = 0; q < BLK_CHUNK; ++q) {
                uint32_t v;
                if constexpr (EXACT) {
                    v = __builtin_amdgcn_alignbit(w1[q], w0[q], static_cast<uint32_t>(bq[q]) & 31u);
                } else {
                    const int32_t b0 = max(bq[q], 0);
                    v = __builtin_amdgcn_alignbit(w1[q], w0[q], static_cast<uint32_t>(b0) & 31u) << (b0 - bq[q]);
                }
                mask |= (v & want[q]) << (5 * q);
            }
            uint64_t mk;
            while ((mk = __ballot(mask != 0u)) != 0ull) {
                int32_t base = 0;
                if (lane == 0) base = atomicAdd(&S.ecnt, static_cast<int32_t>(__popcll(mk)));
                base = __builtin_amdgcn_readfirstlane(base);
                if (base >= BLK_EDGES) return;   // (uniform) the pairs do not fit: the block is added in halves
                if (mask) {
                    const int bit = __builtin_ctz(mask);
                    mask &= mask - 1u;
                    const int q = (bit * 13) >> 6, j = bit - 5 * q;   // bit / 5 for bit < 30
                    const int32_t e = base + static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(
                                                 static_cast<uint32_t>(mk >> 32),
                                                 __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mk), 0u)));
                    if (e < BLK_EDGES) S.et[e] = static_cast<uint32_t>(i | ((c * BLK_CHUNK + q) << 9) | (j << 18));
                }
            }
        }
        g += NW;
        while (g >= groups) {
            g -= groups;
            ++c;
        }
    }
}

// Links nodes u and v: the worse root (smaller cluster before the block, then
// smaller node: a fixed total order) goes below the better one.  Wrap sweep: q
// = x0(u) - x0(v); a pair whose ends already share a root closes a loop, which
// winds around axis 0 when the displacements disagree.
template <typename C>
__device__ __forceinline__ void blk_link(BlkLds<C> &S, uint32_t u, uint32_t v, int32_t q)
{
    using W = typename BlkLds<C>::W;
    for (;;) {
        int32_t Du, Dv;
        uint32_t wa, wb;
        const uint32_t a = blk_find<C>(S, u, wa, Du);
        const uint32_t b = blk_find<C>(S, v, wb, Dv);
        if (a == b) {
            if (C::MODE == BLK_WRAP && Du != q + Dv) S.flag = 1;
            return;
        }
        const uint32_t sa = wa & NZ_SIZE, sb = wb & NZ_SIZE;
        const bool a_up = sa > sb || (sa == sb && a > b);
        const uint32_t lo = a_up ? b : a, hi = a_up ? a : b;
        const int32_t dab = q - Du + Dv;   // x0(a) - x0(b)
        auto expected = W::make(a_up ? wb : wa, 0);
        if (__hip_atomic_compare_exchange_strong(&S.f[lo], &expected, W::make(hi, a_up ? -dab : dab), __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
            return;
    }
}

// Cursor over the buckets of a band.  The counts of 64 buckets are held by the
// lanes of every wave, so a block costs one read of its entries.
struct BlkBand {
    const uint32_t *counts;
    const uint32_t *sites;
    uint32_t cap;
    int32_t nb;
    int32_t base;    // bucket of lane 0
    uint32_t mine;   // its count, by lane
};

__device__ __forceinline__ void blk_counts(BlkBand &bd, int32_t cb)
{
    const int32_t k = cb + static_cast<int32_t>(lane_id());
    bd.base = cb;
    bd.mine = k < bd.nb ? bd.counts[k] : 0u;
}

// Block of the band starting at bucket cb: as many whole buckets (16 at most)
// as B sites hold.  n sites, thread t < n takes entry t into pc, whose bucket
// holds the block's positions b0 .. b1 - 1; nbk buckets consumed.  over: the
// first bucket of the block overflowed its capacity.
template <int B>
__device__ __forceinline__ void blk_fetch(BlkBand &bd, int32_t cb, int &n, int &nbk, bool &over, uint32_t &pc, int &b0, int &b1)
{
    const uint32_t lane = lane_id();
    if (cb + 16 > bd.base + 64 && bd.base + 64 < bd.nb) blk_counts(bd, cb);
    const int32_t left = min(16, bd.nb - cb);
    const bool in = static_cast<int32_t>(lane) < left;
    const uint32_t got = static_cast<uint32_t>(__shfl(static_cast<int>(bd.mine), min(cb - bd.base + static_cast<int>(lane), 63)));
    const uint32_t c = in ? got : 0u;
    const uint64_t badm = __ballot(in && (c > bd.cap || c > static_cast<uint32_t>(B)));
    const int32_t lim = badm ? __builtin_ctzll(badm) : left;
    uint32_t incl = c;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        const uint32_t v = static_cast<uint32_t>(__shfl_up(static_cast<int>(incl), o));
        if (lane >= static_cast<uint32_t>(o)) incl += v;
    }
    const uint64_t ok = __ballot(static_cast<int32_t>(lane) < lim && incl <= static_cast<uint32_t>(B));
    nbk = __popcll(ok);
    n = nbk > 0 ? static_cast<int>(__builtin_amdgcn_readlane(incl, nbk - 1)) : 0;
    over = nbk == 0 && cb < bd.nb;
    const uint32_t t = threadIdx.x;
    uint32_t base = 0, k = 0, end = 0;
    for (int q = 0; q < nbk; ++q) {
        const uint32_t iq = __builtin_amdgcn_readlane(incl, q);
        if (t >= iq) {
            base = iq;
            k = static_cast<uint32_t>(q) + 1u;
        }
        if (end <= t) end = iq;
    }
    b0 = static_cast<int>(base);
    b1 = static_cast<int>(end);
    pc = t < static_cast<uint32_t>(n) ? bd.sites[static_cast<uint64_t>(cb + static_cast<int32_t>(k)) * bd.cap + (t - base)] : 0u;
}

__device__ __forceinline__ uint64_t site_key(const NzSample &d, uint32_t pc)
{
    const uint32_t s = static_cast<uint32_t>(site_of(pc, d.L));
    uint64_t ke, ko;
    site_key_pair(static_cast<uint32_t>(d.seed), static_cast<uint32_t>(d.seed >> 32), static_cast<uint32_t>(d.sample),
                  static_cast<uint32_t>(d.sample >> 32), s >> 1, ke, ko);
    return (s & 1u) ? ko : ke;
}

// Rank by (key, site) of this thread's site S.pcs[t] in the block: t < n lies in
// a bucket that holds positions b0 .. b1 - 1, and buckets are in key order, so
// only those are compared.  Keys are recomputed; their high words decide, full
// keys where two are equal.  `keys`: LDS scratch of n words.  Barriers before
// and after are the caller's (one is inside).
template <typename C>
__device__ __forceinline__ int blk_rank(BlkLds<C> &S, uint32_t *keys, const NzSample &d, int n, int b0, int b1)
{
    const int t = static_cast<int>(threadIdx.x);
    uint64_t K = 0;
    uint32_t pc = 0;
    if (t < n) {
        pc = S.pcs[t];
        K = site_key(d, pc);
        keys[t] = static_cast<uint32_t>(K >> 32);
    }
    __syncthreads();
    int rank = b0;
    if (t < n) {
        const uint32_t mine = static_cast<uint32_t>(K >> 32);
        bool tie = false;
#pragma unroll 8
        for (int j = b0; j < b1; ++j) {
            const uint32_t kj = keys[j];
            rank += kj < mine ? 1 : 0;
            tie = tie || (kj == mine && j != t);
        }
        if (tie)
            for (int j = b0; j < b1; ++j)
                if (keys[j] == mine && j != t) {
                    const uint64_t Kj = site_key(d, S.pcs[j]);
                    if (Kj < K || (Kj == K && S.pcs[j] < pc)) ++rank;
                }
    }
    return rank;
}

// joins[n] of every node: the least time, over all paths of pairs from the nodes
// that start with one, by which the path is there, a node from time_of(n) on.
// (barriers inside, one at the end)
template <typename C, typename Time>
__device__ __forceinline__ void blk_relax(BlkLds<C> &S, uint32_t *joins, int ne, Time &&time_of)
{
    const int t = static_cast<int>(threadIdx.x);
    for (;;) {
        __syncthreads();
        if (t == 0) S.flag = 0;
        __syncthreads();
        bool changed = false;
        for (int e = t; e < ne; e += C::NT) {
            const uint32_t u = S.et[e] & 0xFFFFu, v = S.et[e] >> 16;
            const uint32_t ju = ld_g(&joins[u]), jv = ld_g(&joins[v]);
            const uint32_t there = max(time_of(u), time_of(v));
            const uint32_t a = max(ju, there), b = max(jv, there);
            if (a < jv) atomicMin(&joins[v], a);
            if (b < ju) atomicMin(&joins[u], b);
            changed = changed || a < jv || b < ju;
        }
        if (changed) S.flag = 1;
        __syncthreads();
        if (!S.flag) break;
    }
}

enum { BLK_COMMITTED = 0, BLK_SPANS = 1, BLK_NOFIT = 2 };

// Adds the sites S.pcs[lo .. lo + len) (1 <= len <= B; sorted: in (key, site)
// order, else the whole block, position t in bucket positions b0 .. b1 - 1).  BLK_COMMITTED: merged,
// and no cluster spans.  BLK_NOFIT: nothing has changed (up to path halving).
// BLK_SPANS: T is the smallest number of the block's sites, in (key, site)
// order, after which a cluster spans and S.total that cluster's size (of a
// prefilled sample: its band sites); the sample is over.  Largest-cluster sweep (sites
// in order): the window entries of the block are written and smax carries the
// running maximum; BLK_NOFIT also where its sites have to be added one by one and
// are many.
template <typename C>
__device__ __forceinline__ int blk_step(BlkLds<C> &S, const BlkMem<C::MODE> &m, uint32_t *scratch, const NzSample &d, int32_t L,
                                        int nrows, int lo, int len, bool sorted, int b0, int b1, int max_old, int32_t r,
                                        int32_t win_lo, int32_t win_hi, uint32_t *win, int32_t &smax, int &T)
{
    using W = typename BlkLds<C>::W;
    constexpr int MODE = C::MODE;
    const int t = static_cast<int>(threadIdx.x);
    const bool act = t < len;

    // 1. clear the table; enter the block's sites and set their map bits
    for (uint32_t w = static_cast<uint32_t>(t); w < C::RS; w += C::NT) {
        S.rkey[w] = BLK_EMPTY;
        if constexpr (MODE == BLK_SMAX) S.pos[w] = 0xFFFFu;
    }
    if (t == 0) {
        S.ecnt = 0;
        S.nroots = 0;
        S.flag = 0;
        S.bad = 0;
        if constexpr (MODE == BLK_SMAX) {
            S.nbig = 0;
            for (int c = 0; c < BLK_CURVES; ++c) S.member[c] = 0;
        }
    }
    __syncthreads();
    int32_t site = 0;
    if (act) {
        const uint32_t pc = S.pcs[lo + t];
        site = site_of(pc, L);
        m.occ_set(static_cast<uint32_t>(site));
        const int32_t x0 = pc & 63;
        const uint32_t fl = (MODE != BLK_SPAN) ? 0u : ((x0 == 0 ? NZ_FLO : 0u) | (x0 == L - 1 ? NZ_FHI : 0u));
        bool fresh;
        const uint32_t h = blk_enter<C>(S, static_cast<uint32_t>(site), fresh);   // (the table holds B sites)
        S.f[h] = W::make(NZ_ROOT | fl | 1u, 0);
        S.spos[t] = static_cast<uint16_t>(h);
        if constexpr (MODE == BLK_SMAX) S.pos[h] = static_cast<uint16_t>(t);
    }
    __syncthreads();

    // 2. occupied neighbours
    if (m.mshift == 0) blk_scan<true, C>(S, m, nrows, L, lo, len);
    else blk_scan<false, C>(S, m, nrows, L, lo, len);
    __syncthreads();
    const int ne = S.ecnt;
    int res = ne > BLK_EDGES ? BLK_NOFIT : BLK_COMMITTED;

    // 3. the pairs' neighbours become nodes: a site of the block, or the root of
    //    an earlier cluster, entered into the table
    if (res == BLK_COMMITTED) {
        int nnew = 0;
        for (int e = t; e < ne; e += C::NT) {
            const uint32_t code = S.et[e];
            const int i = static_cast<int>(code & 511u), j = static_cast<int>(code >> 18);
            const NzOffset o = S.rows[(code >> 9) & 511u];
            const uint32_t pc = S.pcs[lo + i];
            int32_t nb = site_of(pc, L) + o.stride - 2 + j;
            if constexpr (C::PER) {
                const uint32_t out = o.code & ~allowed_of(pc, L) & (kRowAxes | (1u << j));
                if (out) nb += wrap_fix(out, L);
            }
            uint32_t node = blk_lookup<C>(S, static_cast<uint32_t>(nb));
            int32_t disp = 0;
            if (node == C::RS) {
                int32_t root;
                uint32_t word;
                m.resolve(nb, root, word, disp);
                bool fresh;
                node = blk_enter<C>(S, static_cast<uint32_t>(root), fresh);
                if (fresh) {
                    S.f[node] = W::make(word, 0);
                    ++nnew;
                }
                if (node == C::RS) S.bad = 1;   // table full
            }
            S.et[e] = static_cast<uint32_t>(S.spos[i]) | (node << 16);
            // x0(site) - x0(node): the neighbour lies at x0(site) + d0 = x0(node) + disp
            if constexpr (MODE == BLK_WRAP) S.eq[e] = disp - (j - 2);
        }
        if (nnew) atomicAdd(&S.nroots, nnew);
        __syncthreads();
        if (S.bad || (S.nroots > max_old && len > 1)) res = BLK_NOFIT;
    }
    if (res == BLK_NOFIT) {
        if (act) m.occ_clear(static_cast<uint32_t>(site));
        __syncthreads();
        return res;
    }

    // from here on the block's sites go by their band nodes (the barrier below)
    const int32_t ord0 = BAND_NODE | (r - m.n0);
    if constexpr (MODE != BLK_WRAP)
        if (act) S.rkey[S.spos[t]] = static_cast<uint32_t>(m.flat ? BAND_NODE | site : ord0 + t);

    // this thread's slots of the table
    constexpr int NODES = static_cast<int>(C::RS) / C::NT;
    bool live[NODES];
    uint32_t root[NODES], word0[NODES];
    int32_t disp[NODES];
    auto node_of = [&](int k) { return static_cast<uint32_t>(k * C::NT + t); };
#pragma unroll
    for (int k = 0; k < NODES; ++k) {
        const uint32_t n = node_of(k);
        live[k] = S.rkey[n] != BLK_EMPTY;   // (a site's key changes from one id to another)
        root[k] = n;
        disp[k] = 0;
        word0[k] = live[k] ? W::lo(S.f[n]) : 0u;
    }
    __syncthreads();   // (the unions rewrite the words)
    // roots of the live nodes; sizes and flags into the roots.  True: a cluster
    // spans.  (two barriers inside, the last one at the end)
    auto gather = [&]() -> bool {
#pragma unroll
        for (int k = 0; k < NODES; ++k) {
            if (!live[k]) continue;
            uint32_t unused;
            root[k] = blk_find<C>(S, node_of(k), unused, disp[k]);
            if (root[k] != node_of(k)) {
                uint32_t *w = reinterpret_cast<uint32_t *>(&S.f[root[k]]);   // (low half: the root word)
                atomicAdd(w, word0[k] & NZ_SIZE);
                if (word0[k] & NZ_FLAGS) atomicOr(w, word0[k] & NZ_FLAGS);
            }
        }
        __syncthreads();
        if constexpr (MODE == BLK_SPAN) {
#pragma unroll
            for (int k = 0; k < NODES; ++k)
                if (live[k] && root[k] == node_of(k) && (W::lo(S.f[root[k]]) & NZ_FLAGS) == NZ_FLAGS) S.flag = 1;
        }
        __syncthreads();
        return S.flag != 0;
    };

    // unions of all pairs (that `take` accepts)
    auto unions = [&](auto &&take) {
        for (int e = t; e < ne; e += C::NT) {
            const uint32_t u = S.et[e] & 0xFFFFu, v = S.et[e] >> 16;
            if (!take(u, v)) continue;
            int32_t q = 0;
            if constexpr (MODE == BLK_WRAP) q = S.eq[e];
            blk_link<C>(S, u, v, q);
        }
        __syncthreads();
    };

    if constexpr (MODE == BLK_SMAX) {
        // 4. all unions at once.  A cluster that ends the block no larger than the
        //    maximum before it never counts.  One that ends larger, but in which
        //    what joins its largest member is no larger than that maximum, counts
        //    by the cluster of that member alone, and this grows by each node's
        //    size at the time the node joins: the least time, over all paths of
        //    pairs, by which the last pair of the path is there.  By one lane, site
        //    by site, the kernel took 4.1 ms for 1000 samples of L = 12, zone 1
        //    (windows of 3800 sites around the threshold); with one such cluster per
        //    block 2.2, with up to four 1.6.
        unions([](uint32_t, uint32_t) { return true; });
        gather();
#pragma unroll
        for (int k = 0; k < NODES; ++k)
            if (live[k] && root[k] == node_of(k)) {
                const uint32_t ends = W::lo(S.f[root[k]]) & NZ_SIZE;
                uint32_t c = BLK_CURVES;
                if (ends > static_cast<uint32_t>(smax)) {
                    c = static_cast<uint32_t>(atomicAdd(&S.nbig, 1));
                    if (c < BLK_CURVES) S.ends[c] = ends;
                }
                S.next[root[k]] = static_cast<uint16_t>(min(c, static_cast<uint32_t>(BLK_CURVES)));
            }
        __syncthreads();
        const int nbig = S.nbig;
        uint32_t curve[NODES];   // of this thread's nodes (BLK_CURVES: none)
        bool at_once = nbig <= BLK_CURVES;
        uint32_t ends = static_cast<uint32_t>(smax);
        if (at_once && nbig > 0) {
#pragma unroll
            for (int k = 0; k < NODES; ++k) {
                curve[k] = live[k] ? S.next[root[k]] : BLK_CURVES;
                if (curve[k] < BLK_CURVES)
                    atomicMax(reinterpret_cast<unsigned long long *>(&S.member[curve[k]]),
                              (static_cast<unsigned long long>(word0[k] & NZ_SIZE) << 32) | node_of(k));
            }
            __syncthreads();
            for (int c = 0; c < nbig; ++c) {
                at_once = at_once && S.ends[c] - static_cast<uint32_t>(S.member[c] >> 32) <= static_cast<uint32_t>(smax);
                ends = max(ends, S.ends[c]);
            }
        }
        const int32_t rr = r + t + 1;   // r + t + 1 sites are occupied after position t
        if (at_once) {
            if (r + len >= win_lo) {
                auto time_of = [&](uint32_t n) {
                    const uint32_t p = S.pos[n];
                    return p == 0xFFFFu ? 0u : p + 1u;
                };
                uint32_t *joins = S.scratch;
                uint32_t best = static_cast<uint32_t>(smax);
                if (nbig) {
                    for (int c = 0; c < nbig; ++c)
                        if (act) S.smax[c * C::B + t] = 0u;
#pragma unroll
                    for (int k = 0; k < NODES; ++k) {
                        const bool first = curve[k] < BLK_CURVES && static_cast<uint32_t>(S.member[curve[k]]) == node_of(k);
                        joins[node_of(k)] = first ? time_of(node_of(k)) : BLK_EMPTY;
                    }
                    blk_relax<C>(S, joins, ne, time_of);
#pragma unroll
                    for (int k = 0; k < NODES; ++k)
                        if (curve[k] < BLK_CURVES) {
                            const uint32_t j = joins[node_of(k)];   // (<= len: every node has joined; 0: the member alone)
                            if (j) atomicAdd(&S.smax[curve[k] * C::B + j - 1u], word0[k] & NZ_SIZE);
                        }
                    __syncthreads();
                    uint32_t grown[BLK_CURVES];
#pragma unroll
                    for (int c = 0; c < BLK_CURVES; ++c) {
                        grown[c] = c < nbig && act ? S.smax[c * C::B + t] : 0u;
                        if (c >= nbig) continue;   // (uniform)
#pragma unroll
                        for (int o = 1; o < 64; o <<= 1) {
                            const uint32_t v = static_cast<uint32_t>(__shfl_up(static_cast<int>(grown[c]), o));
                            if ((t & 63) >= o) grown[c] += v;
                        }
                        if ((t & 63) == 63) S.wsum[c * (C::NT / 64) + (t >> 6)] = grown[c];
                    }
                    __syncthreads();
#pragma unroll
                    for (int c = 0; c < BLK_CURVES; ++c) {
                        if (c >= nbig) continue;
                        for (int w = 0; w < (t >> 6); ++w) grown[c] += S.wsum[c * (C::NT / 64) + w];
                        // (a member that is a site of the block is counted as it joins)
                        const uint64_t mb = S.member[c];
                        if (time_of(static_cast<uint32_t>(mb)) == 0u) grown[c] += static_cast<uint32_t>(mb >> 32);
                        best = max(best, grown[c]);
                    }
                }
                if (act && rr >= win_lo && rr < win_hi) win[rr - win_lo] = best;
            }
            smax = static_cast<int32_t>(ends);
        } else if (len > 32) {
            // in halves: the condition is soon met
            if (act) m.occ_clear(static_cast<uint32_t>(site));
            __syncthreads();
            return BLK_NOFIT;
        } else {
            // one by one, by one lane; the sizes are kept at the roots
            if (act) S.first[t] = BLK_EMPTY;
#pragma unroll
            for (int k = 0; k < NODES; ++k)
                if (live[k]) S.f[node_of(k)] = W::make(word0[k], 0);
            __syncthreads();
            for (int e = t; e < ne; e += C::NT) {
                // kept once, at the later position
                const uint32_t i = S.pos[S.et[e] & 0xFFFFu], j = S.pos[S.et[e] >> 16];
                if (j == 0xFFFFu || j < i)
                    S.next[e] = static_cast<uint16_t>(__hip_atomic_exchange(&S.first[i], static_cast<uint32_t>(e), __ATOMIC_RELAXED,
                                                                            __HIP_MEMORY_SCOPE_WORKGROUP));
            }
            __syncthreads();
            if (t == 0) {
                for (int i = 0; i < len; ++i) {
                    uint32_t a = S.spos[i], sz = 1;
                    for (uint32_t e = S.first[i]; (e & 0xFFFFu) != 0xFFFFu; e = S.next[e]) {
                        int32_t unused;
                        uint32_t wb;
                        const uint32_t b = blk_find<C>(S, S.et[e] >> 16, wb, unused);
                        if (b == a) continue;
                        const uint32_t sb = wb & NZ_SIZE;
                        const uint32_t lo_n = sb > sz ? a : b, hi_n = sb > sz ? b : a;
                        sz += sb;
                        st_g(&S.f[lo_n], W::make(hi_n, 0));
                        st_g(&S.f[hi_n], W::make(NZ_ROOT | sz, 0));
                        a = hi_n;
                    }
                    smax = max(smax, static_cast<int32_t>(sz));
                    S.smax[i] = static_cast<uint32_t>(smax);
                }
            }
            __syncthreads();
            smax = static_cast<int32_t>(S.smax[len - 1]);
            if (act && rr >= win_lo && rr < win_hi) win[rr - win_lo] = S.smax[t];
#pragma unroll
            for (int k = 0; k < NODES; ++k) {
                uint32_t unused;
                if (live[k]) root[k] = blk_find<C>(S, node_of(k), unused, disp[k]);
            }
        }
    } else {
        unions([](uint32_t, uint32_t) { return true; });
        if (gather()) {
            res = BLK_SPANS;
            T = 1;
            const uint32_t own = act ? S.spos[t] : 0u;   // this position's node
            int myrank = t;
            if (len > 1) {
                // 5. the smallest T.  Spanning: the least time by which a path joins a
                //    node on the low border to one on the high border.  Wrapping: by
                //    bisection over the block's first T sites.  A trial is a connected-
                //    components pass over the pairs among the first so many sites; the
                //    last one gives the cluster.  (Nine trials took 20 to 27 us per
                //    sample: 1000 samples of L = 16, zones 1-7, 0.45 ms, and 0.38
                //    with the paths.)
                //    ranks: of every node, 0 for earlier roots, 1 + rank for sites.
                uint16_t *ranks = reinterpret_cast<uint16_t *>(scratch + C::B);
                if (!sorted) myrank = blk_rank<C>(S, scratch, d, len, b0, b1);   // (sorted: positions are ranks)
#pragma unroll
                for (int k = 0; k < NODES; ++k) ranks[node_of(k)] = 0;
                __syncthreads();
                if (act) ranks[own] = static_cast<uint16_t>(myrank + 1);
                __syncthreads();
                uint32_t since[NODES];   // the first T that has this thread's node
#pragma unroll
                for (int k = 0; k < NODES; ++k) since[k] = live[k] ? ranks[node_of(k)] : 0xFFFFu;
                auto trial = [&](int first) -> bool {
                    __syncthreads();
                    if (t == 0) S.flag = 0;
#pragma unroll
                    for (int k = 0; k < NODES; ++k) {
                        live[k] = since[k] <= static_cast<uint32_t>(first);
                        if (live[k]) S.f[node_of(k)] = W::make(word0[k], 0);
                    }
                    __syncthreads();
                    unions([&](uint32_t u, uint32_t v) {
                        return static_cast<int>(ranks[u]) <= first && static_cast<int>(ranks[v]) <= first;
                    });
                    return gather();
                };
                if constexpr (MODE == BLK_SPAN) {
                    uint32_t *joins = scratch + C::B + C::RS / 2;
#pragma unroll
                    for (int k = 0; k < NODES; ++k)
                        joins[node_of(k)] = live[k] && (word0[k] & NZ_FLO) ? since[k] : BLK_EMPTY;
                    if (t == 0) S.total = BLK_EMPTY;
                    blk_relax<C>(S, joins, ne, [&](uint32_t n) { return static_cast<uint32_t>(ranks[n]); });
#pragma unroll
                    for (int k = 0; k < NODES; ++k)
                        if (live[k] && (word0[k] & NZ_FHI)) atomicMin(&S.total, joins[node_of(k)]);
                    __syncthreads();
                    T = static_cast<int>(S.total);
                } else {
                    int none = 0;   // the first `none` sites do not span, the first T do
                    T = len;
                    while (T - none > 1) {
                        const int mid = (none + T) / 2;
                        if (trial(mid)) T = mid;
                        else none = mid;
                    }
                }
                trial(T);
            }
            if (act && myrank == T - 1) {
                uint32_t word;
                int32_t unused;
                S.croot = blk_find<C>(S, own, word, unused);
                S.total = word & NZ_SIZE;
            }
            __syncthreads();
            // the earlier clusters of the spanning one get both border flags, by
            // which their prefilled members are counted
            if (MODE == BLK_SPAN && m.n0 > 0) {
#pragma unroll
                for (int k = 0; k < NODES; ++k)
                    if (live[k] && root[k] == S.croot)
                        m.commit(static_cast<int32_t>(S.rkey[node_of(k)]), true, NZ_ROOT | NZ_FLAGS, 0, 0);
                __syncthreads();
            }
            return res;
        }
    }

    // 6. write back
#pragma unroll
    for (int k = 0; k < NODES; ++k) {
        if (!live[k]) continue;
        const uint32_t n = node_of(k), rt = root[k];
        // (dense: nothing points at a site of the block that is no root)
        if constexpr (MODE != BLK_WRAP)
            if (!m.flat && rt != n && static_cast<uint32_t>(S.rkey[n] - static_cast<uint32_t>(ord0)) < static_cast<uint32_t>(len)) continue;
        m.commit(static_cast<int32_t>(S.rkey[n]), rt == n, W::lo(S.f[n]), static_cast<int32_t>(S.rkey[rt]), disp[k]);
    }
    if constexpr (MODE != BLK_WRAP)
        if (act && !m.flat) {
            uint32_t unused;
            int32_t none;
            st_g(&m.par[site], static_cast<int32_t>(S.rkey[blk_find<C>(S, S.spos[t], unused, none)]) | BLK_LINKED);
        }
    __syncthreads();   // (the stores drain behind the next block's checks)
    return res;
}

// Persistent: every workgroup pops samples (longest first) until the queue is
// empty.  PER: periodic coordinates.
template <typename C>
__global__ __launch_bounds__(C::NT, 4) void nz_sweep_kernel(NzSweepArgs a, SweepOut out)
{
    constexpr int MODE = C::MODE, NT = C::NT, B = C::B;
    extern __shared__ uint32_t blk_map[];
    __shared__ BlkLds<C> S;
    // (a sample that spans needs its map no more)
    uint32_t *scratch = C::OWN_SCRATCH ? S.scratch : C::ID_SCRATCH ? S.rkey : blk_map;
    const int t = static_cast<int>(threadIdx.x);
    for (;;) {
        if (t == 0) S.claim = atomicAdd(a.qhead, 1);
        __syncthreads();
        const int qi = __builtin_amdgcn_readfirstlane(S.claim);
        __syncthreads();
        if (qi >= a.nqueue) break;
        const int sid = a.queue[qi];
        if (a.state[sid].status != NZ_ST_PENDING) continue;   // (uniform)
        const NzSample &d = a.desc[sid];
        const int32_t L = d.L, nrows = d.rows, nb = d.nb;
        const uint32_t N = static_cast<uint32_t>(d.N);
        BlkBand band;
        band.counts = reinterpret_cast<const uint32_t *>(a.ws + d.off_counts);
        band.sites = reinterpret_cast<const uint32_t *>(a.ws + d.off_sites);
        band.cap = static_cast<uint32_t>(d.cap);
        band.nb = nb;
        const NzOffset *rows = a.tabs + d.tab;
        BlkMem<MODE> m;
        m.occ = reinterpret_cast<uint32_t *>(a.ws + d.off_occ);
        m.par = reinterpret_cast<int32_t *>(a.ws + d.off_par);
        m.parc = reinterpret_cast<int32_t *>(a.ws + d.off_parc);
        m.flat = a.state[sid].n0 == 0;
        m.band = m.flat ? m.par : reinterpret_cast<int32_t *>(a.ws + d.off_sites);
        m.pw = reinterpret_cast<uint64_t *>(a.ws + d.off_par);
        m.wrec = reinterpret_cast<const uint2 *>(a.ws + d.off_wrec);
        m.map = blk_map;
        m.mshift = map_shift(N, a.map_words);
        m.occ_words = ((N + 63u) >> 6) << 1;

        for (int k = t; k < (nrows + BLK_CHUNK - 1) / BLK_CHUNK * BLK_CHUNK; k += NT) {
            NzOffset o;
            o.stride = 0;
            o.code = 0u;
            if (k < nrows) o = rows[k];
            S.rows[k] = o;
        }
        const int32_t n0 = a.state[sid].n0;
        int32_t r = n0;                // sites already occupied
        m.n0 = n0;
        // the map of the prefilled sites: from their list while it is shorter
        // than the bitset
        const uint32_t mwords = (((N - 1u) >> m.mshift) >> 5) + 1u;
        const bool by_list = static_cast<uint32_t>(r) < m.occ_words;
        for (uint32_t w = static_cast<uint32_t>(t); w < mwords + MAP_PAD; w += NT) {
            const bool inner = w >= 1u && w <= mwords;
            blk_map[w] = (!by_list && m.mshift == 0 && inner) ? m.occ[w - 1u] : 0u;
        }
        __syncthreads();
        if (by_list) {
            const uint32_t *prefix = reinterpret_cast<const uint32_t *>(a.ws + d.off_prefix);
            for (int32_t k = t; k < n0; k += NT) {
                const uint32_t b = prefix[k] >> m.mshift;
                atomicOr(&blk_map[1 + (b >> 5)], 1u << (b & 31));
            }
        } else if (m.mshift) {
            for (uint32_t w0 = static_cast<uint32_t>(t); w0 < m.occ_words; w0 += 8 * NT) {
                uint32_t v[8];
#pragma unroll
                for (uint32_t q = 0; q < 8; ++q) v[q] = w0 + q * NT < m.occ_words ? m.occ[w0 + q * NT] : 0u;
#pragma unroll
                for (uint32_t q = 0; q < 8; ++q) {
                    if (!v[q]) continue;
                    uint32_t bits = 1u;   // (mshift >= 5: the word is part of one bit)
                    if (m.mshift < 5) {
                        bits = 0u;
                        const uint32_t grp = (1u << (1u << m.mshift)) - 1u;
                        for (uint32_t g = 0; g < (32u >> m.mshift); ++g)
                            if ((v[q] >> (g << m.mshift)) & grp) bits |= 1u << g;
                    }
                    const uint32_t b = ((w0 + q * NT) << 5) >> m.mshift;
                    atomicOr(&blk_map[1 + (b >> 5)], bits << (b & 31));
                }
            }
        }

        int32_t smax = a.state[sid].smax;
        int32_t status = NZ_ST_BAND, nstar = 0, mass = 0;
        const int32_t win_lo = MODE == BLK_SMAX ? d.win_lo : 0, win_hi = MODE == BLK_SMAX ? d.win_hi : 0;
        uint32_t *win = reinterpret_cast<uint32_t *>(a.ws + d.off_win);
        bool done = MODE == BLK_SMAX && r >= win_lo;
        if (done) status = NZ_ST_BACKOFF;   // the prefill covers part of the window: start lower

        int32_t cb = 0;
        int n = 0, nbk = 0;
        bool over = false;
        uint32_t pc = 0;
        int nb0 = 0, nb1 = 0;
        blk_counts(band, 0);
        if (!done) blk_fetch<B>(band, cb, n, nbk, over, pc, nb0, nb1);
        while (!done) {
            while (n == 0 && nbk > 0) {
                cb += nbk;
                blk_fetch<B>(band, cb, n, nbk, over, pc, nb0, nb1);
            }
            if (n == 0) {
                if (over) status = NZ_ST_BUCKET;
                break;
            }
            if (t < n) S.pcs[t] = pc;
            const int all = n, b0 = nb0, b1 = nb1;
            // the next block's entries, loaded while this one is processed
            cb += nbk;
            blk_fetch<B>(band, cb, n, nbk, over, pc, nb0, nb1);
            __syncthreads();
            bool sorted = false;
            auto sort = [&]() {
                if (sorted) return;
                sorted = true;
                const uint32_t mine = t < all ? S.pcs[t] : 0u;
                const int rank = blk_rank<C>(S, S.et, d, all, b0, b1);
                __syncthreads();
                if (t < all) S.pcs[rank] = mine;
                __syncthreads();
            };
            if (MODE == BLK_SMAX) sort();
            int len = all;
            for (int lo = 0; lo < all;) {
                int T = 0;
                const int res = blk_step<C>(S, m, scratch, d, L, nrows, lo, len, sorted, b0, b1, a.blk_old, r, win_lo, win_hi, win,
                                            smax, T);
                if (res == BLK_NOFIT) {
                    sort();
                    len = max(1, len / 2);
                    continue;
                }
                if (res == BLK_SPANS) {
                    status = NZ_ST_DONE;
                    nstar = r + T;
                    mass = static_cast<int32_t>(S.total);
                    // S.total counts the band sites alone (prefilled clusters keep no
                    // sizes): the prefilled members of the cluster, whose roots carry
                    // both flags now
                    if (MODE == BLK_SPAN && n0 > 0 && out.mass) {
                        // Two passes over the list: the former roots (one bit each, kept
                        // where the map was: is it in the spanning cluster), then the
                        // members, by their own root's bit.  A root that is linked is
                        // queued (where the tables were), and 64 links are followed at a
                        // time: one by one every wave waits at nearly every entry for
                        // some lane's link (zone 1 of L = 24, 1.1 M entries, 200
                        // samples: the sweep with masses 6.1 ms, queued 5.75).
                        const uint32_t words = min(a.map_words, (static_cast<uint32_t>(n0) + 31u) >> 5);
                        const int32_t in_bits = static_cast<int32_t>(words << 5);
                        for (uint32_t w = static_cast<uint32_t>(t); w < words; w += NT) blk_map[w] = 0u;
                        __syncthreads();
                        int32_t members = 0;
                        constexpr int QN = static_cast<int>(C::RS) / (NT / 64);   // queue entries per wave
                        static_assert(QN >= 128, "64 left and 64 new");
                        const uint32_t lane = lane_id();
                        uint32_t *qk = &S.rkey[(t >> 6) * QN];
                        uint32_t *qv = reinterpret_cast<uint32_t *>(S.f) + (t >> 6) * QN;
                        int32_t nq = 0;   // (wave-uniform)
                        auto chase = [&](int32_t v) -> bool {   // the cluster an entry leads to
                            while (v >= 0) v = ld_g(m.entry(node_id(v)));
                            return (static_cast<uint32_t>(v) & NZ_FLAGS) == NZ_FLAGS;
                        };
                        auto count_root = [&](int32_t k) {
                            ++members;
                            if (k < in_bits) atomicOr(&blk_map[k >> 5], 1u << (k & 31));
                        };
                        auto follow = [&](int32_t e0, int32_t n) {
                            __builtin_amdgcn_wave_barrier();
                            if (static_cast<int32_t>(lane) < n) {
                                const int32_t k = static_cast<int32_t>(ld_w(&qk[e0 + static_cast<int32_t>(lane)]));
                                if (chase(static_cast<int32_t>(ld_w(&qv[e0 + static_cast<int32_t>(lane)])))) count_root(k);
                            }
                            __builtin_amdgcn_wave_barrier();
                        };
                        // every entry, for all lanes (past the end: no entry); the list's
                        // memory is a multiple of 256 bytes
                        auto each = [&](auto &&visit) {
                            for (int32_t base = 0; base < n0; base += 16 * NT) {
                                int4 v[4];
#pragma unroll
                                for (int q = 0; q < 4; ++q) {
                                    const int32_t k = base + 4 * t + q * 4 * NT;
                                    v[q] = k < n0 ? *reinterpret_cast<const int4 *>(&m.parc[k]) : make_int4(NZ_NONE, NZ_NONE, NZ_NONE, NZ_NONE);
                                }
#pragma unroll
                                for (int q = 0; q < 4; ++q) {
                                    const int32_t k = base + 4 * t + q * 4 * NT;
                                    visit(k, v[q].x);
                                    visit(k + 1, k + 1 < n0 ? v[q].y : NZ_NONE);
                                    visit(k + 2, k + 2 < n0 ? v[q].z : NZ_NONE);
                                    visit(k + 3, k + 3 < n0 ? v[q].w : NZ_NONE);
                                }
                            }
                        };
                        each([&](int32_t k, int32_t v) {
                            if (v < 0 && (static_cast<uint32_t>(v) & NZ_FLAGS) == NZ_FLAGS) count_root(k);
                            const bool linked = v >= 0 && (v & BLK_LINKED);
                            const uint64_t mk = __ballot(linked);
                            if (!mk) return;   // (uniform)
                            if (linked) {
                                const int32_t e = nq + static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(
                                                           static_cast<uint32_t>(mk >> 32),
                                                           __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mk), 0u)));
                                st_w(&qk[e], static_cast<uint32_t>(k));
                                st_w(&qv[e], static_cast<uint32_t>(v));
                            }
                            nq += static_cast<int32_t>(__popcll(mk));
                            if (nq >= 64) {
                                nq -= 64;
                                follow(nq, 64);
                            }
                        });
                        follow(0, nq);
                        __syncthreads();
                        each([&](int32_t, int32_t v) {
                            if (v < 0 || (v & BLK_LINKED)) return;
                            const int32_t root = v - LIST_NODE;
                            if (root < in_bits) members += (blk_map[root >> 5] >> (root & 31)) & 1u;
                            else members += chase(v) ? 1 : 0;
                        });
#pragma unroll
                        for (int o = 1; o < 64; o <<= 1) members += __shfl_xor(members, o);
                        if ((t & 63) == 0 && members) atomicAdd(&S.total, static_cast<uint32_t>(members));
                        __syncthreads();
                        mass = static_cast<int32_t>(S.total);
                    }
                    done = true;
                    break;
                }
                r += len;
                lo += len;
                len = min(len, all - lo);
                if (MODE == BLK_SMAX && r + 1 >= win_hi) {
                    status = NZ_ST_DONE;
                    done = true;
                    break;
                }
            }
        }
        if (status == NZ_ST_BAND && d.full) {
            status = NZ_ST_DONE;   // the whole lattice is occupied and never spans
            nstar = 0;
            mass = 0;
        }
        if (t == 0) {
            a.state[sid].status = status;
            a.state[sid].nstar = nstar;
            a.state[sid].mass = mass;
            if (status == NZ_ST_DONE) {
                const int32_t o = out.out_index[sid];
                out.nstar[o] = nstar;
                if (out.mass) out.mass[o] = mass;
            }
        }
        __syncthreads();   // the tables and the map are free for the next sample
    }
}

}  // namespace nz

// ---------------------------------------------------------------------------
// Host-side launchers (internal to the library).

#include "nz_launch.h"

namespace nz {

hipError_t launch_expand(const NzRun *runs, int32_t nruns, int32_t max_count, NzSample *desc, NzState *state,
                         int32_t *queue, int32_t *out_index, int32_t *list, int32_t *qhead, hipStream_t st)
{
    if (nruns <= 0 || nruns > 65535) return nruns <= 0 ? hipSuccess : hipErrorInvalidValue;
    hipLaunchKernelGGL(nz_expand_kernel, dim3(static_cast<uint32_t>((max_count + 255) / 256), static_cast<uint32_t>(nruns)),
                       dim3(256), 0, st, runs, desc, state, queue, out_index, list, qhead);
    return hipGetLastError();
}

hipError_t launch_clear(NzSample *desc, const int32_t *list, int32_t nsamp, int32_t level, uint8_t *ws, NzState *state,
                        hipStream_t st)
{
    if (nsamp <= 0) return hipSuccess;
    if (list && (level < 0 || level > 1)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(nz_clear_kernel, dim3(nsamp), dim3(256), 0, st, desc, list, nsamp, level, ws, state);
    return hipGetLastError();
}

// The local keys kernel's counters and queues have to fit one CU, and its waves
// have to reach every CU (fewer samples: several workgroups each).
constexpr size_t kKeysLds = 150 * 1024;
constexpr int64_t kKeysLocalWaves = 1024;

hipError_t launch_keys(const NzSample *desc, const int32_t *list, int32_t first, int32_t count, int32_t N, uint8_t *ws,
                       NzState *state, bool by_xcd, int32_t max_nb, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    const int32_t waves = std::min(KEYS_LOCAL_THREADS / 64, (N + KEYS_WAVE_SITES - 1) / KEYS_WAVE_SITES);
    const size_t words = (static_cast<size_t>(max_nb) + 1) / 2 * 2;
    const size_t lds = 4 * (words + 3 * static_cast<size_t>(waves) * KEYS_BQ);
    if (!list && max_nb > 0 && lds <= kKeysLds && static_cast<int64_t>(count) * waves >= kKeysLocalWaves) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(nz_keys_kernel_local),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kKeysLds));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(nz_keys_kernel_local, dim3(static_cast<uint32_t>(count)), dim3(static_cast<uint32_t>(64 * waves)), lds,
                           st, desc, first, static_cast<int32_t>(words), ws, state);
        return hipGetLastError();
    }
    const int32_t bps = (N + KEYS_SITES_PER_BLOCK - 1) / KEYS_SITES_PER_BLOCK;
    const int32_t slots = by_xcd ? (count + 7) / 8 * 8 : count;
    const int64_t blocks = static_cast<int64_t>(bps) * slots;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(nz_keys_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(KEYS_THREADS), 0, st, desc, list,
                       first, count, by_xcd, bps, ws, state);
    return hipGetLastError();
}

// Words of the map of the hook of sparse lists, and whether a list of n0 sites of
// N counts as one: under one set bit in 32 of the map.
constexpr uint32_t kHookMapWords = 136 * 256;

bool hook_map_fits(int64_t N, int64_t n0)
{
    return (n0 << (5 + map_shift(static_cast<uint32_t>(N), kHookMapWords))) < N;
}

hipError_t launch_prefill(const NzSample *desc, const int32_t *list, int32_t nlist, int32_t max_sites,
                          int32_t grid_sites, const NzOffset *tabs, uint8_t *ws, NzState *state, bool smax, bool wrap, bool periodic,
                          int32_t map_N, int cus, hipStream_t st, hipEvent_t *ev)
{
    if (nlist <= 0) return hipSuccess;
    // workgroups per sample: a hook workgroup takes 2048 sites of a large list
    // (few partly filled edge buffers) down to 256 of a small one (more waves in
    // flight): zone 1 at L = 16 (150000 sites) 3.78 / 3.23 / 3.08 ms for 1000
    // samples with 256 / 1024 / 2048, zones 1-7 (2000 sites) 0.46 / 0.57 / 0.62
    const int64_t per_wg = std::max<int64_t>(256, std::min<int64_t>(2048, grid_sites / 16 / 256 * 256));
    const int32_t bx_hook = static_cast<int32_t>(std::max<int64_t>(1, std::min<int64_t>(1024, (grid_sites + per_wg - 1) / per_wg)));
    const int32_t bx_site = static_cast<int32_t>(std::max<int64_t>(1, std::min<int64_t>(1024, (grid_sites + 1023) / 1024)));
    auto mark = [&](int k) {
        if (ev) (void)hipEventRecord(ev[k], st);
    };
    mark(0);
    const uint32_t slots8 = static_cast<uint32_t>((nlist + 7) / 8) * 8u;
    if (wrap) {
        hipLaunchKernelGGL(nz_hookw_kernel, dim3(static_cast<uint32_t>(bx_hook) * slots8), dim3(256), 0, st, desc, list,
                           nlist, bx_hook, tabs, ws, state);
        hipLaunchKernelGGL(nz_compressw_kernel, dim3(static_cast<uint32_t>(bx_site) * slots8), dim3(256), 0, st, desc, list,
                           nlist, bx_site, ws, state);
        hipLaunchKernelGGL(nz_accumw_kernel, dim3(static_cast<uint32_t>(bx_site) * slots8), dim3(256), 0, st, desc, list,
                           nlist, bx_site, ws, state);
        mark(1);
        mark(2);
        mark(3);
        mark(4);
        return hipGetLastError();
    }
    if (map_N > 0) {
        auto k = periodic ? nz_hook_kernel_map<true> : nz_hook_kernel_map<false>;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 static_cast<int>(kHookMapWords * 4));
        if (e != hipSuccess) return e;
        const uint32_t words = std::min(kHookMapWords, ((static_cast<uint32_t>(map_N) - 1u) >> 5) + 1u + MAP_PAD);
        // a few workgroups per CU over all samples, of up to 1024 sites each
        const int32_t nt = static_cast<int32_t>(std::max(64, std::min(1024, (grid_sites + 63) / 64 * 64)));
        const int32_t most = std::max(1, (grid_sites + nt - 1) / nt);
        const int32_t bx = std::max(1, std::min(most, 4 * cus / nlist));
        hipLaunchKernelGGL(k, dim3(static_cast<uint32_t>(bx) * slots8), dim3(static_cast<uint32_t>(nt)), words * 4u, st, desc, list,
                           nlist, bx, words, tabs, ws, state);
    } else if (periodic)
        hipLaunchKernelGGL(nz_hook_kernel<true>, dim3(static_cast<uint32_t>(bx_hook) * slots8), dim3(256), 0, st, desc, list,
                           nlist, bx_hook, tabs, ws, state);
    else
        hipLaunchKernelGGL(nz_hook_kernel<false>, dim3(static_cast<uint32_t>(bx_hook) * slots8), dim3(256), 0, st, desc,
                           list, nlist, bx_hook, tabs, ws, state);
    mark(1);
    hipLaunchKernelGGL(nz_compress_kernel, dim3(static_cast<uint32_t>(bx_site) * slots8), dim3(256), 0, st, desc, list,
                       nlist, bx_site, ws, state);
    mark(2);
    if (smax && max_sites <= SIZES_RANGE * SIZES_RANGES) {
        // (longer lists would be read too often: one atomic per site)
        const int32_t ranges = std::max(1, (max_sites + SIZES_RANGE - 1) / SIZES_RANGE);
        const int32_t range = std::max(64, std::min(SIZES_RANGE, max_sites));
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(nz_sizes_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, SIZES_RANGE * 4);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(nz_sizes_kernel, dim3(static_cast<uint32_t>(ranges) * slots8), dim3(range > 8192 ? 1024 : 256),
                           static_cast<size_t>(range) * 4, st, desc, list, nlist, ranges, range, ws, state);
        mark(3);
        mark(4);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(nz_accum_kernel, dim3(static_cast<uint32_t>(bx_site) * slots8), dim3(256), 0, st, desc, list, nlist,
                       bx_site, ws, state);
    mark(3);
    mark(4);   // (there is no separate expand pass)
    if (smax)
        hipLaunchKernelGGL(nz_rootmax_kernel, dim3(static_cast<uint32_t>(bx_site) * slots8), dim3(256), 0, st, desc, list,
                           nlist, bx_site, ws, state);
    return hipGetLastError();
}

hipError_t launch_winsum(const NzSample *desc, const NzState *state, int32_t nsamp, int32_t w, const uint8_t *ws,
                         uint64_t *out, hipStream_t st)
{
    if (nsamp <= 0 || w <= 0) return hipSuccess;
    const int32_t blocks = (w + 255) / 256;
    const uint32_t grid = static_cast<uint32_t>(blocks < 4096 ? blocks : 4096);
    // some 2048 workgroups, and at least eight samples each
    const int32_t spread = std::max(1, std::min((nsamp + 7) / 8, 2048 / static_cast<int32_t>(grid)));
    hipLaunchKernelGGL(nz_winsum_kernel, dim3(grid, static_cast<uint32_t>(spread)), dim3(256), 0, st, desc, state, nsamp, w, ws,
                       out);
    return hipGetLastError();
}

template <int MODE, bool PER, int NT, int B>
static hipError_t launch_block_n(const NzSweepArgs &a, const SweepOut &o, int cus, size_t lds_per_wg, hipStream_t st)
{
    using C = BlkCfg<MODE, PER, NT, B>;
    static_assert(NT > 256 || sizeof(BlkLds<C>) + BLK_SMALL_MAP * 4 <= 65536, "small maps need no limit of their own");
    if (NT > 256 && a.map_words < C::SCRATCH) return hipErrorInvalidValue;
    auto k = nz_sweep_kernel<C>;
    const size_t lds = static_cast<size_t>(a.map_words) * 4u;
    if constexpr (NT > 256) {
        // the limit is the kernel's, not this launch's: always what a workgroup can
        // have, so that no other thread's smaller lattice lowers it before the launch
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           static_cast<int>(lds_per_wg - sizeof(BlkLds<C>)));
        if (e != hipSuccess) return e;
    }
    // workgroups per CU for this much LDS (one architecture: fixed for the process)
    static std::atomic<uint64_t> last{0};   // lds << 32 | workgroups of the last shape asked for
    uint64_t l = last.load(std::memory_order_relaxed);
    if (l == 0 || (l >> 32) != lds) {
        int n = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, NT, lds);
        if (e != hipSuccess) return e;
        l = (static_cast<uint64_t>(lds) << 32) | static_cast<uint32_t>(n);
        last.store(l, std::memory_order_relaxed);
    }
    const int wgs = static_cast<int>(l & 0xFFFFFFFFu);
    const int grid = std::min(a.nqueue, cus * std::max(1, wgs));
    hipLaunchKernelGGL(k, dim3(grid), dim3(NT), lds, st, a, o);
    return hipGetLastError();
}

// Small maps (up to L = 10): several workgroups of 256 threads share a CU.  Exact
// maps of which a CU holds two (L = 11 to 13): two workgroups of 512 threads, if
// there are samples for both, so that one sample's reads cover the other's
// barriers.  Larger ones leave room for one workgroup per CU, of 1024 threads.
// Sweep kernel, 1000 samples, one / two workgroups per CU: zone 1 plain, L = 11
// 2.42 / 1.71 ms, L = 12 3.74 / 2.64; prefilled, L = 12, zone 1 0.77 / 0.68, zones
// 1-7 0.27 / 0.24, L = 13, zone 1 1.04 / 0.94.  Two maps that are not exact lose
// by the reads behind them: L = 16, zones 1-2 prefilled 0.85 / 1.02 ms, 1-7 0.39 /
// 0.53, L = 24 zones 1-2 2.40 / 3.44 (300 samples).
template <int MODE, bool PER>
static hipError_t launch_block_t(NzSweepArgs a, const SweepOut &o, int cus, uint32_t max_N, size_t lds_per_wg, hipStream_t st)
{
    const uint32_t exact = ((max_N - 1u) >> 5) + 1u + MAP_PAD;
    if (exact <= BLK_SMALL_MAP || MODE == BLK_SMAX) {
        a.map_words = std::min(exact, BLK_SMALL_MAP);
        return launch_block_n<MODE, PER, 256, 256>(a, o, cus, lds_per_wg, st);
    }
    if constexpr (MODE != BLK_SMAX) {
        if (a.nqueue > cus && 2 * (static_cast<size_t>(exact) * 4 + sizeof(BlkLds<BlkCfg<MODE, PER, 512, 512>>)) <= lds_per_wg) {
            a.map_words = exact;
            return launch_block_n<MODE, PER, 512, 512>(a, o, cus, lds_per_wg, st);
        }
        a.map_words = std::min<uint32_t>(exact, static_cast<uint32_t>((lds_per_wg - sizeof(BlkLds<BlkCfg<MODE, PER, 1024, 512>>)) / 4));
        return launch_block_n<MODE, PER, 1024, 512>(a, o, cus, lds_per_wg, st);
    }
}

hipError_t launch_sweep(SweepKind kind, bool periodic, const NzSweepArgs &a, int32_t *nstar, int32_t *mass,
                        const int32_t *out_index, int cus, uint32_t max_N, size_t lds_per_wg, hipStream_t st)
{
    if (a.nqueue <= 0) return hipSuccess;
    if (max_N < 1 || lds_per_wg < 65536) return hipErrorInvalidValue;
    SweepOut o{nstar, mass, out_index};
    switch (kind) {
    case SweepKind::wrap: return launch_block_t<BLK_WRAP, true>(a, o, cus, max_N, lds_per_wg, st);
    case SweepKind::smax:
        return periodic ? launch_block_t<BLK_SMAX, true>(a, o, cus, max_N, lds_per_wg, st)
                        : launch_block_t<BLK_SMAX, false>(a, o, cus, max_N, lds_per_wg, st);
    default: return periodic ? hipErrorInvalidValue : launch_block_t<BLK_SPAN, false>(a, o, cus, max_N, lds_per_wg, st);
    }
}

}  // namespace nz

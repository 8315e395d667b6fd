// nz_internal.h -- records shared by the host planner (nz_api.cpp) and the
// HIP kernels (nz_kernels.hip).  Not part of the public ABI.
#pragma once
#include <stdint.h>

// Root word of the union-find (one int32 per site, Sec. II.B construction):
//   bit 31 set      -> the site is a cluster root; bits 0..28 hold the cluster
//                      size, bit 30 "a member has x0 = 0", bit 29 "a member has
//                      x0 = L-1";
//   bit 31 clear    -> the value is the index of the site's parent.
// Sizes need 29 bits, hence L <= 55 (55^5 < 2^29).
#define NZ_ROOT 0x80000000u
#define NZ_FLO 0x40000000u
#define NZ_FHI 0x20000000u
#define NZ_FLAGS (NZ_FLO | NZ_FHI)
#define NZ_SIZE 0x1FFFFFFFu

// Per-sample status written by the kernels.
enum {
    NZ_ST_PENDING = 0,
    NZ_ST_DONE = 1,       // n*, mass final
    NZ_ST_BAND = 2,       // the key band ran out before the sample spanned: redo wider
    NZ_ST_BUCKET = 3,     // a band bucket overflowed before the sample spanned: redo finer
    NZ_ST_BACKOFF = 4,    // the prefilled state already spans: redo with a smaller n0
    NZ_ST_PREFIX = 5,     // the prefill list overflowed: redo with a larger list
};

// One row of a (zone mask, L) table: the offsets that share their steps along
// axes 1..4.  stride is the change of the linear site index by those steps.
// code: bit d0 + 2 is set for every step d0 along axis 0 in the row, and for
// each axis j >= 1 bit (5*j + d_j + 2); the row lies inside the lattice iff
// (code & ~allowed(x)) has no bit above 4, where allowed(x) has bit (5*j + d +
// 2) set iff 0 <= x_j + d < L, and its d0 bits inside are code & allowed(x).
// The first half of a table holds one row of every +- pair, the second half
// their negations in the same order (the row without steps along axes 1..4 is
// split by the sign of d0).
struct NzOffset {
    int32_t stride;
    uint32_t code;
};

// Per-sample descriptor (one per sample of a chunk), built by the host.
struct NzSample {
    uint64_t seed;
    uint64_t sample;
    uint64_t T0;          // keys below T0 are occupied before the sweep (0: plain)
    uint64_t off_par;     // byte offsets into the workspace
    uint64_t off_occ;
    uint64_t off_sites;
    uint64_t off_counts;
    uint64_t off_prefix;  // prefilled sites in list order (site order within each key block)
    uint64_t off_parc;    // parents of the list entries during the bulk labelling
    uint64_t off_wrec;    // per bitset word: list position of its first prefilled site, prefilled bits (8 bytes)
    int32_t L;
    int32_t N;
    int32_t nb;           // buckets of the key band [T0, T0 + nb << shift)
    int32_t cap;          // capacity of each bucket (entries)
    int32_t tab;          // first entry of this sample's row table
    int32_t rows;         // number of rows (even)
    int32_t prefix_cap;   // capacity of the prefill site list
    uint32_t shift : 8;     // log2 of the bucket width in key units
    uint32_t sum_shift : 8;
    uint32_t full : 1;      // the band reaches 2^64 (exhaustion then means "never spans")
    uint32_t smax_mode : 1; // 1: track the largest cluster over [win_lo, win_hi) instead of stopping at n*
    uint32_t periodic : 1;  // 1: coordinates wrap mod L (L >= 5); no borders, so no border flags
    uint32_t wrap : 1;      // 1: periodic first-wrap sweep; entries of off_par are 64-bit
                            //    (low half the parent word, high half the x0 displacement
                            //    from the parent)
    uint64_t magic;       // ceil(2^64 / L) for exact division of site indices by L
    uint64_t off_win;     // smax mode: S_max(n) for n in [win_lo, win_hi), uint32 each
    int32_t win_lo;
    int32_t win_hi;
    uint64_t off_sum;     // bitset summary: bit k set unless words k << sum_shift .. are all zero
    // the in-chunk backoffs: threshold and buckets at n0 - b and at n0 - 3b (T0b =
    // 0: not planned)
    uint64_t T0b[2];
    int32_t nbb[2];
    int32_t sum_words;    // 32-bit summary words (0: no summary)
};
// (a chunk of 16384 samples needs that many of them beside its smallest sample)
static_assert(sizeof(NzSample) <= 176, "the chunk header does not grow");

// Consecutive samples of one job in a chunk, as the host plans them; the expand
// kernel writes a descriptor, a queue entry and an output index for each.
struct NzRun {
    NzSample first;       // descriptor of the first sample
    uint64_t stride;      // workspace bytes from one sample to the next
    int32_t count;
    int32_t desc0;        // first descriptor index
    int32_t queue0;       // first place in the sweep's queue
    int32_t list0;        // first place in the prefill list (-1: nothing prefilled)
    int32_t out0;         // first output index
};

// Per-sample result/state record written by the kernels.
struct NzState {
    int32_t status;
    int32_t nstar;
    int32_t mass;
    int32_t n0;           // sites occupied by the prefill (count of keys < T0)
    int32_t smax;         // smax mode: largest cluster of the prefilled state
};

// Launch parameters of the sweep (one persistent launch per chunk).
struct NzSweepArgs {
    const NzSample *desc;
    const int32_t *queue;     // sample indices, longest first
    int32_t nqueue;
    int32_t *qhead;           // work counter, zero at launch
    const NzOffset *tabs;
    uint8_t *ws;
    NzState *state;
    int32_t blk_old;          // earlier roots one block of several sites may touch
    uint32_t map_words;       // LDS words of a workgroup's occupancy map (set by the launcher)
};

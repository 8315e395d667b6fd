// nz_api.cpp -- the C ABI of libnz (include/nz.h): argument checking, the
// neighbourhood tables, the per-sample plan (key band, buckets, prefill),
// workspace layout, chunked launches on one stream and the redo loop for the
// rare samples whose band or bucket ran short or whose prefill already spans.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cstdlib>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <future>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "../../include/nz.h"
#include "nz_internal.h"
#include "nz_launch.h"

#define NZ_API extern "C" __attribute__((visibility("default")))

namespace {

// (a fixed buffer: describing a failed allocation allocates nothing)
thread_local char g_err[512] = "no error";
thread_local int64_t g_stats[6] = {0, 0, 0, 0, 0, 0};
thread_local bool g_timing = false;
thread_local double g_ms[6] = {0, 0, 0, 0, 0, 0};
// per job of the last batch (caller's job order): sequential additions and
// sites occupied by the bulk prefill, summed over the final runs of its samples
thread_local std::vector<int64_t> g_job_serial, g_job_pre;
// bulk-labelling kernels of the last batch: milliseconds in hook, compress and
// the flag pass (summed over dispatches), 0 (no separate expand pass) and the
// number of dispatches
thread_local double g_cc_ms[5] = {0, 0, 0, 0, 0};

// Events around each kernel of the bulk labelling; a chunk launches it once per
// group of samples and for its two in-chunk backoffs.
struct PrefillEvents {
    static constexpr int kSets = 24;
    hipEvent_t ev[kSets][5] = {};
    int used = 0;
    bool ok = false;
    PrefillEvents()
    {
        ok = true;
        for (auto &row : ev)
            for (auto &e : row) ok = ok && hipEventCreate(&e) == hipSuccess;
    }
    ~PrefillEvents()
    {
        for (auto &row : ev)
            for (auto &e : row)
                if (e) (void)hipEventDestroy(e);
    }
};

// Events bracketing the phases of one chunk: clearing (0, 1), keys (2, 3), prefill
// (3, 4), sweep (4, 5).  Between 1 and 2 a group may wait for the other's keys.
struct PhaseEvents {
    hipEvent_t ev[6] = {};
    bool ok = false;
    PhaseEvents()
    {
        ok = true;
        for (auto &e : ev) ok = ok && hipEventCreate(&e) == hipSuccess;
    }
    ~PhaseEvents()
    {
        for (auto &e : ev)
            if (e) (void)hipEventDestroy(e);
    }
};

int fail(int code, const char *fmt, ...)
{
    char buf[sizeof g_err] = "";
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    std::memcpy(g_err, buf, sizeof buf);
    return code;
}

#define HIP_TRY(call)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail(NZ_EDEVICE, "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_),   \
                        __FILE__, __LINE__);                                                 \
    } while (0)

int64_t pow5(int64_t L) { return L * L * L * L * L; }

// ---------------------------------------------------------------------------
// Neighbourhoods (Sec. II.A.2, Table I): zone k is the shell |d|^2 = k of Z^5,
// k = 1..7.  Every shell vector has |d_j| <= 2.  The table lists first the
// vectors whose last non-zero coordinate is negative and then their negations
// in the same order, so its first half holds one vector of every +-d pair.

std::vector<std::array<int, 5>> enumerate_zone_vectors(uint32_t mask)
{
    std::vector<std::array<int, 5>> neg;
    for (int k = 1; k <= 7; ++k) {
        if (!(mask >> (k - 1) & 1u)) continue;
        for (int v = 0; v < 3125; ++v) {
            std::array<int, 5> d;
            int r2 = 0, rem = v;
            for (int j = 0; j < 5; ++j) {
                d[j] = rem % 5 - 2;
                rem /= 5;
                r2 += d[j] * d[j];
            }
            if (r2 != k) continue;
            int last = 0;
            for (int j = 4; j >= 0; --j)
                if (d[j] != 0) {
                    last = d[j];
                    break;
                }
            if (last < 0) neg.push_back(d);
        }
    }
    std::vector<std::array<int, 5>> all = neg;
    for (const auto &d : neg) all.push_back({-d[0], -d[1], -d[2], -d[3], -d[4]});
    return all;
}

// The vectors of every mask 1..127, enumerated once per process (mask 0 and
// masks above 127 give the empty list).
const std::vector<std::array<int, 5>> &zone_vectors(uint32_t mask)
{
    static const std::array<std::vector<std::array<int, 5>>, 128> all = [] {
        std::array<std::vector<std::array<int, 5>>, 128> t;
        for (uint32_t m = 1; m < 128; ++m) t[m] = enumerate_zone_vectors(m);
        return t;
    }();
    return all[mask < 128 ? mask : 0];
}

// z(mask) for every mask, enumerated once.
int coordination(uint32_t mask)
{
    static const std::array<int, 128> z = [] {
        std::array<int, 128> t{};
        for (uint32_t m = 1; m < 128; ++m) t[m] = static_cast<int>(zone_vectors(m).size());
        return t;
    }();
    return mask >= 1 && mask <= 127 ? z[mask] : -1;
}

// A neighbourhood's rows: the vectors that share (d1..d4), with the set of
// their d0 as bits d0 + 2.  First one row of every +- pair (the vectors of the
// first half of the enumeration fall into whole rows, but for the row without
// steps along axes 1..4, of which they are the negative d0), then the negated
// rows in the same order.
struct ZoneRow {
    std::array<int, 4> d;
    uint32_t d0;
};

const std::vector<ZoneRow> &zone_rows(uint32_t mask)
{
    static const std::array<std::vector<ZoneRow>, 128> all = [] {
        std::array<std::vector<ZoneRow>, 128> t;
        for (uint32_t m = 1; m < 128; ++m) {
            const auto &v = zone_vectors(m);
            std::map<std::array<int, 4>, size_t> at;
            for (size_t k = 0; k < v.size() / 2; ++k) {
                const std::array<int, 4> d{v[k][1], v[k][2], v[k][3], v[k][4]};
                auto it = at.find(d);
                if (it == at.end()) {
                    it = at.emplace(d, t[m].size()).first;
                    t[m].push_back({d, 0u});
                }
                t[m][it->second].d0 |= 1u << (v[k][0] + 2);
            }
            const size_t half = t[m].size();
            for (size_t k = 0; k < half; ++k) {
                const ZoneRow r = t[m][k];
                uint32_t mirror = 0;
                for (int j = 0; j < 5; ++j)
                    if (r.d0 >> j & 1u) mirror |= 1u << (4 - j);
                t[m].push_back({{-r.d[0], -r.d[1], -r.d[2], -r.d[3]}, mirror});
            }
        }
        return t;
    }();
    return all[mask < 128 ? mask : 0];
}

std::vector<NzOffset> build_table(uint32_t mask, int32_t L)
{
    std::vector<NzOffset> t;
    for (const auto &r : zone_rows(mask)) {
        NzOffset o;
        int64_t stride = 0, p = L;
        uint32_t code = r.d0;
        for (int j = 1; j < 5; ++j) {
            stride += r.d[j - 1] * p;
            p *= L;
            code |= 1u << (5 * j + r.d[j - 1] + 2);
        }
        o.stride = static_cast<int32_t>(stride);
        o.code = code;
        t.push_back(o);
    }
    return t;
}

// ---------------------------------------------------------------------------
// Device facts.

struct Device {
    int id = -1;
    int cus = 256;
    size_t lds_per_block = 65536;
};

int device_info(Device &dev)
{
    int id = 0;
    HIP_TRY(hipGetDevice(&id));
    // one cache for the process (the two-group path queries from a second thread)
    static std::mutex lock;
    static std::map<int, Device> cache;
    {
        std::lock_guard<std::mutex> g(lock);
        auto it = cache.find(id);
        if (it != cache.end()) {
            dev = it->second;
            return NZ_OK;
        }
    }
    hipDeviceProp_t p;
    HIP_TRY(hipGetDeviceProperties(&p, id));
    dev.id = id;
    dev.cus = p.multiProcessorCount;
    dev.lds_per_block = p.sharedMemPerBlock;
    int optin = 0;
    if (hipDeviceGetAttribute(&optin, hipDeviceAttributeSharedMemPerBlockOptin, id) == hipSuccess && optin > 0)
        dev.lds_per_block = std::max(dev.lds_per_block, static_cast<size_t>(optin));
    std::lock_guard<std::mutex> g(lock);
    cache[id] = dev;
    return NZ_OK;
}

// ---------------------------------------------------------------------------
// Per-sample plan.

constexpr int kMaxChunk = 16384;
constexpr size_t kAlign = 256;

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Threshold coefficient of p_c = c / (z + b) fitted over Table I (Sec. III.B:
// c ~ 1.553, b ~ 1.01); used only to size key bands and to order work.
double pc_prior(int z) { return 1.553 / (z + 1.01); }

// 32-bit words of a sample's bitset summary
constexpr int64_t kSumWords = 1024;
// LDS words per wave that the accepted LDS residencies are sized with
constexpr size_t kResWords = 896;
struct Plan {
    int32_t job;
    int64_t sample;      // Philox sample index
    int32_t out;         // index into the caller's output arrays
    int32_t L;
    uint32_t mask;
    int64_t n0;          // current prefill rank (0: plain)
    int64_t backoff;     // backoff step still available (0: next backoff goes to 0)
    int64_t band_hi;     // upper end of the key band in sites
    int32_t shift_adj;   // extra halvings of the bucket width
    int32_t prefix_mul;  // prefill list capacity multiplier
    double prio;
    int64_t win_lo, win_hi;   // smax mode: S_max(n) for n in [win_lo, win_hi) (win_hi = 0: off)
    bool wrap;           // periodic first-wrap sample (64-bit union-find entries)
    bool per;            // periodic coordinates (first-wrap or largest-cluster windows)
};

uint64_t rank_to_key(int64_t n, int64_t N)
{
    // floor(n / N * 2^64) for 0 <= n < N
    unsigned __int128 v = (static_cast<unsigned __int128>(static_cast<uint64_t>(n)) << 64) / static_cast<uint64_t>(N);
    return static_cast<uint64_t>(v);
}

// Prefill key threshold for rank n: rank_to_key rounded down to a multiple of
// 2^32, so that the keys kernel tests keys against it (and against the band's
// end, a whole number of buckets of at least 2^32 keys above it) by their high
// words.  The prefill is whatever lies below the threshold: n* and the mass
// never depend on it, and the rounding moves it by under N / 2^32 sites.
uint64_t prefill_key(int64_t n, int64_t N)
{
    // test hook: the unrounded threshold drives the keys kernel's 64-bit compares
    if (getenv("NZ_DEBUG_EXACT_T0")) return rank_to_key(n, N);
    const uint64_t t = rank_to_key(n, N) & ~0xFFFFFFFFull;
    return t != 0 ? t : rank_to_key(n, N);   // (n >= 1 and N < 2^32 keep it nonzero)
}

struct Sizes {
    uint64_t T0;
    int32_t nb, cap, shift, full, prefix_cap;
    // prefill ranks of the backoffs resolved inside the chunk: n0 - b, then
    // n0 - 3b (0: none planned), their key thresholds and band buckets
    int64_t n0b[2];
    uint64_t T0b[2];
    int32_t nbb[2];
    size_t par, occ, sites, counts, prefix, parc, wrec, win, sum, total;
    int32_t sum_shift, sum_words;
};

Sizes plan_sizes(const Plan &p, int bucket_log2)
{
    Sizes s{};
    const int64_t N = pow5(p.L);
    s.T0 = p.n0 > 0 ? prefill_key(p.n0, N) : 0;
    int lgN = 0;
    while ((int64_t(1) << lgN) < N) ++lgN;
    int shift = 64 + bucket_log2 - lgN - p.shift_adj;
    shift = std::max(1, std::min(63, shift));
    s.shift = shift;
    s.full = p.band_hi >= N ? 1 : 0;
    const uint64_t Thi = s.full ? 0 : rank_to_key(std::max<int64_t>(p.band_hi, p.n0 + 1), N);
    // buckets of width 2^shift covering [T, Thi) (or [T, 2^64) for a full band)
    auto buckets = [&](uint64_t T) {
        const unsigned __int128 top = s.full ? (static_cast<unsigned __int128>(1) << 64) : Thi;
        const unsigned __int128 span = top > T ? top - T : 1;
        const unsigned __int128 w = static_cast<unsigned __int128>(1) << shift;
        return static_cast<int32_t>(std::max<unsigned __int128>(1, (span + w - 1) / w));
    };
    s.nb = buckets(s.T0);
    // two backoffs are resolved inside the chunk, so the band region is sized
    // for the backed-off bands as well
    s.n0b[0] = (p.n0 > 0 && p.backoff > 0 && p.n0 - p.backoff > 0) ? p.n0 - p.backoff : 0;
    s.n0b[1] = (s.n0b[0] > 0 && s.n0b[0] - 2 * p.backoff > 0) ? s.n0b[0] - 2 * p.backoff : 0;
    int32_t nb_alloc = s.nb;
    for (int l = 0; l < 2; ++l) {
        s.T0b[l] = s.n0b[l] > 0 ? prefill_key(s.n0b[l], N) : 0;
        s.nbb[l] = s.n0b[l] > 0 ? buckets(s.T0b[l]) : 0;
        nb_alloc = std::max(nb_alloc, s.nbb[l]);
    }
    const double mean = std::ldexp(static_cast<double>(N), shift - 64);
    int cap = static_cast<int>(std::ceil(mean + 8.0 * std::sqrt(mean) + 16.0));
    cap = (cap + 15) / 16 * 16;
    s.cap = std::max(16, std::min(cap, 4096));
    // test hooks: tiny buckets / prefill lists force the redo paths
    if (const char *e = getenv("NZ_DEBUG_BUCKET_CAP")) s.cap = std::max(1, std::min(4096, atoi(e)));
    if (p.n0 > 0) {
        const double e = static_cast<double>(p.n0);
        double want = e + 8.0 * std::sqrt(e) + 64.0;
        if (const char *dbg = getenv("NZ_DEBUG_PREFIX_CAP")) want = std::max(1, atoi(dbg));
        s.prefix_cap = static_cast<int32_t>(std::min<double>(static_cast<double>(N), want * p.prefix_mul));
    } else {
        s.prefix_cap = 0;
    }
    s.par = align_up(static_cast<size_t>(N) * (p.wrap ? 8 : 4));
    s.occ = align_up(static_cast<size_t>((N + 63) / 64) * 8);
    s.sites = align_up(static_cast<size_t>(nb_alloc) * s.cap * 4);
    s.counts = align_up(static_cast<size_t>(nb_alloc) * 4);
    s.prefix = align_up(static_cast<size_t>(s.prefix_cap) * 4);
    // the bulk labelling's list forest and word records (not for periodic
    // first-wrap samples, whose labelling runs on the lattice entries)
    s.parc = p.wrap ? 0 : align_up(static_cast<size_t>(s.prefix_cap) * 4);
    s.wrec = (p.wrap || s.prefix_cap == 0) ? 0 : 2 * s.occ;
    s.win = p.win_hi > 0 ? align_up(static_cast<size_t>(p.win_hi - p.win_lo) * 4) : 0;
    // bitset summary for the hook of sparse prefills: at most kSumWords words, one
    // bit per 1..16 bitset words (none above that: L > 27, or first-wrap samples)
    {
        const int64_t words = (N + 63) / 64 * 2;
        int gs = 0;
        while (((words >> gs) + 31) / 32 > kSumWords) ++gs;
        s.sum_shift = gs;
        s.sum_words = (gs <= 4 && !p.wrap) ? static_cast<int32_t>(((words >> gs) + 31) / 32 + 1) : 0;
        s.sum = align_up(static_cast<size_t>(s.sum_words) * 4);
    }
    s.total = s.par + s.occ + s.sites + s.counts + s.prefix + s.parc + s.wrec + s.win + s.sum;
    return s;
}

// The plan without its prefill.
Plan plain_plan(Plan p)
{
    p.n0 = p.backoff = 0;
    return p;
}

// The smallest workspace region that runs a sample of plan p.  A prefilled sample
// holds an 8-byte record per bitset word; one that would fit with 4 bytes each is
// swept plainly where it does not fit with 8 (L = 36 in 256 MiB, for instance).
// Only the time and the backoff count depend on that.
size_t smallest_bytes(const Plan &p, int bucket_log2)
{
    const Sizes s = plan_sizes(p, bucket_log2);
    if (s.wrec == 0) return s.total;
    return std::min(s.total, std::max(s.total - s.wrec / 2, plan_sizes(plain_plan(p), bucket_log2).total));
}

// How the keys launch of a sample (its Sizes) spreads, by the share of the
// sites that its band holds: above 3% one workgroup per sample, if there are
// enough samples (launch_keys); above 8% and with too many buckets for that, each
// sample's workgroups on one XCD, from kXcdSamples samples on (fewer would leave
// XCDs idle).  Both sides of each line are measured at the keys kernels.
constexpr int32_t kXcdSamples = 32;
enum { KEYS_NARROW = 0, KEYS_WIDE = 1, KEYS_WIDEST = 2 };
int keys_class(const Sizes &s)
{
    const double share = std::ldexp(static_cast<double>(s.nb), s.shift - 64);
    return share > 0.08 ? KEYS_WIDEST : share > 0.03 ? KEYS_WIDE : KEYS_NARROW;
}

// Samples whose prefill lists hold like numbers of sites (within a factor of
// four) are labelled by one launch: its grid has as many workgroups per sample
// as the first list needs, that of the samples that come first in the queue
// (7 compact neighbourhoods x 1000 of L = 8 1.39 ms; as the mean list needs 1.44,
// as the longest 1.48; longer ones take more passes), and in one launch over lists
// of 2000 and 150000 sites most workgroups would find nothing to do.  An empty
// workgroup costs some 4 ns, a group's three launches some 20 us (the L = 12
// periodic batch of 700 samples: 2.03 ms in groups, 1.75 in one launch), so a class
// joins the group before it unless that adds more than kEmptyWgs empty workgroups.
constexpr int64_t kEmptyWgs = 4096;
int prefill_group(int32_t prefix_cap)
{
    int g = 0;
    while (prefix_cap > 1024) {
        prefix_cap >>= 2;
        ++g;
    }
    return g;
}

int64_t default_band_hi(int32_t L, uint32_t mask, int64_t n0)
{
    const int64_t N = pow5(L);
    if (N <= 8192) return N;
    const int z = coordination(mask);
    const double frac = pc_prior(z) * (1.0 + 4.0 / std::sqrt(static_cast<double>(L)));
    int64_t hi = static_cast<int64_t>(frac * N) + 4096;
    hi = std::max(hi, n0 + 4096);
    return std::min(hi, N);
}

size_t header_bytes(size_t table_entries, int32_t chunk)
{
    return align_up(table_entries * sizeof(NzOffset)) + align_up(chunk * sizeof(NzSample)) +
           align_up(chunk * sizeof(NzState)) + 3 * align_up(chunk * sizeof(int32_t)) + kAlign;
}

struct Tune {
    int residency = 0;
    int wg_waves = 0;
    int bucket_log2 = 7;   // mean keys per band bucket: 64..128 (a block of the sweep takes whole buckets)
    int sweep_mode = 0;
    int split_z = 0;     // widest neighbourhood of the first of two groups side by side (0: kSplitZ)
};

int check_job(const nz_job &j, int idx)
{
    if (j.L < 1 || j.L > 55) return fail(j.L < 1 ? NZ_EINVAL : NZ_EUNSUPPORTED, "job %d: L = %d outside [1, 55]", idx, j.L);
    if (j.zone_mask < 1 || j.zone_mask > 127) return fail(NZ_EINVAL, "job %d: zone_mask %u outside [1, 127]", idx, j.zone_mask);
    if (j.boundary != NZ_FREE && j.boundary != NZ_PERIODIC)
        return fail(NZ_EINVAL, "job %d: boundary %d is neither NZ_FREE nor NZ_PERIODIC", idx, j.boundary);
    if (j.boundary == NZ_PERIODIC && j.L < 5)
        return fail(NZ_EUNSUPPORTED, "job %d: periodic boundaries need L >= 5", idx);
    if (j.nsamples < 0) return fail(NZ_EINVAL, "job %d: nsamples < 0", idx);
    if (j.sample0 < 0) return fail(NZ_EINVAL, "job %d: sample0 < 0", idx);
    const int64_t N = pow5(j.L);
    if (j.n0 < -1 || j.n0 >= N) return fail(NZ_EINVAL, "job %d: n0 = %lld outside [-1, N-1]", idx, (long long)j.n0);
    if (j.backoff < 0) return fail(NZ_EINVAL, "job %d: backoff < 0", idx);
    if (j.band_hi < 0) return fail(NZ_EINVAL, "job %d: band_hi < 0", idx);
    return NZ_OK;
}

int read_tune(const nz_tuning *t, Tune &out)
{
    out = Tune{};
    if (!t) return NZ_OK;
    if (t->residency < 0 || t->residency > 3) return fail(NZ_EINVAL, "tuning: residency %d outside [0, 3]", t->residency);
    if (t->wg_waves < 0 || t->wg_waves > 4) return fail(NZ_EINVAL, "tuning: wg_waves %d outside [0, 4]", t->wg_waves);
    if (t->waves_per_simd < 0 || t->waves_per_simd > 8)
        return fail(NZ_EINVAL, "tuning: waves_per_simd %d outside [0, 8]", t->waves_per_simd);
    if (t->bucket_log2 != 0 && (t->bucket_log2 < 4 || t->bucket_log2 > 10))
        return fail(NZ_EINVAL, "tuning: bucket_log2 %d outside [4, 10]", t->bucket_log2);
    if (t->sweep_mode < 0 || t->sweep_mode > 2) return fail(NZ_EINVAL, "tuning: sweep_mode %d outside [0, 2]", t->sweep_mode);
    out.sweep_mode = t->sweep_mode;
    if (t->summary < 0 || t->summary > 2) return fail(NZ_EINVAL, "tuning: summary %d outside [0, 2]", t->summary);
    if (t->split_z != 0 && (t->split_z < 10 || t->split_z > 892))
        return fail(NZ_EINVAL, "tuning: split_z %d outside [10, 892]", t->split_z);
    out.split_z = t->split_z;
    out.residency = t->residency;
    out.wg_waves = t->wg_waves;
    // (a bucket is part of one block of the sweep: at most 128 keys on average)
    if (t->bucket_log2) out.bucket_log2 = std::min(t->bucket_log2, 7);
    return NZ_OK;
}

// Debug override of the earlier roots one block may touch (tests force the
// block sweep's one-site-at-a-time fallback).
int env_blk_old()
{
    const char *e = getenv("NZ_DEBUG_BLOCK_OLD");
    if (!e) return 1 << 30;
    return std::max(0, atoi(e));
}

// ---------------------------------------------------------------------------
// The batch engine.

struct TablePool {
    std::map<std::pair<uint32_t, int32_t>, int32_t> index;
    std::vector<NzOffset> entries;
    int32_t get(uint32_t mask, int32_t L, int32_t *rows)
    {
        *rows = static_cast<int32_t>(zone_rows(mask).size());
        auto key = std::make_pair(mask, L);
        auto it = index.find(key);
        if (it != index.end()) return it->second;
        auto t = build_table(mask, L);
        const int32_t at = static_cast<int32_t>(entries.size());
        entries.insert(entries.end(), t.begin(), t.end());
        index[key] = at;
        return at;
    }
};

// smax mode of a whole batch: every sample records S_max(n) for n in
// [win_lo, win_hi) and the chunks add the windows of their samples into out.
struct SmaxReq {
    int64_t win_lo, win_hi;
    uint64_t *d_out;
};

// Consecutive samples of one job with one plan: p is the first sample's.
struct Run {
    Plan p;
    int64_t count;
};

// The run goes on with a sample of plan p (its successor, planned the same).
bool follows(const Run &r, const Plan &p)
{
    return p.job == r.p.job && p.sample == r.p.sample + r.count && p.out == r.p.out + r.count && p.n0 == r.p.n0 &&
           p.backoff == r.p.backoff && p.band_hi == r.p.band_hi && p.shift_adj == r.p.shift_adj && p.prefix_mul == r.p.prefix_mul;
}

// A run's samples in one chunk.
struct Part {
    Plan p;
    Sizes s;
    int32_t count, desc0, queue0, list0;
    size_t off;
};

NzRun make_run(const Part &part, const nz_job *jobs, TablePool &pool)
{
    const Plan &p = part.p;
    const Sizes &s = part.s;
    NzRun r;
    std::memset(&r, 0, sizeof r);
    NzSample &d = r.first;
    d.seed = jobs[p.job].seed;
    d.sample = static_cast<uint64_t>(p.sample);
    d.T0 = s.T0;
    d.L = p.L;
    d.N = static_cast<int32_t>(pow5(p.L));
    d.nb = s.nb;
    d.cap = s.cap;
    d.shift = s.shift;
    d.full = s.full;
    d.prefix_cap = s.prefix_cap;
    d.tab = pool.get(p.mask, p.L, &d.rows);
    d.magic = p.L == 1 ? 0 : static_cast<uint64_t>(~0ull / static_cast<uint64_t>(p.L) + 1ull);
    size_t off = part.off;
    d.off_par = off; off += s.par;
    d.off_occ = off; off += s.occ;
    d.off_sites = off; off += s.sites;
    d.off_counts = off; off += s.counts;
    d.off_prefix = off; off += s.prefix;
    d.off_parc = off; off += s.parc;
    d.off_wrec = off; off += s.wrec;
    d.off_sum = off; off += s.sum;
    d.sum_shift = s.sum_shift;
    d.sum_words = s.sum_words;
    d.off_win = off; off += s.win;
    d.smax_mode = p.win_hi > 0 ? 1 : 0;
    d.win_lo = static_cast<int32_t>(p.win_lo);
    d.win_hi = static_cast<int32_t>(p.win_hi);
    d.periodic = p.per ? 1 : 0;
    d.wrap = p.wrap ? 1 : 0;
    for (int lv = 0; lv < 2; ++lv) {
        d.T0b[lv] = s.T0b[lv];
        d.nbb[lv] = s.nbb[lv];
    }
    r.stride = s.total;
    r.count = part.count;
    r.desc0 = part.desc0;
    r.queue0 = part.queue0;
    r.list0 = part.list0;
    r.out0 = p.out;
    return r;
}
static_assert(sizeof(NzRun) <= 4 * kAlign, "a run fits the region of the smallest sample (par, occ, sites, counts)");

// The order of the first keys passes of two groups side by side: the second
// group's stream waits for the first group's event.
struct KeysTurn {
    hipEvent_t done = nullptr;
    bool second = false;
    std::shared_future<void> recorded;    // second: set once the event is recorded, or never will be
    std::promise<void> *record = nullptr; // first

    // before / after the stream's first keys pass
    hipError_t before(hipStream_t st)
    {
        if (!second || !recorded.valid()) return hipSuccess;
        recorded.wait();
        recorded = {};
        return hipStreamWaitEvent(st, done, 0);
    }
    hipError_t after(hipStream_t st)
    {
        if (second || !record) return hipSuccess;
        const hipError_t e = hipEventRecord(done, st);
        pass();
        return e;
    }
    void pass()
    {
        if (record) record->set_value();
        record = nullptr;
    }
};

// Whether the labelling takes the hook of sparse lists.
bool hook_map(const Part &part) { return !part.p.wrap && nz::hook_map_fits(pow5(part.p.L), part.s.prefix_cap); }

// job_out (may be NULL): first output index of every job (default: the
// samples of the jobs in order, from 0).
int run_batch(const nz_job *jobs, int32_t njobs, uint8_t *ws, size_t ws_bytes, int32_t *d_nstar, int32_t *d_mass,
              int32_t *h_backoffs, const Tune &tune, hipStream_t st, const SmaxReq *smax = nullptr,
              const int64_t *job_out = nullptr, KeysTurn *turn = nullptr)
{
    Device dev;
    if (int rc = device_info(dev)) return rc;
    for (int k = 0; k < 6; ++k) g_stats[k] = 0;
    for (int k = 0; k < 6; ++k) g_ms[k] = 0.0;
    for (int k = 0; k < 5; ++k) g_cc_ms[k] = 0.0;
    g_job_serial.assign(static_cast<size_t>(std::max(njobs, 0)), 0);
    g_job_pre.assign(static_cast<size_t>(std::max(njobs, 0)), 0);
    if (h_backoffs)
        for (int j = 0; j < njobs; ++j) h_backoffs[j] = 0;

    // tables for every (mask, L) of the batch live at the start of the workspace
    TablePool pool;
    std::vector<Run> todo;
    std::vector<std::vector<int32_t>> lists;   // host lists whose copies may be under way
    int64_t out = 0, left = 0;   // left: samples in todo
    for (int j = 0; j < njobs; ++j) {
        const nz_job &J = jobs[j];
        int32_t rows = 0;
        pool.get(J.zone_mask, J.L, &rows);
        const int z = coordination(J.zone_mask);
        const int64_t N = pow5(J.L);
        if (J.nsamples <= 0) continue;
        Run run{};
        Plan &p = run.p;
        p.job = j;
        p.sample = J.sample0;
        p.out = static_cast<int32_t>(job_out ? job_out[j] : out);
        p.L = J.L;
        p.mask = J.zone_mask;
        p.n0 = J.n0 > 0 ? J.n0 : 0;
        p.backoff = J.backoff;
        p.band_hi = J.band_hi > 0 ? std::min<int64_t>(J.band_hi, N) : default_band_hi(J.L, J.zone_mask, p.n0);
        if (p.band_hi <= p.n0) p.band_hi = std::min<int64_t>(N, p.n0 + 4096);
        p.shift_adj = 0;
        p.prefix_mul = 1;
        p.prio = J.prio > 0 ? J.prio : static_cast<double>(std::max<int64_t>(1, p.band_hi - p.n0)) * (1.0 + z / 64.0);
        p.win_lo = smax ? smax->win_lo : 0;
        p.win_hi = smax ? smax->win_hi : 0;
        p.per = J.boundary == NZ_PERIODIC;
        p.wrap = p.per && !smax;
        run.count = J.nsamples;
        out += J.nsamples;
        left += J.nsamples;
        todo.push_back(run);
    }
    if (out > 0x7FFFFFFF || (job_out && njobs > 0 && job_out[njobs - 1] + jobs[njobs - 1].nsamples > 0x7FFFFFFF))
        return fail(NZ_EINVAL, "too many samples in one batch");
    const size_t tab_bytes = align_up(pool.entries.size() * sizeof(NzOffset));
    bool tabs_there = false;

    int rounds = 0;
    while (!todo.empty()) {
        if (++rounds > 64) return fail(NZ_EDEVICE, "samples still unfinished after 64 redo rounds");
        // free-boundary samples first, then the periodic ones: a chunk holds one
        // boundary condition only, since the sweep is compiled for each
        std::stable_sort(todo.begin(), todo.end(), [](const Run &a, const Run &b) {
            return a.p.per != b.p.per ? b.p.per : a.p.prio > b.p.prio;
        });
        std::vector<Run> redo;
        int64_t redo_left = 0;
        size_t pos = 0;
        while (pos < todo.size()) {
            // ---- form a chunk: longest first, as many as the workspace holds
            const int32_t cmax = static_cast<int32_t>(std::min<int64_t>(kMaxChunk, left));
            const size_t head = header_bytes(pool.entries.size(), cmax);
            if (head >= ws_bytes) return fail(NZ_EWORKSPACE, "workspace of %zu bytes is smaller than the %zu-byte header", ws_bytes, head);
            std::vector<Part> parts;   // in queue order
            int32_t n = 0;
            size_t used = head;
            while (pos < todo.size() && n < cmax) {
                Run &run = todo[pos];
                if (!parts.empty() && run.p.per != parts.front().p.per) break;
                Part part{};
                part.p = run.p;
                part.s = plan_sizes(run.p, tune.bucket_log2);
                part.count = static_cast<int32_t>(std::min<int64_t>({run.count, cmax - n, static_cast<int64_t>((ws_bytes - used) / part.s.total)}));
                if (part.count <= 0) {
                    if (!parts.empty() || run.p.n0 == 0 || used + smallest_bytes(run.p, tune.bucket_log2) > ws_bytes) break;
                    run.p = plain_plan(run.p);   // (not one sample fits with its prefill)
                    continue;
                }
                part.queue0 = n;
                used += part.s.total * static_cast<size_t>(part.count);
                n += part.count;
                run.p.sample += part.count;
                run.p.out += part.count;
                run.count -= part.count;
                parts.push_back(part);
                if (run.count > 0) break;   // the chunk is full
                ++pos;
            }
            if (parts.empty()) {
                Sizes s = plan_sizes(todo[pos].p, tune.bucket_log2);
                return fail(NZ_EWORKSPACE, "workspace of %zu bytes cannot hold one sample (needs %zu)", ws_bytes, head + s.total);
            }
            left -= n;
            ++g_stats[0];
            const bool wrap_chunk = parts.front().p.wrap;
            const bool per_chunk = parts.front().p.per;

            // ---- descriptors, grouped by L and band width for the keys launches
            const int32_t np = static_cast<int32_t>(parts.size());
            std::vector<int32_t> order(np);   // parts in descriptor order
            for (int32_t i = 0; i < np; ++i) order[i] = i;
            std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
                if (parts[a].p.L != parts[b].p.L) return parts[a].p.L < parts[b].p.L;
                return keys_class(parts[a].s) > keys_class(parts[b].s);
            });
            size_t off = head;
            uint32_t max_N = 0;
            int32_t max_count = 0, di = 0;
            for (int32_t i : order) {
                Part &part = parts[i];
                part.desc0 = di;
                part.off = off;
                di += part.count;
                off += part.s.total * static_cast<size_t>(part.count);
                max_N = std::max(max_N, static_cast<uint32_t>(pow5(part.p.L)));
                max_count = std::max(max_count, part.count);
            }
            // the prefilled parts, in groups of like prefill sizes for the labelling
            std::vector<int32_t> pre;
            for (int32_t i : order)
                if (parts[i].s.T0 != 0) pre.push_back(i);
            std::stable_sort(pre.begin(), pre.end(), [&](int32_t a, int32_t b) {
                if (hook_map(parts[a]) != hook_map(parts[b])) return hook_map(parts[b]);
                return prefill_group(parts[a].s.prefix_cap) > prefill_group(parts[b].s.prefix_cap);
            });
            int32_t nlist = 0;
            for (Part &part : parts) part.list0 = -1;
            for (int32_t i : pre) {
                parts[i].list0 = nlist;
                nlist += parts[i].count;
            }
            std::vector<NzRun> runs;
            runs.reserve(parts.size());
            for (int32_t i : order) runs.push_back(make_run(parts[i], jobs, pool));

            // ---- header layout
            uint8_t *h = ws;
            NzOffset *d_tabs = reinterpret_cast<NzOffset *>(h);
            h += tab_bytes;
            NzSample *d_desc = reinterpret_cast<NzSample *>(h);
            h += align_up(cmax * sizeof(NzSample));
            NzState *d_state = reinterpret_cast<NzState *>(h);
            h += align_up(cmax * sizeof(NzState));
            int32_t *d_queue = reinterpret_cast<int32_t *>(h);
            h += align_up(cmax * sizeof(int32_t));
            int32_t *d_outidx = reinterpret_cast<int32_t *>(h);
            h += align_up(cmax * sizeof(int32_t));
            int32_t *d_list = reinterpret_cast<int32_t *>(h);
            h += align_up(cmax * sizeof(int32_t));
            int32_t *d_qhead = reinterpret_cast<int32_t *>(h);
            // the runs pass through the samples' own region, which nothing uses
            // before they are expanded (every sample's is larger than a run)
            NzRun *d_runs = reinterpret_cast<NzRun *>(ws + head);

            if (!tabs_there) {
                HIP_TRY(hipMemcpyAsync(d_tabs, pool.entries.data(), pool.entries.size() * sizeof(NzOffset), hipMemcpyHostToDevice, st));
                tabs_there = true;
            }
            HIP_TRY(hipMemcpyAsync(d_runs, runs.data(), runs.size() * sizeof(NzRun), hipMemcpyHostToDevice, st));
            HIP_TRY(nz::launch_expand(d_runs, np, max_count, d_desc, d_state, d_queue, d_outidx, d_list, d_qhead, st));

            // ---- launches
            PhaseEvents *pe = nullptr;
            PrefillEvents *pfe = nullptr;
            if (g_timing) {
                static thread_local PhaseEvents events;   // released when the thread ends
                static thread_local PrefillEvents pevents;
                if (events.ok) pe = &events;
                if (pevents.ok) {
                    pfe = &pevents;
                    pfe->used = 0;
                }
            }
            auto prefill_events = [&]() -> hipEvent_t * {
                return pfe && pfe->used < PrefillEvents::kSets ? pfe->ev[pfe->used++] : nullptr;
            };
            if (pe) HIP_TRY(hipEventRecord(pe->ev[0], st));
            HIP_TRY(nz::launch_clear(d_desc, nullptr, n, 0, ws, d_state, st));
            if (pe) HIP_TRY(hipEventRecord(pe->ev[1], st));
            if (turn) HIP_TRY(turn->before(st));
            if (pe) HIP_TRY(hipEventRecord(pe->ev[2], st));
            for (int32_t a = 0; a < np;) {
                const Part &first = parts[order[a]];
                const int cls = keys_class(first.s);
                int32_t b = a, count = 0, max_nb = 0;
                while (b < np && parts[order[b]].p.L == first.p.L && keys_class(parts[order[b]].s) == cls) {
                    max_nb = std::max(max_nb, parts[order[b]].s.nb);
                    count += parts[order[b++]].count;
                }
                HIP_TRY(nz::launch_keys(d_desc, nullptr, first.desc0, count, static_cast<int32_t>(pow5(first.p.L)), ws, d_state,
                                        cls == KEYS_WIDEST && count >= kXcdSamples, cls == KEYS_NARROW ? 0 : max_nb, st));
                a = b;
            }
            if (turn) HIP_TRY(turn->after(st));
            if (pe) HIP_TRY(hipEventRecord(pe->ev[3], st));
            std::vector<NzState> state(n);
            std::vector<uint8_t> level(n, 0);   // in-chunk backoffs of every sample
            if (nlist > 0) {
                for (size_t g = 0; g < pre.size();) {
                    const bool map = hook_map(parts[pre[g]]);
                    const int32_t grid = parts[pre[g]].s.prefix_cap;
                    int32_t count = 0, map_N = 0, most = 0;
                    size_t e = g;
                    while (e < pre.size() && hook_map(parts[pre[e]]) == map) {
                        // the samples of one size class (in no order within it), if a
                        // launch of their own saves enough empty workgroups
                        size_t c = e;
                        int32_t samples = 0, largest = 0;
                        const int cls = prefill_group(parts[pre[e]].s.prefix_cap);
                        int32_t N = 0;
                        while (c < pre.size() && hook_map(parts[pre[c]]) == map && prefill_group(parts[pre[c]].s.prefix_cap) == cls) {
                            N = std::max(N, static_cast<int32_t>(pow5(parts[pre[c]].p.L)));
                            largest = std::max(largest, parts[pre[c]].s.prefix_cap);
                            samples += parts[pre[c++]].count;
                        }
                        const int64_t empty = static_cast<int64_t>(samples) * (grid - parts[pre[e]].s.prefix_cap) / 1024;
                        if (e > g && empty > kEmptyWgs) break;
                        most = std::max(most, largest);
                        count += samples;
                        if (map) map_N = std::max(map_N, N);
                        e = c;
                    }
                    HIP_TRY(nz::launch_prefill(d_desc, d_list + parts[pre[g]].list0, count, most, grid, d_tabs, ws, d_state,
                                               smax != nullptr, wrap_chunk, per_chunk, map_N, dev.cus, st, prefill_events()));
                    g = e;
                }
                // Resolve backoffs inside the chunk: samples whose bulk state already
                // spans are re-keyed and re-labelled from n0 - b, and if that spans
                // too from n0 - 3b, so they join this chunk's sweep instead of a
                // later redo round.
                for (int lv = 0; lv < 2; ++lv) {
                    HIP_TRY(hipMemcpyAsync(state.data(), d_state, n * sizeof(NzState), hipMemcpyDeviceToHost, st));
                    HIP_TRY(hipStreamSynchronize(st));
                    std::vector<int32_t> again;        // descriptors, by L (the order of `order`)
                    std::vector<std::pair<int32_t, int32_t>> sizes;   // (N, count) of every L among them
                    int32_t max_prefix = 0, map_N = 1;
                    for (int32_t i : order) {
                        const Part &part = parts[i];
                        if (part.s.T0b[lv] == 0) continue;   // not planned: the redo round takes it
                        const int32_t N = static_cast<int32_t>(pow5(part.p.L));
                        for (int32_t k = part.desc0; k < part.desc0 + part.count; ++k) {
                            if (state[k].status != NZ_ST_BACKOFF) continue;
                            ++g_stats[3];
                            if (h_backoffs) ++h_backoffs[part.p.job];
                            level[k] = static_cast<uint8_t>(lv + 1);
                            again.push_back(k);
                            if (sizes.empty() || sizes.back().first != N) sizes.emplace_back(N, 0);
                            ++sizes.back().second;
                            max_prefix = std::max(max_prefix, part.s.prefix_cap);
                            map_N = map_N > 0 && hook_map(part) ? std::max(map_N, N) : 0;
                        }
                    }
                    if (again.empty()) break;
                    const int32_t na = static_cast<int32_t>(again.size());
                    HIP_TRY(hipMemcpyAsync(d_list, again.data(), na * sizeof(int32_t), hipMemcpyHostToDevice, st));
                    HIP_TRY(nz::launch_clear(d_desc, d_list, na, lv, ws, d_state, st));
                    int32_t a = 0;
                    for (const auto &e : sizes) {
                        HIP_TRY(nz::launch_keys(d_desc, d_list, a, e.second, e.first, ws, d_state, false, 0, st));
                        a += e.second;
                    }
                    HIP_TRY(nz::launch_prefill(d_desc, d_list, na, max_prefix, max_prefix, d_tabs, ws, d_state, smax != nullptr,
                                               wrap_chunk, per_chunk, map_N, dev.cus, st, prefill_events()));
                    // (`again` stays untouched until the copy has been read: the next
                    // pass synchronises first, and so does the end of the chunk)
                    lists.push_back(std::move(again));
                }
            }
            if (pe) HIP_TRY(hipEventRecord(pe->ev[4], st));

            {
                // The LDS residencies are accepted where the state they name fits a
                // workgroup's LDS (kResWords: the per-wave tables that went with it);
                // the sweep keeps its state in HBM and its tables in LDS.
                if (!wrap_chunk && tune.residency != 0 && tune.residency != 2) {
                    const size_t occ_words = (static_cast<size_t>(max_N) + 63) / 64 * 2;
                    const size_t words = occ_words + (tune.residency == 3 ? max_N : 0) + (per_chunk || tune.sweep_mode == 1 ? 0 : kResWords);
                    const size_t need = words * 4 * static_cast<size_t>(tune.wg_waves ? tune.wg_waves : 1);
                    if (need > dev.lds_per_block)
                        return fail(NZ_EUNSUPPORTED, "residency %d needs %zu bytes of LDS per workgroup; the device allows %zu",
                                    tune.residency, need, dev.lds_per_block);
                }
                NzSweepArgs args{};
                args.desc = d_desc;
                args.queue = d_queue;
                args.nqueue = n;
                args.qhead = d_qhead;
                args.tabs = d_tabs;
                args.ws = ws;
                args.state = d_state;
                args.blk_old = env_blk_old();
                HIP_TRY(nz::launch_sweep(wrap_chunk ? nz::SweepKind::wrap : (smax ? nz::SweepKind::smax : nz::SweepKind::span),
                                         per_chunk, args, d_nstar, d_mass, d_outidx, dev.cus, max_N, dev.lds_per_block, st));
            }
            if (smax)
                HIP_TRY(nz::launch_winsum(d_desc, d_state, n, static_cast<int32_t>(smax->win_hi - smax->win_lo), ws,
                                          smax->d_out, st));
            if (pe) HIP_TRY(hipEventRecord(pe->ev[5], st));

            // ---- read back and schedule the redo of unfinished samples
            HIP_TRY(hipMemcpyAsync(state.data(), d_state, n * sizeof(NzState), hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
            lists.clear();
            if (pe) {
                // (g_ms[2]: the sweep orders its own blocks, there is no sort pass)
                constexpr int phase[5] = {0, -1, 0, 1, 3};
                for (int k = 0; k < 5; ++k) {
                    if (phase[k] < 0) continue;
                    float ms = 0.0f;
                    HIP_TRY(hipEventElapsedTime(&ms, pe->ev[k], pe->ev[k + 1]));
                    g_ms[phase[k]] += ms;
                }
                g_ms[5] += 1.0;
            }
            if (pfe) {
                for (int u = 0; u < pfe->used; ++u) {
                    for (int k = 0; k < 4; ++k) {
                        float ms = 0.0f;
                        HIP_TRY(hipEventElapsedTime(&ms, pfe->ev[u][k], pfe->ev[u][k + 1]));
                        g_cc_ms[k] += ms;
                    }
                    g_cc_ms[4] += 1.0;
                }
            }
            if (getenv("NZ_DEBUG_TRACE")) {
                int cnt[8] = {0};
                for (int32_t k = 0; k < n; ++k) ++cnt[std::max(0, std::min(7, static_cast<int>(state[k].status)))];
                std::fprintf(stderr, "nz: round %d chunk of %d: done %d band %d bucket %d backoff %d prefix %d other %d\n",
                             rounds, n, cnt[NZ_ST_DONE], cnt[NZ_ST_BAND], cnt[NZ_ST_BUCKET], cnt[NZ_ST_BACKOFF],
                             cnt[NZ_ST_PREFIX], n - cnt[NZ_ST_DONE] - cnt[NZ_ST_BAND] - cnt[NZ_ST_BUCKET] -
                                                    cnt[NZ_ST_BACKOFF] - cnt[NZ_ST_PREFIX]);
            }
            for (int32_t i : order) {
                const Part &part = parts[i];
                const int64_t N = pow5(part.p.L);
                for (int32_t k = 0; k < part.count; ++k) {
                    const NzState &end = state[part.desc0 + k];
                    if (end.status == NZ_ST_DONE) {
                        const int64_t serial = (end.nstar > 0 ? end.nstar : N) - end.n0;
                        g_stats[4] += end.n0;
                        g_stats[5] += serial;
                        g_job_pre[part.p.job] += end.n0;
                        g_job_serial[part.p.job] += serial;
                        continue;
                    }
                    Plan p = part.p;
                    p.sample += k;
                    p.out += k;
                    for (int lv = 0; lv < level[part.desc0 + k]; ++lv) {
                        p.n0 = part.s.n0b[lv];
                        p.backoff *= 2;   // the next backoff doubles the step
                    }
                    switch (end.status) {
                    case NZ_ST_BAND:
                        ++g_stats[1];
                        p.band_hi = std::min<int64_t>(N, p.n0 + 2 * std::max<int64_t>(p.band_hi - p.n0, 2048));
                        break;
                    case NZ_ST_BUCKET:
                        ++g_stats[2];
                        p.shift_adj += 1;
                        break;
                    case NZ_ST_BACKOFF:
                        ++g_stats[3];
                        if (h_backoffs) ++h_backoffs[p.job];
                        // back off by the caller's step, doubling it each time
                        // (n0 - b, n0 - 3b, n0 - 7b, ...), until the start would
                        // reach 0; without a step, halve.  A badly predicted lattice
                        // needs only a few rounds, and n0 reaches 0 after at most
                        // log2(N) of them.
                        if (p.backoff > 0) {
                            if (p.n0 - p.backoff > 0) {
                                p.n0 -= p.backoff;
                                p.backoff *= 2;
                            } else {
                                p.n0 = 0;
                                p.backoff = 0;
                            }
                        } else {
                            p.n0 = p.n0 >= 64 ? p.n0 / 2 : 0;
                        }
                        break;
                    case NZ_ST_PREFIX:
                        p.prefix_mul *= 2;
                        break;
                    default:
                        return fail(NZ_EDEVICE, "sample %lld finished with status %d", (long long)p.sample, end.status);
                    }
                    ++redo_left;
                    if (!redo.empty() && follows(redo.back(), p)) ++redo.back().count;
                    else redo.push_back(Run{p, 1});
                }
            }
        }
        todo.swap(redo);
        left = redo_left;
    }
    return NZ_OK;
}

// smax: the jobs run in largest-cluster mode (window entries apart).
size_t batch_bytes(const nz_job *jobs, int32_t njobs, const Tune &tune, bool smax = false)
{
    // all samples of the first chunk resident, plus room for one redo of the
    // largest sample with a full band
    std::vector<std::pair<size_t, int64_t>> per;   // (bytes of one sample, samples) of every job
    std::vector<std::pair<uint32_t, int32_t>> tables;
    size_t tab_entries = 0;
    int32_t maxL = 1;
    bool any_wrap = false;
    for (int j = 0; j < njobs; ++j) {
        const auto key = std::make_pair(jobs[j].zone_mask, jobs[j].L);
        if (std::find(tables.begin(), tables.end(), key) == tables.end()) {
            tables.push_back(key);
            tab_entries += zone_rows(jobs[j].zone_mask).size();
        }
        const bool wrap = jobs[j].boundary == NZ_PERIODIC && !smax;
        any_wrap = any_wrap || wrap;
        Plan p{};
        p.L = jobs[j].L;
        p.mask = jobs[j].zone_mask;
        p.n0 = jobs[j].n0 > 0 ? jobs[j].n0 : 0;
        p.backoff = jobs[j].backoff;   // sizes the band of a first backoff too
        p.wrap = wrap;
        const int64_t N = pow5(p.L);
        p.band_hi = jobs[j].band_hi > 0 ? std::min<int64_t>(jobs[j].band_hi, N) : default_band_hi(p.L, p.mask, p.n0);
        if (p.band_hi <= p.n0) p.band_hi = std::min<int64_t>(N, p.n0 + 4096);
        p.prefix_mul = 1;
        if (jobs[j].nsamples > 0) per.emplace_back(plan_sizes(p, tune.bucket_log2).total, jobs[j].nsamples);
        maxL = std::max(maxL, jobs[j].L);
    }
    // the kMaxChunk largest samples
    std::sort(per.begin(), per.end(), [](const auto &a, const auto &b) { return a.first > b.first; });
    int64_t count = 0;
    size_t sum = 0;
    for (const auto &e : per) {
        const int64_t take = std::min<int64_t>(e.second, kMaxChunk - count);
        sum += e.first * static_cast<size_t>(take);
        count += take;
        if (count == kMaxChunk) break;
    }
    size_t total = header_bytes(tab_entries, static_cast<int32_t>(std::max<int64_t>(count, 1))) + sum;
    Plan full{};
    full.L = maxL;
    full.mask = 127;
    full.band_hi = pow5(maxL);
    full.prefix_mul = 1;
    full.wrap = any_wrap;
    total += plan_sizes(full, tune.bucket_log2).total;
    return total;
}

}  // namespace

namespace nz {
int set_error(int code, const char *msg) { return fail(code, "%s", msg); }

int check_batch_fits(const nz_job *jobs, int32_t njobs, const nz_tuning *tune, size_t ws_bytes)
{
    if (njobs < 0 || (njobs > 0 && !jobs)) return fail(NZ_EINVAL, "bad job array");
    for (int j = 0; j < njobs; ++j)
        if (int rc = check_job(jobs[j], j)) return rc;
    Tune t;
    if (int rc = read_tune(tune, t)) return rc;
    try {
        // a chunk's header (sized for as many samples as the batch engine puts
        // in one chunk) plus the largest single sample of any job, planned as
        // the engine plans it
        std::vector<std::pair<uint32_t, int32_t>> tables;
        size_t tab_entries = 0;
        int64_t total = 0;
        for (int j = 0; j < njobs; ++j) {
            const nz_job &J = jobs[j];
            if (J.nsamples <= 0) continue;
            total += J.nsamples;
            const auto key = std::make_pair(J.zone_mask, J.L);
            if (std::find(tables.begin(), tables.end(), key) == tables.end()) {
                tables.push_back(key);
                tab_entries += zone_rows(J.zone_mask).size();
            }
        }
        if (total == 0) return NZ_OK;
        const size_t head = header_bytes(tab_entries, static_cast<int32_t>(std::min<int64_t>(total, kMaxChunk)));
        // with every prefill as it is, and if that does not fit in the smallest form
        for (bool smallest : {false, true}) {
            size_t largest = 0;
            int32_t worst = -1;
            for (int j = 0; j < njobs; ++j) {
                const nz_job &J = jobs[j];
                if (J.nsamples <= 0) continue;
                Plan p{};
                p.L = J.L;
                p.mask = J.zone_mask;
                p.n0 = J.n0 > 0 ? J.n0 : 0;
                p.backoff = J.backoff;
                p.per = J.boundary == NZ_PERIODIC;
                p.wrap = p.per;
                const int64_t N = pow5(J.L);
                p.band_hi = J.band_hi > 0 ? std::min<int64_t>(J.band_hi, N) : default_band_hi(J.L, J.zone_mask, p.n0);
                if (p.band_hi <= p.n0) p.band_hi = std::min<int64_t>(N, p.n0 + 4096);
                p.prefix_mul = 1;
                const size_t b = smallest ? smallest_bytes(p, t.bucket_log2) : plan_sizes(p, t.bucket_log2).total;
                if (b > largest) {
                    largest = b;
                    worst = j;
                }
            }
            if (head + largest <= ws_bytes) return NZ_OK;
            if (smallest)
                return fail(NZ_EWORKSPACE, "job %d (L = %d) needs %zu bytes for one sample; the buffer holds %zu",
                            worst, jobs[worst].L, head + largest, ws_bytes);
        }
    } catch (...) {
        return fail(NZ_ENOMEM, "host allocation failed while sizing the batch");
    }
    return NZ_OK;
}

int run_batch_one_group(const nz_job *jobs, int32_t njobs, uint8_t *ws, size_t ws_bytes, int32_t *d_nstar,
                        int32_t *d_mass, int32_t *h_backoffs, const nz_tuning *tune, hipStream_t st)
{
    int64_t total = 0;
    for (int j = 0; j < njobs; ++j) total += jobs[j].nsamples;
    if (total == 0) {
        for (int k = 0; k < 6; ++k) g_stats[k] = 0;
        if (h_backoffs)
            for (int j = 0; j < njobs; ++j) h_backoffs[j] = 0;
        return NZ_OK;
    }
    if (!d_nstar) return fail(NZ_EINVAL, "n* output is NULL");
    Tune t;
    if (int rc = read_tune(tune, t)) return rc;
    // no phase events: this path creates no runtime objects
    const bool timing = g_timing;
    g_timing = false;
    int rc;
    try {
        rc = run_batch(jobs, njobs, ws, ws_bytes, d_nstar, d_mass, h_backoffs, t, st);
    } catch (...) {
        rc = fail(NZ_ENOMEM, "host allocation failed");
    }
    g_timing = timing;
    return rc;
}
}  // namespace nz

// ---------------------------------------------------------------------------
// Public entry points.

NZ_API const char *nz_last_error(void) { return g_err; }

NZ_API int nz_abi_version(void) { return NZ_ABI_VERSION; }

NZ_API int nz_coordination(uint32_t zone_mask)
{
    if (zone_mask < 1 || zone_mask > 127) return -1;
    return coordination(zone_mask);
}

NZ_API int nz_last_batch_stats(int64_t stats[6])
{
    if (!stats) return fail(NZ_EINVAL, "stats is NULL");
    for (int k = 0; k < 6; ++k) stats[k] = g_stats[k];
    return NZ_OK;
}

NZ_API int nz_last_batch_job_stats(int64_t *serial, int64_t *prefilled, int32_t njobs)
{
    if (njobs < 0 || (njobs > 0 && (!serial || !prefilled))) return fail(NZ_EINVAL, "NULL output or njobs < 0");
    if (static_cast<size_t>(njobs) != g_job_serial.size())
        return fail(NZ_EINVAL, "the last batch had %zu jobs, not %d", g_job_serial.size(), njobs);
    for (int32_t j = 0; j < njobs; ++j) {
        serial[j] = g_job_serial[j];
        prefilled[j] = g_job_pre[j];
    }
    return NZ_OK;
}

NZ_API int nz_last_batch_cc_timing(double ms[5])
{
    if (!ms) return fail(NZ_EINVAL, "ms is NULL");
    for (int k = 0; k < 5; ++k) ms[k] = g_cc_ms[k];
    return NZ_OK;
}

NZ_API int nz_set_timing(int enable)
{
    g_timing = enable != 0;
    return NZ_OK;
}

NZ_API int nz_last_batch_timing(double ms[6])
{
    if (!ms) return fail(NZ_EINVAL, "ms is NULL");
    for (int k = 0; k < 6; ++k) ms[k] = g_ms[k];
    return NZ_OK;
}

// ---------------------------------------------------------------------------
// Two groups at once.  Narrow neighbourhoods (z <= 64) spend their time in the
// latency of labelling and sweep; a batch that also holds wider ones runs the two
// groups side by side (the wide group on a second host thread and stream), so that
// one group's sweep and host round trips overlap the other's keys and labelling.
// Each group gets its own share of the workspace.  7 compact neighbourhoods, side
// by side / as one group: prefilled L = 16 x 1000 17.7 / 19.0 ms, L = 24 x 200
// 31.0 / 32.2, L = 8 x 1000 1.41 / 1.44; plain, where zone 1's sweep is most of a
// batch, it gives nothing: 33.7 / 33.5, 80.0 / 78.5 and 1.28 / 1.25.

constexpr int64_t kSplitMinSamples = 256;   // on both sides
// widest neighbourhood of the first group (L = 16, 7 compact x 1000, prefilled:
// z <= 10 17.9 ms, 64 17.5, 130 17.5, 242 17.8, 340 18.2)
constexpr int32_t kSplitZ = 64;

struct SplitPlan {
    std::vector<nz_job> job[2];
    std::vector<int32_t> index[2];   // caller's job index of every job of a group
    std::vector<int64_t> out[2];     // first output index of every job of a group
    size_t bytes[2] = {0, 0};
};

bool split_groups(const nz_job *jobs, int32_t njobs, const Tune &tune, SplitPlan &sp)
{
    if (getenv("NZ_DEBUG_NO_SPLIT")) return false;
    int64_t o = 0, count[2] = {0, 0};
    for (int j = 0; j < njobs; ++j) {
        const int g = coordination(jobs[j].zone_mask) <= (tune.split_z ? tune.split_z : kSplitZ) ? 0 : 1;
        if (jobs[j].nsamples > 0) {
            sp.job[g].push_back(jobs[j]);
            sp.index[g].push_back(j);
            sp.out[g].push_back(o);
            count[g] += jobs[j].nsamples;
        }
        o += jobs[j].nsamples;
    }
    if (count[0] < kSplitMinSamples || count[1] < kSplitMinSamples) return false;
    for (int g = 0; g < 2; ++g) sp.bytes[g] = batch_bytes(sp.job[g].data(), static_cast<int32_t>(sp.job[g].size()), tune);
    return true;
}

// The second group's stream, its start event and host thread live per host
// thread and device.
struct SideStream {
    hipStream_t st = nullptr;
    hipEvent_t start = nullptr, keys = nullptr;
    bool ok = false;
};

SideStream *side_stream(int device)
{
    static thread_local std::map<int, SideStream> per_device;
    SideStream &s = per_device[device];
    if (!s.ok && !s.st)
        s.ok = hipStreamCreateWithFlags(&s.st, hipStreamNonBlocking) == hipSuccess &&
               hipEventCreateWithFlags(&s.start, hipEventDisableTiming) == hipSuccess &&
               hipEventCreateWithFlags(&s.keys, hipEventDisableTiming) == hipSuccess;
    return s.ok ? &s : nullptr;
}

int run_split(SplitPlan &sp, int32_t njobs, uint8_t *ws, size_t ws_bytes, int32_t *d_nstar, int32_t *d_mass,
              int32_t *h_backoffs, const Tune &tune, hipStream_t st)
{
    int device = 0;
    HIP_TRY(hipGetDevice(&device));
    SideStream *side = side_stream(device);
    if (!side) return fail(NZ_EDEVICE, "could not create the second stream");
    // workspace shares in proportion to the groups' resident sizes
    const size_t wa = static_cast<size_t>(static_cast<long double>(ws_bytes) * sp.bytes[0] /
                                          (sp.bytes[0] + sp.bytes[1])) / kAlign * kAlign;
    std::vector<int32_t> back[2];
    for (int g = 0; g < 2; ++g) back[g].assign(sp.job[g].size(), 0);
    // the second group starts after the work already queued on the caller's stream
    HIP_TRY(hipEventRecord(side->start, st));
    HIP_TRY(hipStreamWaitEvent(side->st, side->start, 0));
    // Both groups' keys are bound by the same vector ALUs, so the second group's
    // first keys pass follows the first group's, whose labelling and sweep are the
    // longer chain, and runs beside its labelling.  At once, one group's small
    // workgroups starve the other's large ones (L = 16, 7 compact neighbourhoods
    // x 1000: prefilled 22.1 ms, in turn 19.9; plain 36.2 and 34.4).
    std::promise<void> recorded;
    KeysTurn turn_a, turn_b;
    turn_a.done = turn_b.done = side->keys;
    turn_a.record = &recorded;
    turn_b.second = true;
    turn_b.recorded = recorded.get_future().share();
    int rc_b = NZ_OK;
    char err_b[sizeof g_err] = "";
    int64_t stats_b[6] = {0, 0, 0, 0, 0, 0};
    double ms_b[6] = {0, 0, 0, 0, 0, 0};
    double cc_b[5] = {0, 0, 0, 0, 0};
    std::vector<int64_t> serial_b, pre_b;
    const bool timing = g_timing;
    std::thread worker([&]() {
        try {
            if (hipSetDevice(device) != hipSuccess) {
                rc_b = fail(NZ_EDEVICE, "hipSetDevice failed on the second thread");
            } else {
                g_timing = timing;
                rc_b = run_batch(sp.job[1].data(), static_cast<int32_t>(sp.job[1].size()), ws + wa, ws_bytes - wa,
                                 d_nstar, d_mass, back[1].data(), tune, side->st, nullptr, sp.out[1].data(), &turn_b);
            }
        } catch (...) {
            rc_b = fail(NZ_ENOMEM, "host allocation failed");
        }
        if (rc_b != NZ_OK) std::memcpy(err_b, g_err, sizeof err_b);
        for (int k = 0; k < 6; ++k) {
            stats_b[k] = g_stats[k];
            ms_b[k] = g_ms[k];
        }
        for (int k = 0; k < 5; ++k) cc_b[k] = g_cc_ms[k];
        serial_b.swap(g_job_serial);
        pre_b.swap(g_job_pre);
    });
    int rc_a;
    try {
        rc_a = run_batch(sp.job[0].data(), static_cast<int32_t>(sp.job[0].size()), ws, wa, d_nstar, d_mass,
                         back[0].data(), tune, st, nullptr, sp.out[0].data(), &turn_a);
    } catch (...) {
        rc_a = fail(NZ_ENOMEM, "host allocation failed");
    }
    turn_a.pass();   // (whatever happened, the worker does not wait)
    worker.join();
    for (int k = 0; k < 6; ++k) {
        g_stats[k] += stats_b[k];
        g_ms[k] += ms_b[k];
    }
    for (int k = 0; k < 5; ++k) g_cc_ms[k] += cc_b[k];
    {
        // per-job figures back in the caller's job order
        std::vector<int64_t> serial(static_cast<size_t>(njobs), 0), pre(static_cast<size_t>(njobs), 0);
        for (size_t k = 0; k < sp.job[0].size() && k < g_job_serial.size(); ++k) {
            serial[sp.index[0][k]] = g_job_serial[k];
            pre[sp.index[0][k]] = g_job_pre[k];
        }
        for (size_t k = 0; k < sp.job[1].size() && k < serial_b.size(); ++k) {
            serial[sp.index[1][k]] = serial_b[k];
            pre[sp.index[1][k]] = pre_b[k];
        }
        g_job_serial.swap(serial);
        g_job_pre.swap(pre);
    }
    if (rc_a != NZ_OK) return rc_a;
    if (rc_b != NZ_OK) return fail(rc_b, "%s", err_b);
    if (h_backoffs) {
        for (int j = 0; j < njobs; ++j) h_backoffs[j] = 0;
        for (int g = 0; g < 2; ++g)
            for (size_t k = 0; k < sp.job[g].size(); ++k) h_backoffs[sp.index[g][k]] = back[g][k];
    }
    return NZ_OK;
}

NZ_API int nz_batch_workspace_bytes(const nz_job *jobs, int32_t njobs, const nz_tuning *tune, size_t *bytes)
{
    if (!bytes) return fail(NZ_EINVAL, "bytes is NULL");
    if (njobs < 0 || (njobs > 0 && !jobs)) return fail(NZ_EINVAL, "bad job array");
    for (int j = 0; j < njobs; ++j)
        if (int rc = check_job(jobs[j], j)) return rc;
    Tune t;
    if (int rc = read_tune(tune, t)) return rc;
    try {
        SplitPlan sp;
        *bytes = split_groups(jobs, njobs, t, sp) ? sp.bytes[0] + sp.bytes[1] + kAlign : batch_bytes(jobs, njobs, t);
    } catch (...) {
        return fail(NZ_ENOMEM, "host allocation failed while sizing the workspace");
    }
    return NZ_OK;
}

NZ_API int nz_sweep_batch(const nz_job *jobs, int32_t njobs, void *d_ws, size_t ws_bytes, int32_t *d_nstar,
                          int32_t *d_mass, int32_t *h_backoffs, const nz_tuning *tune, void *stream)
{
    if (njobs < 0 || (njobs > 0 && !jobs)) return fail(NZ_EINVAL, "bad job array");
    int64_t total = 0;
    for (int j = 0; j < njobs; ++j) {
        if (int rc = check_job(jobs[j], j)) return rc;
        total += jobs[j].nsamples;
    }
    if (total == 0) return NZ_OK;
    if (!d_ws || !d_nstar) return fail(NZ_EINVAL, "workspace or n* output is NULL");
    if (reinterpret_cast<uintptr_t>(d_ws) % kAlign) return fail(NZ_EINVAL, "workspace must be 256-byte aligned");
    Tune t;
    if (int rc = read_tune(tune, t)) return rc;
    // a workspace that cannot hold one sample is refused before any device call
    if (int rc = nz::check_batch_fits(jobs, njobs, tune, ws_bytes)) return rc;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (g_timing) {
        HIP_TRY(hipEventCreate(&e0));
        HIP_TRY(hipEventCreate(&e1));
        HIP_TRY(hipEventRecord(e0, static_cast<hipStream_t>(stream)));
    }
    int rc;
    try {
        // two groups side by side when the workspace holds both resident
        SplitPlan sp;
        if (split_groups(jobs, njobs, t, sp) && ws_bytes >= sp.bytes[0] + sp.bytes[1] + kAlign)
            rc = run_split(sp, njobs, static_cast<uint8_t *>(d_ws), ws_bytes, d_nstar, d_mass, h_backoffs, t,
                           static_cast<hipStream_t>(stream));
        else
            rc = run_batch(jobs, njobs, static_cast<uint8_t *>(d_ws), ws_bytes, d_nstar, d_mass, h_backoffs, t,
                           static_cast<hipStream_t>(stream));
    } catch (...) {
        rc = fail(NZ_ENOMEM, "host allocation failed");
    }
    if (e0) {
        float ms = 0.0f;
        if (rc == NZ_OK && hipEventRecord(e1, static_cast<hipStream_t>(stream)) == hipSuccess &&
            hipEventSynchronize(e1) == hipSuccess && hipEventElapsedTime(&ms, e0, e1) == hipSuccess)
            g_ms[4] = ms;
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    return rc;
}

// Device memory of the host entry points (nz_sweep, nz_smax_window), kept from
// one call to the next on the same thread: mapping and unmapping it cost more
// than the sweep itself (L = 12, 1000 samples of zone 1, 2 GB: 9 ms or 60 ms of
// a call, by the state of the allocator).  Blocks up to kKeepBytes are kept, at
// most kKeepTotal over all threads; larger ones are freed with the call, and a
// kept block by nz_release, when its thread ends, when the thread turns to
// another device or a larger block, or when an allocation fails.
constexpr size_t kKeepBytes = size_t(4) << 30;
constexpr size_t kKeepTotal = size_t(8) << 30;

class DeviceBlock {
public:
    ~DeviceBlock() { release(); }
    // `bytes` of memory on `device` (current), NULL if there is none
    void *get(int device, size_t bytes)
    {
        if (p_ && device_ == device && bytes_ >= bytes) return p_;
        release();
        void *p = nullptr;
        if (hipMalloc(&p, bytes) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        p_ = p;
        device_ = device;
        bytes_ = bytes;
        counted_ = false;
        return p_;
    }
    // the call is over: keeps the block if the bounds allow it
    void done()
    {
        if (!p_ || counted_) return;
        if (bytes_ <= kKeepBytes && kept_.fetch_add(bytes_) + bytes_ <= kKeepTotal) {
            counted_ = true;
            return;
        }
        if (bytes_ <= kKeepBytes) kept_.fetch_sub(bytes_);
        release();
    }
    void release()
    {
        if (!p_) return;
        (void)hipFree(p_);
        if (counted_) kept_.fetch_sub(bytes_);
        p_ = nullptr;
        counted_ = false;
    }

private:
    void *p_ = nullptr;
    size_t bytes_ = 0;
    int device_ = -1;
    bool counted_ = false;
    static std::atomic<size_t> kept_;
};
std::atomic<size_t> DeviceBlock::kept_{0};

DeviceBlock &thread_block()
{
    static thread_local DeviceBlock block;
    return block;
}

NZ_API int nz_release(void)
{
    thread_block().release();
    return NZ_OK;
}

// Workspace of at most `want` bytes (`samples` samples resident at once) followed
// by `extra` bytes of outputs.  One beyond the kept size is cut to it while it
// still holds kEnough samples: the chunks then fill the chip all the same, and
// an extra chunk costs less than the mapping.  Else it is limited to half of the
// free memory.
constexpr int64_t kEnough = 512;
int host_block(size_t want, int64_t samples, size_t extra, uint8_t **ws, size_t *ws_bytes, uint8_t **tail)
{
    int device = 0;
    HIP_TRY(hipGetDevice(&device));
    want = align_up(want);
    if (extra < kKeepBytes / 2 && want + extra > kKeepBytes) {
        const size_t cut = (kKeepBytes - extra) / kAlign * kAlign;
        if (static_cast<double>(samples) * (static_cast<double>(cut) / static_cast<double>(want)) >= static_cast<double>(kEnough)) want = cut;
    }
    for (int attempt = 0; attempt < 2; ++attempt) {
        if (want + extra > kKeepBytes || attempt > 0) {
            thread_block().release();   // (it counts as free memory)
            size_t freeb = 0, totalb = 0;
            HIP_TRY(hipMemGetInfo(&freeb, &totalb));
            want = std::min(want, freeb / 2 / kAlign * kAlign);
        }
        if (void *p = thread_block().get(device, want + extra)) {
            *ws = static_cast<uint8_t *>(p);
            *ws_bytes = want;
            *tail = *ws + want;
            return NZ_OK;
        }
    }
    return fail(NZ_ENOMEM, "hipMalloc of %zu workspace bytes failed", want + extra);
}

NZ_API int nz_sweep(int32_t L, uint32_t zone_mask, int32_t boundary, int64_t nsamples, uint64_t seed, int32_t *nstar,
                    int32_t *mass)
{
    nz_job j{};
    j.L = L;
    j.zone_mask = zone_mask;
    j.boundary = boundary;
    j.seed = seed;
    j.sample0 = 0;
    j.nsamples = nsamples;
    j.n0 = -1;
    if (int rc = check_job(j, 0)) return rc;
    if (nsamples == 0) return NZ_OK;
    if (!nstar) return fail(NZ_EINVAL, "nstar is NULL");
    if (nsamples > 0x7FFFFFFF) return fail(NZ_EINVAL, "nsamples too large");
    Tune t;
    size_t bytes = 0;
    try {
        bytes = batch_bytes(&j, 1, t);
    } catch (...) {
        return fail(NZ_ENOMEM, "host allocation failed");
    }
    uint8_t *ws = nullptr, *tail = nullptr;
    const size_t out_bytes = static_cast<size_t>(nsamples) * 4;
    if (int rc = host_block(bytes, std::min<int64_t>(nsamples, kMaxChunk), 2 * out_bytes, &ws, &bytes, &tail)) return rc;
    int32_t *dn = reinterpret_cast<int32_t *>(tail), *dm = dn + nsamples;
    int rc;
    try {
        rc = run_batch(&j, 1, ws, bytes, dn, mass ? dm : nullptr, nullptr, t, nullptr);
        if (rc == NZ_OK) {
            // n* and masses lie one behind the other: one copy
            std::vector<int32_t> both(static_cast<size_t>(nsamples) * (mass ? 2 : 1));
            if (hipMemcpy(both.data(), dn, both.size() * 4, hipMemcpyDeviceToHost) != hipSuccess) {
                rc = fail(NZ_EDEVICE, "copy of results failed");
            } else {
                std::memcpy(nstar, both.data(), out_bytes);
                if (mass) std::memcpy(mass, both.data() + nsamples, out_bytes);
            }
        }
    } catch (...) {
        rc = fail(NZ_ENOMEM, "host allocation failed");
    }
    thread_block().done();
    return rc;
}

NZ_API int nz_smax_window(int32_t L, uint32_t zone_mask, int32_t boundary, uint64_t seed, int64_t sample0,
                          int64_t nsamples, int64_t n0, int64_t n_lo, int64_t n_hi, uint64_t *smax_sum)
{
    nz_job j{};
    j.L = L;
    j.zone_mask = zone_mask;
    j.boundary = boundary;
    j.seed = seed;
    j.sample0 = sample0;
    j.nsamples = nsamples;
    j.n0 = n0 > 0 ? n0 : -1;
    j.backoff = 0;   // a prefill that reaches the window halves n0
    if (int rc = check_job(j, 0)) return rc;
    const int64_t N = pow5(L);
    if (n_lo < 1 || n_hi <= n_lo || n_hi > N)
        return fail(NZ_EINVAL, "window [%lld, %lld) outside [1, N = %lld]", (long long)n_lo, (long long)n_hi,
                    (long long)N);
    if (n0 >= n_lo) return fail(NZ_EINVAL, "n0 = %lld must lie below the window start %lld", (long long)n0, (long long)n_lo);
    if (!smax_sum) return fail(NZ_EINVAL, "smax_sum is NULL");
    if (nsamples > 0x7FFFFFFF) return fail(NZ_EINVAL, "nsamples too large");
    const int64_t W = n_hi - n_lo;
    for (int64_t k = 0; k < W; ++k) smax_sum[k] = 0;
    if (nsamples == 0) return NZ_OK;
    // the key band ends a little beyond the window, so a band that runs short is rare
    j.band_hi = std::min<int64_t>(N, n_hi + 4 * static_cast<int64_t>(std::sqrt(static_cast<double>(n_hi))) + 1024);
    Tune t;
    size_t bytes = 0;
    try {
        bytes = batch_bytes(&j, 1, t, true) + static_cast<size_t>(std::min<int64_t>(nsamples, kMaxChunk) + 1) *
                                                  align_up(static_cast<size_t>(W) * 4);
    } catch (...) {
        return fail(NZ_ENOMEM, "host allocation failed");
    }
    uint8_t *ws = nullptr, *tail = nullptr;
    if (int rc = host_block(bytes, std::min<int64_t>(nsamples, kMaxChunk), static_cast<size_t>(W) * 8 + static_cast<size_t>(nsamples) * 4,
                            &ws, &bytes, &tail)) return rc;
    uint64_t *dsum = reinterpret_cast<uint64_t *>(tail);
    int32_t *dn = reinterpret_cast<int32_t *>(tail + W * 8);
    int rc = NZ_OK;
    if (hipMemset(dsum, 0, W * 8) != hipSuccess) rc = fail(NZ_EDEVICE, "clearing the window sums failed");
    SmaxReq req{n_lo, n_hi, dsum};
    if (rc == NZ_OK) {
        try {
            rc = run_batch(&j, 1, ws, bytes, dn, nullptr, nullptr, t, nullptr, &req);
        } catch (...) {
            rc = fail(NZ_ENOMEM, "host allocation failed");
        }
    }
    if (rc == NZ_OK && hipMemcpy(smax_sum, dsum, W * 8, hipMemcpyDeviceToHost) != hipSuccess)
        rc = fail(NZ_EDEVICE, "copy of the window sums failed");
    thread_block().done();
    return rc;
}

// Walks the binomial weights w(n) = C(N,n) p^n (1-p)^(N-n) / that of the mode
// (1 at the mode), 0 < p < 1, from the mode outward by their ratio: up first,
// then down.  term(n, w) adds a term, done(n, w) may end a direction once no
// later term of it can change a sum.  Terms below 1e-300 are dropped.  The
// ratios of eight steps are formed together (their divisions overlap); the
// product runs through them one by one, in the same order as step by step.
// UNROLL: so are the products and terms (the window convolution's 7% faster, the
// canonical one's steps, which search, 7% slower).
template <bool UNROLL, typename Term, typename Done>
void binomial_walk(int64_t N, double p, int64_t mode, Term &&term, Done &&done)
{
    const double up = p / (1.0 - p);
    double r[8];
    double w = 1.0;
    // step(k) for k = 0 .. m - 1, while it says so
    const auto steps = [&](int m, auto &&step) {
        if constexpr (UNROLL) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (k == m) return true;
                if (!step(k)) return false;
            }
        } else {
            for (int k = 0; k < m; ++k)
                if (!step(k)) return false;
        }
        return true;
    };
    for (int64_t n = mode; n < N; n += 8) {
        const int m = static_cast<int>(std::min<int64_t>(8, N - n));
        for (int k = 0; k < 8; ++k) r[k] = static_cast<double>(N - n - k) / static_cast<double>(n + k + 1) * up;
        const bool on = steps(m, [&](int k) {
            w *= r[k];
            if (w < 1e-300) return false;
            term(n + k + 1, w, true);
            return true;
        });
        if (!on || done(n + m, w, true)) break;
    }
    w = 1.0;
    for (int64_t n = mode; n > 0; n -= 8) {
        const int m = static_cast<int>(std::min<int64_t>(8, n));
        for (int k = 0; k < 8; ++k) r[k] = static_cast<double>(n - k) / static_cast<double>(N - n + k + 1) / up;
        const bool on = steps(m, [&](int k) {
            w *= r[k];
            if (w < 1e-300) return false;
            term(n - k - 1, w, false);
            return true;
        });
        if (!on || done(n - m, w, false)) return;
    }
}

// Adding less than this times a sum leaves the sum as it is (half an ulp of it
// is at least 2^-54 of it), and the weights only fall on the way outward.
constexpr double kNoChange = 0x1p-55;

// Binomial convolution of an observable on a window (eqs. (5)-(6) need
// P_max(p) = <S_max(n)>/N convolved with the binomial of (N, p)): the same
// weights as nz_canonical, summed over n in [n_lo, n_hi) only.
NZ_API int nz_convolve_window(const double *Q, int64_t n_lo, int64_t n_hi, int64_t N, const double *p_grid, int64_t np,
                              double *out, double *cover)
{
    if (N < 1 || n_lo < 0 || n_hi > N + 1 || n_lo >= n_hi || !Q)
        return fail(NZ_EINVAL, "window [%lld, %lld) outside [0, N + 1 = %lld]", (long long)n_lo, (long long)n_hi,
                    (long long)(N + 1));
    if (np < 0 || (np > 0 && (!p_grid || !out))) return fail(NZ_EINVAL, "bad p grid or output");
    for (int64_t k = 0; k < np; ++k)
        if (!(p_grid[k] >= 0.0 && p_grid[k] <= 1.0)) return fail(NZ_EINVAL, "p_grid[%lld] outside [0, 1]", (long long)k);
    // Largest |Q| (NaN or infinite: the walks are not cut short inside the window).  An
    // entry costs as much here as a step of a walk, of which a walk cut short saves
    // some 57 standard deviations' worth, so windows wider than the walks gain
    // from it are not looked through (N = 16^5, 200000 entries, one p: 0.58 ms with
    // the look, 0.08 without; 65 p on 4000 entries: 1.5 and 4.3).
    double reach = 0.0;
    for (int64_t k = 0; k < np; ++k) reach += 57.0 * std::sqrt(static_cast<double>(N) * p_grid[k] * (1.0 - p_grid[k]));
    double most = static_cast<double>(n_hi - n_lo) <= reach ? 0.0 : HUGE_VAL;
    for (int64_t n = 0; n < n_hi - n_lo && most < HUGE_VAL; ++n) {
        const double q = std::fabs(Q[n]);
        if (!(q <= most)) most = q;
    }
    for (int64_t k = 0; k < np; ++k) {
        const double p = p_grid[k];
        int64_t mode = p == 0.0 ? 0 : (p == 1.0 ? N : static_cast<int64_t>(std::floor((N + 1) * p)));
        if (mode > N) mode = N;
        const bool inside = mode >= n_lo && mode < n_hi;
        double sw = 1.0, swq = inside ? Q[mode - n_lo] : 0.0, swin = inside ? 1.0 : 0.0;
        if (p > 0.0 && p < 1.0)
            binomial_walk<true>(
                N, p, mode,
                [&](int64_t n, double w, bool) {
                    sw += w;
                    const bool in = n >= n_lo && n < n_hi;
                    swq += w * (in ? Q[n - n_lo] : 0.0);
                    swin += w * (in ? 1.0 : 0.0);
                },
                [&](int64_t n, double w, bool upward) {
                    if (!(w < kNoChange * sw)) return false;
                    if (upward ? n >= n_hi - 1 : n <= n_lo) return true;   // past the window
                    return w < kNoChange * swin && w * most < kNoChange * std::fabs(swq);
                });
        out[k] = swq / sw;
        if (cover) cover[k] = swin / sw;
    }
    return NZ_OK;
}

// ---------------------------------------------------------------------------
// Learned-prefill planning: the MLP's input rows, its training targets and the
// turn of its outputs into the jobs' prefill depth, backoff step and key band.

// The size input: L enters through the finite-size-scaling variable
// L^(-1/nu), nu = 0.5720 (the 5D correlation-length exponent quoted in
// Sec. II.A.1): the mean of n*/N approaches p_c roughly linearly in it.
constexpr double kNu5 = 0.5720;

double size_variable(int32_t L) { return std::exp(-std::log(static_cast<double>(L)) / kNu5); }

NZ_API int nz_mlp_size_stats(const int32_t *L, int32_t B, double out[2])
{
    if (B < 1 || !L || !out) return fail(NZ_EINVAL, "nz_mlp_size_stats: NULL pointer or B < 1");
    for (int32_t b = 0; b < B; ++b)
        if (L[b] < 1 || L[b] > 55) return fail(NZ_EINVAL, "nz_mlp_size_stats: L[%d] = %d outside [1, 55]", b, L[b]);
    double sum = 0.0;
    for (int32_t b = 0; b < B; ++b) sum += size_variable(L[b]);
    const double mean = sum / B;
    double ss = 0.0;
    for (int32_t b = 0; b < B; ++b) ss += (size_variable(L[b]) - mean) * (size_variable(L[b]) - mean);
    const double sd = std::sqrt(ss / B);
    out[0] = mean;
    out[1] = sd > 0.0 ? sd : 1.0;
    return NZ_OK;
}

NZ_API int nz_mlp_features(const uint32_t *zone_mask, const int32_t *L, int32_t B, double size_mean, double size_std,
                           float *x)
{
    if (B < 1 || !zone_mask || !L || !x) return fail(NZ_EINVAL, "nz_mlp_features: NULL pointer or B < 1");
    if (!(size_std > 0.0)) return fail(NZ_EINVAL, "nz_mlp_features: size_std must be positive");
    for (int32_t b = 0; b < B; ++b) {
        if (zone_mask[b] < 1 || zone_mask[b] > 127 || L[b] < 1 || L[b] > 55)
            return fail(NZ_EINVAL, "nz_mlp_features: row %d has zone_mask %u, L %d", b, zone_mask[b], L[b]);
        for (int k = 0; k < 7; ++k) x[8 * b + k] = static_cast<float>((zone_mask[b] >> k) & 1u);
        x[8 * b + 7] = static_cast<float>((size_variable(L[b]) - size_mean) / size_std);
    }
    return NZ_OK;
}

NZ_API int nz_prefill_target(const int32_t *nstar, int64_t nsamples, int32_t L, double out[5])
{
    if (nsamples < 0 || (nsamples > 0 && !nstar) || !out || L < 1 || L > 55)
        return fail(NZ_EINVAL, "nz_prefill_target: bad arguments");
    const double N = static_cast<double>(pow5(L));
    long double s1 = 0.0L;
    int64_t count = 0;
    for (int64_t k = 0; k < nsamples; ++k)
        if (nstar[k] > 0) {
            s1 += static_cast<long double>(nstar[k]) / N;
            ++count;
        }
    if (count == 0) return fail(NZ_EINVAL, "nz_prefill_target: no sample spans");
    const long double mean = s1 / count;
    long double ss = 0.0L;
    for (int64_t k = 0; k < nsamples; ++k)
        if (nstar[k] > 0) {
            const long double d = static_cast<long double>(nstar[k]) / N - mean;
            ss += d * d;
        }
    const double sd = std::max(static_cast<double>(std::sqrt(ss / count)), 0.5 / N);
    out[0] = static_cast<double>(count);
    out[1] = static_cast<double>(mean);
    out[2] = sd;
    out[3] = std::log(out[1]);
    out[4] = std::log(sd);
    return NZ_OK;
}

NZ_API int nz_prefill_plan(const float *y, nz_job *jobs, int32_t njobs, double k_sigma, double band_sigma,
                           int32_t plain)
{
    if (njobs < 0 || (njobs > 0 && (!y || !jobs))) return fail(NZ_EINVAL, "nz_prefill_plan: NULL pointer or njobs < 0");
    if (!(k_sigma >= 0.0) || !(band_sigma >= 0.0)) return fail(NZ_EINVAL, "nz_prefill_plan: negative sigma factor");
    for (int32_t j = 0; j < njobs; ++j)
        if (jobs[j].L < 1 || jobs[j].L > 55) return fail(NZ_EINVAL, "nz_prefill_plan: job %d has L = %d", j, jobs[j].L);
    for (int32_t j = 0; j < njobs; ++j) {
        nz_job &J = jobs[j];
        const int64_t N = pow5(J.L);
        const double mean = std::exp(static_cast<double>(y[2 * j]));
        const double sd = std::exp(static_cast<double>(y[2 * j + 1]));
        const double hi = std::ceil((mean + band_sigma * sd) * static_cast<double>(N)) + 1024.0;
        J.band_hi = hi >= static_cast<double>(N) ? N : static_cast<int64_t>(hi);
        if (plain) {
            J.n0 = -1;
            continue;
        }
        const double d0 = std::floor((mean - k_sigma * sd) * static_cast<double>(N));
        J.n0 = d0 <= 0.0 ? 0 : (d0 >= static_cast<double>(N - 1) ? N - 1 : static_cast<int64_t>(d0));
        const double b = std::ceil(k_sigma * sd * static_cast<double>(N));
        J.backoff = b >= static_cast<double>(N) ? N : static_cast<int64_t>(b);
    }
    return NZ_OK;
}

// Whether more than an eighth of the entries hold counts: all of them up to 4096
// entries, else 64 blocks of 64 spread over the histogram.
static bool dense_histogram(const uint64_t *hist, int64_t N)
{
    const int64_t stride = N < 4096 ? 64 : N / 64;
    int64_t seen = 0, held = 0;
    for (int64_t b = 0; b <= N; b += stride)
        for (int64_t n = b; n < std::min<int64_t>(b + 64, N + 1); ++n) {
            ++seen;
            held += hist[n] != 0 ? 1 : 0;
        }
    return 8 * held > seen;
}

// Binomial convolution (Sec. II.B): weights C(N,n) p^n (1-p)^(N-n) are formed
// from the mode outward with the ratio w(n+1)/w(n) = (N-n)/(n+1) * p/(1-p) and
// normalised by their sum.  Terms below 1e-300 of the mode weight are dropped.
//
// F(n) = (samples with 1 <= n* <= n) / total is a step function.  The n* of a run
// lie in a few thousand of the N + 1 entries, and the steps alone are kept, in one
// pass over the histogram (L = 16, 1000 samples, 101 points, one core: 2.0 ms, and
// 10.2 with F at every n).  A histogram with counts in more than an eighth of its
// entries is taken as F at every n: as steps it costs three arrays instead of one
// and a search per term.  L = 16, steps / every n: all entries held, one point 14.6
// / 2.2 ms, 101 points 15.5 / 3.7; a seventh of them, 3.4 / 2.2 and 5.9 / 3.7; a
// tenth, as steps, 2.7 and 4.7.
NZ_API int nz_canonical(const uint64_t *hist, int64_t hist_len, const double *p_grid, int64_t np, double *R)
{
    if (!hist || hist_len < 2) return fail(NZ_EINVAL, "hist must have at least 2 entries");
    if (np < 0 || (np > 0 && (!p_grid || !R))) return fail(NZ_EINVAL, "bad p grid or output");
    for (int64_t k = 0; k < np; ++k)
        if (!(p_grid[k] >= 0.0 && p_grid[k] <= 1.0)) return fail(NZ_EINVAL, "p_grid[%lld] outside [0, 1]", (long long)k);
    const int64_t N = hist_len - 1;
    bool dense = dense_histogram(hist, N);
    std::vector<int64_t> at;      // the steps: n, samples up to n
    std::vector<uint64_t> upto;
    std::vector<double> F;        // before the first step and at every step; dense: at every n
    double total = 0.0;
    try {
        uint64_t run = 0, exact = 0;
        bool whole = true;   // the total is an exact integer below 2^53
        for (int64_t n0 = 0; n0 <= N && !dense; n0 += 64) {
            const int64_t n1 = std::min<int64_t>(n0 + 64, N + 1);
            uint64_t any = 0;
            for (int64_t n = n0; n < n1; ++n) any |= hist[n];
            if (!any) continue;
            for (int64_t n = n0; n < n1; ++n) {
                if (!hist[n]) continue;
                total += static_cast<double>(hist[n]);
                exact += hist[n];
                whole = whole && hist[n] < (1ull << 53) && exact < (1ull << 53);
                if (n == 0) continue;
                run += hist[n];
                at.push_back(n);
                upto.push_back(run);
            }
            dense = static_cast<int64_t>(at.size()) > N / 8 + 64;   // (the blocks looked at were not typical)
        }
        if (dense) {
            total = 0.0;
            uint64_t any = 0;
            exact = run = 0;
            for (int64_t n = 0; n <= N; ++n) {
                any |= hist[n];
                exact += hist[n];
            }
            if (any < (1ull << 53) / static_cast<uint64_t>(N + 1)) total = static_cast<double>(exact);
            else
                for (int64_t n = 0; n <= N; ++n) total += static_cast<double>(hist[n]);
            F.resize(static_cast<size_t>(N) + 1);
            for (int64_t n = 1; n <= N; ++n) {
                run += hist[n];
                F[n] = static_cast<double>(run) / total;
            }
        } else {
            if (whole) total = static_cast<double>(exact);
            // (integers, divided once, so F is exact to rounding)
            F.resize(upto.size() + 1);
            for (size_t i = 0; i < upto.size(); ++i) F[i + 1] = static_cast<double>(upto[i]) / total;
        }
    } catch (...) {
        return fail(NZ_ENOMEM, "host allocation failed");
    }
    if (total <= 0.0) return fail(NZ_EINVAL, "empty histogram");
    const auto step_of = [&](int64_t n) {   // steps at or below n
        return static_cast<size_t>(std::upper_bound(at.begin(), at.end(), n) - at.begin());
    };
    // f_mode = F(mode), F_at(n, upward) = F(n), none_below(n): F = 0 below n
    const auto convolve = [&](double p, int64_t mode, double f_mode, auto &&F_at, auto &&none_below) {
        double sw = 1.0, swf = f_mode;
        binomial_walk<false>(
            N, p, mode,
            [&](int64_t n, double w, bool upward) {
                sw += w;
                swf += w * F_at(n, upward);
            },
            [&](int64_t n, double w, bool upward) {
                if (!(w < kNoChange * sw)) return false;
                if (w < kNoChange * swf) return true;   // F <= 1
                return upward ? F.back() == 0.0 : none_below(n);
            });
        return swf / sw;
    };
    for (int64_t k = 0; k < np; ++k) {
        const double p = p_grid[k];
        if (p == 0.0 || p == 1.0) {
            R[k] = p == 0.0 ? 0.0 : F.back();   // F(0) = 0, F(N)
            continue;
        }
        const int64_t mode = std::min(N, static_cast<int64_t>(std::floor((N + 1) * p)));
        if (dense) {
            R[k] = convolve(
                p, mode, F[mode], [&](int64_t n, bool) { return F[n]; }, [&](int64_t n) { return n == 0 || F[n - 1] == 0.0; });
            continue;
        }
        const size_t mode_step = step_of(mode);
        size_t i = mode_step;   // steps at or below the current n
        bool was_up = true;
        R[k] = convolve(
            p, mode, F[mode_step],
            [&](int64_t n, bool upward) {
                if (upward != was_up) {
                    was_up = upward;
                    i = mode_step;
                }
                if (upward)
                    while (i < at.size() && at[i] <= n) ++i;
                else
                    while (i > 0 && at[i - 1] > n) --i;
                return F[i];
            },
            [&](int64_t n) { return at.empty() || n <= at.front(); });
    }
    return NZ_OK;
}

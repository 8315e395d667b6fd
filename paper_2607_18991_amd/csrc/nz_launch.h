// nz_launch.h -- kernel launchers of nz_kernels.hip used by the host planner.
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/nz.h"
#include "nz_internal.h"

namespace nz {

// Descriptors, pending states, queue, output indexes and prefill list of a
// chunk's samples from runs[0..nruns), none longer than max_count; *qhead = 0.
hipError_t launch_expand(const NzRun *runs, int32_t nruns, int32_t max_count, NzSample *desc, NzState *state,
                         int32_t *queue, int32_t *out_index, int32_t *list, int32_t *qhead, hipStream_t st);

// Clears the bucket counters and summaries of samples 0..nsamp-1; with a list
// those of list[0..nsamp), which start over at their backoff `level`.
hipError_t launch_clear(NzSample *desc, const int32_t *list, int32_t nsamp, int32_t level, uint8_t *ws, NzState *state,
                        hipStream_t st);

// Keys for samples [first, first + count) of the descriptor array, all of
// lattice size N.
// (list != NULL: samples list[first .. first + count) instead).
// by_xcd: all workgroups of a sample on one XCD (for bands that hold many sites).
// max_nb > 0: no sample has more than max_nb buckets, and one workgroup per sample
// is preferred where the samples are enough and the counters fit.
hipError_t launch_keys(const NzSample *desc, const int32_t *list, int32_t first, int32_t count, int32_t N, uint8_t *ws,
                       NzState *state, bool by_xcd, int32_t max_nb, hipStream_t st);

// Bulk connected components for the samples listed in list[0..nlist), whose
// prefill lists hold max_sites sites at most.  The grids are sized for lists of
// grid_sites: longer ones take more passes.
// smax: also the largest cluster of each smax-mode sample's prefilled state.
// wrap: the listed samples are periodic first-wrap samples (64-bit entries).
// periodic: the listed samples have periodic coordinates (all or none of them).
// ev (may be NULL): five events recorded before the hook, after it, after
// compress and after the flag pass, the fifth with the fourth (there is no
// separate expand pass).
bool hook_map_fits(int64_t N, int64_t n0);
hipError_t launch_prefill(const NzSample *desc, const int32_t *list, int32_t nlist, int32_t max_sites,
                          int32_t grid_sites, const NzOffset *tabs, uint8_t *ws, NzState *state, bool smax, bool wrap, bool periodic,
                          int32_t map_N, int cus, hipStream_t st, hipEvent_t *ev = nullptr);

// out[0..w) += sum over the chunk's finished samples 0..nsamp-1 of their S_max windows.
hipError_t launch_winsum(const NzSample *desc, const NzState *state, int32_t nsamp, int32_t w, const uint8_t *ws,
                         uint64_t *out, hipStream_t st);

// What the sweep looks for: the first spanning cluster (free boundaries), the
// first cluster wrapping around axis 0 (periodic; 64-bit entries), or the
// largest cluster over a window of n (either).
enum class SweepKind { span, wrap, smax };

// The samples of a.queue, all of one kind and boundary condition, at most max_N
// sites each, on a device of `cus` compute units whose workgroups may use
// lds_per_wg bytes of LDS.
hipError_t launch_sweep(SweepKind kind, bool periodic, const NzSweepArgs &a, int32_t *nstar, int32_t *mass,
                        const int32_t *out_index, int cus, uint32_t max_N, size_t lds_per_wg, hipStream_t st);

// Host side of nz_sweep_batch_static (nz_api.cpp): whether a chunk header and
// the largest single sample of the jobs fit a buffer of ws_bytes; and
// the batch engine run as one group on one stream with no events, threads or
// streams of its own.
int set_error(int code, const char *msg);
int check_batch_fits(const nz_job *jobs, int32_t njobs, const nz_tuning *tune, size_t ws_bytes);
int run_batch_one_group(const nz_job *jobs, int32_t njobs, uint8_t *ws, size_t ws_bytes, int32_t *d_nstar,
                        int32_t *d_mass, int32_t *h_backoffs, const nz_tuning *tune, hipStream_t st);

}  // namespace nz

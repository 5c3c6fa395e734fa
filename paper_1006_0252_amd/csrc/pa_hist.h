// The energy histogram of a +-1 population, in the run's work area.
//
// Between calls every run's histogram is zero and its range is reset (slots of the misc area):
// pa_init_couplings leaves them so, and whoever takes a histogram puts them back (k_normalise and k_moments
// as they read it).  Cleared by a launch of its own before each count, a step of 5 10^4 replicas was two
// launches of 4 us longer.  (The reader as the last block of the count itself was no gain: the memory
// fence before its ticket cost each block as much as the launch.)
#pragma once

#include "pa_common.h"

namespace pa {
namespace hist {

// int64 slots of the misc area: the range of the energies counted so far, then ln Q, S and E_lo of the
// step (FP64 bits), kept there until k_finish commits it
constexpr int kMiscEmin = 0, kMiscEmax = 1, kMiscLnQ = 2, kMiscS = 3, kMiscElo = 4;

// by one thread
__device__ __forceinline__ void reset_range(int64_t* misc)
{
    misc[kMiscEmin] = INT32_MAX;
    misc[kMiscEmax] = INT32_MIN;
}

// all of a run's histogram, by the threads of `blocks` blocks
__device__ __forceinline__ void clear(const pa_state* st, int block, int blocks)
{
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    int64_t* hist = work_ptr<int64_t>(st, wl.hist);
    for (int i = block * blockDim.x + threadIdx.x; i < st->n_bins; i += blocks * blockDim.x) hist[i] = 0;
    if (block == 0 && threadIdx.x == 0) reset_range(work_ptr<int64_t>(st, wl.misc));
}

// the histogram of the run's overlaps with a partner, cleared by one block before they are counted
__device__ __forceinline__ void clear_overlaps(const pa_state* st)
{
    int64_t* qh = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).qhist);
    for (int i = threadIdx.x; i <= st->N; i += blockDim.x) qh[i] = 0;
}

}  // namespace hist
}  // namespace pa

// The energy histogram of a +-1 population, in the run's work area, which is scratch: nothing in it is kept
// from one call to the next, so that a caller may share it between runs or overwrite it.  The histogram and
// its range (slots of the misc area) are therefore cleared by a launch of their own within the call that
// counts.  (Left zero by the reader of the last call, a step of 5 10^4 replicas is two launches, 3% of it,
// shorter, but the scratch is then state; the reader as the last block of the count was no gain: the memory
// fence before its ticket cost each block as much as the launch.)
#pragma once

#include "pa_common.h"

namespace pa {
namespace hist {

// int64 slots of the misc area: the range of the energies counted so far, then ln Q, S and E_lo of the
// step (FP64 bits), kept there until k_finish commits it
constexpr int kMiscEmin = 0, kMiscEmax = 1, kMiscLnQ = 2, kMiscS = 3, kMiscElo = 4;

// all of a run's histogram and its range, by the threads of `blocks` blocks
__device__ __forceinline__ void clear(const pa_state* st, int block, int blocks)
{
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    int64_t* hist = work_ptr<int64_t>(st, wl.hist);
    for (int i = block * blockDim.x + threadIdx.x; i < st->n_bins; i += blocks * blockDim.x) hist[i] = 0;
    if (block == 0 && threadIdx.x == 0) {
        int64_t* misc = work_ptr<int64_t>(st, wl.misc);
        misc[kMiscEmin] = INT32_MAX;
        misc[kMiscEmax] = INT32_MIN;
    }
}

// the histogram of the run's overlaps with a partner, before they are counted, by `blocks` blocks
__device__ __forceinline__ void clear_overlaps(const pa_state* st, int block, int blocks)
{
    int64_t* qh = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).qhist);
    for (int i = block * blockDim.x + threadIdx.x; i <= st->N; i += blocks * blockDim.x) qh[i] = 0;
}

}  // namespace hist
}  // namespace pa

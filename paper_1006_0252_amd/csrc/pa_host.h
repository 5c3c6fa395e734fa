// Host side of libpa: the launch functions of the .hip files.
#pragma once

#include "pa_common.h"

namespace pa {

// A launch of 2^32 threads or more along x is cut short without an error.  blocks of threads each go in parts:
// go(first block, blocks of the part).
constexpr int64_t kLaunchThreads = (int64_t)1 << 31;

template <class F>
void launch_parts(int64_t blocks, int threads, F go)
{
    const int64_t most = kLaunchThreads / threads;
    for (int64_t first = 0; first < blocks; first += most)
        go((uint32_t)first, (unsigned)(blocks - first < most ? blocks - first : most));
}

// host launch helpers (defined in the .hip files)
// initialise n runs with consecutive states on one stream, of one dim, layout and coupling kind (any sizes)
int launch_init(const pa_run* runs, int n, const int8_t* const* J_host, hipStream_t s);
int launch_init_group(int L, int layout, pa_state* base, const BatchOrder& order, int n, int64_t cap, hipStream_t s);
int launch_sweep(const pa_run& run, const pa_step& step, hipStream_t s);
// n > 1 chain runs (dim 1) with consecutive states, one length and layout, one stream
int launch_sweep_chain_batch(const pa_run* runs, int n, const pa_step& step, hipStream_t s);
bool launch_sweep_chain(int N, int layout, const pa_state* base, int n, int64_t cap, const SweepParams& p, hipStream_t s);
int launch_sweep_fast(const pa_run& run, const SweepParams& p, int lpr, int wpb, hipStream_t s);
// the group kernel (cube sides 4 to 20 and 24, both layouts): one run, or a group of equal-L runs of a
// batch (items, groups: 64-replica groups of the runs' capacities and of their target sizes)
int launch_sweep_group(const pa_run& run, const SweepParams& p, hipStream_t s);
int launch_sweep_group_batch(int L, int layout, pa_state* base, int pos0, int pos1, const BatchOrder& order,
                             const SweepParams& p, int64_t items, int64_t groups, hipStream_t s);
// batched launchers: n runs whose device states are contiguous (runs[r].state == runs[0].state + r)
int launch_resample(const pa_run* runs, int n, const pa_step& step, hipStream_t s);
void launch_hist(const pa_run* runs, int n, bool overlap, hipStream_t s);
int launch_measure(const pa_run* runs, int n, const pa_run* partner, int pair_xor, hipStream_t s);
int launch_free_energy(const pa_run* runs, int n, double* out, hipStream_t s);
int launch_sweep_batch(const pa_run* runs, int n, const SweepParams& p, hipStream_t s);
bool fast_sweep_supported(int dim, int L);
bool group_sweep_supported(int dim, int L);
// the fast cube sweep compares first looks against top + 1 in 16 bits: tops up to 0xFFFE (a move
// of dE = 4 accepted with probability below 1 - 2^-16, i.e. beta above about 4e-6)
inline bool fast_sweep_thresholds_ok(const SweepParams& p) { return p.thi[4] <= 0xFFFEu; }
int build_sweep_params(const pa_step& step, int z, SweepParams* p);
int launch_weighted_average_dev(int n_sets, int M, const double* x, const double* R, const double* A, int n_obs,
                                double* out, hipStream_t s);
int launch_overlap_average_dev(int n_sets, int n_pairs, const double* x, const double* R, const double* Q,
                               double* out, hipStream_t s);
int launch_bootstrap_dev(int n_sets, int M, const double* x, const double* R, const double* A, int n_obs, int n_boot,
                         const int32_t* idx, double* rep, double* err, hipStream_t s);
int build_thresholds(double beta, int z, uint64_t* T, uint8_t* always);
int launch_features(const pa_run* runs, int n, float* x, hipStream_t s);
int launch_rho(const pa_run* runs, int n, const double* args, int n_args, int mode, double cap, int64_t ld,
               double* out, hipStream_t s);
int upload_ladder(hipStream_t s);

// Gaussian-coupling path (separate kernels; n > 1 runs: consecutive states on one stream)
int gauss_couplings_upload(const pa_run* runs, int n, hipStream_t s);
int launch_energy_gauss(const pa_run* runs, int n, hipStream_t s);
// consecutive: the runs' states are consecutive and share runs[0].stream (one launch for all)
int launch_sweep_gauss(const pa_run* runs, int n_runs, bool consecutive, const pa_step& step, hipStream_t s);
int launch_resample_gauss(const pa_run* runs, int n, const pa_step& step, hipStream_t s);
int launch_measure_gauss(const pa_run* runs, int n, const pa_run* partner, int pair_xor, hipStream_t s);
int launch_moments_gauss(const pa_run* runs, int n, bool overlap, hipStream_t s);

}  // namespace pa

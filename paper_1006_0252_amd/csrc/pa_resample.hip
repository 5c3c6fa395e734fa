// Resampling between temperatures (Sec. II, eqs. Q and wn; Poisson copy numbers with mean
// (R_target / R~) tau_j; the new population of R~' replicas).
//
// Chain of kernels on the run's stream, all sized by capacity and reading the population size
// from the device, with no host synchronisation:
//   hist      energy histogram h (width-4 bins from E_base), E_lo, E_hi      (cleared, integer atomics)
//   normalise S = sum_E h(E) w(E - E_lo) in ascending E (FP64, one thread, fixed order),
//             ln Q, and per bin the mean copy number lambda = R_target w / S split into
//             Poisson(64) blocks q, ladder level m and thinning threshold
//   copies    Poisson(lambda) per replica from its Philox stream (integer compares only), and the sum
//             of each tile of kScanTile replicas
//   offsets   exclusive scan of the copy numbers -> offsets, R~'; source replica of every new replica
//   gather    copy spins and energies into the other buffer
//   finish    swap buffers, R~ = R~', accumulate ln Q, record; or, where R~' does not fit, the
//             capacity / extinction flag
// Every kernel is a no-op once the run's sticky status is set.  The status is written only by launches of
// one block per run, after every wave of it has read it: the blocks of a launch that change it under each
// other could leave some waves of a block at its first line and take the rest on.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "pa_common.h"
#include "pa_hist.h"
#include "pa_host.h"

#pragma clang fp contract(off)

namespace pa {

using namespace hist;

// Poisson(2^m) inversion tables, m = kLadderMin .. kLadderMax (host-built, uploaded once)
__device__ uint64_t g_ladder[kLadderLevels][kLadderCap];

// ------------------------------------------------------------------ host tables
// C[n] = floor(CDF_{2^m}(n) 2^32) with pmf recursion p_0 = exp(-Lambda), p_n = p_{n-1} Lambda / n;
// the table ends at the first n >= Lambda with p_n < 2^-40, that entry forced to 2^32.
static int ladder_host(int m, uint64_t* C, int cap)
{
    const double Lam = ldexp(1.0, m);
    double p = exp(-Lam);
    double F = 0.0;
    const double tail = ldexp(1.0, -40);
    int n = 0;
    for (;;) {
        F += p;
        if ((double)n >= Lam && p < tail) {
            C[n] = (uint64_t)1 << 32;
            return n + 1;
        }
        const double c = floor(ldexp(F, 32));
        C[n] = c >= 4294967296.0 ? ((uint64_t)1 << 32) : (uint64_t)c;
        ++n;
        p = p * Lam / (double)n;
        if (n >= cap - 1) {
            C[n] = (uint64_t)1 << 32;
            return n + 1;
        }
    }
}

static uint64_t g_ladder_host[kLadderLevels][kLadderCap];
static bool g_ladder_built = false;
static int g_ladder_device_mask = 0;  // devices that hold the table

int upload_ladder(hipStream_t s)
{
    if (!g_ladder_built) {
        for (int m = kLadderMin; m <= kLadderMax; ++m) {
            uint64_t* C = g_ladder_host[m - kLadderMin];
            const int n = ladder_host(m, C, kLadderCap);
            for (int k = n; k < kLadderCap; ++k) C[k] = (uint64_t)1 << 32;
        }
        g_ladder_built = true;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return PA_ERR_HIP;
    if (dev < 31 && (g_ladder_device_mask >> dev) & 1) return PA_OK;
    if (hipMemcpyToSymbolAsync(HIP_SYMBOL(g_ladder), g_ladder_host, sizeof(g_ladder_host), 0,
                               hipMemcpyHostToDevice, s) != hipSuccess)
        return PA_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return PA_ERR_HIP;
    if (dev < 31) g_ladder_device_mask |= 1 << dev;
    return PA_OK;
}

// ------------------------------------------------------------------ kernels
// the histograms before the count; overlap: those of the overlaps too
__global__ void __launch_bounds__(256) k_hist_clear(pa_state* base, bool overlap)
{
    pa_state* st = base + blockIdx.y;
    if (overlap) clear_overlaps(st, blockIdx.x, gridDim.x);
    if (st->status) return;
    clear(st, blockIdx.x, gridDim.x);
}

constexpr int kHistLoads = 8;

// histogram of the current population's energies, counted in an LDS copy of cap_bins entries
// when the run's bins fit there (the LDS is sized for the call, whose runs may differ in size),
// else directly in global memory
__global__ void __launch_bounds__(256) k_hist(pa_state* base, int cap_bins)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    extern __shared__ uint32_t sh[];
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    int64_t* hist = work_ptr<int64_t>(st, wl.hist);
    int64_t* misc = work_ptr<int64_t>(st, wl.misc);
    const int nb = st->n_bins;
    const bool priv = nb <= cap_bins;
    const int64_t R = st->R;
    // a run takes only the blocks its energies fill (kHistLoads per thread): in a batch, a small
    // run left the rest to clear, scan and merge a histogram each for a few energies
    const int64_t per_block = (int64_t)blockDim.x * kHistLoads;
    const int nblk = (int)min((int64_t)gridDim.x, (R + per_block - 1) / per_block);
    if ((int)blockIdx.x >= nblk) return;  // the same for the whole block
    const int32_t* E = st->energy[st->cur];
    const int Eb = st->E_base;
    if (priv)
        for (int i = threadIdx.x; i < nb; i += blockDim.x) sh[i] = 0;
    __syncthreads();
    int emin = INT32_MAX, emax = INT32_MIN;
    // kHistLoads energies per thread are loaded before any of them is counted, so that many loads
    // are in flight at once (a load and its count in turn wait out the memory latency each time)
    const int64_t stride = (int64_t)nblk * blockDim.x;
    for (int64_t j0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j0 < R; j0 += kHistLoads * stride) {
        int e[kHistLoads];
#pragma unroll
        for (int u = 0; u < kHistLoads; ++u) e[u] = j0 + u * stride < R ? E[j0 + u * stride] : 0;
#pragma unroll
        for (int u = 0; u < kHistLoads; ++u) {
            if (j0 + u * stride >= R) break;
            const int b = (e[u] - Eb) >> 2;
            if (priv) atomicAdd(&sh[b], 1u);
            else atomicAdd((unsigned long long*)&hist[b], 1ull);
            emin = min(emin, e[u]);
            emax = max(emax, e[u]);
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        emin = min(emin, __shfl_xor(emin, off, 64));
        emax = max(emax, __shfl_xor(emax, off, 64));
    }
    if ((threadIdx.x & 63) == 0 && emin <= emax) {
        atomicMin((long long*)&misc[kMiscEmin], (long long)emin);
        atomicMax((long long*)&misc[kMiscEmax], (long long)emax);
    }
    __syncthreads();
    if (priv)
        for (int i = threadIdx.x; i < nb; i += blockDim.x)
            if (sh[i]) atomicAdd((unsigned long long*)&hist[i], (unsigned long long)sh[i]);
}

struct ResampleParams {
    double beta_from, beta_to, R_target;
    const double* w;
    int32_t k;
};

// S plus x[0 .. n - 1] in order by one thread, 16 LDS loads ahead of the chain of dependent additions
__device__ inline double add_in_order(double S, const double* x, int n)
{
    int i = 0;
    for (; i + 16 <= n; i += 16) {
        double c[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) c[u] = x[i + u];
#pragma unroll
        for (int u = 0; u < 16; ++u) S = S + c[u];
    }
    for (; i < n; ++i) S = S + x[i];
    return S;
}

constexpr int kNoCopies = 1000;  // the level of a bin of zero weight: no draws, copy number 0

// smallest m in [kLadderMin, kLadderMax] with 2^m >= x (0 < x <= 64)
__device__ inline int ladder_level(double x)
{
    int e;
    const double f = frexp(x, &e);
    const int m = (f == 0.5) ? e - 1 : e;
    return m < kLadderMin ? kLadderMin : m;
}

// one block: S in ascending energy order, ln Q, per-bin Poisson parameters (the step's record is
// written by k_finish, once the new population is known to fit)
constexpr int kNormBins = 1024;

__global__ void __launch_bounds__(256) k_normalise(pa_state* base, ResampleParams p)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    __shared__ double prod[kNormBins];
    __shared__ double S_sh;
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    const int64_t* hist = work_ptr<int64_t>(st, wl.hist);
    int64_t* misc = work_ptr<int64_t>(st, wl.misc);
    int64_t* bin_q = work_ptr<int64_t>(st, wl.bin_q);
    uint64_t* bin_keep = work_ptr<uint64_t>(st, wl.bin_keep);
    int32_t* bin_m = work_ptr<int32_t>(st, wl.bin_m);
    const int E_lo = (int)misc[kMiscEmin], E_hi = (int)misc[kMiscEmax];
    const int ilo = (E_lo - st->E_base) >> 2, ihi = (E_hi - st->E_base) >> 2;
    const int n = ihi - ilo + 1;
    const double dbeta = p.beta_to - p.beta_from;
    // S = sum_i h_i w_i, i ascending; products in parallel (each rounded once), sum by one thread
    double S = 0.0;
    for (int b0 = 0; b0 < n; b0 += kNormBins) {
        const int cnt = min(kNormBins, n - b0);
        for (int t = threadIdx.x; t < cnt; t += blockDim.x) prod[t] = (double)hist[ilo + b0 + t] * p.w[b0 + t];
        __syncthreads();
        if (threadIdx.x == 0) S = add_in_order(S, prod, cnt);
        __syncthreads();
    }
    if (threadIdx.x == 0) S_sh = S;
    __syncthreads();
    S = S_sh;
    const double R = (double)st->R;
    const double Rt = p.R_target > 0.0 ? p.R_target : (double)st->R0;
    const bool bad = !isfinite(S) || !(S > 0.0);
    if (threadIdx.x == 0) {
        const double lnQ = -dbeta * (double)E_lo + log(S) - log(R);
        *reinterpret_cast<double*>(&misc[kMiscElo]) = (double)E_lo;
        if (bad) {
            st->status |= PA_FLAG_NONFINITE;
        } else {
            *reinterpret_cast<double*>(&misc[kMiscLnQ]) = lnQ;
            *reinterpret_cast<double*>(&misc[kMiscS]) = S;
            st->E_lo = E_lo;
            st->E_hi = E_hi;
        }
    }
    if (bad) return;
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
        const double lam = (Rt * p.w[t]) / S;
        const int b = ilo + t;
        if (!(lam > 0.0)) {
            bin_q[b] = 0;
            bin_m[b] = kNoCopies;
            bin_keep[b] = 0;
            continue;
        }
        int64_t q = 0;
        double rem = lam;
        if (lam > 64.0) {
            q = (int64_t)ceil(lam / 64.0) - 1;
            rem = lam - 64.0 * (double)q;
        }
        const int m = ladder_level(rem);
        bin_q[b] = q;
        bin_m[b] = m;
        bin_keep[b] = (uint64_t)floor(ldexp(rem, 32 - m));
    }
}

// Poisson(2^m) by inversion: the smallest n with u < C[n] (C non-decreasing, its last entries 2^32 > u).
// The first 16 entries of the levels below 2^3, less one so that they fit 32 bits, are kept in LDS: eight
// at a time in two loads, counting the entries below u; a walk through the table waits out a load per
// step.  From 2^3 on, a branch-free binary search: n counts the entries <= u.
constexpr int kLowLevels = 3 - kLadderMin, kLowEntries = 16;

__device__ inline void load_low(uint32_t* low)
{
    for (int i = threadIdx.x; i < kLowLevels * kLowEntries; i += blockDim.x)
        low[i] = (uint32_t)(g_ladder[i / kLowEntries][i % kLowEntries] - 1);
}

__device__ inline int invert_ladder(int m, uint32_t u, const uint32_t* low)
{
    const uint64_t* C = g_ladder[m - kLadderMin];
    int n = 0;
    if (m < 3) {
        const uint4* L = reinterpret_cast<const uint4*>(low + (m - kLadderMin) * kLowEntries);
#pragma unroll
        for (int i = 0; i < kLowEntries / 8; ++i) {
            if (n < 8 * i) break;
            const uint4 a = L[2 * i], b = L[2 * i + 1];
            n += (u > a.x) + (u > a.y) + (u > a.z) + (u > a.w) + (u > b.x) + (u > b.y) + (u > b.z) + (u > b.w);
        }
        if (n == kLowEntries)
            while (!((uint64_t)u < C[n])) ++n;
        return n;
    }
    static_assert(kLadderCap == 256, "binary search over 256 entries");
#pragma unroll
    for (int step = 128; step > 0; step >>= 1)
        if (C[n + step - 1] <= (uint64_t)u) n += step;
    return n;
}

// Copy numbers: replica j's Poisson(lambda_j) count at step k is the sum of q Poisson(64) blocks and
// a Poisson(2^m) count K thinned by K draws against keep = rem 2^(32 - m).  Draw d (blocks d = 0 ..
// q - 1, K at d = q, the thinning draws at d = q + 1 ..) is word d mod 4 of Philox(d / 4, j, k, 4).
// Every lane finds its own K, and thins it itself up to kOwnDraws draws (most in the call that gave K);
// the wave takes the other lanes' draws together, a call per lane (the draws are counter-based, so any lane
// can make any of them, and the count is an integer sum).
// Walking the table in global memory draw by draw, with the wave on each lane of mean 8 and more in turn:
// 5 10^4 replicas of L = 8 at beta 0 14 us, 2 10^4 of L = 20 at beta 3 28 us, 10^6 of L = 16 31 us; this 9, 6.5, 22.
constexpr int kOwnDraws = 27;

struct CopyDraws {
    uint32_t j, k, k0, k1;
    __device__ uint4v call(uint32_t c) const { return philox10(c, j, k, kTagPoisson, k0, k1); }
};

// every lane of the wave calls this (lanes without a replica or copies with drawn = false); v0: call 0, made
// while the loads that lead to lambda are in flight
__device__ inline int64_t draw_copies(bool drawn, const CopyDraws& mine, uint4v v0, int m, int64_t q, uint64_t keep,
                                      const uint32_t* low)
{
    int64_t n = 0;
    int K = 0;
    if (drawn) {
        uint4v v = q < 4 ? v0 : mine.call((uint32_t)q >> 2);
        K = invert_ladder(m, word_of(v, (int)(q & 3)), low);
        if (q == 0 && K <= kOwnDraws) {
            n = (K > 0 && v.y < keep) + (K > 1 && v.z < keep) + (K > 2 && v.w < keep);
            for (int d = 4; d <= K; d += 4) {
                v = mine.call((uint32_t)d >> 2);
                n += (v.x < keep) + (d + 1 <= K && v.y < keep) + (d + 2 <= K && v.z < keep) + (d + 3 <= K && v.w < keep);
            }
        }
    }
    uint64_t todo = __ballot(drawn && (q > 0 || K > kOwnDraws));
    while (todo) {
        const int lane = (int)(threadIdx.x & 63), h = __builtin_ctzll(todo);
        todo &= todo - 1;
        CopyDraws cd = mine;
        cd.j = (uint32_t)__shfl((int)mine.j, h, 64);
        const int64_t qh = __shfl(q, h, 64);
        const uint64_t keeph = (uint64_t)__shfl((int64_t)keep, h, 64);
        const int64_t d0 = qh + 1, d1 = qh + __shfl(K, h, 64);  // the thinning draws
        int64_t part = 0;
        for (int64_t blk = lane; blk < qh; blk += 64)
            part += invert_ladder(kLadderMax, word_of(cd.call((uint32_t)blk >> 2), (int)(blk & 3)), low);
        for (int64_t c = (d0 >> 2) + lane; 4 * c <= d1; c += 64) {
            const uint4v v = cd.call((uint32_t)c);
#pragma unroll
            for (int w = 0; w < 4; ++w) part += 4 * c + w >= d0 && 4 * c + w <= d1 && word_of(v, w) < keeph;
        }
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
        if (lane == h) n = part;
    }
    return n;
}

// sum of the block's copy numbers into its tile's slot (every thread of the block calls this)
__device__ inline void tile_sum(const pa_state* st, int64_t c)
{
    __shared__ int64_t part[kScanTile / 64];
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x != 0) return;
    int64_t s = 0;
    for (int w = 0; w < kScanTile / 64; ++w) s += part[w];
    work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).scan)[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kScanTile) k_copies(pa_state* base, int32_t k)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t R = st->R;
    if ((int64_t)blockIdx.x * kScanTile >= R) return;  // the whole block past R
    __shared__ __attribute__((aligned(16))) uint32_t low[kLowLevels * kLowEntries];
    load_low(low);
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    const int64_t* bin_q = work_ptr<int64_t>(st, wl.bin_q);
    const uint64_t* bin_keep = work_ptr<uint64_t>(st, wl.bin_keep);
    const int32_t* bin_m = work_ptr<int32_t>(st, wl.bin_m);
    const bool live = j < R;
    const CopyDraws cd = {(uint32_t)j, (uint32_t)k, (uint32_t)st->seed, (uint32_t)(st->seed >> 32)};
    const uint4v v0 = cd.call(0);
    int m = kNoCopies;
    int64_t q = 0;
    uint64_t keep = 0;
    if (live) {
        const int b = (st->energy[st->cur][j] - st->E_base) >> 2;
        m = bin_m[b];
        if (m != kNoCopies) {
            q = bin_q[b];
            keep = bin_keep[b];
        }
    }
    __syncthreads();
    const int64_t n = draw_copies(live && m != kNoCopies, cd, v0, m, q, keep, low);
    const int32_t c = (int32_t)min(n, (int64_t)INT32_MAX);
    if (live) st->counts[j] = c;
    tile_sum(st, live ? c : 0);
}

// Offsets and sources, a block per tile of kScanTile consecutive sources.  The block adds the sums of the
// tiles before it (and all of them, for R~', which block 0 records, and for the capacity and extinction
// checks, which every block makes alike and k_finish turns into the flag), scans its own copy numbers into
// offsets[j] (offsets[R] = R~'), and its new replicas offsets[j0] .. offsets[j0 + 256] - 1 each find their
// source in the block's offsets in LDS (largest j with offsets[j] <= r', 8 LDS steps) and are written in
// order.  Per new replica over the whole array, the same search took ~20 dependent global loads; per
// source, the writes of uneven copy numbers were scattered and slower still.  As four launches (sums,
// their scan, offsets, sources) 27 us at 10^6 replicas and 16 at 5 10^4; this 16 (with the scan) and 5.
// SCANNED: k_scan_tiles has turned the sums into the copies before each tile, and the total after the last.
template <bool SCANNED>
__global__ void __launch_bounds__(kScanTile) k_offsets(pa_state* base)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    const int64_t R = st->R;
    const int64_t j0 = (int64_t)blockIdx.x * kScanTile;
    if (j0 >= R) return;
    __shared__ int64_t red[2][kScanTile / 64];
    __shared__ int64_t off[kScanTile + 1];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    const int64_t* sums = work_ptr<int64_t>(st, wl.scan);
    const int tiles = (int)((R + kScanTile - 1) / kScanTile), mine = (int)blockIdx.x;
    int64_t before = 0, total = 0;
    if constexpr (SCANNED) {
        before = sums[mine];
        total = sums[tiles];
    } else {
#pragma unroll 4
        for (int i = tid; i < tiles; i += kScanTile) {
            const int64_t v = sums[i];
            total += v;
            before += i < mine ? v : 0;
        }
        for (int o = 32; o > 0; o >>= 1) {
            total += __shfl_xor(total, o, 64);
            before += __shfl_xor(before, o, 64);
        }
        if (lane == 0) {
            red[0][wv] = total;
            red[1][wv] = before;
        }
        __syncthreads();
        total = before = 0;
        for (int w = 0; w < kScanTile / 64; ++w) {
            total += red[0][w];
            before += red[1][w];
        }
    }
    if (mine == 0 && tid == 0) st->R_new = total;
    if (total > st->capacity || total == 0) return;  // the same for every block
    const int64_t j = j0 + tid;
    const int64_t v = j < R ? st->counts[j] : 0;
    int64_t x = v;  // inclusive wave scan
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    __syncthreads();  // red has been read
    if (lane == 63) red[0][wv] = x;
    __syncthreads();
    int64_t pre = before;
    for (int w = 0; w < wv; ++w) pre += red[0][w];
    off[tid] = pre + x - v;
    if (tid == kScanTile - 1) off[kScanTile] = pre + x;
    if (j < R) st->offsets[j] = pre + x - v;
    if (j == R - 1) st->offsets[R] = total;
    __syncthreads();
    const int n = (int)(R - j0 < kScanTile ? R - j0 : kScanTile);
    int32_t* src = work_ptr<int32_t>(st, wl.src);
    for (int64_t d = before + tid; d < off[n]; d += kScanTile) {
        int lo = 0, hi = n;  // off[lo] <= d < off[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (off[mid] <= d) lo = mid;
            else hi = mid;
        }
        src[d] = (int32_t)(j0 + lo);
    }
}

// The exclusive scan of a run's tile sums in place, their total after them, by one block.
constexpr int kScanThreads = 1024, kScanLoads = 8;

__global__ void __launch_bounds__(kScanThreads) k_scan_tiles(pa_state* base)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    __shared__ int64_t red[kScanThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int tiles = (int)((st->R + kScanTile - 1) / kScanTile);
    int64_t* sums = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).scan);
    int64_t carry = 0;
    for (int i0 = 0; i0 < tiles; i0 += kScanThreads * kScanLoads) {
        const int first = i0 + tid * kScanLoads;
        int64_t v[kScanLoads], own = 0;
#pragma unroll
        for (int u = 0; u < kScanLoads; ++u) v[u] = first + u < tiles ? sums[first + u] : 0;
#pragma unroll
        for (int u = 0; u < kScanLoads; ++u) own += v[u];
        int64_t x = own;  // inclusive wave scan
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) red[wv] = x;
        __syncthreads();
        int64_t before = carry + x - own;
        for (int w = 0; w < kScanThreads / 64; ++w) {
            before += w < wv ? red[w] : 0;
            carry += red[w];
        }
#pragma unroll
        for (int u = 0; u < kScanLoads; ++u) {
            if (first + u < tiles) sums[first + u] = before;
            before += v[u];
        }
        __syncthreads();  // red has been read
    }
    if (tid == 0) sums[tiles] = carry;
}

// Every block adding all the sums grows with the square of the population, so from kDirectTiles tiles of the
// largest capacity on they are scanned first.  A whole resampling of L = 4, bit-packed, with the sums added
// and scanned: 2 10^5 replicas 39.0 and 39.9 us, 5 10^5 51.2 and 51.3, 10^6 70.7 and 67.1, 2 10^6 108 and 95,
// 10^7 926 and 378, 10^8 65.7 and 3.72 ms.
constexpr int64_t kDirectTiles = 2048;

static void launch_offsets(pa_state* base, int n, unsigned tiles, hipStream_t s)
{
    if (tiles <= kDirectTiles) {
        hipLaunchKernelGGL(k_offsets<false>, dim3(tiles, n), dim3(kScanTile), 0, s, base);
        return;
    }
    hipLaunchKernelGGL(k_scan_tiles, dim3(1, n), dim3(kScanThreads), 0, s, base);
    hipLaunchKernelGGL(k_offsets<true>, dim3(tiles, n), dim3(kScanTile), 0, s, base);
}

// whether the step's new population is to be formed (offsets has run, finish has not)
__device__ __forceinline__ bool accepted(const pa_state* st)
{
    return !st->status && st->R_new > 0 && st->R_new <= st->capacity;
}

// u8 gather: one thread per 16 bytes of a destination row; first: the first block of this part of the grid
__global__ void __launch_bounds__(256) k_gather_u8(pa_state* base, uint32_t first)
{
    pa_state* st = base + blockIdx.y;
    if (!accepted(st)) return;
    const int per_row = st->row_stride / 16;
    const int64_t t = (int64_t)(first + blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t rn = t / per_row;
    const int c = (int)(t - rn * per_row);
    if (rn >= st->R_new) return;
    const int32_t* src = work_ptr<int32_t>(st, work_layout(st->N, st->n_bins, st->capacity).src);
    const int64_t j = src[rn];
    const int cur = st->cur;
    const uint4* a = (const uint4*)((const uint8_t*)st->spins[cur] + j * st->row_stride) + c;
    uint4* b = (uint4*)((uint8_t*)st->spins[cur ^ 1] + rn * st->row_stride) + c;
    *b = *a;
    if (c == 0) {
        if (st->couplings == PA_GAUSS)
            reinterpret_cast<double*>(st->energy[cur ^ 1])[rn] = reinterpret_cast<const double*>(st->energy[cur])[j];
        else
            st->energy[cur ^ 1][rn] = st->energy[cur][j];
    }
}

// bit-packed gather of rows row0 .. row1 - 1 of one replica; a row word of replica j sits at
// (j/64 * n_rows + rho) * 64 + j mod 64 (row words of 1, 2 or 4 bytes by lattice size)
// (16 loads in flight per lane: one dependent load-store pair per row leaves the copy latency-
// bound, a few hundred bytes in flight per wave against the microseconds of HBM latency)
template <typename Wt>
__device__ inline void gather_rows(const pa_state* st, int64_t j, int64_t rn, int n_rows, int row0, int row1)
{
    constexpr int U = 16;
    const int cur = st->cur;
    const Wt* a = (const Wt*)st->spins[cur] + ((j >> 6) * n_rows) * 64 + (j & 63);
    Wt* b = (Wt*)st->spins[cur ^ 1] + ((rn >> 6) * n_rows) * 64 + (rn & 63);
    int rho = row0;
    for (; rho + U <= row1; rho += U) {
        Wt v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = a[(int64_t)(rho + u) * 64];
#pragma unroll
        for (int u = 0; u < U; ++u) b[(int64_t)(rho + u) * 64] = v[u];
    }
    for (; rho < row1; ++rho) b[(int64_t)rho * 64] = a[(int64_t)rho * 64];
}

// commit an accepted step: swap the buffers, accumulate ln Q (eq. sumQ) and write record[k]; a step
// refused by a sticky flag leaves state and records as they were
__device__ inline void commit_step(pa_state* st, const ResampleParams& p, double lnQ, double S, double E_lo)
{
    pa_record* rec = st->record + p.k;
    rec->beta = p.beta_to;
    rec->lnQ = lnQ;
    rec->minus_betaF = st->ln_omega + (st->acc + lnQ);
    rec->S = S;
    rec->R = (double)st->R_new;
    rec->E_lo = E_lo;
    st->acc = st->acc + lnQ;
    st->cur ^= 1;
    st->R = st->R_new;
    st->k = p.k;
    st->beta = p.beta_to;
}

__global__ void k_finish(pa_state* base, ResampleParams p)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    if (!accepted(st)) {
        st->status |= st->R_new > 0 ? PA_FLAG_CAPACITY : PA_FLAG_EXTINCT;
        return;
    }
    const int64_t* misc = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).misc);
    const double* kept = reinterpret_cast<const double*>(misc);
    commit_step(st, p, kept[kMiscLnQ], kept[kMiscS], kept[kMiscElo]);
}

// Launch shapes cover the largest run of the call; grid.y indexes the runs, whose states
// are contiguous (state r at runs[0].state + r).  A single run is n = 1.
struct BatchShape {
    int64_t cap_max = 0, pieces_max = 0, rows_max = 0;  // pieces: 16 bytes of a run's byte rows
};

static BatchShape batch_shape(const pa_run* runs, int n)
{
    BatchShape b;
    for (int r = 0; r < n; ++r) {
        pa_sizes sz;
        pa_buffer_sizes(runs[r].dim, runs[r].L, runs[r].layout, runs[r].couplings, runs[r].capacity, runs[r].n_records, &sz);
        b.cap_max = std::max(b.cap_max, runs[r].capacity);
        b.pieces_max = std::max(b.pieces_max, runs[r].capacity * (sz.row_stride / 16));
        b.rows_max = std::max<int64_t>(b.rows_max, runs[r].dim == 1 ? (runs[r].L + 31) / 32 : runs[r].L * runs[r].L);
    }
    return b;
}

// the energy histograms of n runs (overlap: those of their overlaps are cleared as well)
void launch_hist(const pa_run* runs, int n, bool overlap, hipStream_t s)
{
    const BatchShape b = batch_shape(runs, n);
    // an LDS histogram of up to 16384 bins, sized for the largest run of the call that fits (runs
    // with more bins count in global memory)
    int64_t cap_bins = 0;
    for (int r = 0; r < n; ++r) {
        pa_sizes sz;
        pa_buffer_sizes(runs[r].dim, runs[r].L, runs[r].layout, runs[r].couplings, runs[r].capacity, runs[r].n_records, &sz);
        if (sz.n_bins <= 16384) cap_bins = std::max(cap_bins, sz.n_bins);
    }
    // few blocks: each block zeroes and scans all bins of its LDS histogram and merges the occupied
    // ones with global atomics that land on the same few bins (L = 16, 1e6 replicas: 1024 blocks
    // 98 us, 256 blocks 29 us, 128 blocks 21 us; with eight loads in flight per thread, 128 blocks
    // 17.5 us, 256 blocks 28 us, and 64, 32, 16 blocks were slower already before)
    const unsigned hist_blocks = (unsigned)std::min<int64_t>(128, (b.cap_max + 255) / 256);
    hipLaunchKernelGGL(k_hist_clear, dim3(32, n), dim3(256), 0, s, runs[0].state, overlap);
    hipLaunchKernelGGL(k_hist, dim3(hist_blocks, n), dim3(256), (size_t)cap_bins * 4, s, runs[0].state, (int)cap_bins);
}

// Bit-packed gather, a block of kStageThreads consecutive destination replicas at a time.  The
// sources of consecutive destinations are non-decreasing, so the block's sources lie in a few
// consecutive source groups; row by row (kStageRows rows per pass) the block stages those groups'
// whole rows in LDS with 16-byte loads and each thread then takes its replica's word from LDS into
// the destination row.  A source row is read from HBM once per block instead of once per
// destination group that needs it (a group's sources straddle two source groups about a third of
// the time).  A block whose sources span more than kStageGroups groups (large copy numbers next to
// long runs of zeros) gathers per replica with gather_rows.
// A replica's rows are split over the blocks of grid.z, whole passes each, up to kGatherBlocks blocks in
// all: 2 10^4 replicas of L = 20 are 40 blocks of destinations, whose 400 rows in turn took 93 us (64 MB
// moved), split 14; 10^6 of L = 16 have blocks enough and take 205 us (1.02 GB) either way.
constexpr int kGatherBlocks = 2048;
constexpr int kStageThreads = 512;  // destination replicas per block (eight bit-packed groups)
constexpr int kStageGroups = 16;
constexpr int kStageRows = 8;

template <typename Wt>
__device__ __forceinline__ void gather_staged(pa_state* st, int rows_per, uint4* stage)
{
    constexpr int LPL = 64 * (int)sizeof(Wt) / 16;  // 16-byte pieces of a 64-replica row
    const int64_t R_new = st->R_new;
    const int64_t d0 = (int64_t)blockIdx.x * kStageThreads;
    if (d0 >= R_new) return;
    const int64_t d1 = d0 + kStageThreads - 1 < R_new ? d0 + kStageThreads - 1 : R_new - 1;
    const int32_t* src = work_ptr<int32_t>(st, work_layout(st->N, st->n_bins, st->capacity).src);
    const int64_t rn = d0 + threadIdx.x;
    const bool valid = rn < R_new;
    const int64_t j = valid ? src[rn] : 0;
    const int n_rows = st->dim == 1 ? (st->N + 31) / 32 : st->L * st->L;
    const int row0 = (int)blockIdx.z * rows_per, row1 = min(row0 + rows_per, n_rows);
    if (row0 >= row1) return;  // a small lattice of a batch
    const bool first = row0 == 0;  // moves the energies
    const int64_t g_lo = src[d0] >> 6, g_hi = src[d1] >> 6;  // the same for every thread
    const int cur = st->cur;
    if (g_hi - g_lo + 1 > kStageGroups) {
        if (valid) {
            gather_rows<Wt>(st, j, rn, n_rows, row0, row1);
            if (first) st->energy[cur ^ 1][rn] = st->energy[cur][j];
        }
        return;
    }
    const int nsrc = (int)(g_hi - g_lo + 1);
    const uint4* A = reinterpret_cast<const uint4*>((const Wt*)st->spins[cur] + g_lo * n_rows * 64);
    Wt* B = (Wt*)st->spins[cur ^ 1] + ((rn >> 6) * n_rows) * 64 + (rn & 63);
    const Wt* S = reinterpret_cast<const Wt*>(stage);
    const int64_t jl = j - g_lo * 64;  // the source's place among the staged groups' replicas
    const int jg = (int)(jl >> 6), jo = (int)(jl & 63);
    for (int r0 = row0; r0 < row1; r0 += kStageRows) {
        const int nr = row1 - r0 < kStageRows ? row1 - r0 : kStageRows;
        // staged piece e: group e / (nr LPL), row r0 + (e / LPL) mod nr, piece e mod LPL
        for (int e = threadIdx.x; e < nsrc * nr * LPL; e += kStageThreads) {
            const int line = e / LPL, part = e - line * LPL;
            const int gi = line / nr, q = line - gi * nr;
            stage[(gi * kStageRows + q) * LPL + part] = A[((int64_t)gi * n_rows + r0 + q) * LPL + part];
        }
        __syncthreads();
        if (valid) {
            for (int q = 0; q < nr; ++q) B[(int64_t)(r0 + q) * 64] = S[(jg * kStageRows + q) * 64 + jo];
        }
        __syncthreads();
    }
    if (valid && first) st->energy[cur ^ 1][rn] = st->energy[cur][j];
}

// one block of kStageThreads destinations of run blockIdx.y and a slice of its rows; the row word's width is the run's (a
// batch may mix lattice sizes), the staging buffer sized for the widest
__global__ void __launch_bounds__(kStageThreads, 8) k_gather_bits_staged(pa_state* base, int rows_per)
{
    __shared__ uint4 stage[kStageGroups * kStageRows * 16];
    pa_state* st = base + blockIdx.y;
    if (!accepted(st)) return;
    const int WB = st->dim == 1 ? 4 : (st->L <= 8 ? 1 : (st->L <= 16 ? 2 : 4));
    if (WB == 1) gather_staged<uint8_t>(st, rows_per, stage);
    else if (WB == 2) gather_staged<uint16_t>(st, rows_per, stage);
    else gather_staged<uint32_t>(st, rows_per, stage);
}

static void launch_gather(const pa_run* runs, int n, hipStream_t s)
{
    const BatchShape b = batch_shape(runs, n);
    pa_state* base = runs[0].state;
    if (runs[0].layout == PA_U8) {
        launch_parts((b.pieces_max + 255) / 256, 256, [&](uint32_t first, unsigned blocks) {
            hipLaunchKernelGGL(k_gather_u8, dim3(blocks, n), dim3(256), 0, s, base, first);
        });
    } else {
        const int64_t blocks = (b.cap_max + kStageThreads - 1) / kStageThreads;
        const int64_t passes = (b.rows_max + kStageRows - 1) / kStageRows;
        const int64_t slices = std::max<int64_t>(1, std::min(passes, kGatherBlocks / (blocks * n)));
        const int64_t per = (passes + slices - 1) / slices;  // passes of a slice
        const dim3 grid((unsigned)blocks, n, (unsigned)((passes + per - 1) / per));
        hipLaunchKernelGGL(k_gather_bits_staged, grid, dim3(kStageThreads), 0, s, base, (int)per * kStageRows);
    }
}

// ------------------------------------------------------------------ small populations
// +-1 runs of up to kSmallCap replicas and kSmallBins energy bins (every run of the call): a block per run
// does the whole resampling with the population's energies, weights, copy numbers and offsets in
// registers and LDS.  The chain of kernels above is bound by its launches there: ten of 3 to 5 us each for
// a few us of work (1000 rings of 64 sites: 36 us a step, this 9 us; the 200 runs of that ensemble 50 us,
// this 12 us).  Same histogram, sums in the same order, same draws.
// Bound by its own chain of latencies, so everything it reads is asked for at once: the state's fields
// (one by one where they are used, 14 us), energies, weights, rows; the replicas' first draws are made
// meanwhile.
// GATHER: the block also moves the rows and commits the step (byte rows of up to kSmallRows bytes per
// run); otherwise it leaves the source map and the step's ln Q and S for the gather kernel and k_finish.
constexpr int kSmallCap = 4096, kSmallBins = 8192, kSmallThreads = 1024, kSmallPer = kSmallCap / kSmallThreads;
constexpr int64_t kSmallRows = 192 << 10;
constexpr int kStagePieces = 4096;  // 16-byte pieces of rows kept in LDS (64 KB)
constexpr int kCommit = kSmallThreads - 1;  // the thread of the step's one-thread work, in the wave with the fewest replicas

// the parts of mean copy number lam: Poisson(64) blocks q, ladder level m and thinning threshold keep;
// false (no copies) unless lam > 0
__device__ inline bool poisson_parts(double lam, int* m, int64_t* q, uint64_t* keep)
{
    if (!(lam > 0.0)) return false;
    double rem = lam;
    *q = 0;
    if (lam > 64.0) {
        *q = (int64_t)ceil(lam / 64.0) - 1;
        rem = lam - 64.0 * (double)*q;
    }
    *m = ladder_level(rem);
    *keep = (uint64_t)floor(ldexp(rem, 32 - *m));
    return true;
}

// x combined over the wave's lanes up to each lane (DPP): a lane without a source combines with none
template <int CTRL, int ROWS, class F>
__device__ __forceinline__ int dpp_step(int x, int none, F f)
{
    return f(x, __builtin_amdgcn_update_dpp(none, x, CTRL, ROWS, 0xF, false));
}

template <class F>
__device__ __forceinline__ int wave_scan(int x, int none, F f)
{
    x = dpp_step<0x111, 0xF>(x, none, f);  // row_shr 1, 2, 4, 8, then the rows before
    x = dpp_step<0x112, 0xF>(x, none, f);
    x = dpp_step<0x114, 0xF>(x, none, f);
    x = dpp_step<0x118, 0xF>(x, none, f);
    x = dpp_step<0x142, 0xA>(x, none, f);
    return dpp_step<0x143, 0xC>(x, none, f);
}

// pointers known to be global: loads and stores through the state's pointers are flat ones, which the
// scalar loads after them wait for
template <typename T>
using glob = T __attribute__((address_space(1)))*;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool GATHER>
__global__ void __launch_bounds__(kSmallThreads) k_resample_small(pa_state* base, ResampleParams p)
{
    constexpr int kBig = 1 << 24;  // sums of 64 numbers below it fit 31 bits; larger ones overflow the run
    static_assert(kSmallCap < kBig && kSmallPer * (kSmallThreads / 64) == 64, "a lane per wave's total");
    pa_state* st = base + blockIdx.x;
    if (st->status) return;
    extern __shared__ double dyn[];  // products of a chunk of bins, the first weights, then the histogram
    __shared__ __attribute__((aligned(16))) uint32_t low[kLowLevels * kLowEntries];
    __shared__ uint16_t src_of[kSmallCap];
    __shared__ u32x4 stage[GATHER ? kStagePieces : 1];  // the first rows, asked for at the start
    __shared__ int64_t totals[64];  // copies of replicas 64 i ..
    __shared__ int lohi[2];
    __shared__ double S_sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the state's fields, all read at once
    int cur = st->cur, nb = st->n_bins, Eb = st->E_base, stride = st->row_stride, R = (int)st->R;
    int64_t capacity = st->capacity, R0 = st->R0;
    uint64_t seed = st->seed;
    int32_t *E0 = st->energy[0], *E1 = st->energy[1], *counts = st->counts;
    int64_t* offsets = st->offsets;
    void *s0 = st->spins[0], *s1 = st->spins[1];
    asm volatile("" : "+s"(cur), "+s"(nb), "+s"(Eb), "+s"(stride), "+s"(R), "+s"(capacity), "+s"(R0), "+s"(seed), "+s"(E0),
                 "+s"(E1), "+s"(counts), "+s"(offsets), "+s"(s0), "+s"(s1));
    const double Rt = p.R_target > 0.0 ? p.R_target : (double)R0;
    const CopyDraws cd0 = {0u, (uint32_t)p.k, (uint32_t)seed, (uint32_t)(seed >> 32)};
    const glob<int32_t> E = (glob<int32_t>)(cur ? E1 : E0), E_new = (glob<int32_t>)(cur ? E0 : E1);
    const int per_row = stride / 16;
    double* prod = dyn;
    double* w_sh = dyn + kSmallThreads;
    uint32_t* hist = reinterpret_cast<uint32_t*>(dyn + 2 * kSmallThreads);

    // the energies' histogram and range; everything that the kernel reads is asked for here
    int e[kSmallPer], lo = INT32_MAX, hi = INT32_MIN;
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) e[i] = tid + i * kSmallThreads < R ? E[tid + i * kSmallThreads] : 0;
    const double w_mine = tid < nb ? p.w[tid] : 0.0;
    uint4v v0[kSmallPer];  // the replicas' first draws
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        CopyDraws cd = cd0;
        cd.j = (uint32_t)(tid + i * kSmallThreads);
        if (i * kSmallThreads < R) v0[i] = cd.call(0);
    }
    const glob<u32x4> A = (glob<u32x4>)(cur ? s1 : s0), B = (glob<u32x4>)(cur ? s0 : s1);
    const int staged = GATHER ? min(R * per_row, kStagePieces) : 0;
    u32x4 rows[kStagePieces / kSmallThreads];
#pragma unroll
    for (int u = 0; u < kStagePieces / kSmallThreads; ++u)
        if (tid + u * kSmallThreads < staged) rows[u] = A[tid + u * kSmallThreads];
    const double lnR = tid == kCommit ? log((double)R) : 0.0;
    load_low(low);
    for (int b = tid; b < nb; b += kSmallThreads) hist[b] = 0;
    if (tid == 0) {
        lohi[0] = INT32_MAX;
        lohi[1] = INT32_MIN;
    }
    w_sh[tid] = w_mine;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        if (tid + i * kSmallThreads >= R) break;
        atomicAdd(&hist[(e[i] - Eb) >> 2], 1u);
        lo = min(lo, e[i]);
        hi = max(hi, e[i]);
    }
    lo = wave_scan(lo, INT32_MAX, [](int a, int b) { return min(a, b); });
    hi = wave_scan(hi, INT32_MIN, [](int a, int b) { return max(a, b); });
    if (lane == 63 && lo <= hi) {
        atomicMin(&lohi[0], lo);
        atomicMax(&lohi[1], hi);
    }
    __syncthreads();
    lo = lohi[0];
    hi = lohi[1];
    const int ilo = R > 0 ? (lo - Eb) >> 2 : 0, n = R > 0 ? ((hi - Eb) >> 2) - ilo + 1 : 0;

    // S, energies ascending (thread 0)
    double sum = 0.0;
    for (int b0 = 0; b0 < n; b0 += kSmallThreads) {
        if (b0 > 0) __syncthreads();  // the last chunk has been added
        if (b0 + tid < n) prod[tid] = (double)hist[ilo + b0 + tid] * (b0 == 0 ? w_mine : p.w[b0 + tid]);
        __syncthreads();
        if (tid == 0) sum = add_in_order(sum, prod, min(kSmallThreads, n - b0));
    }
    if (tid == 0) S_sh = sum;
    __syncthreads();
    const double S = S_sh;
    if (!isfinite(S) || !(S > 0.0)) {  // the same for the whole block
        if (tid == 0) st->status |= PA_FLAG_NONFINITE;
        return;
    }
    if (tid == 0) {
        st->E_lo = lo;
        st->E_hi = hi;
    }

#pragma unroll
    for (int u = 0; u < kStagePieces / kSmallThreads; ++u)
        if (tid + u * kSmallThreads < staged) stage[tid + u * kSmallThreads] = rows[u];

    // copy numbers c and, o, their exclusive sum within the wave
    int c[kSmallPer], o[kSmallPer];
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        c[i] = o[i] = 0;
        if (i * kSmallThreads >= R) {
            if (lane == 0) totals[i * (kSmallThreads / 64) + wave] = 0;
            continue;
        }
        const int j = tid + i * kSmallThreads, b = (e[i] - lo) >> 2;
        int m = kLadderMin;
        int64_t q = 0;
        uint64_t keep = 0;
        const double w = j < R ? (b < kSmallThreads ? w_sh[b] : p.w[b]) : 0.0;
        const bool drawn = poisson_parts((Rt * w) / S, &m, &q, &keep);
        CopyDraws cd = cd0;
        cd.j = (uint32_t)j;
        c[i] = (int32_t)min(draw_copies(drawn, cd, v0[i], m, q, keep, low), (int64_t)INT32_MAX);
        if (j < R) ((glob<int32_t>)counts)[j] = c[i];
        int64_t total;
        if (__ballot(c[i] >= kBig)) {
            total = c[i];
            for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
        } else {
            const int x = wave_scan(c[i], 0, [](int a, int b) { return a + b; });
            o[i] = x - c[i];
            total = x;  // lane 63's is the wave's
        }
        if (lane == 63) totals[i * (kSmallThreads / 64) + wave] = total;
    }
    __syncthreads();
    int64_t R_all = totals[lane];
    int before = (int)R_all;
    if (__ballot(R_all >= kBig)) {
        for (int off = 32; off > 0; off >>= 1) R_all += __shfl_xor(R_all, off, 64);
    } else {
        before = wave_scan(before, 0, [](int a, int b) { return a + b; });
        R_all = __builtin_amdgcn_readlane(before, 63);
        before -= (int)totals[lane];
    }
    const bool over = R_all > capacity;
    if (tid == 0) {
        st->R_new = R_all;
        if (over) st->status |= PA_FLAG_CAPACITY;
        else if (R_all == 0) st->status |= PA_FLAG_EXTINCT;
    }
    if (over || R_all == 0) return;  // the same for the whole block
    const int R_new = (int)R_all;

    // offsets, and each replica's place in the new population: its lane writes up to kOwnCopies copies, the
    // wave the rest of a replica with more
    constexpr int kOwnCopies = 8;
    const glob<int64_t> off_out = (glob<int64_t>)offsets;
    const WorkLayout wl = work_layout(st->N, nb, capacity);
    const glob<int32_t> src = (glob<int32_t>)work_ptr<int32_t>(st, wl.src);
    if (tid == 0) off_out[R] = R_new;
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        if (i * kSmallThreads >= R) break;
        const int j = tid + i * kSmallThreads;
        const int first = o[i] + __builtin_amdgcn_readlane(before, i * (kSmallThreads / 64) + wave);
        if (j < R) off_out[j] = first;
        auto put = [&](int d, int from, int energy) {
            if constexpr (GATHER) {
                src_of[d] = (uint16_t)from;
                E_new[d] = energy;
            } else {
                src[d] = from;
            }
        };
        for (int t = 0; t < min(c[i], kOwnCopies); ++t) put(first + t, j, e[i]);
        uint64_t todo = __ballot(c[i] > kOwnCopies);
        while (todo) {
            const int h = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int ch = __builtin_amdgcn_readlane(c[i], h), fh = __builtin_amdgcn_readlane(first, h);
            const int eh = __builtin_amdgcn_readlane(e[i], h);
            for (int t = kOwnCopies + lane; t < ch; t += 64) put(fh + t, j - lane + h, eh);
        }
    }
    const double E_lo = (double)lo;
    double lnQ = 0.0;
    auto set_lnQ = [&] {  // one thread's work (kept there: else every thread takes the logarithm)
        double x = S;
        asm volatile("" : "+v"(x));
        lnQ = -(p.beta_to - p.beta_from) * E_lo + log(x) - lnR;
    };
    if constexpr (!GATHER) {
        if (tid == kCommit) {
            set_lnQ();
            int64_t* misc = work_ptr<int64_t>(st, wl.misc);
            *reinterpret_cast<double*>(&misc[kMiscElo]) = E_lo;
            *reinterpret_cast<double*>(&misc[kMiscLnQ]) = lnQ;
            *reinterpret_cast<double*>(&misc[kMiscS]) = S;
        }
    } else {
        const int pieces = R_new * per_row;
        // t / per_row: exact, as (t + 0.5) / per_row is at least 0.5 / per_row from a whole number, against an error
        // of t / per_row 2^-22, and t < 12288
        const float inv = 1.0f / (float)per_row;
        __syncthreads();
        constexpr int U = 4;  // loads in flight per thread
        for (int t0 = tid; t0 - tid < pieces; t0 += U * kSmallThreads) {
            u32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + u * kSmallThreads, rn = (int)(((float)t + 0.5f) * inv);
                if (t >= pieces) continue;
                const int from = src_of[rn] * per_row + (t - rn * per_row);
                if (from < kStagePieces) v[u] = stage[from];
                else v[u] = A[from];
            }
            if (t0 == kCommit) set_lnQ();  // while the loads are in flight
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t0 + u * kSmallThreads < pieces) B[t0 + u * kSmallThreads] = v[u];
        }
        __syncthreads();  // every thread has read the state
        if (tid == kCommit) commit_step(st, p, lnQ, S, E_lo);
    }
}

// launches the resampling of small populations; false when a run of the call is not small
static bool launch_resample_small(const pa_run* runs, int n, const ResampleParams& p, hipStream_t s)
{
    int64_t cap = 0, bins = 0, rows = 0;
    for (int r = 0; r < n; ++r) {
        pa_sizes sz;
        pa_buffer_sizes(runs[r].dim, runs[r].L, runs[r].layout, runs[r].couplings, runs[r].capacity, runs[r].n_records, &sz);
        cap = std::max(cap, runs[r].capacity);
        bins = std::max(bins, sz.n_bins);
        rows = std::max(rows, runs[r].capacity * sz.row_stride);
    }
    if (cap > kSmallCap || bins > kSmallBins) return false;
    pa_state* base = runs[0].state;
    const bool gather = runs[0].layout == PA_U8 && rows <= kSmallRows;
    const size_t lds = kSmallThreads * 16 + (size_t)bins * 4;
    const dim3 g((unsigned)n), b(kSmallThreads);
    if (gather) hipLaunchKernelGGL(k_resample_small<true>, g, b, lds, s, base, p);
    else hipLaunchKernelGGL(k_resample_small<false>, g, b, lds, s, base, p);
    if (!gather) {
        launch_gather(runs, n, s);
        hipLaunchKernelGGL(k_finish, dim3(1, (unsigned)n), dim3(1), 0, s, base, p);
    }
    return true;
}

int launch_resample(const pa_run* runs, int n, const pa_step& step, hipStream_t s)
{
    const BatchShape b = batch_shape(runs, n);
    ResampleParams p;
    p.beta_from = step.beta_from;
    p.beta_to = step.beta_to;
    p.R_target = step.R_target;
    p.w = step.weights;
    p.k = step.k;
    if (launch_resample_small(runs, n, p, s)) return hip_status(hipGetLastError());
    pa_state* base = runs[0].state;
    const unsigned tiles = (unsigned)((b.cap_max + kScanTile - 1) / kScanTile);
    launch_hist(runs, n, false, s);
    hipLaunchKernelGGL(k_normalise, dim3(1, n), dim3(256), 0, s, base, p);
    hipLaunchKernelGGL(k_copies, dim3(tiles, n), dim3(kScanTile), 0, s, base, (int32_t)step.k);
    launch_offsets(base, n, tiles, s);
    launch_gather(runs, n, s);
    hipLaunchKernelGGL(k_finish, dim3(1, n), dim3(1), 0, s, base, p);
    return hip_status(hipGetLastError());
}

// ------------------------------------------------------------------ Gaussian couplings
// Real energies: per-replica weights instead of the energy histogram.  E_lo = min E (exact);
// w_j = expd(-(dbeta (E_j - E_lo))); S = sum of w_j over j = 0, 1, ... in replica order (eq. Q);
// ln Q = -dbeta E_lo + ln S - ln R~; copies of j ~ Poisson((R_target w_j) / S) by the same ladder
// and draws as the histogram path.  The weights are kept in the inactive energy buffer (FP64,
// [capacity]) between their evaluation and the copy numbers; the gather overwrites them.
constexpr int kMiscGaussS = kMiscS;  // misc slot: S (FP64 bits)

__global__ void __launch_bounds__(256) k_gauss_min(pa_state* base)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    __shared__ double red[256];
    const double* E = reinterpret_cast<const double*>(st->energy[st->cur]);
    double m = INFINITY;
    for (int64_t j = threadIdx.x; j < st->R; j += blockDim.x) m = fmin(m, E[j]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        int64_t* misc = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).misc);
        *reinterpret_cast<double*>(&misc[kMiscElo]) = red[0];
    }
}

// thread per replica: its weight w_j into the inactive energy buffer
__global__ void __launch_bounds__(256) k_gauss_weights(pa_state* base, double dbeta)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= st->R) return;
    const int64_t* misc = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).misc);
    const double E_lo = *reinterpret_cast<const double*>(&misc[kMiscElo]);
    const double* E = reinterpret_cast<const double*>(st->energy[st->cur]);
    double* w = reinterpret_cast<double*>(st->energy[st->cur ^ 1]);
    w[j] = expd(-(dbeta * (E[j] - E_lo)));
}

// ln Q and S of a step, kept for k_finish (one thread)
__device__ inline void gauss_keep(pa_state* st, const ResampleParams& p, int64_t* misc, double S, double E_lo)
{
    if (!isfinite(S) || !(S > 0.0)) {
        st->status |= PA_FLAG_NONFINITE;
        return;
    }
    *reinterpret_cast<double*>(&misc[kMiscLnQ]) = -(p.beta_to - p.beta_from) * E_lo + log(S) - log((double)st->R);
    *reinterpret_cast<double*>(&misc[kMiscGaussS]) = S;
}

// a block per run: S in replica order, ln Q (the step's record is written by k_finish).  The block
// loads the weights a chunk at a time into LDS with coalesced loads, and one thread adds them in order
constexpr int kNormChunk = 4096;

__global__ void __launch_bounds__(256) k_gauss_normalise(pa_state* base, ResampleParams p)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    __shared__ double chunk[kNormChunk];
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    int64_t* misc = work_ptr<int64_t>(st, wl.misc);
    const double* w = reinterpret_cast<const double*>(st->energy[st->cur ^ 1]);
    const int64_t R = st->R;
    double S = 0.0;
    for (int64_t j0 = 0; j0 < R; j0 += kNormChunk) {
        const int n = (int)(R - j0 < kNormChunk ? R - j0 : kNormChunk);
        for (int i = threadIdx.x; i < n; i += blockDim.x) chunk[i] = w[j0 + i];
        __syncthreads();
        if (threadIdx.x == 0) S = add_in_order(S, chunk, n);
        __syncthreads();
    }
    if (threadIdx.x == 0) gauss_keep(st, p, misc, S, *reinterpret_cast<const double*>(&misc[kMiscElo]));
}

// The three above for populations of up to kWeighCap replicas, a block per run with the weights in LDS: one
// launch instead of three (8 runs of 2000: 24 us as three, 21 as one, and two gaps between launches fewer).  With
// 512 threads it takes 15 us, but such blocks wait for room beside the other stream's sweeps where runs go
// in halves: a step of 200 chains is then 1.2% longer.
constexpr int kWeighCap = 8192, kWeighThreads = 256, kWeighLoads = 8;

__global__ void __launch_bounds__(kWeighThreads) k_gauss_weigh(pa_state* base, ResampleParams p)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    extern __shared__ double w_sh[];  // [capacity]
    __shared__ double red[kWeighThreads / 64];
    int64_t* misc = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).misc);
    const int R = (int)st->R;
    const glob<double> E = (glob<double>)st->energy[st->cur], w = (glob<double>)st->energy[st->cur ^ 1];
    double E_lo = INFINITY;
    for (int j0 = threadIdx.x; j0 < R; j0 += kWeighLoads * kWeighThreads) {
        double e[kWeighLoads];
#pragma unroll
        for (int u = 0; u < kWeighLoads; ++u) e[u] = E[min(j0 + u * kWeighThreads, R - 1)];
#pragma unroll
        for (int u = 0; u < kWeighLoads; ++u) {
            if (j0 + u * kWeighThreads < R) w_sh[j0 + u * kWeighThreads] = e[u];
            E_lo = fmin(E_lo, e[u]);
        }
    }
    for (int o = 32; o > 0; o >>= 1) E_lo = fmin(E_lo, __shfl_xor(E_lo, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = E_lo;
    __syncthreads();
    E_lo = red[0];
    for (int i = 1; i < kWeighThreads / 64; ++i) E_lo = fmin(E_lo, red[i]);
    const double dbeta = p.beta_to - p.beta_from;
#pragma unroll 4
    for (int j = threadIdx.x; j < R; j += kWeighThreads) w[j] = w_sh[j] = expd(-(dbeta * (w_sh[j] - E_lo)));
    __syncthreads();
    if (threadIdx.x != 0) return;
    *reinterpret_cast<double*>(&misc[kMiscElo]) = E_lo;
    gauss_keep(st, p, misc, add_in_order(0.0, w_sh, R), E_lo);
}

// copy numbers from the replica weights, drawn as in k_copies
__global__ void __launch_bounds__(kScanTile) k_gauss_copies(pa_state* base, ResampleParams p)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t R = st->R;
    if ((int64_t)blockIdx.x * kScanTile >= R) return;  // the whole block past R
    __shared__ __attribute__((aligned(16))) uint32_t low[kLowLevels * kLowEntries];
    load_low(low);
    const int64_t* misc = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).misc);
    const double S = *reinterpret_cast<const double*>(&misc[kMiscGaussS]);
    const double* w = reinterpret_cast<const double*>(st->energy[st->cur ^ 1]);
    const double Rt = p.R_target > 0.0 ? p.R_target : (double)st->R0;
    const bool live = j < R;
    const double lam = live ? (Rt * w[j]) / S : 0.0;
    int m = kLadderMin;
    int64_t q = 0;
    uint64_t keep = 0;
    const bool drawn = poisson_parts(lam, &m, &q, &keep);
    const CopyDraws cd = {(uint32_t)j, (uint32_t)p.k, (uint32_t)st->seed, (uint32_t)(st->seed >> 32)};
    const uint4v v0 = cd.call(0);
    __syncthreads();
    const int64_t n = draw_copies(drawn, cd, v0, m, q, keep, low);
    const int32_t c = (int32_t)min(n, (int64_t)INT32_MAX);
    if (live) st->counts[j] = c;
    tile_sum(st, live ? c : 0);
}

// runs: n runs with consecutive states on one stream (grid.y = run), or a single run
int launch_resample_gauss(const pa_run* runs, int n, const pa_step& step, hipStream_t s)
{
    ResampleParams p;
    p.beta_from = step.beta_from;
    p.beta_to = step.beta_to;
    p.R_target = step.R_target;
    p.w = nullptr;
    p.k = step.k;
    pa_state* base = runs[0].state;
    int64_t cap = 0;
    for (int r = 0; r < n; ++r) cap = std::max<int64_t>(cap, runs[r].capacity);
    const unsigned cap_blocks = (unsigned)((cap + 255) / 256);
    const unsigned tiles = (unsigned)((cap + kScanTile - 1) / kScanTile);
    const unsigned ny = (unsigned)n;
    if (cap <= kWeighCap) {
        hipLaunchKernelGGL(k_gauss_weigh, dim3(1, ny), dim3(kWeighThreads), (size_t)cap * 8, s, base, p);
    } else {
        hipLaunchKernelGGL(k_gauss_min, dim3(1, ny), dim3(256), 0, s, base);
        hipLaunchKernelGGL(k_gauss_weights, dim3(cap_blocks, ny), dim3(256), 0, s, base, step.beta_to - step.beta_from);
        hipLaunchKernelGGL(k_gauss_normalise, dim3(1, ny), dim3(256), 0, s, base, p);
    }
    hipLaunchKernelGGL(k_gauss_copies, dim3(tiles, ny), dim3(kScanTile), 0, s, base, p);
    launch_offsets(base, n, tiles, s);
    launch_gather(runs, n, s);
    hipLaunchKernelGGL(k_finish, dim3(1, ny), dim3(1), 0, s, base, p);
    return hip_status(hipGetLastError());
}

}  // namespace pa

extern "C" int pa_ladder_table(int m, uint64_t* C, int cap, int* len)
{
    if (!C || !len || cap < 2 || m < pa::kLadderMin || m > pa::kLadderMax) return PA_ERR_ARG;
    *len = pa::ladder_host(m, C, cap);
    return PA_OK;
}

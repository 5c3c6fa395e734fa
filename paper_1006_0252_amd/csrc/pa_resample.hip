// Resampling between temperatures (Sec. II, eqs. Q and wn; Poisson copy numbers with mean
// (R_target / R~) tau_j; the new population of R~' replicas).
//
// Chain of kernels on the run's stream, all sized by capacity and reading the population size
// from the device, with no host synchronisation:
//   hist      energy histogram h (width-4 bins from E_base), E_lo, E_hi      (integer atomics)
//   normalise S = sum_E h(E) w(E - E_lo) in ascending E (FP64, one thread, fixed order),
//             ln Q, and per bin the mean copy number lambda = R_target w / S split into
//             Poisson(64) blocks q, ladder level m and thinning threshold
//   copies    Poisson(lambda) per replica from its Philox stream (integer compares only), and the sum
//             of each tile of kScanTile replicas
//   offsets   exclusive scan of the copy numbers -> offsets, R~', capacity/extinction flags; source
//             replica of every new replica
//   gather    copy spins and energies into the other buffer
//   finish    swap buffers, R~ = R~', accumulate ln Q, record
// Every kernel is a no-op once the run's sticky status is set.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "pa_common.h"
#include "pa_host.h"

#pragma clang fp contract(off)

namespace pa {

// Poisson(2^m) inversion tables, m = kLadderMin .. kLadderMax (host-built, uploaded once)
__device__ uint64_t g_ladder[kLadderLevels][kLadderCap];

// int64 slots of the misc area: E_lo and E_hi of the population being resampled (FP64 bits of E_lo
// with Gaussian couplings), then ln Q and S of the step (FP64 bits), kept there until k_finish
// commits the step to the run's state and record
constexpr int kMiscEmin = 0, kMiscEmax = 1, kMiscLnQ = 2, kMiscS = 3;

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
__global__ void k_hist_clear(pa_state* base)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    int64_t* hist = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).hist);
    int64_t* misc = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).misc);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < st->n_bins; i += gridDim.x * blockDim.x) hist[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        misc[kMiscEmin] = INT32_MAX;
        misc[kMiscEmax] = INT32_MIN;
    }
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
__global__ void __launch_bounds__(256) k_normalise(pa_state* base, ResampleParams p)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    __shared__ double prod[1024];
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
    for (int b0 = 0; b0 < n; b0 += 1024) {
        const int cnt = min(1024, n - b0);
        for (int t = threadIdx.x; t < cnt; t += blockDim.x) prod[t] = (double)hist[ilo + b0 + t] * p.w[b0 + t];
        __syncthreads();
        if (threadIdx.x == 0)
            for (int t = 0; t < cnt; ++t) S = S + prod[t];
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
            bin_m[b] = 1000;  // no draws: copy number 0
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

// the smallest n with u < C[n] (C non-decreasing, its last entries 2^32 > u).  Small means walk
// the table from 0 (a few steps); from 2^3 on, a branch-free binary search: n counts the entries
// <= u, eight dependent loads instead of about 2^m (a Poisson(64) block took ~64)
__device__ inline int64_t invert_ladder(int m, uint32_t u)
{
    const uint64_t* C = g_ladder[m - kLadderMin];
    if (m < 3) {
        int64_t n = 0;
        while (!((uint64_t)u < C[n])) ++n;
        return n;
    }
    static_assert(kLadderCap == 256, "binary search over 256 entries");
    int n = 0;
#pragma unroll
    for (int step = 128; step > 0; step >>= 1)
        if (C[n + step - 1] <= (uint64_t)u) n += step;
    return n;
}

// Copy numbers: replica j's Poisson(lambda_j) count at step k is the sum of q Poisson(64) blocks and
// a Poisson(2^m) count K thinned by K draws against keep = rem 2^(32 - m).  Draw d (blocks d = 0 ..
// q - 1, K at d = q, the thinning draws at d = q + 1 ..) is word d mod 4 of Philox(d / 4, j, k, 4).
// Light lanes (no blocks, 2^m < 16) draw in turn; the wave takes each heavy lane's draws
// together, spread over its 64 lanes (the draws are counter-based, so any lane can make any of
// them, and the count is an integer sum), instead of waiting for one lane to make them one by one.
constexpr int kCopiesHeavyM = 4;

struct CopyDraws {
    uint32_t j, k, k0, k1;
    __device__ uint32_t at(uint32_t d) const
    {
        return word_of(philox10(d >> 2, j, k, kTagPoisson, k0, k1), (int)(d & 3));
    }
};

__device__ inline int64_t copies_light(const CopyDraws& cd, int m, uint64_t keep)
{
    uint32_t d = 0;
    uint4v v = {0, 0, 0, 0};
    auto draw = [&]() -> uint32_t {
        if ((d & 3) == 0) v = philox10(d >> 2, cd.j, cd.k, kTagPoisson, cd.k0, cd.k1);
        const uint32_t u = word_of(v, d & 3);
        ++d;
        return u;
    };
    const int64_t K = invert_ladder(m, draw());
    int64_t n = 0;
    for (int64_t e = 0; e < K; ++e)
        if ((uint64_t)draw() < keep) ++n;
    return n;
}

// every lane of the wave calls this (lanes without a replica with heavy = false); returns the
// count of a heavy lane's replica, n unchanged elsewhere
__device__ inline int64_t copies_heavy_by_wave(bool heavy, int64_t n, const CopyDraws& mine, int m, int64_t q,
                                               uint64_t keep)
{
    const int lane = (int)(threadIdx.x & 63);
    uint64_t todo = __ballot(heavy);
    while (todo) {
        const int h = __builtin_ctzll(todo);
        todo &= todo - 1;
        CopyDraws cd = mine;
        cd.j = (uint32_t)__shfl((int)mine.j, h, 64);
        const int mh = __shfl(m, h, 64);
        const int64_t qh = __shfl(q, h, 64);
        const uint64_t keeph = (uint64_t)__shfl((int64_t)keep, h, 64);
        int64_t part = 0;
        for (int64_t blk = lane; blk < qh; blk += 64) part += invert_ladder(kLadderMax, cd.at((uint32_t)blk));
        const int64_t K = invert_ladder(mh, cd.at((uint32_t)qh));
        for (int64_t e = lane; e < K; e += 64)
            if ((uint64_t)cd.at((uint32_t)(qh + 1 + e)) < keeph) ++part;
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
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    const int64_t* bin_q = work_ptr<int64_t>(st, wl.bin_q);
    const uint64_t* bin_keep = work_ptr<uint64_t>(st, wl.bin_keep);
    const int32_t* bin_m = work_ptr<int32_t>(st, wl.bin_m);
    const bool live = j < R;
    int m = 1000;  // bins of zero weight carry m = 1000: no copies
    int64_t q = 0;
    uint64_t keep = 0;
    if (live) {
        const int b = (st->energy[st->cur][j] - st->E_base) >> 2;
        m = bin_m[b];
        if (m != 1000) {
            q = bin_q[b];
            keep = bin_keep[b];
        }
    }
    const CopyDraws cd = {(uint32_t)j, (uint32_t)k, (uint32_t)st->seed, (uint32_t)(st->seed >> 32)};
    const bool drawn = live && m != 1000;
    const bool heavy = drawn && (q > 0 || m >= kCopiesHeavyM);
    int64_t n = drawn && !heavy ? copies_light(cd, m, keep) : 0;
    n = copies_heavy_by_wave(heavy, n, cd, m, q, keep);
    const int32_t c = (int32_t)min(n, (int64_t)INT32_MAX);
    if (live) st->counts[j] = c;
    tile_sum(st, live ? c : 0);
}

// Offsets and sources, a block per tile of kScanTile consecutive sources.  The block adds the sums of the
// tiles before it (and all of them, for R~' and the capacity and extinction checks, which every block
// makes alike and block 0 records), scans its own copy numbers into offsets[j] (offsets[R] = R~'), and its
// new replicas offsets[j0] .. offsets[j0 + 256] - 1 each find their source in the block's offsets in LDS
// (largest j with offsets[j] <= r', 8 LDS steps) and are written in order.  Per new replica over the whole
// array, the same search took ~20 dependent global loads; per source, the writes of uneven copy numbers
// were scattered and slower still.  As separate launches (sums, their scan, offsets, sources) 27 us at
// 10^6 replicas and four launches of 4 us at 5 10^4; this 18 and 5.
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
    const bool over = total > st->capacity;
    if (mine == 0 && tid == 0) {
        st->R_new = total;
        if (over) st->status |= PA_FLAG_CAPACITY;
        else if (total == 0) st->status |= PA_FLAG_EXTINCT;
    }
    if (over || total == 0) return;  // the same for every block
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

// u8 gather: one thread per 16 bytes of a destination row
__global__ void __launch_bounds__(256) k_gather_u8(pa_state* base)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    const int per_row = st->row_stride / 16;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
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
    const int64_t* misc = work_ptr<int64_t>(st, work_layout(st->N, st->n_bins, st->capacity).misc);
    const double E_lo = st->couplings == PA_GAUSS ? *reinterpret_cast<const double*>(&misc[kMiscEmin])
                                                  : (double)misc[kMiscEmin];
    commit_step(st, p, *reinterpret_cast<const double*>(&misc[kMiscLnQ]), *reinterpret_cast<const double*>(&misc[kMiscS]), E_lo);
}

// Launch shapes cover the largest run of the call; grid.y indexes the runs, whose states
// are contiguous (state r at runs[0].state + r).  A single run is n = 1.
struct BatchShape {
    int64_t cap_max = 0, stride_max = 0, rows_max = 0;
};

static BatchShape batch_shape(const pa_run* runs, int n)
{
    BatchShape b;
    for (int r = 0; r < n; ++r) {
        pa_sizes sz;
        pa_buffer_sizes(runs[r].dim, runs[r].L, runs[r].layout, runs[r].couplings, runs[r].capacity, runs[r].n_records, &sz);
        b.cap_max = std::max(b.cap_max, runs[r].capacity);
        b.stride_max = std::max(b.stride_max, sz.row_stride);
        b.rows_max = std::max<int64_t>(b.rows_max, runs[r].dim == 1 ? (runs[r].L + 31) / 32 : runs[r].L * runs[r].L);
    }
    return b;
}

int launch_hist(const pa_run* runs, int n, hipStream_t s)
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
    const size_t hist_lds = (size_t)cap_bins * 4;
    // few blocks: each block zeroes and scans all bins of its LDS histogram and merges the occupied
    // ones with global atomics that land on the same few bins (L = 16, 1e6 replicas: 1024 blocks
    // 98 us, 256 blocks 29 us, 128 blocks 21 us; with eight loads in flight per thread, 128 blocks
    // 17.5 us, 256 blocks 28 us, and 64, 32, 16 blocks were slower already before)
    const unsigned hist_blocks = (unsigned)std::min<int64_t>(128, (b.cap_max + 255) / 256);
    hipLaunchKernelGGL(k_hist_clear, dim3(32, n), dim3(256), 0, s, runs[0].state);
    hipLaunchKernelGGL(k_hist, dim3(hist_blocks, n), dim3(256), hist_lds, s, runs[0].state, (int)cap_bins);
    return PA_OK;
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
    if (st->status) return;
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
        const int64_t threads = b.cap_max * (b.stride_max / 16);
        hipLaunchKernelGGL(k_gather_u8, dim3((unsigned)((threads + 255) / 256), n), dim3(256), 0, s, base);
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
// +-1 runs of up to kSmallCap replicas and kSmallBins energy bins (every run of the call): a block per run does the whole resampling with the population's energies, weights, copy
// numbers and offsets in registers and LDS.  The chain of kernels above is bound by its launches there:
// ten of 3 to 5 us each for a few us of work (1000 rings of 64 sites: 36 us a step, this 13 us; the 200 runs
// of that ensemble 50 us, this 17 us).  Same histogram, sums in the same order, same draws.
// GATHER: the block also moves the rows and commits the step (byte rows of up to kSmallRows bytes per
// run); otherwise it leaves the source map and the step's ln Q and S for the gather kernel and k_finish.
constexpr int kSmallCap = 4096, kSmallBins = 8192, kSmallThreads = 1024, kSmallPer = kSmallCap / kSmallThreads;
constexpr int64_t kSmallRows = 192 << 10;

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

template <typename T, class F>
__device__ __forceinline__ T block_reduce(T x, T* red, F f)
{
    for (int o = 32; o > 0; o >>= 1) x = f(x, __shfl_xor(x, o, 64));
    __syncthreads();  // red may be in use
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    T v = red[0];
    for (int w = 1; w < kSmallThreads / 64; ++w) v = f(v, red[w]);
    return v;
}

template <bool GATHER>
__global__ void __launch_bounds__(kSmallThreads) k_resample_small(pa_state* base, ResampleParams p)
{
    pa_state* st = base + blockIdx.x;
    if (st->status) return;
    extern __shared__ double dyn[];  // products of a chunk of bins, then the histogram
    __shared__ int32_t off[kSmallCap + 1];
    __shared__ uint16_t src_of[kSmallCap];
    __shared__ int64_t red[kSmallThreads / 64];
    __shared__ double S_sh;
    const int tid = threadIdx.x;
    const int R = (int)st->R;
    const int cur = st->cur;
    const double dbeta = p.beta_to - p.beta_from;
    const double Rt = p.R_target > 0.0 ? p.R_target : (double)st->R0;
    const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
    int64_t* misc = work_ptr<int64_t>(st, wl.misc);

    // E_lo, the weights and S in its fixed order
    double wt[kSmallPer];
    double* prod = dyn;
    uint32_t* hist = reinterpret_cast<uint32_t*>(dyn + kSmallThreads);
    const int32_t* E = st->energy[cur];
    const int nb = st->n_bins, Eb = st->E_base;
    int e[kSmallPer], lo = INT32_MAX, hi = INT32_MIN;
    for (int b = tid; b < nb; b += kSmallThreads) hist[b] = 0;
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        const int j = tid + i * kSmallThreads;
        e[i] = j < R ? E[j] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        if (tid + i * kSmallThreads >= R) break;
        atomicAdd(&hist[(e[i] - Eb) >> 2], 1u);
        lo = min(lo, e[i]);
        hi = max(hi, e[i]);
    }
    int* redi = reinterpret_cast<int*>(red);
    lo = block_reduce(lo, redi, [](int a, int b) { return min(a, b); });
    hi = block_reduce(hi, redi, [](int a, int b) { return max(a, b); });
    const double E_lo = (double)lo;
    const int ilo = R > 0 ? (lo - Eb) >> 2 : 0, n = R > 0 ? ((hi - Eb) >> 2) - ilo + 1 : 0;
    double sum = 0.0;  // energies ascending (thread 0)
    for (int b0 = 0; b0 < n; b0 += kSmallThreads) {
        if (b0 + tid < n) prod[tid] = (double)hist[ilo + b0 + tid] * p.w[b0 + tid];
        __syncthreads();
        if (tid == 0) {
            const int cnt = min(kSmallThreads, n - b0);
            for (int t = 0; t < cnt; ++t) sum = sum + prod[t];
        }
        __syncthreads();
    }
    if (tid == 0) S_sh = sum;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) wt[i] = tid + i * kSmallThreads < R ? p.w[(e[i] - lo) >> 2] : 0.0;
    if (tid == 0 && isfinite(sum) && sum > 0.0) {
        st->E_lo = lo;
        st->E_hi = hi;
    }
    const double S = S_sh;
    if (!isfinite(S) || !(S > 0.0)) {  // the same for the whole block
        if (tid == 0) st->status |= PA_FLAG_NONFINITE;
        return;
    }

    // copy numbers and their exclusive scan, 1024 replicas at a time in order
    const CopyDraws cd0 = {0u, (uint32_t)p.k, (uint32_t)st->seed, (uint32_t)(st->seed >> 32)};
    int64_t carry = 0;
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        if (i * kSmallThreads >= R) break;
        const int j = tid + i * kSmallThreads;
        const bool live = j < R;
        int m = kLadderMin;
        int64_t q = 0;
        uint64_t keep = 0;
        const bool drawn = live && poisson_parts((Rt * wt[i]) / S, &m, &q, &keep);
        CopyDraws cd = cd0;
        cd.j = (uint32_t)j;
        const bool heavy = drawn && (q > 0 || m >= kCopiesHeavyM);
        int64_t n = drawn && !heavy ? copies_light(cd, m, keep) : 0;
        n = copies_heavy_by_wave(heavy, n, cd, m, q, keep);
        const int32_t c = (int32_t)min(n, (int64_t)INT32_MAX);
        if (live) st->counts[j] = c;
        int64_t x = live ? c : 0;  // inclusive wave scan
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(x, o, 64);
            if ((tid & 63) >= o) x += y;
        }
        __syncthreads();
        if ((tid & 63) == 63) red[tid >> 6] = x;
        __syncthreads();
        int64_t pre = carry, all = 0;
        for (int w = 0; w < kSmallThreads / 64; ++w) {
            if (w < (tid >> 6)) pre += red[w];
            all += red[w];
        }
        const int64_t o = pre + x - (live ? c : 0);
        if (live) off[j] = (int32_t)min(o, (int64_t)INT32_MAX);
        carry += all;
    }
    if (tid == 0) {
        st->R_new = carry;
        if (carry > st->capacity) st->status |= PA_FLAG_CAPACITY;
        else if (carry == 0) st->status |= PA_FLAG_EXTINCT;
    }
    if (carry > st->capacity || carry == 0) return;  // the same for the whole block
    const int R_new = (int)carry;
    if (tid == 0) off[R] = R_new;
    __syncthreads();
    for (int j = tid; j <= R; j += kSmallThreads) st->offsets[j] = off[j];

    // the source of each new replica: the largest j with off[j] <= d
    int32_t* src = work_ptr<int32_t>(st, wl.src);
    for (int d = tid; d < R_new; d += kSmallThreads) {
        int lo = 0, hi = R;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (off[mid] <= d) lo = mid;
            else hi = mid;
        }
        if (GATHER) src_of[d] = (uint16_t)lo;
        else src[d] = lo;
    }
    const double lnQ = -dbeta * E_lo + log(S) - log((double)R);
    if constexpr (!GATHER) {
        if (tid == 0) {
            misc[kMiscEmin] = lo;
            *reinterpret_cast<double*>(&misc[kMiscLnQ]) = lnQ;
            *reinterpret_cast<double*>(&misc[kMiscS]) = S;
        }
        return;
    } else {
        __syncthreads();
        const int per_row = st->row_stride / 16, pieces = R_new * per_row;
        const uint4* A = reinterpret_cast<const uint4*>(st->spins[cur]);
        uint4* B = reinterpret_cast<uint4*>(st->spins[cur ^ 1]);
        constexpr int U = 4;  // loads in flight per thread
        for (int t0 = tid; t0 < pieces; t0 += U * kSmallThreads) {
            uint4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + u * kSmallThreads, rn = t / per_row;
                if (t < pieces) v[u] = A[src_of[rn] * per_row + (t - rn * per_row)];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t0 + u * kSmallThreads < pieces) B[t0 + u * kSmallThreads] = v[u];
        }
        for (int d = tid; d < R_new; d += kSmallThreads) st->energy[cur ^ 1][d] = st->energy[cur][src_of[d]];
        __syncthreads();  // every thread has read the state
        if (tid == 0) commit_step(st, p, lnQ, S, E_lo);
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
    const size_t lds = kSmallThreads * 8 + (size_t)bins * 4;
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
    launch_hist(runs, n, s);
    hipLaunchKernelGGL(k_normalise, dim3(1, n), dim3(256), 0, s, base, p);
    hipLaunchKernelGGL(k_copies, dim3(tiles, n), dim3(kScanTile), 0, s, base, (int32_t)step.k);
    hipLaunchKernelGGL(k_offsets, dim3(tiles, n), dim3(kScanTile), 0, s, base);
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
        *reinterpret_cast<double*>(&misc[kMiscEmin]) = red[0];
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
    const double E_lo = *reinterpret_cast<const double*>(&misc[kMiscEmin]);
    const double* E = reinterpret_cast<const double*>(st->energy[st->cur]);
    double* w = reinterpret_cast<double*>(st->energy[st->cur ^ 1]);
    w[j] = expd(-(dbeta * (E[j] - E_lo)));
}

// a block per run: S in replica order, ln Q (the step's record is written by k_finish).  The block
// loads the weights a chunk at a time into LDS with coalesced loads, and one thread adds them in
// order from there, 16 LDS loads ahead of the chain of dependent FP64 additions
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
        if (threadIdx.x == 0) {
            int i = 0;
            for (; i + 16 <= n; i += 16) {
                double c[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) c[u] = chunk[i + u];
#pragma unroll
                for (int u = 0; u < 16; ++u) S = S + c[u];
            }
            for (; i < n; ++i) S = S + chunk[i];
        }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double dbeta = p.beta_to - p.beta_from;
    const double E_lo = *reinterpret_cast<const double*>(&misc[kMiscEmin]);
    if (!isfinite(S) || !(S > 0.0)) {
        st->status |= PA_FLAG_NONFINITE;
        return;
    }
    *reinterpret_cast<double*>(&misc[kMiscLnQ]) = -dbeta * E_lo + log(S) - log((double)R);
    *reinterpret_cast<double*>(&misc[kMiscGaussS]) = S;
}

// copy numbers from the replica weights, drawn as in k_copies
__global__ void __launch_bounds__(kScanTile) k_gauss_copies(pa_state* base, ResampleParams p)
{
    pa_state* st = base + blockIdx.y;
    if (st->status) return;
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t R = st->R;
    if ((int64_t)blockIdx.x * kScanTile >= R) return;  // the whole block past R
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
    const bool heavy = drawn && (q > 0 || m >= kCopiesHeavyM);
    int64_t n = drawn && !heavy ? copies_light(cd, m, keep) : 0;
    n = copies_heavy_by_wave(heavy, n, cd, m, q, keep);
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
    hipLaunchKernelGGL(k_gauss_min, dim3(1, ny), dim3(256), 0, s, base);
    hipLaunchKernelGGL(k_gauss_weights, dim3(cap_blocks, ny), dim3(256), 0, s, base, step.beta_to - step.beta_from);
    hipLaunchKernelGGL(k_gauss_normalise, dim3(1, ny), dim3(256), 0, s, base, p);
    hipLaunchKernelGGL(k_gauss_copies, dim3(tiles, ny), dim3(kScanTile), 0, s, base, p);
    hipLaunchKernelGGL(k_offsets, dim3(tiles, ny), dim3(kScanTile), 0, s, base);
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

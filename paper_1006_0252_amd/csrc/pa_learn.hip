// Learned temperature steps: population features, resampled-fraction step labels, and the
// 6-64-64-64-1 network that proposes the next dbeta (forward, loss gradient, Adam).
//
// The paper leaves the schedule to the user (Sec. II: every temperature sequence gives an
// exact method; Sec. III: Var(beta F~) measures how well it worked).  Here a network reads
// (beta, ln N, ln R, E/N, var E/N, skew E) of the population and proposes dbeta; it is
// trained towards the step at which the resampling of Sec. II (normalised weights tau_j,
// eq. wn) replaces a fixed fraction rho* of the population.  Resampling itself is unchanged,
// so every schedule the network produces is an exact schedule.
#include <math.h>

#include <mutex>
#include <type_traits>

#include "pa_common.h"
#include "pa_hist.h"
#include "pa_host.h"

namespace pa {

// ------------------------------------------------------------------ network geometry
constexpr int kIn = 6, kH = 64;
constexpr int kOffW1 = 0, kOffB1 = 384, kOffW2 = 448, kOffB2 = 4544, kOffW3 = 4608, kOffB3 = 8704, kOffW4 = 8768,
              kOffB4 = 8832, kParams = 8833;
static_assert(kOffB4 + 1 == kParams && kParams == PA_MLP_PARAMS, "parameter layout");

// Work memory of a gradient: the formula of pa_mlp_work_bytes is part of the interface and larger than the
// partial gradients need (kTile samples per tile, one partial of kParams + 1 floats per block of at most
// kMaxBlocks).
constexpr int kRows = 396;
constexpr int kChunk = 1024;
constexpr int64_t kMaxSamples = (int64_t)65535 * kChunk;  // samples of a gradient (more are refused)
constexpr int kTile = 32;
constexpr int kMaxBlocks = 512;

__host__ __device__ inline int64_t mlp_ld(int64_t B) { return (B + 63) & ~(int64_t)63; }
__host__ __device__ inline int64_t mlp_chunks(int64_t B) { return (B + kChunk - 1) / kChunk; }
__host__ inline int64_t mlp_tiles(int64_t B) { return (B + kTile - 1) / kTile; }
static_assert((kParams + 1) * (64 / kTile) <= kRows * 64, "the partial gradients of 64 samples fit their work memory");

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// round to nearest, ties to even; NaN -> quiet NaN
__device__ inline uint16_t f32_to_bf16(float x)
{
    const uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return 0x7FC0;
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// fixed affine input map (the same for every trained network)
__device__ inline void normalise(const float* x, float* xh)
{
    xh[0] = (x[0] - 2.5f) / 2.5f;    // beta
    xh[1] = (x[1] - 6.0f) / 2.0f;    // ln N
    xh[2] = (x[2] - 10.0f) / 2.5f;   // ln R
    xh[3] = x[3] + 1.0f;             // E / N
    xh[4] = x[4] - 1.0f;             // var E / N
    xh[5] = x[5] / 2.0f;             // skew E
}

__device__ inline float softplus(float z) { return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z))); }
__device__ inline float sigmoid(float z) { return 1.0f / (1.0f + expf(-z)); }

// ------------------------------------------------------------------ forward and gradient
// A block of four waves takes tiles of 32 samples through the whole network: the weights in LDS as FP32, the
// layers as FP32 matrix products on the matrix cores (v_mfma_f32_16x16x4_f32: wave w computes rows 16 w ..
// 16 w + 15 of every layer), activations and deltas of the tile in LDS.  With TRAIN the outer products of
// deltas and layer inputs accumulate in registers over the block's tiles, and the block writes one partial
// gradient; k_mlp_grad_sum adds the partials in block order.  All sums have a fixed order.
//
// Bound by the latency of one tile's chain of layers: at B = 10160 (318 tiles, one per block) the matrix
// products take 3 us, the weights' way to LDS, tanh and the LDS round trips between layers the rest of 27.
// One sample per lane, its activations in registers and the per-sample matrices written to memory for 40
// blocks of outer products, took 131 + 706 us a gradient, this 27 + 5.

typedef float f32x4 __attribute__((ext_vector_type(4)));

// LDS pitches: the lanes of an operand read (row l mod 16, column l / 16, or the other way round) spread over
// the banks
constexpr int kPitchW = 68, kPitchW1 = 12, kPitchS = 36;

struct MlpSmem {
    float W2[kH * kPitchW], W3[kH * kPitchW], W1[kH * kPitchW1];  // W1: columns 6, 7 zero
    float b1[kH], b2[kH], b3[kH], w4[kH];
    float X[8 * kPitchS];                                          // normalised inputs, rows 6, 7 zero
    float H1[kH * kPitchS], H2[kH * kPitchS], H3[kH * kPitchS], D[kH * kPitchS];
    float part[8 * kTile], gz[kTile], ls[kTile];
    float b4;
};

// C (+)= A B over K columns for the wave's 16 rows and n tiles of 16 columns; lane l supplies A[l mod 16][k +
// l / 16] = a(k) and B[k + l / 16][16 t + l mod 16] = b(t, k), and holds C[4 (l / 16) + i][16 t + l mod 16]
template <int K, int NT, class FA, class FB>
__device__ __forceinline__ void mfma_tiles(f32x4 (&acc)[NT], FA a, FB b)
{
#pragma unroll
    for (int k = 0; k < K; k += 4) {
        const float av = a(k);
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, b(t, k), acc[t], 0, 0, 0);
    }
}

template <bool TRAIN>
__global__ void __launch_bounds__(256) k_mlp(const uint16_t* __restrict__ w, const float* __restrict__ x, int64_t B,
                                             float dmin, float dmax, float* __restrict__ out,
                                             const double* __restrict__ target, float* __restrict__ partial)
{
    __shared__ MlpSmem sm;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lk = lane >> 4;   // operand row or column, and k offset
    const int j0 = 16 * wave;                   // the wave's rows
    for (int p = tid; p < kH * kIn; p += 256) sm.W1[(p / kIn) * kPitchW1 + p % kIn] = bf16_to_f32(w[kOffW1 + p]);
    for (int p = tid; p < kH * kH; p += 256) {
        sm.W2[(p >> 6) * kPitchW + (p & 63)] = bf16_to_f32(w[kOffW2 + p]);
        sm.W3[(p >> 6) * kPitchW + (p & 63)] = bf16_to_f32(w[kOffW3 + p]);
    }
    if (tid < kH) {
        sm.W1[tid * kPitchW1 + 6] = sm.W1[tid * kPitchW1 + 7] = 0.0f;
        sm.b1[tid] = bf16_to_f32(w[kOffB1 + tid]);
        sm.b2[tid] = bf16_to_f32(w[kOffB2 + tid]);
        sm.b3[tid] = bf16_to_f32(w[kOffB3 + tid]);
        sm.w4[tid] = bf16_to_f32(w[kOffW4 + tid]);
        if (tid == 0) sm.b4 = bf16_to_f32(w[kOffB4]);
    }
    // gradient sums over the block's tiles: W3, W2 (rows j0 .., four column tiles), W1 (one), and per thread one
    // row of w4 / b3 / b2 / b1 (threads 0.., 64.., 128.., 192..); thread 0 adds b4 and the loss
    f32x4 g3[4] = {}, g2[4] = {}, g1[1] = {};
    float g_vec = 0.0f, g_b4 = 0.0f, g_loss = 0.0f;

    for (int64_t tile = blockIdx.x; tile * kTile < B; tile += gridDim.x) {
        const int64_t b0 = tile * kTile;
        __syncthreads();  // the weights; the last tile's readers
        if (tid < kTile) {
            float xr[kIn], xh[kIn];
#pragma unroll
            for (int k = 0; k < kIn; ++k) xr[k] = b0 + tid < B ? x[(b0 + tid) * kIn + k] : 0.0f;
            normalise(xr, xh);
#pragma unroll
            for (int k = 0; k < 8; ++k) sm.X[k * kPitchS + tid] = k < kIn ? xh[k] : 0.0f;
        }
        __syncthreads();
        // out[j][s] = tanh(bias[j] + sum_i W[j][i] in[i][s])
        auto layer = [&](auto K, const float* W, int pitch, const float* bias, const float* in, float* o) {
            f32x4 acc[2];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[0][i] = acc[1][i] = bias[j0 + 4 * lk + i];
            mfma_tiles<decltype(K)::value, 2>(
                acc, [&](int k) { return W[(j0 + lr) * pitch + k + lk]; },
                [&](int t, int k) { return in[(k + lk) * kPitchS + 16 * t + lr]; });
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) o[(j0 + 4 * lk + i) * kPitchS + 16 * t + lr] = tanhf(acc[t][i]);
            __syncthreads();
        };
        layer(std::integral_constant<int, 8>{}, sm.W1, kPitchW1, sm.b1, sm.X, sm.H1);
        layer(std::integral_constant<int, kH>{}, sm.W2, kPitchW, sm.b2, sm.H1, sm.H2);
        layer(std::integral_constant<int, kH>{}, sm.W3, kPitchW, sm.b3, sm.H2, sm.H3);
        {
            const int s = tid & 31, q = tid >> 5;
            float z = 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) z = fmaf(sm.w4[8 * q + i], sm.H3[(8 * q + i) * kPitchS + s], z);
            sm.part[q * kTile + s] = z;
        }
        __syncthreads();
        if (tid < kTile) {
            float z = sm.b4;
#pragma unroll
            for (int q = 0; q < 8; ++q) z += sm.part[q * kTile + tid];
            const int64_t b = b0 + tid;
            const float ln_n = b < B ? x[b * kIn + 1] : 0.0f, v = b < B ? x[b * kIn + 4] : 0.0f;
            const bool has_sigma = v > 0.0f;
            const float log_sigma = has_sigma ? 0.5f * (ln_n + logf(v)) : 0.0f;
            const float sp = softplus(z);
            if (!TRAIN) {
                float d = has_sigma ? sp * expf(-log_sigma) : dmax;
                d = d != d ? dmax : fminf(fmaxf(d, dmin), dmax);
                if (b < B) out[b] = d;
            } else {
                const double t = b < B ? target[b] : 0.0;
                const bool valid = has_sigma && t > 0.0 && t <= 1.0e300;
                float gz = 0.0f, ls = 0.0f;
                if (valid) {
                    const float err = logf(sp) - log_sigma - (float)log(t);
                    ls = err * err / (float)B;
                    gz = (2.0f / (float)B) * err * sigmoid(z) / sp;
                }
                sm.gz[tid] = gz;
                sm.ls[tid] = ls;
            }
        }
        if constexpr (TRAIN) {
            __syncthreads();
            // delta3 = gz w4 (1 - h3^2)
            for (int e = tid; e < kH * kTile; e += 256) {
                const int j = e >> 5, s = e & 31;
                const float h = sm.H3[j * kPitchS + s];
                sm.D[j * kPitchS + s] = sm.gz[s] * sm.w4[j] * (1.0f - h * h);
            }
            // row sums of a matrix of the tile by 64 threads
            auto row_sum = [&](const float* M, int r) {
                float v = 0.0f;
#pragma unroll
                for (int s = 0; s < kTile; ++s) v += M[r * kPitchS + s];
                return v;
            };
            if (wave == 0) {
                float v = 0.0f;
#pragma unroll
                for (int s = 0; s < kTile; ++s) v = fmaf(sm.gz[s], sm.H3[lane * kPitchS + s], v);
                g_vec += v;
            }
            if (tid == 0) {
#pragma unroll
                for (int s = 0; s < kTile; ++s) {
                    g_b4 += sm.gz[s];
                    g_loss += sm.ls[s];
                }
            }
            __syncthreads();
            // G[a][c] += sum_s D[a][s] in[c][s]
            auto outer = [&](auto& acc, const float* D, const float* in) {
                mfma_tiles<kTile>(
                    acc, [&](int k) { return D[(j0 + lr) * kPitchS + k + lk]; },
                    [&](int t, int k) { return in[(16 * t + lr) * kPitchS + k + lk]; });
            };
            // d[i][s] = (sum_j W[j][i] D[j][s]) (1 - h[i][s]^2)
            auto back = [&](const float* W, const float* D, const float* h, float* d) {
                f32x4 acc[2] = {};
                mfma_tiles<kH, 2>(
                    acc, [&](int k) { return W[(k + lk) * kPitchW + j0 + lr]; },
                    [&](int t, int k) { return D[(k + lk) * kPitchS + 16 * t + lr]; });
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int e = (j0 + 4 * lk + i) * kPitchS + 16 * t + lr;
                        d[e] = acc[t][i] * (1.0f - h[e] * h[e]);
                    }
                __syncthreads();
            };
            if (wave == 1) g_vec += row_sum(sm.D, lane);
            outer(g3, sm.D, sm.H2);
            back(sm.W3, sm.D, sm.H2, sm.H3);  // delta2 in H3's place
            if (wave == 2) g_vec += row_sum(sm.H3, lane);
            outer(g2, sm.H3, sm.H1);
            back(sm.W2, sm.H3, sm.H1, sm.D);  // delta1 in delta3's place
            if (wave == 3) g_vec += row_sum(sm.D, lane);
            // the inputs' 8 rows as a tile of 16 (rows past them: zero)
            mfma_tiles<kTile>(
                g1, [&](int k) { return sm.D[(j0 + lr) * kPitchS + k + lk]; },
                [&](int, int k) { return lr < 8 ? sm.X[lr * kPitchS + k + lk] : 0.0f; });
        }
    }
    if constexpr (TRAIN) {
        float* o = partial + (int64_t)blockIdx.x * (kParams + 1);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = (j0 + 4 * lk + i) * kH + 16 * t + lr;
                o[kOffW3 + e] = g3[t][i];
                o[kOffW2 + e] = g2[t][i];
            }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (lr < kIn) o[kOffW1 + (j0 + 4 * lk + i) * kIn + lr] = g1[0][i];
        const int off = wave == 0 ? kOffW4 : (wave == 1 ? kOffB3 : (wave == 2 ? kOffB2 : kOffB1));
        o[off + lane] = g_vec;
        if (tid == 0) {
            o[kOffB4] = g_b4;
            o[kParams] = g_loss;
        }
    }
}

// grad[p] = sum over the partials: 16 slices of every 16th partial each, then the slices in order; the loss sum
// goes to loss[0]
constexpr int kSumSlices = 16;

__global__ void __launch_bounds__(64 * kSumSlices) k_mlp_grad_sum(const float* __restrict__ partial, int n,
                                                                  float* __restrict__ grad, float* __restrict__ loss)
{
    __shared__ float part[kSumSlices][64];
    const int c = threadIdx.x & 63, slice = threadIdx.x >> 6, p = blockIdx.x * 64 + c;
    float s = 0.0f;
    if (p <= kParams) {
#pragma unroll 8
        for (int i = slice; i < n; i += kSumSlices) s += partial[(int64_t)i * (kParams + 1) + p];
    }
    part[slice][c] = s;
    __syncthreads();
    if (slice != 0 || p > kParams) return;
    s = 0.0f;
#pragma unroll
    for (int i = 0; i < kSumSlices; ++i) s += part[i][c];
    if (p < kParams) grad[p] = s;
    else if (loss) loss[0] = s;
}

// Adam (Kingma and Ba, ICLR 2015): FP32 master weights and moments, BF16 copy for the network
__global__ void k_adam(float* __restrict__ theta, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ grad, uint16_t* __restrict__ w, int64_t n, float bc1, float bc2,
                       float lr, float beta1, float beta2, float eps)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const float g = grad[p];
    const float mp = beta1 * m[p] + (1.0f - beta1) * g;
    const float vp = beta2 * v[p] + (1.0f - beta2) * (g * g);
    m[p] = mp;
    v[p] = vp;
    const float th = theta[p] - lr * (mp / bc1) / (sqrtf(vp / bc2) + eps);
    theta[p] = th;
    w[p] = f32_to_bf16(th);
}

__global__ void k_bf16_round(const float* __restrict__ x, uint16_t* __restrict__ out, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = f32_to_bf16(x[i]);
}

// ------------------------------------------------------------------ population side

// x[r] = (beta, ln N, ln R, E_mean / N, E_var / N, E_skew) of record[k] of run r
__global__ void k_features(const pa_state* base, int n, float* __restrict__ x)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const pa_state* st = base + r;
    const pa_record* rec = st->record + st->k;
    const double N = (double)st->N;
    float* o = x + (int64_t)r * kIn;
    o[0] = (float)st->beta;
    o[1] = (float)log(N);
    o[2] = (float)log((double)st->R);
    o[3] = (float)(rec->E_mean / N);
    o[4] = (float)(rec->E_var / N);
    o[5] = (float)rec->E_skew;
}

constexpr int kMaxRho = 8;
struct RhoArgs { double v[kMaxRho]; };

// block-wide sum in a fixed order (256 lanes)
__device__ inline double block_sum(double x, double* red)
{
    const int t = threadIdx.x;
    red[t] = x;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// rho(dbeta) = 1 - (1/R) sum over energy bins i of h_i min(1, R w_i / S), w_i = exp(-4 dbeta (i - ilo)),
// S = sum_i h_i w_i (the population's normalised weights tau of eq. wn, per energy)
__device__ double rho_of(const int64_t* hist, int ilo, int ihi, double R, double dbeta, double* red)
{
    double s = 0.0;
    for (int i = ilo + threadIdx.x; i <= ihi; i += blockDim.x) {
        const int64_t h = hist[i];
        if (h) s += (double)h * exp(-4.0 * dbeta * (double)(i - ilo));
    }
    const double S = block_sum(s, red);
    double kept = 0.0;
    for (int i = ilo + threadIdx.x; i <= ihi; i += blockDim.x) {
        const int64_t h = hist[i];
        if (h) kept += (double)h * fmin(1.0, R * exp(-4.0 * dbeta * (double)(i - ilo)) / S);
    }
    return 1.0 - block_sum(kept, red) / R;
}

// mode 0: out[r * n + j] = rho(arg_j); mode 1: out[j * ld + r] = dbeta with rho = arg_j in [0, cap]
// (64 halvings; cap when rho(cap) <= arg_j).  NaN for runs with a raised status bit.
__global__ void __launch_bounds__(256) k_rho(pa_state* base, RhoArgs args, int n_args, int mode, double cap,
                                             int64_t ld, double* __restrict__ out)
{
    __shared__ double red[256];
    const pa_state* st = base + blockIdx.y;
    const int j = blockIdx.x;
    double result;
    if (st->status) {
        result = NAN;
    } else {
        const WorkLayout wl = work_layout(st->N, st->n_bins, st->capacity);
        const int64_t* h = work_ptr<int64_t>(st, wl.hist);
        const int64_t* misc = work_ptr<int64_t>(st, wl.misc);
        const int ilo = (int)((misc[hist::kMiscEmin] - st->E_base) >> 2), ihi = (int)((misc[hist::kMiscEmax] - st->E_base) >> 2);
        const double R = (double)st->R;
        if (mode == 0) {
            result = rho_of(h, ilo, ihi, R, args.v[j], red);
        } else if (rho_of(h, ilo, ihi, R, cap, red) <= args.v[j]) {
            result = cap;
        } else {
            double lo = 0.0, hi = cap;
            for (int it = 0; it < 64; ++it) {
                const double mid = 0.5 * (lo + hi);
                if (rho_of(h, ilo, ihi, R, mid, red) < args.v[j]) lo = mid;
                else hi = mid;
            }
            result = 0.5 * (lo + hi);
        }
    }
    if (threadIdx.x == 0) {
        if (mode == 0) out[(int64_t)blockIdx.y * n_args + j] = result;
        else out[(int64_t)j * ld + blockIdx.y] = result;
    }
}

int launch_features(const pa_run* runs, int n, float* x, hipStream_t s)
{
    hipLaunchKernelGGL(k_features, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, (const pa_state*)runs[0].state,
                       n, x);
    return hip_status(hipGetLastError());
}

int launch_rho(const pa_run* runs, int n, const double* args, int n_args, int mode, double cap, int64_t ld,
               double* out, hipStream_t s)
{
    RhoArgs a;
    for (int j = 0; j < kMaxRho; ++j) a.v[j] = j < n_args ? args[j] : 0.0;
    launch_hist(runs, n, false, s);
    hipLaunchKernelGGL(k_rho, dim3((unsigned)n_args, (unsigned)n), dim3(256), 0, s, runs[0].state, a, n_args, mode,
                       cap, ld, out);
    return hip_status(hipGetLastError());
}

// The loss gradient of a batch of at most kStaticMaxB samples with its partial gradients in a fixed device
// array (of pa_mlp_work_bytes' size) instead of caller memory, for callers that cannot allocate.
// Every call on a device shares that device's array: calls that overlap on one GPU race.  Nothing
// in it needs clearing between calls (every element a call reads, it has written first).
constexpr int64_t kStaticMaxB = 4096;
constexpr int64_t kStaticFloats = (int64_t)kRows * kStaticMaxB + ((kStaticMaxB + kChunk - 1) / kChunk) * (kParams + 1);
static __device__ __align__(256) float scratch[kStaticFloats];

constexpr int kMaxDevices = 64;
static float* g_scratch_dev[kMaxDevices];  // device address of `scratch` on each device, once looked up
static std::mutex g_scratch_lock;

// the current device's address of `scratch` (the host-side name is not a device address)
static int scratch_address(float** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PA_ERR_HIP;
    std::lock_guard<std::mutex> g(g_scratch_lock);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PA_ERR_HIP;
        g_scratch_dev[dev] = (float*)p;
    }
    *out = g_scratch_dev[dev];
    return PA_OK;
}

// the kernels of pa_mlp_grad on a given work area
static int mlp_grad_launch(const uint16_t* w, const float* x, const double* target, int64_t B, float* wk, float* grad,
                           float* loss, hipStream_t s)
{
    if (B > kMaxSamples) return PA_ERR_ARG;
    const int64_t tiles = mlp_tiles(B);
    const int blocks = (int)(tiles < kMaxBlocks ? tiles : kMaxBlocks);
    hipLaunchKernelGGL(k_mlp<true>, dim3((unsigned)blocks), dim3(256), 0, s, w, x, B, 0.0f, 0.0f, (float*)nullptr, target,
                       wk);
    hipLaunchKernelGGL(k_mlp_grad_sum, dim3((kParams + 1 + 63) / 64), dim3(64 * kSumSlices), 0, s, (const float*)wk, blocks,
                       grad, loss);
    return hip_status(hipGetLastError());
}

}  // namespace pa

using namespace pa;

extern "C" int pa_mlp_work_bytes(int64_t B, int64_t* bytes)
{
    if (B <= 0 || !bytes) return PA_ERR_ARG;
    *bytes = (int64_t)kRows * mlp_ld(B) * 4 + mlp_chunks(B) * (int64_t)(kParams + 1) * 4;
    return PA_OK;
}

extern "C" int pa_mlp_forward(const uint16_t* w, const float* x, int64_t B, float dbeta_min, float dbeta_max,
                              float* dbeta, void* stream)
{
    if (!w || !x || !dbeta || B <= 0 || B > ((int64_t)1 << 30)) return PA_ERR_ARG;
    if (!(dbeta_min >= 0.0f) || !(dbeta_max >= dbeta_min) || !isfinite(dbeta_max)) return PA_ERR_ARG;
    const int64_t tiles = mlp_tiles(B);
    hipLaunchKernelGGL(k_mlp<false>, dim3((unsigned)(tiles < kMaxBlocks ? tiles : kMaxBlocks)), dim3(256), 0,
                       (hipStream_t)stream, w, x, B,
                       dbeta_min, dbeta_max, dbeta, (const double*)nullptr, (float*)nullptr);
    return hip_status(hipGetLastError());
}

extern "C" int pa_mlp_grad(const uint16_t* w, const float* x, const double* target, int64_t B, void* work,
                           float* grad, float* loss, void* stream)
{
    if (!w || !x || !target || !work || !grad || B <= 0 || B > ((int64_t)1 << 30)) return PA_ERR_ARG;
    return mlp_grad_launch(w, x, target, B, (float*)work, grad, loss, (hipStream_t)stream);
}

extern "C" int pa_mlp_grad_static(const uint16_t* w, const float* x, const double* target, int64_t B, float* grad,
                                  float* loss, void* stream)
{
    if (!w || !x || !target || !grad || B <= 0) return PA_ERR_ARG;
    if (B > kStaticMaxB) return PA_ERR_SIZE;
    float* wk = nullptr;
    const int st = scratch_address(&wk);
    if (st != PA_OK) return st;
    return mlp_grad_launch(w, x, target, B, wk, grad, loss, (hipStream_t)stream);
}

extern "C" int pa_mlp_adam(float* theta, float* m, float* v, const float* grad, uint16_t* w, int64_t n, int t,
                           float lr, float beta1, float beta2, float eps, void* stream)
{
    if (!theta || !m || !v || !grad || !w || n <= 0 || t < 1) return PA_ERR_ARG;
    if (!(lr > 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps >= 0.0f))
        return PA_ERR_ARG;
    // bias corrections 1 - beta^t of the moment estimates
    const float bc1 = (float)(1.0 - pow((double)beta1, (double)t));
    const float bc2 = (float)(1.0 - pow((double)beta2, (double)t));
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, theta, m, v, grad,
                       w, n, bc1, bc2, lr, beta1, beta2, eps);
    return hip_status(hipGetLastError());
}

extern "C" int pa_bf16_round(const float* x, uint16_t* out, int64_t n, void* stream)
{
    if (!x || !out || n <= 0) return PA_ERR_ARG;
    hipLaunchKernelGGL(k_bf16_round, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, x, out, n);
    return hip_status(hipGetLastError());
}

// Gaussian couplings (the model of Sec. IV: J_ij normal with mean 0 and variance 1).
// Energies are real numbers, so the path fixes every floating-point step in order and in the
// operations used: couplings drawn on the host (Box-Muller, libm), energies summed in bond order
// and recomputed after every call of sweeps, local fields summed in incident-bond order, the
// acceptance probability floor(expd(-beta dE) 2^64) / 2^64 with exp written out (expd), and no
// fused multiply-adds.  Population layout: one byte per spin.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "pa_common.h"
#include "pa_hist.h"
#include "pa_host.h"
#include "pa_lattice.h"
#include "pa_sweep_strings.h"
#include "pa_sweep_util.h"

#pragma clang fp contract(off)

namespace pa {

// ------------------------------------------------------------------ host: couplings
// Philox4x32-10 (Salmon et al., SC'11), host side
static void philox_host(uint32_t c[4], uint32_t k0, uint32_t k1)
{
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
        c[1] = (uint32_t)p1;
        c[3] = (uint32_t)p0;
        c[0] = n0;
        c[2] = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// J_b = sqrt(-2 ln u1) cos(2 pi u2) from Philox(ctr (b, 0, 0, 6), key disorder seed): u1 from
// the top 27 + 26 bits of words 0, 1 (plus one, so u1 > 0), u2 from words 2, 3
static void couplings_host(uint64_t seed, std::vector<double>& J)
{
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    for (size_t b = 0; b < J.size(); ++b) {
        uint32_t w[4] = {(uint32_t)b, 0u, 0u, 6u};
        philox_host(w, k0, k1);
        const uint64_t m1 = ((uint64_t)(w[0] >> 5) << 26) | (uint64_t)(w[1] >> 6);
        const uint64_t m2 = ((uint64_t)(w[2] >> 5) << 26) | (uint64_t)(w[3] >> 6);
        const double u1 = ldexp((double)(m1 + 1), -53);
        const double u2 = ldexp((double)m2, -53);
        J[b] = sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
    }
}

// the couplings of run blockIdx.y from those of run src.run[blockIdx.y] (the same realization)
__global__ void __launch_bounds__(256) k_copy_couplings(pa_state* base, BatchOrder src)
{
    const pa_state* st = base + blockIdx.y;
    const int from = src.run[blockIdx.y];
    if (from == (int)blockIdx.y) return;
    const double* a = reinterpret_cast<const double*>(base[from].J);
    double* b = reinterpret_cast<double*>(st->J);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < st->n_bonds; i += gridDim.x * blockDim.x) b[i] = a[i];
}

// Couplings of n runs with consecutive states, the states already written on s.  Up to kMaxBatch runs at
// a time, a realization that several of them share is drawn and uploaded once (for its first run) and
// copied on the device for the others.
int gauss_couplings_upload(const pa_run* runs, int n, hipStream_t s)
{
    for (int r0 = 0; r0 < n; r0 += kMaxBatch) {
        const int m = n - r0 < kMaxBatch ? n - r0 : kMaxBatch;
        const pa_run* q = runs + r0;
        BatchOrder src;
        std::vector<std::vector<double>> J;
        J.reserve((size_t)m);
        int64_t most = 0;
        bool copies = false;
        for (int r = 0; r < m; ++r) {
            int from = 0;
            while (from < r && !(src.run[from] == from && q[from].L == q[r].L && q[from].disorder_seed == q[r].disorder_seed)) ++from;
            src.run[r] = (uint16_t)from;
            const int64_t B = q[r].dim == 1 ? q[r].L : 3 * (int64_t)q[r].L * q[r].L * q[r].L;
            most = B > most ? B : most;
            if (from != r) {
                copies = true;
                continue;
            }
            J.emplace_back((size_t)B);
            couplings_host(q[r].disorder_seed, J.back());
            if (hipMemcpyAsync(q[r].J, J.back().data(), (size_t)B * 8, hipMemcpyHostToDevice, s) != hipSuccess) {
                (void)hipStreamSynchronize(s);  // the copies before it read the host vectors
                return PA_ERR_HIP;
            }
        }
        if (copies)
            hipLaunchKernelGGL(k_copy_couplings, dim3((unsigned)((most + 255) / 256), (unsigned)m), dim3(256), 0, s,
                               runs[r0].state, src);
        // the host vectors are released on return
        if (hipStreamSynchronize(s) != hipSuccess) return PA_ERR_HIP;
    }
    return PA_OK;
}

// ------------------------------------------------------------------ device helpers
__device__ inline int gauss_colour(const pa_state* st, int i)
{
    if (st->dim == 1) return i & 1;
    const int L = st->L;
    return ((i % L) + (i / L) % L + i / (L * L)) & 1;
}

// E = sum over bonds b = 0, 1, ... of J_b s_i s_j, in bond order from 0 (s = 1 means sigma = -1)
__device__ double energy_gauss(const pa_state* st, const uint8_t* s)
{
    const double* J = reinterpret_cast<const double*>(st->J);
    const int N = st->N, L = st->L;
    double E = 0.0;
    if (st->dim == 1) {
        for (int i = 0; i < N; ++i) {
            const int j = i + 1 == N ? 0 : i + 1;
            E = E + ((s[i] ^ s[j]) ? -J[i] : J[i]);
        }
    } else {
        for (int i = 0; i < N; ++i) {
            int nb[3];
            plus_neighbours3(i, L, nb);
            for (int a = 0; a < 3; ++a) E = E + ((s[i] ^ s[nb[a]]) ? -J[3 * i + a] : J[3 * i + a]);
        }
    }
    return E;
}

// thread per replica of the current population
__global__ void __launch_bounds__(64) k_energy_gauss(const pa_state* __restrict__ base)
{
    const pa_state* st = base + blockIdx.y;
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= st->R) return;
    const uint8_t* s = (const uint8_t*)st->spins[st->cur] + r * st->row_stride;
    reinterpret_cast<double*>(st->energy[st->cur])[r] = energy_gauss(st, s);
}

// N_S checkerboard sweeps of one replica per thread; the draws are those of the +-1 path
__global__ void __launch_bounds__(64) k_sweep_gauss(const pa_state* __restrict__ st, double beta, int64_t t0, int ns)
{
    if (st->status) return;
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= st->R) return;
    const int N = st->N, L = st->L, dim = st->dim;
    const double* J = reinterpret_cast<const double*>(st->J);
    uint8_t* s = (uint8_t*)st->spins[st->cur] + r * st->row_stride;
    const uint32_t k0 = (uint32_t)st->seed, k1 = (uint32_t)(st->seed >> 32), rr = (uint32_t)r;
    for (int64_t t = t0; t < t0 + ns; ++t) {
        for (int col = 0; col < 2; ++col) {
            const uint32_t ctr2 = (uint32_t)(2 * t + col);
            int cached = -1;
            uint4v v = {0, 0, 0, 0};
            for (int i = 0; i < N; ++i) {
                if (gauss_colour(st, i) != col) continue;
                // local field, incident bonds in the order +x, +y, +z, -x, -y, -z (chain: +1, -1)
                double h = 0.0;
                if (dim == 1) {
                    const int ip = i + 1 == N ? 0 : i + 1, im = i == 0 ? N - 1 : i - 1;
                    h = h + (s[ip] ? -J[i] : J[i]);
                    h = h + (s[im] ? -J[im] : J[im]);
                } else {
                    int nb[3];
                    plus_neighbours3(i, L, nb);
                    const int x = i % L, y = (i / L) % L, z = i / (L * L);
                    const int m[3] = {(x == 0 ? L - 1 : x - 1) + L * (y + L * z), x + L * ((y == 0 ? L - 1 : y - 1) + L * z),
                                      x + L * (y + L * (z == 0 ? L - 1 : z - 1))};
                    for (int a = 0; a < 3; ++a) h = h + (s[nb[a]] ? -J[3 * i + a] : J[3 * i + a]);
                    for (int a = 0; a < 3; ++a) h = h + (s[m[a]] ? -J[3 * m[a] + a] : J[3 * m[a] + a]);
                }
                const double dE = s[i] ? 2.0 * h : -2.0 * h;
                bool accept = dE <= 0.0;
                if (!accept) {
                    const double p = expd(-(beta * dE));
                    if (p >= 1.0) {
                        accept = true;
                    } else {
                        const uint64_t T64 = (uint64_t)ldexp(p, 64);
                        const int hh = i >> 1;
                        if ((hh >> 3) != cached) {
                            cached = hh >> 3;
                            v = philox10((uint32_t)cached, rr, ctr2, kTagMet, k0, k1);
                        }
                        const uint32_t u16 = (word_of(v, (hh & 7) >> 1) >> (16 * (hh & 1))) & 0xFFFFu;
                        const uint32_t thi = (uint32_t)(T64 >> 48);
                        if (u16 != thi) {
                            accept = u16 < thi;
                        } else {
                            const uint4v w = philox10((uint32_t)i, rr, ctr2, kTagTie, k0, k1);
                            const uint64_t U = ((uint64_t)u16 << 48) | (uint64_t)w.x | ((uint64_t)(w.y & 0xFFFFu) << 32);
                            accept = U < T64;
                        }
                    }
                }
                if (accept) s[i] ^= 1;
            }
        }
    }
    if (ns > 0) reinterpret_cast<double*>(st->energy[st->cur])[r] = energy_gauss(st, s);
}

// ------------------------------------------------------------------ tabled sweep
// The same sweeps with lane = replica: 64 replicas side by side in LDS, each as its two colour
// strings (pa_sweep_strings.h; on the chain bit b of the colour-c string is site 2 b + c), and a word
// of 32 sites of a colour at a time.
//
// dE of an attempt depends only on the site and on the pattern b of the bits s_j xor s_i of
// its neighbours in field order: flipping every spin negates each term of h exactly, hence h,
// and leaves dE unchanged.  Per call, k_gauss_table tabulates for every site and pattern
// T64 = floor(p 2^64) with p = expd(-(beta dE)) computed as in k_sweep_gauss (s_i = 0, s_j = bit
// of b), or all ones where the flip is always accepted (dE <= 0 or p >= 1; a p below 1 gives at
// most 2^64 - 2^11), and the bound min(T16, 0xFFFE) + 1 of its top T16 = T64 >> 48.  An attempt
// compares its 16-bit draw u with the bound: bound - u saturated is 2 or more where u < T16 (accept), 1
// where u = T16 (a tie: the 64-bit draw against T64 decides, as in k_sweep_gauss) and 0 where u > T16
// (reject).  With T16 = 0xFFFF the bound is one too low: u = 0xFFFE comes out as a tie and u = 0xFFFF as a
// rejection, so both are looked at again with T64 (a running maximum of the draws finds the
// latter).  The outcome of every attempt is therefore the same as there.
//
// Table layout (after the work layout): u16 [colour c][call m][pattern b][k], k = 0..7 the sites of
// half-index 8 m + k, the eight sites whose draws are the fields of Philox call m.  The lanes of a wave
// work on the same word at the same time, so lane b loads the 16-byte row [c][m][b] of each of the
// word's four calls: coalesced 1 KB loads whose addresses do not depend on the spins, issued a word
// ahead.  Each attempt then takes its entry from lane b = its pattern with ds_bpermute, a lane-to-lane
// read at the latency of LDS, instead of a gather from the cache at the latency of memory.
// ds_bpermute reads only bits 2..7 of its address, and an 8 x 8 bit transpose of the six neighbour
// words puts the patterns of sites k, 8 + k, 16 + k, 24 + k into bits 2..7 of the four bytes of one
// word, so an address is one shift.  The u64 table of T64 follows in the same order.
//
// Bound by the vector ALU and the latency of a wave's own chain: 10.7 VALU and 1.27 LDS instructions per
// attempt at side 8, of which Philox 4.7; the 73 registers leave six waves per SIMD.  126 runs of side
// 8, R = 2000, 100 sweeps: 4.05 ms, 3.1e12 attempts/s; with one wave per group (as the kernel before, on
// 16-site segments of both colours: 13.9 VALU) 5.23 ms, and a second round of blocks as soon as some
// runs have more than 32 groups (R = 2060: 4.30 ms against 6.62 ms).  50 runs: 4.12 -> 2.08 ms.  The
// sides other than 4 and 8 took one thread per replica: side 6, 8 runs, 20 sweeps 40 ms -> 0.09 ms.
// Chain of 256 sites, 200 runs of 1000, 50 sweeps 1.13 -> 0.87 ms; 64 sites 0.31 -> 0.24 ms.

// h of site i for neighbour pattern b (bit a: neighbour a in field order has s_j != s_i); LC: the
// cube side as a constant (its divisions become shifts or multiplications), 0 for L at run time
template <int NB, int LC = 0>
__device__ double gauss_field_pattern(const double* __restrict__ J, int i, int b, int L_rt, int N)
{
    const int L = LC ? LC : L_rt;
    double h = 0.0;
    if constexpr (NB == 2) {
        const int im = i == 0 ? N - 1 : i - 1;
        h = h + ((b & 1) ? -J[i] : J[i]);
        h = h + ((b & 2) ? -J[im] : J[im]);
    } else {
        const int x = i % L, y = (i / L) % L, z = i / (L * L);
        const int m[3] = {(x == 0 ? L - 1 : x - 1) + L * (y + L * z), x + L * ((y == 0 ? L - 1 : y - 1) + L * z),
                          x + L * (y + L * (z == 0 ? L - 1 : z - 1))};
        for (int a = 0; a < 3; ++a) h = h + (((b >> a) & 1) ? -J[3 * i + a] : J[3 * i + a]);
        for (int a = 0; a < 3; ++a) h = h + (((b >> (3 + a)) & 1) ? -J[3 * m[a] + a] : J[3 * m[a] + a]);
    }
    return h;
}

// true if the flip is always accepted; otherwise *T64 = floor(p 2^64) with p < 1 (s_i = 0)
__device__ inline bool gauss_threshold(double h, double beta, uint64_t* T64)
{
    const double dE = -2.0 * h;
    if (dE <= 0.0) return true;
    const double p = expd(-(beta * dE));
    if (p >= 1.0) return true;
    *T64 = (uint64_t)ldexp(p, 64);
    return false;
}

__device__ __forceinline__ uint16_t* gauss_table(const pa_state* st)
{
    return reinterpret_cast<uint16_t*>(st->work + work_layout(st->N, st->n_bins, st->capacity).total);
}

// calls per colour (the last one may have fewer than eight sites: its entries past them are zero)
__host__ __device__ inline int gauss_calls(int N) { return (N / 2 + 7) / 8; }

// the u64 table of full thresholds, after the NB-pattern u16 table (8-byte aligned)
template <int NB>
__device__ __forceinline__ uint64_t* gauss_table64(const pa_state* st)
{
    return reinterpret_cast<uint64_t*>(gauss_table(st) + ((size_t)(16 * gauss_calls(st->N)) << NB));
}

// grid (entries / 256, runs): entry e = (c, m, b, k) of run blockIdx.y; LC as in gauss_field_pattern
template <int NB, int LC>
__global__ void __launch_bounds__(256) k_gauss_table(pa_state* __restrict__ states, double beta)
{
    const pa_state* st = states + blockIdx.y;
    if (st->status) return;
    const int N = st->N, L = LC ? LC : st->L;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    const int half = (8 * gauss_calls(N)) << NB;
    if (e >= 2 * half) return;
    const int c = e >= half, rem = e - c * half;
    const int b = (rem >> 3) & ((1 << NB) - 1), hh = 8 * (rem >> (NB + 3)) + (rem & 7);
    uint64_t T64 = 0;
    uint32_t bound = 0;
    if (hh < N / 2) {
        const int i0 = 2 * hh;
        const int col0 = NB == 2 ? 0 : ((i0 % L) + (i0 / L) % L + i0 / (L * L)) & 1;
        const int i = i0 + (col0 != c);
        const double h = gauss_field_pattern<NB, LC>(reinterpret_cast<const double*>(st->J), i, b, L, N);
        if (gauss_threshold(h, beta, &T64)) T64 = ~0ull;
        const uint32_t T16 = (uint32_t)(T64 >> 48);
        bound = (T16 < 0xFFFEu ? T16 : 0xFFFEu) + 1u;
    }
    gauss_table(st)[e] = (uint16_t)bound;
    gauss_table64<NB>(st)[e] = T64;
}

typedef uint32_t gu32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) gu32x4* grow_ptr;  // table rows, global memory

// Lane addresses of the 32 sites' table entries from the neighbour words X (each xor the own word, in
// field order): the pattern of site 8 i + k in bits 2 .. NB + 1 of what site_address gives for it
// (other bits arbitrary; on the chain, bits 4..7 too: lanes that agree mod 4 hold the same row).
template <int NB>
struct Patterns {
    uint32_t P[NB == 6 ? 8 : 2];
    __device__ __forceinline__ void make(const uint32_t (&X)[NB])
    {
        using words::select_bits;
        if constexpr (NB == 6) {
            // rows 2..7 of the transpose are the neighbour words, rows 0 and 1 arbitrary
            constexpr uint32_t M4 = 0x0F0F0F0Fu, M2 = 0x33333333u, M1 = 0x55555555u;
            uint32_t A[8];
            A[0] = X[2] << 4;
            A[1] = X[3] << 4;
            A[2] = select_bits(M4, X[0], X[4] << 4);
            A[3] = select_bits(M4, X[1], X[5] << 4);
            A[4] = X[2];
            A[5] = X[3];
            A[6] = select_bits(M4, X[0] >> 4, X[4]);
            A[7] = select_bits(M4, X[1] >> 4, X[5]);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                if (r & 2) continue;
                const uint32_t lo = A[r], hi = A[r + 2];
                A[r] = select_bits(M2, lo, hi << 2);
                A[r + 2] = select_bits(M2, lo >> 2, hi);
            }
#pragma unroll
            for (int r = 0; r < 8; r += 2) {
                P[r] = select_bits(M1, A[r], A[r + 1] << 1);
                P[r + 1] = select_bits(M1, A[r] >> 1, A[r + 1]);
            }
        } else {
            // even sites j at bits j, j + 1 of P[0], odd ones at bits j - 1, j of P[1]
            P[0] = select_bits(0x55555555u, X[0], X[1] << 1);
            P[1] = select_bits(0xAAAAAAAAu, X[1], X[0] >> 1);
        }
    }
    __device__ __forceinline__ uint32_t address(int i, int k) const  // constants after unrolling
    {
        if constexpr (NB == 6) {
            return P[k] >> (8 * i);
        } else {
            const int s = 8 * i + (k & ~1);
            return s >= 2 ? P[k & 1] >> (s - 2) : P[k & 1] << (2 - s);
        }
    }
};

// v_pk_max_u16, written out as first_look's minimum is
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("v_pk_max_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// A cube's energy in bond order.  A bond's term is +-J, added as fma(+-1, J, E): the product is exact, so
// the sum rounds once, as E + (+-J).  The wave holds a lattice row's couplings, one per lane, and reads each
// from its lane as a scalar.  Loaded as scalars two sites at a time, they had the wave wait most of the time:
// a call of one sweep of 2000 replicas took, side 6 36 us, 8 61 us, 10 107 us; so 27, 45 and 71.
__device__ __forceinline__ double lane_of(double x, int lane)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// E plus J, or less J where bit x of d is set.  sign and one: 2^31 and the high half of 1.0, kept in
// registers by the caller (as literals they cost the and and the or an instruction each)
struct SignWords {
    uint32_t sign = 0x80000000u, one = 0x3FF00000u;
    __device__ __forceinline__ SignWords() { asm volatile("" : "+v"(sign), "+v"(one)); }
};

__device__ __forceinline__ double bond_sign(uint32_t d, int x, const SignWords& k)
{
    return __builtin_bit_cast(double, (uint64_t)words::select_bits(k.sign, d << (31 - x), k.one) << 32);
}

// E of a cube from its strings (E0, E1 at word 0, S dwords from word to word): site i, then axis +x, +y, +z.
// A row is taken as its even and its odd sites (bit m: x = 2 m, 2 m + 1), which the strings hold side by side.
// The rows next to row i + 1 are asked for before the bonds of row i, the couplings four rows ahead, and a
// bond's sign and coupling are made kAhead bonds before they are used and kept there.
template <int L, int S>
__device__ __forceinline__ double cube_energy(const double* couplings, const uint32_t* E0, const uint32_t* E1)
{
    constexpr int H2 = L / 2, kAhead = 4, kRows = 4;
    static_assert(L % 2 == 0, "whole rounds of kRows rows");
    const __attribute__((address_space(1))) double* J = (const __attribute__((address_space(1))) double*)couplings;
    struct Row {
        uint32_t e0, e1, o0, o1;
        int sh;
        __device__ __forceinline__ uint32_t ev() const { return __builtin_amdgcn_alignbit(e1, e0, sh); }
        __device__ __forceinline__ uint32_t od() const { return __builtin_amdgcn_alignbit(o1, o0, sh); }
    };
    auto load = [&](int y, int z) {  // colour 0 takes x = 2 m + (y + z) mod 2
        const int b = H2 * (y + L * z), k = (b >> 5) * S, to1 = (int)(E1 - E0);
        const int e = k + (((y + z) & 1) ? to1 : 0), o = k + (((y + z) & 1) ? 0 : to1);
        return Row{E0[e], E0[e + S], E0[o], E0[o + S], b & 31};
    };
    const int lane = threadIdx.x & 63;
    auto row_J = [&](int i) { return J[3 * L * (i < L * L ? i : L * L - 1) + (lane < 3 * L ? lane : 0)]; };
    double Jq[kRows];
#pragma unroll
    for (int n = 0; n < kRows; ++n) Jq[n] = row_J(n);
    const SignWords sw;
    double E = 0.0;
    Row ny = load(1, 0), nz = load(0, 1);
    const Row r0 = load(0, 0);
    uint32_t ev = r0.ev(), od = r0.od(), ev_z = 0, od_z = 0;  // this row, and the first row of the next plane
    int y = 0, z = 0;
#pragma unroll 1
    for (int i = 0; i < L * L; i += kRows) {
#pragma unroll
        for (int n = 0; n < kRows; ++n) {
            const uint32_t evy = ny.ev(), ody = ny.od(), evz = nz.ev(), odz = nz.od();
            ev_z = y == 0 ? evz : ev_z;
            od_z = y == 0 ? odz : od_z;
            // bit m: the bond of x = 2 m (e) and of x = 2 m + 1 (o) along each axis
            const uint32_t next = words::select_bits(1u << (H2 - 1), ev << (H2 - 1), ev >> 1);
            const uint32_t e[3] = {ev ^ od, ev ^ evy, ev ^ evz};
            const uint32_t o[3] = {od ^ next, od ^ ody, od ^ odz};
            const bool wrap = y + 1 == L;
            ev = wrap ? ev_z : evy;
            od = wrap ? od_z : ody;
            y = wrap ? 0 : y + 1;
            z = wrap ? z + 1 : z;
            ny = load(y + 1 < L ? y + 1 : 0, z < L ? z : 0);
            nz = load(y, z + 1 < L ? z + 1 : 0);
            double sg[3 * L], Jb[3 * L];
#pragma unroll
            for (int b = -kAhead; b < 3 * L; ++b) {
                if (b >= 0) E = __builtin_fma(sg[b], Jb[b], E);
                if (b + kAhead < 3 * L) {
                    const int c = b + kAhead, x = c / 3;
                    sg[c] = bond_sign(x & 1 ? o[c % 3] : e[c % 3], x >> 1, sw);
                    Jb[c] = lane_of(Jq[n], c);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            Jq[n] = row_J(i + n + kRows);
        }
    }
    return E;
}

struct GaussX { uint32_t w[6]; };

// The attempts of a word that the bounds leave open, decided exactly: ties (bits with u = bound - 1) and the
// sites with u = 0xFFFF of the calls in tops (bit i: call i, which is drawn again to find them).  Either way
// u follows from the threshold, so no other call is drawn again but for the low bits of a true tie (one
// word in 16 of a wave comes here; with every call of the word and of its ties drawn again, side 8 and 126
// runs took 3% longer).  T64w: the word's rows of the u64 table; sites is the mask of the word's sites, odd
// that of the sites 2 h + 1.  Returns the accepted ones.
template <int NB>
__device__ __forceinline__ uint32_t gauss_resolve(const uint64_t* __restrict__ T64w, const GaussX& X, uint32_t ties, uint32_t tops,
                                                  uint32_t sites, uint32_t odd, uint32_t k, uint32_t rr, uint32_t ctr2,
                                                  uint32_t k0, uint32_t k1)
{
    uint32_t high = 0;  // sites with u = 0xFFFF
    while (tops) {
        const int i = __builtin_ctz(tops);
        tops &= tops - 1;
        const uint4v v = philox10(4 * k + i, rr, ctr2, kTagMet, k0, k1);
        for (int f = 0; f < 8; ++f) high |= (uint32_t)(field16(v, f) == 0xFFFFu) << (8 * i + f);
    }
    uint32_t open = (ties | high) & sites;
    uint32_t F = 0;
    while (open) {
        const int j = __builtin_ctz(open);
        open &= open - 1;
        int b = 0;
        for (int a = 0; a < NB; ++a) b |= (int)((X.w[a] >> j) & 1u) << a;
        const uint64_t T = T64w[((((j >> 3) << NB) + b) << 3) + (j & 7)];
        const uint32_t T16 = (uint32_t)(T >> 48);
        const uint32_t u = (high >> j) & 1u ? 0xFFFFu : min(T16, 0xFFFEu);
        bool accept = T == ~0ull || u < T16;
        if (!accept && u == T16) accept = tie_accept(u, T, 2u * (32u * k + j) + ((odd >> j) & 1u), rr, ctr2, k0, k1);
        F |= (uint32_t)accept << j;
    }
    return F;
}

// The same out of line, for the kernels of small populations: shorter code matters more there than registers
// (in line, two runs of side 8 took 1.3% longer; in the others the values kept over a call took the registers
// past what six waves per SIMD leave: 200 chains of 256 sites 0.90 ms a call, 0.86 in line).
template <int NB>
static __device__ __noinline__ uint32_t gauss_resolve_call(const uint64_t* __restrict__ T64w, GaussX X, uint32_t ties, uint32_t tops,
                                                           uint32_t sites, uint32_t odd, uint32_t k, uint32_t rr, uint32_t ctr2,
                                                           uint32_t k0, uint32_t k1)
{
    return gauss_resolve<NB>(T64w, X, ties, tops, sites, odd, k, rr, ctr2, k0, k1);
}

// whether either half of a word is 0xFFFF
__device__ __forceinline__ bool any_top(uint32_t u) { return (u | 0xFFFFu) == 0xFFFFFFFFu || (u & 0xFFFFu) == 0xFFFFu; }

// The attempts of word w of a colour (bits `sites` of it): X the neighbour words xor w in field order,
// rows the table rows of the word's calls in this lane, T64w the word's rows of the u64 table.  Returns
// the new word.  CALLS: the calls with sites (0: nbytes of them, known at run time).
template <int NB, int CALLS, int NR>
__device__ __forceinline__ uint32_t gauss_word(uint32_t w, const uint32_t (&X)[NB], const gu32x4 (&rows)[NR], uint32_t sites,
                                               uint32_t odd, int nbytes, const uint64_t* __restrict__ T64w, uint32_t k,
                                               const words::Lane& c)
{
    using words::select_bits;
    Patterns<NB> pt;
    pt.make(X);
    uint32_t raw[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (CALLS ? i >= CALLS : i >= nbytes) break;
#pragma unroll
        for (int t = 0; t < 8; ++t)
            raw[i][t] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)pt.address(i, t), (int)rows[i][t >> 1]);
    }
    // outcomes and their places as in words::decide_word
    uint32_t ra = 0, rb = 0, umax[4] = {0, 0, 0, 0};  // umax: of a call's draws
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (CALLS ? i >= CALLS : i >= nbytes) break;
        const uint4v v = words::philox10_lane(4 * k + i, c.rr, c.ctr2, kTagMet, c.k0, c.k1);
        const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
        uint32_t e[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            // site 2 t's entry is the low half of its word, site 2 t + 1's the high half
            const uint32_t bound = __builtin_amdgcn_perm(raw[i][2 * t + 1], raw[i][2 * t], 0x07060100u);
            e[t] = words::first_look(bound, vw[t]);
            umax[i] = t == 0 ? vw[t] : pk_max_u16(umax[i], vw[t]);
        }
        const int o = 8 * (i & 1);
        uint32_t r = i < 2 ? ra : rb;
        r = (i & 1) ? words::lshl_or(e[0], o, r) : e[0];
        r = words::lshl_or(e[1], o + 2, r);
        r = words::lshl_or(e[2], o + 4, r);
        r = words::lshl_or(e[3], o + 6, r);
        if (i < 2) ra = r;
        else rb = r;
    }
    uint32_t acc = select_bits(0x0000FFFFu, select_bits(0x5555u, ra >> 1, ra >> 16), select_bits(0x55550000u, rb << 15, rb));
    uint32_t all = umax[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) {
        if (CALLS ? i >= CALLS : i >= nbytes) break;
        all = pk_max_u16(all, umax[i]);
    }
    const bool top = any_top(all);
    if (((ra | rb) & 0x55555555u) != 0 || top) {
        const uint32_t ties = select_bits(0x0000FFFFu, select_bits(0x5555u, ra, ra >> 15),
                                          select_bits(0x55550000u, rb << 16, rb << 1));
        if ((ties & sites) || top) {
            GaussX gx = {};
#pragma unroll
            for (int a = 0; a < NB; ++a) gx.w[a] = X[a];
            const uint32_t tops = (uint32_t)any_top(umax[0]) | (uint32_t)any_top(umax[1]) << 1 | (uint32_t)any_top(umax[2]) << 2 |
                                  (uint32_t)any_top(umax[3]) << 3;
            acc |= gauss_resolve<NB>(T64w, gx, ties, tops, sites, odd, k, c.rr, c.ctr2, c.k0, c.k1);
        }
    }
    return w ^ (acc & sites);
}

// The attempts of call i of word k alone, in place in the word's byte i; row: the call's row in this lane
template <int NB>
__device__ __forceinline__ uint32_t gauss_byte(uint32_t w, const uint32_t (&X)[NB], gu32x4 row, uint32_t sites, uint32_t odd,
                                               const uint64_t* __restrict__ T64w, uint32_t k, int i, const words::Lane& c)
{
    using words::select_bits;
    const int sh = 8 * i;
    uint32_t XI[NB];  // the byte's neighbour patterns as a word's first byte
#pragma unroll
    for (int a = 0; a < NB; ++a) XI[a] = (X[a] >> sh) & 0xFFu;
    Patterns<NB> pt;
    pt.make(XI);
    uint32_t raw[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) raw[t] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)pt.address(0, t), (int)row[t >> 1]);
    const uint4v v = words::philox10_lane(4 * k + i, c.rr, c.ctr2, kTagMet, c.k0, c.k1);
    const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
    uint32_t ra = 0, umax = vw[0];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        ra = words::lshl_or(words::first_look(__builtin_amdgcn_perm(raw[2 * t + 1], raw[2 * t], 0x07060100u), vw[t]), 2 * t, ra);
        if (t > 0) umax = pk_max_u16(umax, vw[t]);
    }
    sites &= 0xFFu << sh;
    uint32_t acc = (select_bits(0x5555u, ra >> 1, ra >> 16) & 0xFFu) << sh;
    const bool top = any_top(umax);
    if ((ra & 0x55555555u) != 0 || top) {
        const uint32_t ties = (select_bits(0x5555u, ra, ra >> 15) & 0xFFu) << sh;
        if ((ties & sites) || top) {
            GaussX gx = {};
#pragma unroll
            for (int a = 0; a < NB; ++a) gx.w[a] = X[a];
            acc |= gauss_resolve_call<NB>(T64w, gx, ties, (uint32_t)top << i, sites, odd, k, c.rr, c.ctr2, c.k0, c.k1);
        }
    }
    return (w ^ (acc & sites)) >> sh;  // (the byte: the rest of the word arbitrary)
}

// A block takes four waves: 4 / NWV groups of 64 replicas, the words of each split by NWV waves.  1-D
// grid; block -> (run, block of the run): with 8 or more runs, the (run, block) items are split into 8
// contiguous ranges and the blocks of range x are those with id = x mod 8 (blocks go round-robin to the
// 8 XCDs, so a run's table stays in one L2, or in two where a run straddles ranges).  Every lane of a
// wave takes part in the lane reads of the table (lanes past R compute and store nothing), so no
// branch may split a wave around them.
constexpr int kGaussWaves = 4;
constexpr int kGaussCallWaves = 16;  // most waves of a block whose waves take calls instead of words

__device__ __forceinline__ bool gauss_place(int n_runs, int blocks, int* run, int* block)
{
    const int items = n_runs * blocks;
    const int item = n_runs >= 8 ? (int)(blockIdx.x & 7) * ((items + 7) / 8) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const int end = n_runs >= 8 ? min(items, (int)((blockIdx.x & 7) + 1) * ((items + 7) / 8)) : items;
    if (item >= end) return false;
    *run = item / blocks;
    *block = item % blocks;
    return true;
}

template <int NWV>
__device__ __forceinline__ void gauss_sync()
{
    if constexpr (NWV == 1) wave_sync();
    else __syncthreads();
}

template <int L, int NWV>
struct GaussCubeSmem {
    static constexpr int GPB = kGaussWaves / NWV;
    uint32_t E[GPB][2 * strings::Geo<L>::EW * 64];                       // the extended strings, [word][replica]
    uint32_t tab[2 * strings::Geo<L>::NW * strings::Geo<L>::TW];         // geometry masks
};

// Waves per SIMD that the registers must leave room for: six at sides 6 and 8 (126 runs, 20 sweeps of side 6 598
// -> 582 us, 100 of side 8 4.19 -> 4.11 ms); the others are faster with the five they happen to get (side 4 162 and
// 181 us, side 10, 40 runs, 795 and 891).
constexpr int gauss_cube_waves(int L) { return L == 6 || L == 8 ? 6 : 1; }

template <int L, int NWV>
__global__ void __launch_bounds__(kGaussWaves * 64, gauss_cube_waves(L)) k_sweep_gauss_cube(pa_state* __restrict__ states, int n_runs,
                                                                       int blocks, int64_t t0, int ns)
{
    using Gm = strings::Geo<L>;
    constexpr int G = Gm::G, EW = Gm::EW, NW = Gm::NW, TW = Gm::TW, GPB = kGaussWaves / NWV;
    constexpr bool WHOLE = Gm::NH % 32 == 0;
    constexpr int M = (Gm::NH + 7) / 8;  // calls per colour
    __shared__ GaussCubeSmem<L, NWV> sm;
    int run, block;
    if (!gauss_place(n_runs, blocks, &run, &block)) return;
    const pa_state* st = states + run;
    const int64_t R = st->R;
    if (st->status || (int64_t)block * GPB * 64 >= R) return;
    const int lane = threadIdx.x & 63, w4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    strings::build_tables<L, false>(nullptr, sm.tab, lane, w4, kGaussWaves);
    __syncthreads();
    const int gi = w4 / NWV, wave = w4 % NWV;
    const int64_t r = ((int64_t)block * GPB + gi) * 64 + lane;
    if (r - lane >= R) return;  // (NWV = 1: no barrier of the block follows)
    const bool valid = r < R;
    uint32_t* E0 = sm.E[gi] + lane;
    uint32_t* E1 = E0 + EW * 64;
    uint8_t* row = (uint8_t*)st->spins[st->cur] + r * Gm::STRIDE;
    auto put = [&](uint32_t* S, int k, uint32_t v) {
        S[(G + k) * 64] = v;
        if constexpr (WHOLE) {
            if (k < G) S[(G + NW + k) * 64] = v;
            if (k >= NW - G) S[(k - (NW - G)) * 64] = v;
        }
    };
#pragma unroll 1
    for (int k = wave; k < NW; k += NWV) {
        uint32_t ev, od;
        strings::load_word_u8(row, Gm::STRIDE, k, &ev, &od);
        const uint32_t sig0 = sm.tab[k * TW + 6], in = sm.tab[k * TW + 11];  // colour 0: x even, sites
        put(E0, k, words::select_bits(sig0, ev, od) & in);
        put(E1, k, words::select_bits(sig0, od, ev) & in);
    }
    gauss_sync<NWV>();
    if constexpr (!WHOLE) {
        strings::refresh_ghosts<L, 64>(E0, wave, NWV);
        strings::refresh_ghosts<L, 64>(E1, wave, NWV);
        gauss_sync<NWV>();
    }

    const uint16_t* __restrict__ Tab = gauss_table(st);
    const uint64_t* __restrict__ Tab64 = gauss_table64<6>(st);
    words::Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    // this lane's rows of the calls of word k of a colour (calls past the last one: the last one's)
    auto load_rows = [&](int col, int k, gu32x4 (&rows)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = WHOLE || 4 * k + i < M ? 4 * k + i : M - 1;
            rows[i] = ((grow_ptr)Tab)[((col * M + m) << 6) + lane];
        }
    };
    gu32x4 rows[4];
    if (wave < NW) load_rows(0, wave, rows);
    for (int64_t t = t0; t < t0 + ns; ++t) {
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * t + col);
            uint32_t* W = col ? E1 : E0;
            const uint32_t* O = col ? E0 : E1;
#pragma unroll 1
            for (int k = wave; k < NW; k += NWV) {
                // the rows of the wave's next word (of the other colour after its last one)
                gu32x4 next[4];
                const bool last = k + NWV >= NW;
                load_rows(last ? col ^ 1 : col, last ? wave : k + NWV, next);
                const uint32_t* T = sm.tab + (col * NW + k) * TW;
                const uint32_t w = W[(G + k) * 64];
                uint32_t nb[6];
                strings::neighbours<L, 64>(O + (G + k) * 64, T, nb);  // +x, -x, +y, -y, +z, -z
                const uint32_t X[6] = {w ^ nb[0], w ^ nb[2], w ^ nb[4], w ^ nb[1], w ^ nb[3], w ^ nb[5]};
                const uint32_t sites = WHOLE ? 0xFFFFFFFFu : T[11];
                put(W, k, gauss_word<6, 4>(w, X, rows, sites, ~T[6], 4, Tab64 + ((size_t)(col * M + 4 * k) << 9), k, c));
#pragma unroll
                for (int i = 0; i < 4; ++i) rows[i] = next[i];
            }
            gauss_sync<NWV>();
            if constexpr (!WHOLE) {
                strings::refresh_ghosts<L, 64>(W, wave, NWV);
                gauss_sync<NWV>();
            }
        }
    }

    // spins back, and (the group's first wave) E in bond order: site i, then axis +x, +y, +z
#pragma unroll 1
    for (int k = wave; k < NW; k += NWV) {
        const uint32_t sig0 = sm.tab[k * TW + 6], in = sm.tab[k * TW + 11];
        const uint32_t a = E0[(G + k) * 64], b = E1[(G + k) * 64];
        if (valid)
            strings::store_word_u8(row, Gm::STRIDE, k, words::select_bits(sig0, a, b) & in, words::select_bits(sig0, b, a) & in);
    }
    if (wave != 0) return;
    const double E = cube_energy<L, 64>(reinterpret_cast<const double*>(st->J), E0 + G * 64, E1 + G * 64);
    if (valid) reinterpret_cast<double*>(st->energy[st->cur])[r] = E;
}

// Small populations of sides 8 and 10: 16 replicas per block and a thread per (replica, call), so that a
// population is four times as many blocks and a phase is one call long.  The lanes of a wave then work on
// four calls, so the table lies in LDS (read there instead of from lane to lane), [colour][call][k][pattern]:
// a site's 64 bounds take 32 banks, and a call's stride puts neighbouring calls on alternate halves.
constexpr int kSplitReplicas = 16;
constexpr int kSplitCall = 8 * 64 + 64;  // u16 of a call (128 bytes of padding)

template <int L>
struct GaussSplitSmem {
    static constexpr int M = (strings::Geo<L>::NH + 7) / 8;
    static constexpr int UNITS = (M + 3) / 4 * 4;  // calls at once: whole waves
    uint32_t E[2 * strings::Geo<L>::EW * kSplitReplicas];
    uint32_t tab[2 * strings::Geo<L>::NW * strings::Geo<L>::TW];
    uint16_t bound[2 * M * kSplitCall];
};

// base plus byte B of v, an LDS address of this lane (one SDWA op)
template <int B>
__device__ __forceinline__ uint32_t add_byte(uint32_t base, uint32_t v)
{
    uint32_t r;
    if constexpr (B == 0)
        asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(base), "v"(v));
    else if constexpr (B == 1)
        asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(base), "v"(v));
    else if constexpr (B == 2)
        asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(base), "v"(v));
    else
        asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(base), "v"(v));
    return r;
}

template <int L>
__global__ void __launch_bounds__(kSplitReplicas * GaussSplitSmem<L>::UNITS)
k_sweep_gauss_split(pa_state* __restrict__ states, int n_runs, int blocks, int64_t t0, int ns)
{
    using Gm = strings::Geo<L>;
    using words::select_bits;
    using words::xor3;
    constexpr int Q = kSplitReplicas, G = Gm::G, EW = Gm::EW, NW = Gm::NW, TW = Gm::TW, M = GaussSplitSmem<L>::M;
    constexpr int UNITS = GaussSplitSmem<L>::UNITS, THREADS = Q * UNITS;
    constexpr bool WHOLE = Gm::NH % 32 == 0;
    __shared__ GaussSplitSmem<L> sm;
    int run, block;
    if (!gauss_place(n_runs, blocks, &run, &block)) return;
    const pa_state* st = states + run;
    const int64_t R = st->R, r0 = (int64_t)block * Q;
    if (st->status || r0 >= R) return;  // the same for the whole block
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = threadIdx.x % Q, unit = threadIdx.x / Q;
    const int64_t r = r0 + q;
    const bool valid = r < R;
    strings::build_tables<L, false>(nullptr, sm.tab, lane, wave, THREADS / 64);
    const uint16_t* __restrict__ Tab = gauss_table(st);
    const uint64_t* __restrict__ Tab64 = gauss_table64<6>(st);
    for (int e = ns > 0 ? (int)threadIdx.x : 2 * M * 64; e < 2 * M * 64; e += THREADS) {
        const gu32x4 v = ((grow_ptr)Tab)[e];  // call e / 64, pattern e mod 64
        uint16_t* t = sm.bound + (e >> 6) * kSplitCall + (e & 63);
#pragma unroll
        for (int k = 0; k < 8; ++k) t[64 * k] = (uint16_t)(v[k >> 1] >> (16 * (k & 1)));
    }
    uint32_t* E0 = sm.E + q;
    uint32_t* E1 = E0 + EW * Q;
    uint8_t* row = (uint8_t*)st->spins[st->cur] + (valid ? r : R - 1) * Gm::STRIDE;
    __syncthreads();
    for (int k = unit; k < NW; k += UNITS) {
        uint32_t ev, od;
        strings::load_word_u8(row, Gm::STRIDE, k, &ev, &od);
        const uint32_t sig0 = sm.tab[k * TW + 6], in = sm.tab[k * TW + 11];  // colour 0: x even, sites
        const uint32_t v[2] = {select_bits(sig0, ev, od) & in, select_bits(sig0, od, ev) & in};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint32_t* S = c ? E1 : E0;
            S[(G + k) * Q] = v[c];
            if constexpr (WHOLE) {
                if (k < G) S[(G + NW + k) * Q] = v[c];
                if (k >= NW - G) S[(k - (NW - G)) * Q] = v[c];
            }
        }
    }
    __syncthreads();
    if constexpr (!WHOLE) {
        strings::refresh_ghosts<L, Q>(E0, unit, UNITS);
        strings::refresh_ghosts<L, Q>(E1, unit, UNITS);
        __syncthreads();
    }

    words::Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    // this thread's call: byte i of word k
    const int m = unit, k = m >> 2, i = m & 3;
    // bytes i of two words to bytes 1, 2 and, after them, byte i of a third to byte 3
    const uint32_t two = 0x0C04000Cu + (uint32_t)i * 0x010100u, three = 0x04020100u + ((uint32_t)i << 24);
    for (int64_t t = t0; t < t0 + ns; ++t) {
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * t + col);
            uint32_t* W = col ? E1 : E0;
            const uint32_t* O = col ? E0 : E1;
            if (m < M) {
                const uint4v v = philox10((uint32_t)m, c.rr, c.ctr2, kTagMet, c.k0, c.k1);
                const uint32_t* T = sm.tab + (col * NW + k) * TW;
                const uint32_t w = W[(G + k) * Q];
                uint32_t nb[6];
                strings::neighbours<L, Q>(O + (G + k) * Q, T, nb);
                const uint32_t X[6] = {w ^ nb[0], w ^ nb[2], w ^ nb[4], w ^ nb[1], w ^ nb[3], w ^ nb[5]};
                // rows 1..6 of an 8 x 8 bit matrix, transposed: byte s of (x, y) is twice site s's pattern
                uint32_t x = __builtin_amdgcn_perm(X[2], __builtin_amdgcn_perm(X[1], X[0], two), three);
                uint32_t y = __builtin_amdgcn_perm(X[5], __builtin_amdgcn_perm(X[4], X[3], two), three) >> 8;
                uint32_t d;
                d = (x ^ (x >> 7)) & 0x00AA00AAu;
                x = xor3(x, d, d << 7);
                d = (y ^ (y >> 7)) & 0x00AA00AAu;
                y = xor3(y, d, d << 7);
                d = (x ^ (x >> 14)) & 0x0000CCCCu;
                x = xor3(x, d, d << 14);
                d = (y ^ (y >> 14)) & 0x0000CCCCu;
                y = xor3(y, d, d << 14);
                d = (x ^ __builtin_amdgcn_alignbit(y, x, 28)) & 0xF0F0F0F0u;
                x ^= d;
                y ^= d >> 4;
                const char* tb = reinterpret_cast<const char*>(sm.bound + (col * M + m) * kSplitCall);
                auto bound = [&](auto B, uint32_t z, int s) -> uint32_t {
                    constexpr int b = decltype(B)::value;
                    const uint32_t a = add_byte<b>((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)tb, z);
                    return *(const __attribute__((address_space(3))) uint16_t*)(uintptr_t)(a + 128 * s);
                };
                const uint32_t bd[8] = {bound(std::integral_constant<int, 0>{}, x, 0), bound(std::integral_constant<int, 1>{}, x, 1),
                                        bound(std::integral_constant<int, 2>{}, x, 2), bound(std::integral_constant<int, 3>{}, x, 3),
                                        bound(std::integral_constant<int, 0>{}, y, 4), bound(std::integral_constant<int, 1>{}, y, 5),
                                        bound(std::integral_constant<int, 2>{}, y, 6), bound(std::integral_constant<int, 3>{}, y, 7)};
                const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
                uint32_t ra = 0, umax = vw[0];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    ra = words::lshl_or(words::first_look(bd[2 * s] | bd[2 * s + 1] << 16, vw[s]), 2 * s, ra);
                    if (s > 0) umax = pk_max_u16(umax, vw[s]);
                }
                const int sh = 8 * i;
                const uint32_t sites = (WHOLE ? 0xFFFFFFFFu : T[11]) & (0xFFu << sh);
                uint32_t acc = (select_bits(0x5555u, ra >> 1, ra >> 16) & 0xFFu) << sh;
                const bool top = any_top(umax);
                if ((ra & 0x55555555u) != 0 || top) {
                    const uint32_t ties = (select_bits(0x5555u, ra, ra >> 15) & 0xFFu) << sh;
                    if ((ties & sites) || top) {
                        GaussX gx = {};
#pragma unroll
                        for (int a = 0; a < 6; ++a) gx.w[a] = X[a];
                        acc |= gauss_resolve_call<6>(Tab64 + ((size_t)(col * M + 4 * k) << 9), gx, ties, (uint32_t)top << i, sites, ~T[6], (uint32_t)k,
                                                c.rr, c.ctr2, c.k0, c.k1);
                    }
                }
                // only this thread's byte of the word, whose other readers in this phase use their own bytes alone
                const uint8_t out = (uint8_t)((w ^ (acc & sites)) >> sh);
                auto byte = [&](int e) -> uint8_t& { return reinterpret_cast<uint8_t*>(W + e * Q)[i]; };
                byte(G + k) = out;
                if constexpr (WHOLE) {
                    if (k < G) byte(G + NW + k) = out;
                    if (k >= NW - G) byte(k - (NW - G)) = out;
                }
            }
            __syncthreads();
            if constexpr (!WHOLE) {
                strings::refresh_ghosts<L, Q>(W, unit, UNITS);
                __syncthreads();
            }
        }
    }

    // spins back, and (16 lanes of a wave) E
    for (int w = unit; w < NW; w += UNITS) {
        const uint32_t sig0 = sm.tab[w * TW + 6], in = sm.tab[w * TW + 11];
        const uint32_t a = E0[(G + w) * Q], b = E1[(G + w) * Q];
        if (valid) strings::store_word_u8(row, Gm::STRIDE, w, select_bits(sig0, a, b) & in, select_bits(sig0, b, a) & in);
    }
    // the blocks of a CU, one of every 256, leave E to different waves, which lie on different SIMDs
    if (wave != (int)(blockIdx.x >> 8) % (THREADS / 64)) return;
    const double E = cube_energy<L, Q>(reinterpret_cast<const double*>(st->J), E0 + G * Q, E1 + G * Q);
    if (valid && lane < Q) reinterpret_cast<double*>(st->energy[st->cur])[r] = E;
}

// Chains: the two strings of a 64-replica group in dynamic LDS ([colour][word][64]), its words split by
// the block's waves.  No ghost words: the bits of a word past its ends come from the words on both
// sides, periodically.
// WHOLE: N is a multiple of 64, every word has 32 sites.  CALLS: a wave takes a call of eight sites at a time
// instead of a word, for small populations, where it is the wave's own chain that takes the time.
template <bool WHOLE, bool CALLS>
__global__ void __launch_bounds__((CALLS ? kGaussCallWaves : kGaussWaves) * 64)
k_sweep_gauss_chain(pa_state* __restrict__ states, int n_runs, int blocks, int64_t t0, int ns)
{
    const int NWV = CALLS ? (int)(blockDim.x >> 6) : kGaussWaves;
    extern __shared__ uint32_t lds[];
    int run, block;
    if (!gauss_place(n_runs, blocks, &run, &block)) return;
    const pa_state* st = states + run;
    const int64_t R = st->R;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = (int64_t)block * 64 + lane;
    if (st->status || r - lane >= R) return;  // the same for the whole block
    const bool valid = r < R;
    const int N = st->N, NH = N >> 1, NW = (NH + 31) >> 5, M = gauss_calls(N);
    const int end = (NH - 1) & 31;  // bit of the string's last site in its last word
    const uint32_t last_sites = 0xFFFFFFFFu >> (31 - end);
    const int last_bytes = (end >> 3) + 1;
    uint32_t* E0 = lds + lane;
    uint32_t* E1 = E0 + NW * 64;
    const int stride = st->row_stride;
    uint8_t* row = (uint8_t*)st->spins[st->cur] + r * stride;
#pragma unroll 1
    for (int k = wave; k < NW; k += NWV) {
        uint32_t ev, od;
        strings::load_word_u8(row, stride, k, &ev, &od);
        const uint32_t in = k + 1 == NW ? last_sites : 0xFFFFFFFFu;
        E0[k * 64] = ev & in;
        E1[k * 64] = od & in;
    }
    __syncthreads();
    // the string's word k shifted by one site: bit b holds bit b + 1 or b - 1, periodically
    auto up = [&](const uint32_t* S, int k, uint32_t a) {
        return k + 1 < NW ? __builtin_amdgcn_alignbit(S[(k + 1) * 64], a, 1) : (a >> 1) | (S[0] << end);
    };
    auto down = [&](const uint32_t* S, int k, uint32_t a) {
        return k > 0 ? __builtin_amdgcn_alignbit(a, S[(k - 1) * 64], 31) : (a << 1) | (S[(NW - 1) * 64] >> end);
    };
    const uint16_t* __restrict__ Tab = gauss_table(st);
    const uint64_t* __restrict__ Tab64 = gauss_table64<2>(st);
    words::Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    auto load_rows = [&](int col, int k, gu32x4 (&rows)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = WHOLE || 4 * k + i < M ? 4 * k + i : M - 1;
            rows[i] = ((grow_ptr)Tab)[((col * M + m) << 2) + (lane & 3)];
        }
    };
    auto call_row = [&](int col, int m) { return ((grow_ptr)Tab)[((col * M + m) << 2) + (lane & 3)]; };
    gu32x4 rows[4];
    if constexpr (CALLS) {
        if (wave < M) rows[0] = call_row(0, wave);
    } else {
        if (wave < NW) load_rows(0, wave, rows);
    }
    for (int64_t t = t0; t < t0 + ns; ++t) {
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * t + col);
            uint32_t* W = col ? E1 : E0;
            const uint32_t* O = col ? E0 : E1;
            if constexpr (CALLS) {
#pragma unroll 1
                for (int m = wave; m < M; m += NWV) {
                    const bool last = m + NWV >= M;
                    const gu32x4 next = call_row(last ? col ^ 1 : col, last ? wave : m + NWV);
                    const int k = m >> 2, i = m & 3;
                    const uint32_t w = W[k * 64], a = O[k * 64];
                    const uint32_t X[2] = {w ^ (col ? up(O, k, a) : a), w ^ (col ? a : down(O, k, a))};
                    const uint32_t sites = WHOLE || k + 1 < NW ? 0xFFFFFFFFu : last_sites;
                    reinterpret_cast<uint8_t*>(W + k * 64)[i] =
                        (uint8_t)gauss_byte<2>(w, X, rows[0], sites, col ? 0xFFFFFFFFu : 0u,
                                               Tab64 + ((size_t)(col * M + 4 * k) << 5), (uint32_t)k, i, c);
                    rows[0] = next;
                }
            } else {
#pragma unroll 1
                for (int k = wave; k < NW; k += NWV) {
                    gu32x4 next[4];
                    const bool last = k + NWV >= NW;
                    load_rows(last ? col ^ 1 : col, last ? wave : k + NWV, next);
                    const uint32_t w = W[k * 64], a = O[k * 64];
                    // neighbours +1 and -1 of site 2 b + col
                    const uint32_t X[2] = {w ^ (col ? up(O, k, a) : a), w ^ (col ? a : down(O, k, a))};
                    const uint64_t* T64w = Tab64 + ((size_t)(col * M + 4 * k) << 5);
                    const uint32_t odd = col ? 0xFFFFFFFFu : 0u;
                    const bool full = WHOLE || k + 1 < NW;
                    W[k * 64] = gauss_word<2, WHOLE ? 4 : 0>(w, X, rows, full ? 0xFFFFFFFFu : last_sites, odd, full ? 4 : last_bytes,
                                                     T64w, k, c);
#pragma unroll
                    for (int i = 0; i < 4; ++i) rows[i] = next[i];
                }
            }
            __syncthreads();
        }
    }
#pragma unroll 1
    for (int k = wave; k < NW; k += NWV)
        if (valid) strings::store_word_u8(row, stride, k, E0[k * 64], E1[k * 64]);
    if (wave != 0) return;
    // E in bond order: bond i joins sites i and i + 1
    const double* __restrict__ J = reinterpret_cast<const double*>(st->J);
    double E = 0.0;
#pragma unroll 1
    for (int k = 0; k < NW; ++k) {
        const uint32_t a = E0[k * 64], b = E1[k * 64];
        const uint32_t d0 = a ^ b, d1 = b ^ up(E0, k, a);
        const int n = k + 1 == NW ? end + 1 : 32;
        const double* Jk = J + 64 * k;
#pragma unroll 4
        for (int j = 0; j < n; ++j) {
            E = E + (((d0 >> j) & 1u) ? -Jk[2 * j] : Jk[2 * j]);
            E = E + (((d1 >> j) & 1u) ? -Jk[2 * j + 1] : Jk[2 * j + 1]);
        }
    }
    if (valid) reinterpret_cast<double*>(st->energy[st->cur])[r] = E;
}

// Chains of up to 128 sites: a replica's two strings are one or two registers each, and so are the rows
// of all their calls (CALLS per colour), so a sweep touches no memory; four groups of one wave per block.
template <int CALLS>
__global__ void __launch_bounds__(kGaussWaves * 64) k_sweep_gauss_short(pa_state* __restrict__ states, int n_runs,
                                                                        int blocks, int64_t t0, int ns)
{
    constexpr int NW = (CALLS + 3) / 4, LAST = CALLS - 4 * (NW - 1);  // words, calls of the last one
    int run, block;
    if (!gauss_place(n_runs, blocks, &run, &block)) return;
    const pa_state* st = states + run;
    const int64_t R = st->R;
    const int lane = threadIdx.x & 63, w4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = ((int64_t)block * kGaussWaves + w4) * 64 + lane;
    if (st->status || r - lane >= R) return;
    const int end = (st->N / 2 - 1) & 31;  // the last site's bit in the last word
    const uint32_t sites = 0xFFFFFFFFu >> (31 - end);
    const int stride = st->row_stride;
    uint8_t* row = (uint8_t*)st->spins[st->cur] + r * stride;
    uint32_t s[2][NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) strings::load_word_u8(row, stride, k, &s[0][k], &s[1][k]);
    s[0][NW - 1] &= sites;
    s[1][NW - 1] &= sites;
    // a string's word k shifted by one site, periodically (bits past the last site arbitrary)
    auto up = [&](const uint32_t (&v)[NW], int k) {
        return k + 1 < NW ? __builtin_amdgcn_alignbit(v[NW - 1], v[k], 1) : (v[k] >> 1) | (v[0] << end);
    };
    auto down = [&](const uint32_t (&v)[NW], int k) {
        return k > 0 ? __builtin_amdgcn_alignbit(v[k], v[0], 31) : (v[0] << 1) | (v[NW - 1] >> end);
    };
    const uint16_t* __restrict__ Tab = gauss_table(st);
    const uint64_t* __restrict__ Tab64 = gauss_table64<2>(st);
    gu32x4 rows[2][CALLS];
#pragma unroll
    for (int i = 0; i < 2 * CALLS; ++i) rows[i / CALLS][i % CALLS] = ((grow_ptr)Tab)[(i << 2) + (lane & 3)];
    words::Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    for (int64_t t = t0; t < t0 + ns; ++t) {
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * t + col);
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                // site 2 b: neighbours 2 b + 1 and 2 b - 1; site 2 b + 1: 2 b + 2 and 2 b
                const uint32_t w = s[col][k], a = s[col ^ 1][k];
                const uint32_t X[2] = {w ^ (col ? up(s[0], k) : a), w ^ (col ? a : down(s[1], k))};
                const uint64_t* T64w = Tab64 + ((size_t)(col * CALLS + 4 * k) << 5);
                const uint32_t odd = col ? 0xFFFFFFFFu : 0u;
                if (k + 1 < NW) {
                    const gu32x4 (&rw)[4] = *reinterpret_cast<const gu32x4 (*)[4]>(&rows[col][0]);
                    s[col][k] = gauss_word<2, 4>(w, X, rw, 0xFFFFFFFFu, odd, 4, T64w, (uint32_t)k, c);
                } else {
                    const gu32x4 (&rw)[LAST] = *reinterpret_cast<const gu32x4 (*)[LAST]>(&rows[col][4 * (NW - 1)]);
                    s[col][k] = gauss_word<2, LAST>(w, X, rw, sites, odd, LAST, T64w, (uint32_t)k, c);
                }
            }
        }
    }
    if (r < R)
#pragma unroll
        for (int k = 0; k < NW; ++k) strings::store_word_u8(row, stride, k, s[0][k], s[1][k]);
    // E in bond order: bond i joins sites i and i + 1
    const double* __restrict__ J = reinterpret_cast<const double*>(st->J);
    double E = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const uint32_t d0 = s[0][k] ^ s[1][k], d1 = s[1][k] ^ up(s[0], k);
        const int n = k + 1 < NW ? 32 : end + 1;
#pragma unroll 4
        for (int j = 0; j < n; ++j) {
            E = E + (((d0 >> j) & 1u) ? -J[64 * k + 2 * j] : J[64 * k + 2 * j]);
            E = E + (((d1 >> j) & 1u) ? -J[64 * k + 2 * j + 1] : J[64 * k + 2 * j + 1]);
        }
    }
    if (r < R) reinterpret_cast<double*>(st->energy[st->cur])[r] = E;
}

// the tabled kernels cover cubes of even side 4 to 16 and chains of up to 4096 sites
static bool gauss_tab_shape(int dim, int L) { return dim == 3 ? L >= 4 && L <= 16 : L <= 4096; }

// energy mean, variance, skewness of the population, the overlap histogram cleared where one will be counted
// (one block; any summation order: these are
// compared to 1e-12, not bit for bit)
__global__ void __launch_bounds__(256) k_moments_gauss(pa_state* base, bool overlap)
{
    pa_state* st = base + blockIdx.y;
    if (overlap) hist::clear_overlaps(st, 0, 1);
    if (st->status) return;
    __shared__ double red[256];
    const int64_t R = st->R;
    const double* E = reinterpret_cast<const double*>(st->energy[st->cur]);
    auto bsum = [&](double x) {
        red[threadIdx.x] = x;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
            __syncthreads();
        }
        const double v = red[0];
        __syncthreads();
        return v;
    };
    double a = 0.0;
    for (int64_t j = threadIdx.x; j < R; j += blockDim.x) a += E[j];
    const double mean = bsum(a) / (double)R;
    double b2 = 0.0, b3 = 0.0;
    for (int64_t j = threadIdx.x; j < R; j += blockDim.x) {
        const double d = E[j] - mean;
        b2 += d * d;
        b3 += d * d * d;
    }
    const double m2 = bsum(b2) / (double)R;
    const double m3 = bsum(b3) / (double)R;
    if (threadIdx.x == 0) {
        pa_record* rec = st->record + st->k;
        rec->E_mean = mean;
        rec->E_var = m2;
        rec->E_skew = m2 > 0.0 ? m3 / (m2 * sqrt(m2)) : 0.0;
    }
}

// ------------------------------------------------------------------ launchers
// n runs of one shape with consecutive states from base on stream s; cap the largest capacity
struct GaussLaunch {
    pa_state* base;
    int n;
    int64_t cap;
    hipStream_t s;
};

// Where the population (its capacity, in groups of 64, over the runs of the launch) leaves most of the chip
// idle with a wave per word, its blocks are made of calls.  Chains of more than two calls, 20 sweeps: 64 sites,
// 2 runs of 1000 (42 groups) 47.7 and 39.4 us, 16 runs (336) 49.4 and 43.7, 32 runs 50.2 and 54.1; 128 sites 86.4
// and 48.5, 16 runs 87.3 and 61.7; 512 sites 142 and 108, 16 runs 184 and 118, 24 runs 189 and 205; 32 sites have
// two calls and lose (32.1 and 35.9).  Cubes of side 8, 2 runs of 2000 (82 groups) 160 and 96 us, 4 runs 161
// and 102, 8 runs 166 and 181; side 10, whose block fills a CU's LDS, 2 runs 288 and 115, 6 runs 297 and 321,
// and a whole step with 4 runs of 1500 is 1.2 times as long.  Sides 4 and 6 would sweep faster too, but a step of
// theirs is bound by its launches and gained nothing.
constexpr int64_t kCallGroupsChain = 336;
constexpr int64_t call_groups_cube(int L) { return L == 8 ? 168 : (L == 10 ? 96 : 0); }

// per_block: replicas of a block of `waves` waves
template <class K>
static int launch_gauss_sweep(K kernel, int64_t per_block, int waves, size_t lds, const GaussLaunch& a, const pa_step& step)
{
    const int64_t blocks = (a.cap + per_block - 1) / per_block;
    const int64_t grid = a.n >= 8 ? (a.n * blocks + 7) / 8 * 8 : a.n * blocks;
    if (grid > INT32_MAX) return PA_ERR_ARG;
    if (grid * waves * 64 > kLaunchThreads && a.n > 1) {  // (the runs of a launch all take the largest one's blocks)
        GaussLaunch lo = a, hi = a;
        lo.n = a.n / 2;
        hi.n = a.n - lo.n;
        hi.base += lo.n;
        const int st = launch_gauss_sweep(kernel, per_block, waves, lds, lo, step);
        return st != PA_OK ? st : launch_gauss_sweep(kernel, per_block, waves, lds, hi, step);
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3((unsigned)waves * 64), lds, a.s, a.base, a.n, (int)blocks, step.t0,
                       step.n_sweeps);
    return hip_status(hipGetLastError());
}

template <int NB, int LC>
static void launch_gauss_table(int N, const GaussLaunch& a, double beta)
{
    const unsigned blocks = (unsigned)((((16 * gauss_calls(N)) << NB) + 255) / 256);
    hipLaunchKernelGGL((k_gauss_table<NB, LC>), dim3(blocks, (unsigned)a.n), dim3(256), 0, a.s, a.base, beta);
}

template <int L>
static int launch_gauss_cube(const GaussLaunch& a, const pa_step& step)
{
    if (step.n_sweeps > 0) launch_gauss_table<6, L>(L * L * L, a, step.beta_to);
    constexpr int NWV = L == 4 ? 1 : 4;  // (side 4: one word per colour)
    if constexpr (call_groups_cube(L) > 0)
        if (a.n * (a.cap / 64) <= call_groups_cube(L))
            return launch_gauss_sweep(k_sweep_gauss_split<L>, kSplitReplicas, kSplitReplicas * GaussSplitSmem<L>::UNITS / 64, 0, a, step);
    return launch_gauss_sweep(k_sweep_gauss_cube<L, NWV>, 64 * (kGaussWaves / NWV), kGaussWaves, 0, a, step);
}

static int launch_gauss_chain(int N, const GaussLaunch& a, const pa_step& step)
{
    if (step.n_sweeps > 0) launch_gauss_table<2, 0>(N, a, step.beta_to);
    const size_t lds = (size_t)2 * ((N / 2 + 31) / 32) * 64 * 4;
    if (gauss_calls(N) > 2 && a.n * (a.cap / 64) <= kCallGroupsChain) {
        const int waves = std::min(kGaussCallWaves, (gauss_calls(N) + 3) / 4 * 4);
        return N % 64 == 0 ? launch_gauss_sweep(k_sweep_gauss_chain<true, true>, 64, waves, lds, a, step)
                           : launch_gauss_sweep(k_sweep_gauss_chain<false, true>, 64, waves, lds, a, step);
    }
    switch (gauss_calls(N)) {
        case 1: return launch_gauss_sweep(k_sweep_gauss_short<1>, 64 * kGaussWaves, kGaussWaves, 0, a, step);
        case 2: return launch_gauss_sweep(k_sweep_gauss_short<2>, 64 * kGaussWaves, kGaussWaves, 0, a, step);
        case 3: return launch_gauss_sweep(k_sweep_gauss_short<3>, 64 * kGaussWaves, kGaussWaves, 0, a, step);
        case 4: return launch_gauss_sweep(k_sweep_gauss_short<4>, 64 * kGaussWaves, kGaussWaves, 0, a, step);
        case 5: return launch_gauss_sweep(k_sweep_gauss_short<5>, 64 * kGaussWaves, kGaussWaves, 0, a, step);
        case 6: return launch_gauss_sweep(k_sweep_gauss_short<6>, 64 * kGaussWaves, kGaussWaves, 0, a, step);
        case 7: return launch_gauss_sweep(k_sweep_gauss_short<7>, 64 * kGaussWaves, kGaussWaves, 0, a, step);
        case 8: return launch_gauss_sweep(k_sweep_gauss_short<8>, 64 * kGaussWaves, kGaussWaves, 0, a, step);
        default: break;
    }
    return N % 64 == 0 ? launch_gauss_sweep(k_sweep_gauss_chain<true, false>, 64, kGaussWaves, lds, a, step)
                       : launch_gauss_sweep(k_sweep_gauss_chain<false, false>, 64, kGaussWaves, lds, a, step);
}

int launch_sweep_gauss(const pa_run* runs, int n_runs, bool consecutive, const pa_step& step, hipStream_t s)
{
    const int dim = runs[0].dim, L = runs[0].L;
    bool same = true;
    for (int r = 1; r < n_runs; ++r) same = same && runs[r].dim == dim && runs[r].L == L;
    if (n_runs > 1 && !(consecutive && same)) {
        for (int r = 0; r < n_runs; ++r) {
            const int st = launch_sweep_gauss(&runs[r], 1, true, step, (hipStream_t)runs[r].stream);
            if (st != PA_OK) return st;
        }
        return PA_OK;
    }
    if (!gauss_tab_shape(dim, L)) {
        for (int r = 0; r < n_runs; ++r) {
            hipLaunchKernelGGL(k_sweep_gauss, dim3((unsigned)((runs[r].capacity + 63) / 64)), dim3(64), 0, s,
                               (const pa_state*)runs[r].state, step.beta_to, step.t0, step.n_sweeps);
            const int st = hip_status(hipGetLastError());
            if (st != PA_OK) return st;
        }
        return PA_OK;
    }
    GaussLaunch a = {runs[0].state, n_runs, 0, s};
    for (int r = 0; r < n_runs; ++r) a.cap = runs[r].capacity > a.cap ? runs[r].capacity : a.cap;
    if (dim == 1) return launch_gauss_chain(L, a, step);
    switch (L) {
        case 4: return launch_gauss_cube<4>(a, step);
        case 6: return launch_gauss_cube<6>(a, step);
        case 8: return launch_gauss_cube<8>(a, step);
        case 10: return launch_gauss_cube<10>(a, step);
        case 12: return launch_gauss_cube<12>(a, step);
        case 14: return launch_gauss_cube<14>(a, step);
        default: return launch_gauss_cube<16>(a, step);
    }
}

// energies of the current populations of n runs with consecutive states: the tabled kernels with no
// sweeps, which hold 64 replicas' spins in LDS (one thread per replica over byte rows took 156 us for
// 2000 replicas of side 8, whatever the number of runs), one thread per replica past their shapes
int launch_energy_gauss(const pa_run* runs, int n, hipStream_t s)
{
    bool tab = true;
    int64_t cap = 0;
    for (int r = 0; r < n; ++r) {
        tab = tab && gauss_tab_shape(runs[r].dim, runs[r].L) && runs[r].L == runs[0].L;
        cap = runs[r].capacity > cap ? runs[r].capacity : cap;
    }
    if (tab) {
        pa_step none = {};
        return launch_sweep_gauss(runs, n, true, none, s);
    }
    hipLaunchKernelGGL(k_energy_gauss, dim3((unsigned)((cap + 63) / 64), (unsigned)n), dim3(64), 0, s,
                       (const pa_state*)runs[0].state);
    return hip_status(hipGetLastError());
}

int launch_moments_gauss(const pa_run* runs, int n, bool overlap, hipStream_t s)
{
    hipLaunchKernelGGL(k_moments_gauss, dim3(1, (unsigned)n), dim3(256), 0, s, runs[0].state, overlap);
    return hip_status(hipGetLastError());
}

}  // namespace pa

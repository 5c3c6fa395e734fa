// Metropolis sweeps of chains with +-1 couplings: the same sample as the generic kernel (same Philox
// fields, same acceptance rule, same order of colours).
//
// A replica's sites of one colour are a bit string: bit b of colour c is site 2 b + c, whose Metropolis
// field is field b mod 8 of Philox call b / 8, so a 32-bit word is four whole calls.  The neighbours of
// bit b of colour 0 are bits b and b - 1 of colour 1, those of bit b of colour 1 are bits b + 1 and b
// of colour 0.  A flip is free unless both bonds are satisfied (in the kernels' convention: both bond
// bits set), and then one bound serves every site, so the decision needs no table (words::decide_word
// with one bound).  Lane = replica, so the words' call indices are the same over a wave.
//
// Bound by the vector ALU where the population fills the chip (6.9 instructions per attempt, Philox 4.7)
// and by a wave's own chain of instructions where it does not (hence the second pair of kernels, with a
// lane per call).  The generic kernel takes a site at a
// time and moves byte rows a byte at a time: N = 64, 5 sweeps, 1000 replicas 29 us (here
// 4.6), 200 runs of them 80 (here 24).
#include "pa_common.h"
#include "pa_host.h"
#include "pa_sweep_strings.h"
#include "pa_sweep_util.h"

namespace pa {

namespace chain {

using namespace strings;

constexpr int kWaves = 4;

// word k of a replica's two strings (sites 64 k ..) from its byte row, or from the row words 2 k and
// 2 k + 1 of its bit-packed group (rows: its bytes or its word of row 0; n_rows rows of 32 sites)
template <int LAYOUT>
__device__ __forceinline__ void load_word(const uint8_t* rows, int stride, int n_rows, int k, uint32_t* ev, uint32_t* od)
{
    if constexpr (LAYOUT == PA_U8) {
        load_word_u8(rows, stride, k, ev, od);
    } else {
        const uint32_t* a = reinterpret_cast<const uint32_t*>(rows) + 128 * k;
        const uint32_t lo = a[0], hi = 2 * k + 1 < n_rows ? a[64] : 0u;
        uint32_t o_lo, o_hi;
        const uint32_t e_lo = split_row(lo, &o_lo), e_hi = split_row(hi, &o_hi);
        *ev = e_lo | (e_hi << 16);
        *od = o_lo | (o_hi << 16);
    }
}

template <int LAYOUT>
__device__ __forceinline__ void store_word(uint8_t* rows, int stride, int n_rows, int k, uint32_t ev, uint32_t od)
{
    if constexpr (LAYOUT == PA_U8) {
        store_word_u8(rows, stride, k, ev, od);
    } else {
        uint32_t* a = reinterpret_cast<uint32_t*>(rows) + 128 * k;
        a[0] = merge_row(ev & 0xFFFFu, od & 0xFFFFu);
        if (2 * k + 1 < n_rows) a[64] = merge_row(ev >> 16, od >> 16);
    }
}

// this lane's replica in the current population's buffer
template <int LAYOUT>
__device__ __forceinline__ uint8_t* replica_rows(const pa_state* st, int64_t r, int n_rows)
{
    uint8_t* base = (uint8_t*)st->spins[st->cur];
    return LAYOUT == PA_U8 ? base + r * st->row_stride : base + (((r >> 6) * n_rows) * 64 + (r & 63)) * 4;
}

// The coupling masks of word k (bit b set where J = -1), formed by the wave: j[0] bond 2 b (site 2 b to
// 2 b + 1), j[1] bond 2 b + 1, j[2] bond 2 b - 1
__device__ __forceinline__ void bond_masks(const int8_t* J, int N, int k, int lane, uint32_t (&j)[3])
{
    const int i = 64 * k + 2 * (lane & 31) + (lane >> 5);  // lanes 0..31: bond 2 b, lanes 32..63: bond 2 b + 1
    const uint64_t m = __ballot(i < N && J[i < N ? i : 0] < 0);
    const int before = k == 0 ? N - 1 : 64 * k - 1;
    j[0] = (uint32_t)m;
    j[1] = (uint32_t)(m >> 32);
    j[2] = (j[1] << 1) | (uint32_t)(J[before] < 0);
}

// one colour's attempts in a word: X the bond words of +1 and -1 (set: J s s = -1)
template <int MODE, int NBYTES, bool TIES_IN_LINE = true>
__device__ __forceinline__ uint32_t update(uint32_t w, uint32_t b0, uint32_t b1, uint32_t sites, uint32_t k, int col,
                                           const Lane& c, const Thr& th)
{
    const uint32_t cand = b0 & b1 & sites;
    const uint32_t nw = decide_word<MODE, true, NBYTES, TIES_IN_LINE>(w, 0u, 0u, cand, 4u * k, 1u, nullptr, c, th, [&]() {
        return WordSites{4u * k, 1u, 64u * k, 16u, col ? 0xFFFFFFFFu : 0u};
    });
    return select_bits(sites, nw, w);
}

// Chains of up to 128 sites: the strings and the coupling masks in registers, so a sweep touches no
// memory.  CALLS: Philox calls per colour; grid (blocks of four groups of one wave each, runs).
template <int CALLS, int MODE, int LAYOUT>
__global__ void __launch_bounds__(64 * kWaves) k_sweep_chain_short(const pa_state* __restrict__ base, SweepParams p, Thr th)
{
    constexpr int NW = (CALLS + 3) / 4, LAST = CALLS - 4 * (NW - 1);
    const pa_state* __restrict__ st = base + blockIdx.y;
    const int lane = threadIdx.x & 63, w4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t R = st->R, r = ((int64_t)blockIdx.x * kWaves + w4) * 64 + lane;
    if (st->status || r - lane >= R) return;  // sticky error: the population stays as it is
    const int N = st->N, n_rows = (N + 31) / 32, stride = st->row_stride;
    const int end = (N / 2 - 1) & 31;  // the last site's bit in the last word
    const uint32_t last_sites = 0xFFFFFFFFu >> (31 - end);
    uint8_t* rows = replica_rows<LAYOUT>(st, r, n_rows);
    uint32_t s[2][NW], j[NW][3];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const uint32_t in = k + 1 < NW ? 0xFFFFFFFFu : last_sites;
        load_word<LAYOUT>(rows, stride, n_rows, k, &s[0][k], &s[1][k]);
        s[0][k] &= in;
        s[1][k] &= in;
        bond_masks(st->J, N, k, lane, j[k]);
    }
    // a string's word k shifted by one site, periodically (bits past the last site arbitrary)
    auto up = [&](const uint32_t (&v)[NW], int k) {
        return k + 1 < NW ? __builtin_amdgcn_alignbit(v[NW - 1], v[k], 1) : (v[k] >> 1) | (v[0] << end);
    };
    auto down = [&](const uint32_t (&v)[NW], int k) {
        return k > 0 ? __builtin_amdgcn_alignbit(v[k], v[0], 31) : (v[0] << 1) | (v[NW - 1] >> end);
    };
    Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    for (int t = 0; t < p.n_sweeps; ++t) {
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * (p.t0 + t) + col);
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                const uint32_t w = s[col][k], a = s[col ^ 1][k];
                const uint32_t b0 = col ? xor3(w, up(s[0], k), j[k][1]) : xor3(w, a, j[k][0]);
                const uint32_t b1 = col ? xor3(w, a, j[k][0]) : xor3(w, down(s[1], k), j[k][2]);
                s[col][k] = k + 1 < NW ? update<MODE, 4>(w, b0, b1, 0xFFFFFFFFu, (uint32_t)k, col, c, th)
                                       : update<MODE, LAST>(w, b0, b1, last_sites, (uint32_t)k, col, c, th);
            }
        }
    }
    if (r >= R) return;
    int neg = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const uint32_t in = k + 1 < NW ? 0xFFFFFFFFu : last_sites;
        neg += __popc(xor3(s[0][k], s[1][k], j[k][0]) & in) + __popc(xor3(s[1][k], up(s[0], k), j[k][1]) & in);
        store_word<LAYOUT>(rows, stride, n_rows, k, s[0][k], s[1][k]);
    }
    st->energy[st->cur][r] = N - 2 * neg;
}

// Longer chains: the strings of a block's 64 replicas in LDS ([colour][word][replica]) and the masks of
// every word ([word][4]), the words split by four waves that meet after each colour.  first: the first block
// of this part of the grid.
template <int MODE, int LAYOUT>
__global__ void __launch_bounds__(64 * kWaves) k_sweep_chain(const pa_state* __restrict__ base, uint32_t first, SweepParams p,
                                                             Thr th)
{
    extern __shared__ uint32_t lds[];
    const pa_state* __restrict__ st = base + blockIdx.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t R = st->R, r = (int64_t)(first + blockIdx.x) * 64 + lane;
    if (st->status || r - lane >= R) return;  // the same for the whole block
    const bool valid = r < R;
    const int N = st->N, n_rows = (N + 31) / 32, stride = st->row_stride, NW = (N / 2 + 31) / 32;
    const int end = (N / 2 - 1) & 31;
    const uint32_t last_sites = 0xFFFFFFFFu >> (31 - end);
    uint32_t* S0 = lds + lane;
    uint32_t* S1 = S0 + NW * 64;
    uint32_t* masks = lds + 2 * NW * 64;
    int* neg_sum = reinterpret_cast<int*>(masks + 4 * NW);
    if (threadIdx.x < 64) neg_sum[threadIdx.x] = 0;
    uint8_t* rows = replica_rows<LAYOUT>(st, r, n_rows);
#pragma unroll 1
    for (int k = wave; k < NW; k += kWaves) {
        const uint32_t in = k + 1 < NW ? 0xFFFFFFFFu : last_sites;
        uint32_t ev, od, j[3];
        load_word<LAYOUT>(rows, stride, n_rows, k, &ev, &od);
        S0[k * 64] = ev & in;
        S1[k * 64] = od & in;
        bond_masks(st->J, N, k, lane, j);
        if (lane < 3) masks[4 * k + lane] = lane == 0 ? j[0] : (lane == 1 ? j[1] : j[2]);
    }
    __syncthreads();
    auto up = [&](const uint32_t* S, int k, uint32_t a) {
        return k + 1 < NW ? __builtin_amdgcn_alignbit(S[(k + 1) * 64], a, 1) : (a >> 1) | (S[0] << end);
    };
    auto down = [&](const uint32_t* S, int k, uint32_t a) {
        return k > 0 ? __builtin_amdgcn_alignbit(a, S[(k - 1) * 64], 31) : (a << 1) | (S[(NW - 1) * 64] >> end);
    };
    Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    for (int t = 0; t < p.n_sweeps; ++t) {
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * (p.t0 + t) + col);
            uint32_t* W = col ? S1 : S0;
            const uint32_t* O = col ? S0 : S1;
#pragma unroll 1
            for (int k = wave; k < NW; k += kWaves) {
                const uint32_t w = W[k * 64], a = O[k * 64];
                const uint32_t* j = masks + 4 * k;
                const uint32_t b0 = col ? xor3(w, up(O, k, a), j[1]) : xor3(w, a, j[0]);
                const uint32_t b1 = col ? xor3(w, a, j[0]) : xor3(w, down(O, k, a), j[2]);
                W[k * 64] = update<MODE, 4, false>(w, b0, b1, k + 1 < NW ? 0xFFFFFFFFu : last_sites, (uint32_t)k, col, c, th);
            }
            __syncthreads();
        }
    }
    int neg = 0;
#pragma unroll 1
    for (int k = wave; k < NW; k += kWaves) {
        const uint32_t in = k + 1 < NW ? 0xFFFFFFFFu : last_sites;
        const uint32_t a = S0[k * 64], b = S1[k * 64];
        neg += __popc(xor3(a, b, masks[4 * k]) & in) + __popc(xor3(b, up(S0, k, a), masks[4 * k + 1]) & in);
        if (valid) store_word<LAYOUT>(rows, stride, n_rows, k, a, b);
    }
    atomicAdd(&neg_sum[lane], neg);
    __syncthreads();
    if (wave == 0 && valid) st->energy[st->cur][r] = N - 2 * neg_sum[lane];
}

// 16 consecutive sites (byte i of word k's two strings) of a replica's rows
template <int LAYOUT>
__device__ __forceinline__ void load_piece(const uint8_t* rows, int stride, int n_rows, int k, int i, uint32_t* ev, uint32_t* od)
{
    *ev = *od = 0;
    if constexpr (LAYOUT == PA_U8) {
        if (64 * k + 16 * i >= stride) return;
        const uint4 q = *reinterpret_cast<const uint4*>(rows + 64 * k + 16 * i);
        *ev = pack4(__builtin_amdgcn_perm(q.y, q.x, 0x06040200u)) | (pack4(__builtin_amdgcn_perm(q.w, q.z, 0x06040200u)) << 4);
        *od = pack4(__builtin_amdgcn_perm(q.y, q.x, 0x07050301u)) | (pack4(__builtin_amdgcn_perm(q.w, q.z, 0x07050301u)) << 4);
    } else {
        const int row = 2 * k + (i >> 1);
        if (row >= n_rows) return;
        *ev = split_row(reinterpret_cast<const uint32_t*>(rows)[64 * row] >> (16 * (i & 1)) & 0xFFFFu, od);
    }
}

// the same sites back from the whole words (bit-packed: one store per row, by its first piece)
template <int LAYOUT>
__device__ __forceinline__ void store_piece(uint8_t* rows, int stride, int n_rows, int k, int i, uint32_t ev, uint32_t od)
{
    if constexpr (LAYOUT == PA_U8) {
        if (64 * k + 16 * i >= stride) return;
        const uint32_t e0 = unpack4(ev >> (8 * i)), o0 = unpack4(od >> (8 * i));
        const uint32_t e1 = unpack4(ev >> (8 * i + 4)), o1 = unpack4(od >> (8 * i + 4));
        *reinterpret_cast<uint4*>(rows + 64 * k + 16 * i) =
            make_uint4(__builtin_amdgcn_perm(o0, e0, 0x05010400u), __builtin_amdgcn_perm(o0, e0, 0x07030602u),
                       __builtin_amdgcn_perm(o1, e1, 0x05010400u), __builtin_amdgcn_perm(o1, e1, 0x07030602u));
    } else {
        const int row = 2 * k + (i >> 1);
        if ((i & 1) || row >= n_rows) return;
        reinterpret_cast<uint32_t*>(rows)[64 * row] = merge_row((ev >> (8 * i)) & 0xFFFFu, (od >> (8 * i)) & 0xFFFFu);
    }
}

// byte i of one colour's updated word k: one call
template <int MODE>
__device__ __forceinline__ uint32_t update_byte(uint32_t w, uint32_t cand, int k, int i, int col, const Lane& c, const Thr& th)
{
    const uint32_t call = (uint32_t)(4 * k + i);
    const uint32_t nb = decide_word<MODE, false, 1>((w >> (8 * i)) & 0xFFu, 0u, 0u, (cand >> (8 * i)) & 0xFFu, call, 1u, nullptr,
                                                    c, th, [&]() { return WordSites{call, 1u, 16u * call, 16u, col ? 0xFFFFFFFFu : 0u}; });
    return nb & 0xFFu;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

// A lane per call instead of one per replica, where the population has too few groups to fill the chip.
// Up to 128 sites: four or eight neighbouring lanes hold the replica's words, each decides its byte, and
// the lanes put the word together among themselves.  NW: words per colour; a block of kWaves waves takes
// 256 / (4 NW) replicas.
template <int NW, int MODE, int LAYOUT>
__global__ void __launch_bounds__(64 * kWaves) k_sweep_chain_short_split(const pa_state* __restrict__ base, SweepParams p, Thr th)
{
    constexpr int LPR = 4 * NW;
    const pa_state* __restrict__ st = base + blockIdx.y;
    const int64_t R = st->R, r = ((int64_t)blockIdx.x * (64 * kWaves) + threadIdx.x) / LPR;
    if (st->status || ((int64_t)blockIdx.x * (64 * kWaves) + (threadIdx.x & ~63u)) / LPR >= R) return;  // the whole wave
    const int N = st->N, n_rows = (N + 31) / 32, stride = st->row_stride;
    const int l = threadIdx.x % LPR, k = l >> 2, i = l & 3;  // this lane's word and byte
    const int end = (N / 2 - 1) & 31;  // the last site's bit in the last word
    const bool last = k + 1 == NW;
    const uint32_t sites = last ? 0xFFFFFFFFu >> (31 - end) : 0xFFFFFFFFu;
    uint8_t* rows = replica_rows<LAYOUT>(st, r < R ? r : R - 1, n_rows);
    // the two colours' words: this lane's, and the replica's other one (the same where there is one)
    uint32_t own[2], oth[2], j[3];
    auto whole = [&](uint32_t byte) {  // the word of the quad's bytes
        uint32_t x = byte << (8 * i);
        x |= dpp<0xB1>(x);
        x |= dpp<0x4E>(x);
        return x;
    };
    auto other = [&](uint32_t v) { return NW == 1 ? v : dpp<0x141>(v); };
    load_piece<LAYOUT>(rows, stride, n_rows, k, i, &own[0], &own[1]);
#pragma unroll
    for (int col = 0; col < 2; ++col) {
        own[col] = whole(own[col]) & sites;
        oth[col] = other(own[col]);
    }
    {
        uint32_t m[NW][3];
#pragma unroll
        for (int q = 0; q < NW; ++q) bond_masks(st->J, N, q, threadIdx.x & 63, m[q]);
#pragma unroll
        for (int d = 0; d < 3; ++d) j[d] = last ? m[NW - 1][d] : m[0][d];
    }
    // the other word's bit that comes in at the top (up) and at the bottom (down) of a shifted word
    const int top = last ? end : 31, bottom = k > 0 ? 31 : end;
    Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    for (int t = 0; t < p.n_sweeps; ++t) {
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * (p.t0 + t) + col);
            const uint32_t w = own[col], a = own[col ^ 1], o = oth[col ^ 1];
            const uint32_t b0 = xor3(w, a, j[0]);
            const uint32_t b1 = col ? xor3(w, (a >> 1) | (o << top), j[1]) : xor3(w, (a << 1) | (o >> bottom), j[2]);
            own[col] = select_bits(sites, whole(update_byte<MODE>(w, b0 & b1 & sites, k, i, col, c, th)), w);
            oth[col] = other(own[col]);
        }
    }
    int neg = __popc(xor3(own[0], own[1], j[0]) & sites) +
              __popc(xor3(own[1], (own[0] >> 1) | (oth[0] << top), j[1]) & sites);
    neg += NW == 1 ? 0 : (int)dpp<0x141>((uint32_t)neg);
    if (r >= R) return;
    store_piece<LAYOUT>(rows, stride, n_rows, k, i, own[0], own[1]);
    if (l == 0) st->energy[st->cur][r] = N - 2 * neg;
}

// Longer chains: Q replicas per block, their words in LDS ([colour][word][replica]), each byte of a colour
// taken by one thread.  Q = 16 where 16 calls are all of a colour (up to 256 sites), else 4 (N = 1024, 1000
// replicas, five sweeps: 16 replicas a block 22.4 us, 8 15.9, 4 11.7).
template <int Q, int MODE, int LAYOUT>
__global__ void __launch_bounds__(64 * kWaves) k_sweep_chain_split(const pa_state* __restrict__ base, SweepParams p, Thr th)
{
    constexpr int UNITS = 64 * kWaves / Q;
    extern __shared__ uint32_t lds[];
    const pa_state* __restrict__ st = base + blockIdx.y;
    const int q = threadIdx.x % Q, unit = threadIdx.x / Q;
    const int64_t R = st->R, r0 = (int64_t)blockIdx.x * Q, r = r0 + q;
    if (st->status || r0 >= R) return;  // the same for the whole block
    const int N = st->N, n_rows = (N + 31) / 32, stride = st->row_stride, NW = (N / 2 + 31) / 32;
    const int calls = (N / 2 + 7) / 8, end = (N / 2 - 1) & 31;
    const uint32_t last_sites = 0xFFFFFFFFu >> (31 - end);
    uint32_t* S0 = lds + q;
    uint32_t* S1 = S0 + NW * Q;
    uint32_t* masks = lds + 2 * NW * Q;
    int* neg_sum = reinterpret_cast<int*>(masks + 4 * NW);
    if (threadIdx.x < Q) neg_sum[threadIdx.x] = 0;
    uint8_t* rows = replica_rows<LAYOUT>(st, r < R ? r : R - 1, n_rows);
    for (int b = unit; b < 4 * NW; b += UNITS) {  // bytes past the last site are zero
        const int k = b >> 2, i = b & 3;
        const uint32_t in = ((k + 1 < NW ? 0xFFFFFFFFu : last_sites) >> (8 * i)) & 0xFFu;
        uint32_t ev, od;
        load_piece<LAYOUT>(rows, stride, n_rows, k, i, &ev, &od);
        reinterpret_cast<uint8_t*>(S0 + k * Q)[i] = (uint8_t)(ev & in);
        reinterpret_cast<uint8_t*>(S1 + k * Q)[i] = (uint8_t)(od & in);
    }
    for (int k = threadIdx.x >> 6; k < NW; k += kWaves) {
        const int lane = threadIdx.x & 63;
        uint32_t j[3];
        bond_masks(st->J, N, k, lane, j);
        if (lane < 3) masks[4 * k + lane] = lane == 0 ? j[0] : (lane == 1 ? j[1] : j[2]);
    }
    __syncthreads();
    auto up = [&](const uint32_t* S, int k, uint32_t a) {
        return k + 1 < NW ? __builtin_amdgcn_alignbit(S[(k + 1) * Q], a, 1) : (a >> 1) | (S[0] << end);
    };
    auto down = [&](const uint32_t* S, int k, uint32_t a) {
        return k > 0 ? __builtin_amdgcn_alignbit(a, S[(k - 1) * Q], 31) : (a << 1) | (S[(NW - 1) * Q] >> end);
    };
    Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    for (int t = 0; t < p.n_sweeps; ++t) {
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * (p.t0 + t) + col);
            uint32_t* W = col ? S1 : S0;
            const uint32_t* O = col ? S0 : S1;
            // a thread writes only its byte of a word, and the byte's other readers in this phase use
            // their own bytes of it alone
#pragma unroll 1
            for (int b = unit; b < calls; b += UNITS) {
                const int k = b >> 2, i = b & 3;
                const uint32_t w = W[k * Q], a = O[k * Q];
                const uint32_t* j = masks + 4 * k;
                const uint32_t b0 = xor3(w, a, j[0]);
                const uint32_t b1 = col ? xor3(w, up(O, k, a), j[1]) : xor3(w, down(O, k, a), j[2]);
                const uint32_t sites = k + 1 < NW ? 0xFFFFFFFFu : last_sites;
                const uint32_t x = update_byte<MODE>(w, b0 & b1 & sites, k, i, col, c, th);
                reinterpret_cast<uint8_t*>(W + k * Q)[i] = (uint8_t)select_bits(sites >> (8 * i), x, w >> (8 * i));
            }
            __syncthreads();
        }
    }
    int neg = 0;
    for (int b = unit; b < 4 * NW; b += UNITS) {
        const int k = b >> 2, i = b & 3;
        const uint32_t a = S0[k * Q], d = S1[k * Q];
        if (i == 0) {
            const uint32_t in = k + 1 < NW ? 0xFFFFFFFFu : last_sites;
            neg += __popc(xor3(a, d, masks[4 * k]) & in) + __popc(xor3(d, up(S0, k, a), masks[4 * k + 1]) & in);
        }
        if (r < R) store_piece<LAYOUT>(rows, stride, n_rows, k, i, a, d);
    }
    if (neg) atomicAdd(&neg_sum[q], neg);
    __syncthreads();
    if (threadIdx.x < Q && r < R) st->energy[st->cur][r] = N - 2 * neg_sum[q];
}

// Where the population (its capacity, in groups of 64, over the runs of the call) is too small for a lane
// per replica to fill the chip, a lane per call (five sweeps at beta 0.5 after one another, capacities 1.6 times
// 1000 replicas a run, lane per replica and per call).  Chains of up to 128 sites, more than one call: N = 64,
// 1 run 7.7 and 4.6 us, 32 runs (800 groups) 8.5 and 7.0, 64 runs (1600) 11.6 and 10.7, 100 runs 12.5 and 13.5;
// N = 128, 1 run 13.4 and 4.7, 64 runs 21.7 and 15.8; N = 16 has one call and gains nothing (4.4 and 4.6).  Longer
// ones: N = 200, 1 run 11.3 and 7.3, 8 runs (200 groups) 12.0 and 9.6, 16 runs 14.7 and 12.8; N = 1024, 1 run 35.2
// and 8.4, 8 runs 37.1 and 20.0.
constexpr int64_t kSplitShort = 1536, kSplitLong = 256;

template <int MODE, int LAYOUT>
static void launch(int N, const pa_state* base, int n, int64_t cap, const SweepParams& p, const Thr& th, hipStream_t s)
{
    const int calls = (N / 2 + 7) / 8;
    const int NW = (N / 2 + 31) / 32;
    const int64_t groups = n * (cap / 64);
    if (NW <= 2 && calls > 1 && groups <= kSplitShort) {
        const dim3 b(64 * kWaves), g((unsigned)((cap * 4 * NW + b.x - 1) / b.x), (unsigned)n);
        if (NW == 1) hipLaunchKernelGGL((k_sweep_chain_short_split<1, MODE, LAYOUT>), g, b, 0, s, base, p, th);
        else hipLaunchKernelGGL((k_sweep_chain_short_split<2, MODE, LAYOUT>), g, b, 0, s, base, p, th);
        return;
    }
    if (NW > 2 && groups <= kSplitLong) {
        const int Q = calls <= 16 ? 16 : 4;
        const size_t lds = ((size_t)2 * NW * Q + 4 * NW + Q) * 4;
        const dim3 b(64 * kWaves), g((unsigned)(cap / Q), (unsigned)n);
        if (Q == 16) hipLaunchKernelGGL((k_sweep_chain_split<16, MODE, LAYOUT>), g, b, lds, s, base, p, th);
        else hipLaunchKernelGGL((k_sweep_chain_split<4, MODE, LAYOUT>), g, b, lds, s, base, p, th);
        return;
    }
    const dim3 b(64 * kWaves), g((unsigned)((cap / 64 + kWaves - 1) / kWaves), (unsigned)n);
    switch (calls) {
        case 1: hipLaunchKernelGGL((k_sweep_chain_short<1, MODE, LAYOUT>), g, b, 0, s, base, p, th); return;
        case 2: hipLaunchKernelGGL((k_sweep_chain_short<2, MODE, LAYOUT>), g, b, 0, s, base, p, th); return;
        case 3: hipLaunchKernelGGL((k_sweep_chain_short<3, MODE, LAYOUT>), g, b, 0, s, base, p, th); return;
        case 4: hipLaunchKernelGGL((k_sweep_chain_short<4, MODE, LAYOUT>), g, b, 0, s, base, p, th); return;
        case 5: hipLaunchKernelGGL((k_sweep_chain_short<5, MODE, LAYOUT>), g, b, 0, s, base, p, th); return;
        case 6: hipLaunchKernelGGL((k_sweep_chain_short<6, MODE, LAYOUT>), g, b, 0, s, base, p, th); return;
        case 7: hipLaunchKernelGGL((k_sweep_chain_short<7, MODE, LAYOUT>), g, b, 0, s, base, p, th); return;
        case 8: hipLaunchKernelGGL((k_sweep_chain_short<8, MODE, LAYOUT>), g, b, 0, s, base, p, th); return;
        default: break;
    }
    const size_t lds = ((size_t)2 * NW * 64 + 4 * NW + 64) * 4;
    launch_parts(cap / 64, (int)b.x, [&](uint32_t first, unsigned blocks) {
        hipLaunchKernelGGL((k_sweep_chain<MODE, LAYOUT>), dim3(blocks, (unsigned)n), b, lds, s, base, first, p, th);
    });
}

}  // namespace chain

// n chains of N sites with consecutive states from base (cap: their largest capacity); false for a length
// or thresholds the kernels do not take (the LDS of 64 replicas of 4096 sites is 33 KB, four blocks per
// CU; tops above 0xFFFE leave no room for the + 1 of the bound)
bool launch_sweep_chain(int N, int layout, const pa_state* base, int n, int64_t cap, const SweepParams& p, hipStream_t s)
{
    if (N > 4096 || p.thi[2] > 0xFFFEu) return false;
    words::Thr th = {};
    th.thi4 = p.thi[2];  // a chain's one class that needs a draw
    th.T4 = p.T64[2];
    if (p.thi[2] == 0) {
        if (layout == PA_U8) chain::launch<2, PA_U8>(N, base, n, cap, p, th, s);
        else chain::launch<2, PA_BITS64>(N, base, n, cap, p, th, s);
    } else {
        if (layout == PA_U8) chain::launch<1, PA_U8>(N, base, n, cap, p, th, s);
        else chain::launch<1, PA_BITS64>(N, base, n, cap, p, th, s);
    }
    return true;
}

}  // namespace pa

// Metropolis sweeps of cubes: the replicas of a block side by side in LDS, and the block's waves split
// the words of a colour between them.  The same sample as the generic kernel (same Philox fields,
// same acceptance rule, same checkerboard order).
//
// A replica's spins are kept in LDS as its two colour strings (pa_sweep_strings.h), so a block takes its
// replicas' worth of LDS however many waves work on it.  LPR = 1: 64 replicas per block, lane =
// replica in every wave, and a wave takes the words w, w + waves, ..: the word is the same over the
// wave's lanes, so the generator's uniform rounds stay on the scalar unit, and a word load hits 64
// banks.  LPR = 4: 16 replicas per block and four consecutive words per wave (again 64 banks), for
// populations with too few 64-replica groups to fill the chip; the rounds that were uniform then run
// on the vector unit (5% more instructions).  A colour phase reads only the other colour's string, so
// the waves meet at one barrier per phase (and one more where the string's length is not a whole
// number of words and its ghost words are funnels of other waves' words).
//
// Bound by the vector ALU (VALUBusy 100%; 7.5 instructions per attempt at L = 16, of which Philox 4.7).
// Measured, ten sweeps at beta 0.5 or 1, against the kernels it replaced (one wave per group, four lanes
// per replica with rows or colour words, and the generic kernel): L = 16, 10^6 replicas 8.10 -> 7.55 ms
// (5.4e12 attempts/s); L = 12, 2 10^5 replicas 1.10 -> 0.75 ms; L = 10, 3 10^4 0.25 -> 0.089 ms; L = 8 in
// bytes, 5 10^4 152 -> 71 us; L = 14, 10^5 5.6 -> 0.65 ms; L = 20, 2 10^4 6.8 -> 0.41 ms.
#include <algorithm>
#include <type_traits>

#include "pa_common.h"
#include "pa_host.h"
#include "pa_sweep_strings.h"
#include "pa_sweep_util.h"

namespace pa {

namespace group {

using namespace strings;

// Waves per block.  Multiples of four where a block has more than two waves: the waves go round the
// four SIMDs of the CU, and a SIMD with one wave more holds the others up at every barrier (L = 12,
// 2 10^5 replicas, 3 waves 896 us, 4 waves 762 us, 9 waves 1004 us a launch of ten sweeps).  Within that, as
// few as keep the CU full with the blocks its LDS holds (L = 16, 10^6 replicas: 4 waves 10.5 ms, 8
// waves 7.7 ms, 16 waves 9.7 ms), dividing the words of a colour with little left over (words: 1, 4, 8,
// 16, 27, 43, 64, 92, 125, 216).  L = 4 and 6: one wave has enough to do in a phase to need no partner
// (L = 6, 10^6 replicas: 1 wave 0.49 ms, 2 waves 0.51, 4 waves 0.57).
__host__ __device__ constexpr int waves_of(int L, int LPR)
{
    switch (L) {
        case 4:
        case 6: return 1;
        case 8: return LPR == 1 ? 4 : 2;
        case 10: return 4;
        case 12: return LPR == 1 ? 4 : 8;
        case 14: return LPR == 1 ? 8 : 4;
        case 18: return LPR == 1 ? 12 : 8;
        default: return 8;
    }
}

// Four lanes per replica instead of one: where the population has fewer 64-replica groups than four
// per CU (ten sweeps at beta 0.5 or 1, one lane and four lanes: L = 6, 157 groups 62 and 22 us; L = 8, 782
// groups 80 and 71 us, 3125 groups 216 and 219 us; L = 12, 157 groups 130 and 66 us, 782 groups 272 and 243,
// 1563 groups 432 and 456; L = 16, 782 groups 536 and 484, 1563 groups 899 and 911), and from L = 20
// on for every size: a CU's LDS holds one block of 64 replicas there, whose waves all wait at its
// barriers (L = 20, 6250 groups 7.9 and 7.5 ms; L = 24, 625 groups 1.58 and 1.33 ms).
// Up to three sweeps it is the blocks' tables and transfers that count, which four lanes per replica repeat four
// times as often: there fewer than 384 groups (one and four lanes, L = 16, 313 groups, one sweep 45 and 41 us,
// three 101 and 77; 469 groups, one 46 and 57, three 101 and 113; L = 8, 469 groups, one 11.0 and 13.5, three
// 20.7 and 21.3; L = 6 is faster with four).
constexpr int64_t kSplitGroups = 1024, kShortGroups = 384;
constexpr int kShortSweeps = 3;
__host__ __device__ constexpr bool always_split(int L) { return L >= 20; }

// groups of a block (a one-wave group needs no barrier: four share a bound table)
__host__ __device__ constexpr int groups_of(int L, int LPR) { return waves_of(L, LPR) == 1 ? 4 : 1; }
__host__ __device__ constexpr int threads_of(int L, int LPR) { return 64 * waves_of(L, LPR) * groups_of(L, LPR); }

template <int L, int LPR>
struct GroupSmem {
    static constexpr int Q = 64 / LPR;         // replicas
    uint32_t E[2 * Geo<L>::EW * Q];            // the two extended strings, [word][replica]
    uint32_t tab[2 * Geo<L>::NW * Geo<L>::TW]; // per (colour, word): coupling and geometry masks
    uint32_t neg[Q];                           // unsatisfied bonds per replica
};

template <int L, int LPR>
struct BlockSmem {
    GroupSmem<L, LPR> g[groups_of(L, LPR)];
    uint2 tt[256];  // first-look bounds
};

// Rows that fill their words (sides 8 and 16): the half-sites of word k are the site bits 64 k .. of the
// replica, whole rows whose even and odd sites are taken a dword at a time (one sweep, row by row and so: L = 16,
// 3 10^5 replicas 363 and 332 us; L = 8, 10^7 1605 and 1304).
template <int L>
constexpr bool whole_rows()
{
    return 8 * Geo<L>::WB == L;
}

// Sites 2 h (ev) and 2 h + 1 (od) of the 32 half-sites h of word k from the bit-packed rows of the
// group (base: the lane's word of row 0): half-sites 32 k ..
// lie in the rows 32 k / (L/2) ..
template <int L>
__device__ __forceinline__ void load_word_bits(const uint8_t* base, int k, uint32_t* ev, uint32_t* od)
{
    using Gm = Geo<L>;
    constexpr int H2 = Gm::H2, MAXR = whole_rows<L>() ? 64 / L : (31 + H2 - 1) / H2 + 1;
    const int r0 = 32 * k / H2;
    uint32_t v[MAXR];
#pragma unroll
    for (int i = 0; i < MAXR; ++i) {
        const int r = r0 + i < Gm::NR ? r0 + i : Gm::NR - 1;
        const uint8_t* a = base + (int64_t)r * 64 * Gm::WB;
        v[i] = Gm::WB == 1 ? (uint32_t)*a : (Gm::WB == 2 ? (uint32_t)*(const uint16_t*)a : *(const uint32_t*)a);
    }
    if constexpr (whole_rows<L>()) {
        uint32_t d[2] = {0, 0}, o_lo, o_hi;
#pragma unroll
        for (int i = 0; i < MAXR; ++i) d[L * i / 32] |= v[i] << (L * i % 32);
        const uint32_t e_lo = split_row(d[0], &o_lo), e_hi = split_row(d[1], &o_hi);
        *ev = e_lo | (e_hi << 16);
        *od = o_lo | (o_hi << 16);
        return;
    }
    uint32_t e = 0, o = 0;
#pragma unroll
    for (int i = 0; i < MAXR; ++i) {
        if (r0 + i >= Gm::NR) break;
        uint32_t od_r;
        const uint32_t ev_r = split_row(v[i], &od_r);
        const int sh = H2 * (r0 + i) - 32 * k;  // the row's first half-site in the word
        if (sh >= 32) break;
        if (sh >= 0) {
            e |= ev_r << sh;
            o |= od_r << sh;
        } else {
            e |= ev_r >> -sh;
            o |= od_r >> -sh;
        }
    }
    *ev = e;
    *od = o;
}

// bit-packed row r of the lane's replica from its strings (E0, E1 at word 0 of the string)
template <int L, int S>
__device__ __forceinline__ void store_row_bits(uint8_t* base, int r, const uint32_t* E0, const uint32_t* E1)
{
    using Gm = Geo<L>;
    const uint32_t v = string_row<L, S>(r % L, r / L, E0, E1);
    uint8_t* a = base + (int64_t)r * 64 * Gm::WB;
    if (Gm::WB == 1) *a = (uint8_t)v;
    else if (Gm::WB == 2) *(uint16_t*)a = (uint16_t)v;
    else *(uint32_t*)a = v;
}

// the rows of word k's sites 2 h (ev) and 2 h + 1 (od), where they are whole
template <int L>
__device__ __forceinline__ void store_word_bits(uint8_t* base, int k, uint32_t ev, uint32_t od)
{
    using Gm = Geo<L>;
    static_assert(whole_rows<L>() && Gm::WB <= 2, "sides 8 and 16");
    const uint32_t d[2] = {merge_row(ev & 0xFFFFu, od & 0xFFFFu), merge_row(ev >> 16, od >> 16)};
    uint8_t* a = base + (int64_t)k * (64 / L) * 64 * Gm::WB;
#pragma unroll
    for (int i = 0; i < 64 / L; ++i) {
        const uint32_t v = d[L * i / 32] >> (L * i % 32);
        if (Gm::WB == 1) a[64 * i] = (uint8_t)v;
        else reinterpret_cast<uint16_t*>(a)[64 * i] = (uint16_t)v;
    }
}

// The rows of a lane's replica between memory (base: its word of row 0) and its two strings, each row once and
// the strings in registers, for a wave that has the whole replica.  By words, the rows that lie in two of
// them are read twice and a word's loads wait for the last word's: 10^5 replicas of L = 6, one sweep 23.6 us,
// ten 90.4; so 18.2 and 85.0; 10^7 of L = 4, one 267, so 227.
template <int L>
__device__ __forceinline__ void load_replica_bits(const uint8_t* base, uint32_t (&s0)[Geo<L>::NW], uint32_t (&s1)[Geo<L>::NW])
{
    using Gm = Geo<L>;
    constexpr int H2 = Gm::H2;
    constexpr uint32_t HM = (1u << H2) - 1u;
    static_assert(Gm::WB == 1, "rows of a byte");
    uint32_t v[Gm::NR];
#pragma unroll
    for (int r = 0; r < Gm::NR; ++r) v[r] = base[64 * r];
#pragma unroll
    for (int k = 0; k < Gm::NW; ++k) s0[k] = s1[k] = 0;
#pragma unroll
    for (int r = 0; r < Gm::NR; ++r) {
        uint32_t odd;
        const uint32_t even = split_colours(v[r], &odd) & HM;
        const bool flip = (r % L + r / L) & 1;  // colour 0 takes x = 2 m + (y + z) mod 2
        const uint32_t c0 = flip ? odd & HM : even, c1 = flip ? even : odd & HM;
        const int k = H2 * r / 32, sh = H2 * r % 32;
        s0[k] |= c0 << sh;
        s1[k] |= c1 << sh;
        if (sh + H2 > 32) {
            s0[k + 1] |= c0 >> (32 - sh);
            s1[k + 1] |= c1 >> (32 - sh);
        }
    }
}

template <int L>
__device__ __forceinline__ void store_replica_bits(uint8_t* base, const uint32_t (&s0)[Geo<L>::NW], const uint32_t (&s1)[Geo<L>::NW])
{
    using Gm = Geo<L>;
    constexpr int H2 = Gm::H2;
    constexpr uint32_t HM = (1u << H2) - 1u;
#pragma unroll
    for (int r = 0; r < Gm::NR; ++r) {
        const int k = H2 * r / 32, sh = H2 * r % 32;
        uint32_t c0 = s0[k] >> sh, c1 = s1[k] >> sh;
        if (sh + H2 > 32) {
            c0 |= s0[k + 1] << (32 - sh);
            c1 |= s1[k + 1] << (32 - sh);
        }
        const bool flip = (r % L + r / L) & 1;
        base[64 * r] = (uint8_t)merge_colours((flip ? c1 : c0) & HM, (flip ? c0 : c1) & HM);
    }
}

// the initial spins of word k's sites 2 h (ev) and 2 h + 1 (od): 64 consecutive bits of the replica's
// stream, half of a call
__device__ __forceinline__ void init_word(int k, uint32_t r, bool valid, uint32_t k0, uint32_t k1, uint32_t* ev,
                                          uint32_t* od)
{
    const uint4v v = philox10((uint32_t)(k >> 1), r, 0u, kTagInit, k0, k1);
    const uint32_t lo = valid ? ((k & 1) ? v.z : v.x) : 0u, hi = valid ? ((k & 1) ? v.w : v.y) : 0u;
    uint32_t o_lo, o_hi;
    const uint32_t e_lo = split_row(lo, &o_lo), e_hi = split_row(hi, &o_hi);
    *ev = e_lo | (e_hi << 16);
    *od = o_lo | (o_hi << 16);
}

// N_S sweeps of the Q replicas from r0 on of one run by the group's waves.  INIT: no sweeps; the spins
// are the run's initial draws instead of loads (spin i of replica r is bit i mod 128 of Philox(ctr
// (i / 128, r, 0, 1), key seed); zero past R), and in the bit-packed layout the whole group is stored.
template <int L, int MODE, int LAYOUT, int LPR, bool INIT = false>
__device__ __forceinline__ void sweep_shared(const pa_state* st, int64_t r0, int wave, GroupSmem<L, LPR>& sm,
                                             const uint2* tt, const SweepParams& p, const Thr& th)
{
    using Gm = Geo<L>;
    constexpr int G = Gm::G, EW = Gm::EW, NW = Gm::NW, TW = Gm::TW, NWV = waves_of(L, LPR), Q = 64 / LPR;
    constexpr int UNITS = NWV * LPR;          // words taken at once
    constexpr bool WHOLE = Gm::NH % 32 == 0;  // the string is a whole number of words
    const int lane = threadIdx.x & 63, q = lane % Q;
    const int unit = wave * LPR + (LPR == 1 ? 0 : lane / Q);
    auto sync = [] {
        if constexpr (NWV == 1) wave_sync();
        else __syncthreads();
    };
    if constexpr (INIT && LAYOUT == PA_BITS64) {
        if (r0 >= st->R) {  // the same for the whole group
            uint8_t* a = (uint8_t*)st->spins[0] + ((r0 >> 6) * Gm::NR * 64 + (r0 & 63) + q) * Gm::WB;
            for (int i = unit; i < Gm::NR; i += UNITS) {
                uint8_t* w = a + (int64_t)i * 64 * Gm::WB;
                if (Gm::WB == 1) *w = 0;
                else if (Gm::WB == 2) *(uint16_t*)w = 0;
                else *(uint32_t*)w = 0;
            }
            return;
        }
    }
    if (wave == 0 && lane < Q) sm.neg[lane] = 0;
    build_tables<L>(st->J, sm.tab, lane, wave, NWV);
    uint32_t* E0 = sm.E + q;
    uint32_t* E1 = sm.E + EW * Q + q;
    const int64_t R = st->R, r = r0 + q;
    const bool valid = r < R;
    uint8_t* rows = (uint8_t*)st->spins[st->cur] +
                    (LAYOUT == PA_U8 ? r * Gm::STRIDE : ((r >> 6) * Gm::NR * 64 + (r & 63)) * Gm::WB);
    // a word and, where ghost words are copies of whole words, its ghost copies
    auto put = [&](uint32_t* S, int k, uint32_t v) {
        S[(G + k) * Q] = v;
        if constexpr (WHOLE) {
            if (k < G) S[(G + NW + k) * Q] = v;
            if (k >= NW - G) S[(k - (NW - G)) * Q] = v;
        }
    };
    // a wave with the whole bit-packed replica moves it at once
    constexpr bool AT_ONCE = LAYOUT == PA_BITS64 && UNITS == 1;
    sync();  // the tables
    if constexpr (AT_ONCE && !INIT) {
        uint32_t s0[NW], s1[NW];
        load_replica_bits<L>(rows, s0, s1);
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            put(E0, k, s0[k]);
            put(E1, k, s1[k]);
        }
    }
#pragma unroll 1
    for (int k = AT_ONCE && !INIT ? NW : unit; k < NW; k += UNITS) {
        uint32_t ev, od;
        if constexpr (INIT) init_word(k, (uint32_t)r, valid, (uint32_t)st->seed, (uint32_t)(st->seed >> 32), &ev, &od);
        else if constexpr (LAYOUT == PA_U8) load_word_u8(rows, Gm::STRIDE, k, &ev, &od);
        else load_word_bits<L>(rows, k, &ev, &od);
        const uint32_t sig0 = sm.tab[k * TW + 6], in = sm.tab[k * TW + 11];  // colour 0: x even, sites
        put(E0, k, select_bits(sig0, ev, od) & in);
        put(E1, k, select_bits(sig0, od, ev) & in);
    }
    sync();
    if constexpr (!WHOLE) {
        refresh_ghosts<L, Q>(E0, unit, UNITS);
        refresh_ghosts<L, Q>(E1, unit, UNITS);
        sync();
    }

    Lane c;
    c.rr = (uint32_t)r;
    c.k0 = (uint32_t)st->seed;
    c.k1 = (uint32_t)(st->seed >> 32);
    for (int s = 0; s < (INIT ? 0 : p.n_sweeps); ++s) {
        for (int col = 0; col < 2; ++col) {
            c.ctr2 = (uint32_t)(2 * (p.t0 + s) + col);
            uint32_t* W = col ? E1 : E0;
            const uint32_t* O = col ? E0 : E1;
            auto word = [&](int k, auto nbytes) {
                const uint32_t* T = sm.tab + (col * NW + k) * TW;
                const uint32_t w = W[(G + k) * Q];
                uint32_t nb[6];
                neighbours<L, Q>(O + (G + k) * Q, T, nb);
                uint32_t c0, c1, c2;
                bond_count(xor3(w, nb[0], T[0]), xor3(w, nb[1], T[1]), xor3(w, nb[2], T[2]), xor3(w, nb[3], T[3]),
                           xor3(w, nb[4], T[4]), xor3(w, nb[5], T[5]), c0, c1, c2);
                if constexpr (!WHOLE) c2 &= T[11];  // bits past the string are no candidates
                const uint32_t call0 = 4u * (uint32_t)k;
                const uint32_t nw = decide_word<MODE, LPR == 1, decltype(nbytes)::value>(w, c0, c1, c2, call0, 1u, tt, c,
                                                                                         th, [&]() {
                    // bit b is half-site 32 k + b: site 2 (32 k + b) + sigma
                    return WordSites{call0, 1u, 64u * (uint32_t)k, 16u, ~T[6] & T[11]};
                });
                put(W, k, nw);
            };
            // a partial last word draws only the calls of its bytes with sites (LPR = 1: the word is the
            // wave's alone)
            constexpr bool SHORT = !WHOLE && LPR == 1;
            constexpr int LASTB = (Gm::NH % 32 + 7) / 8;
            constexpr int FULL = SHORT ? NW - 1 : NW;
#pragma unroll 1
            for (int k = unit; k < FULL; k += UNITS) word(k, std::integral_constant<int, 4>{});
            if constexpr (SHORT) {
                if (wave == FULL % NWV) word(NW - 1, std::integral_constant<int, LASTB>{});
            }
            sync();
            if constexpr (!WHOLE) {
                refresh_ghosts<L, Q>(W, unit, UNITS);
                sync();
            }
        }
    }

    // energy: every bond joins a colour-0 and a colour-1 site, so the six bonds of the colour-0
    // sites count each bond once.  E = n_bonds - 2 (bonds whose word bit is set)
    int neg = 0;
#pragma unroll 1
    for (int k = unit; k < NW; k += UNITS) {
        const uint32_t* T = sm.tab + k * TW;
        const uint32_t w = E0[(G + k) * Q];
        uint32_t nb[6];
        neighbours<L, Q>(E1 + (G + k) * Q, T, nb);
#pragma unroll
        for (int d = 0; d < 6; ++d) neg += __popc(xor3(w, nb[d], T[d]) & T[11]);
    }
    atomicAdd(&sm.neg[q], (uint32_t)neg);
    constexpr bool WORDS = LAYOUT == PA_U8 || (whole_rows<L>() && !AT_ONCE);
    if constexpr (WORDS) {
#pragma unroll 1
        for (int k = unit; k < NW; k += UNITS) {
            const uint32_t sig0 = sm.tab[k * TW + 6], in = sm.tab[k * TW + 11];
            const uint32_t a = E0[(G + k) * Q], b = E1[(G + k) * Q];
            const uint32_t ev = select_bits(sig0, a, b) & in, od = select_bits(sig0, b, a) & in;
            if constexpr (LAYOUT == PA_U8) {
                if (valid) store_word_u8(rows, Gm::STRIDE, k, ev, od);
            } else {
                if (valid || INIT) store_word_bits<L>(rows, k, ev, od);
            }
        }
    } else if constexpr (AT_ONCE) {
        uint32_t s0[NW], s1[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            s0[k] = E0[(G + k) * Q];
            s1[k] = E1[(G + k) * Q];
        }
        if (valid || INIT) store_replica_bits<L>(rows, s0, s1);
    } else {
#pragma unroll 1
        for (int i = unit; i < Gm::NR; i += UNITS)
            if (valid || INIT) store_row_bits<L, Q>(rows, i, E0 + G * Q, E1 + G * Q);
    }
    sync();
    if (wave == 0 && lane < Q && valid) st->energy[st->cur][r] = st->n_bonds - 2 * (int)sm.neg[lane];
}

// the calling thread's group in its block and wave in the group, as scalars
template <int L, int LPR>
__device__ __forceinline__ void place(int* group, int* wave)
{
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    *group = w / waves_of(L, LPR);
    *wave = w % waves_of(L, LPR);
}

// one run: group i of the grid takes replicas 64 / LPR i ..; first: the first block of this part of the grid
template <int L, int MODE, int LAYOUT, int LPR>
__global__ void __launch_bounds__(threads_of(L, LPR)) k_sweep_group(const pa_state* __restrict__ st, uint32_t first, SweepParams p,
                                                                    Thr th)
{
    __shared__ BlockSmem<L, LPR> sm;
    constexpr int GPB = groups_of(L, LPR);
    if (st->status) return;  // sticky error: the population stays as it is
    int gi, wave;
    place<L, LPR>(&gi, &wave);
    const int64_t r0 = ((int64_t)(first + blockIdx.x) * GPB + gi) * (64 / LPR);
    if (GPB == 1 && r0 >= st->R) return;
    if (MODE != 2) build_bounds(sm.tt, th, threadIdx.x, threads_of(L, LPR));
    if constexpr (GPB > 1) {
        __syncthreads();
        if (r0 >= st->R) return;
    }
    sweep_shared<L, MODE, LAYOUT, LPR>(st, r0, wave, sm.g[gi], sm.tt, p, th);
}

// a group of equal-L runs of a batch: the LPR groups from LPR b on take item b of the work list
// (k_batch_tiles: 64 replicas each)
template <int L, int MODE, int LAYOUT, int LPR>
__global__ void __launch_bounds__(threads_of(L, LPR)) k_sweep_group_batch(pa_state* base, uint32_t first, int pos0,
                                                                          int pos1, BatchOrder order, SweepParams p,
                                                                          Thr th)
{
    __shared__ BlockSmem<L, LPR> sm;
    constexpr int GPB = groups_of(L, LPR);
    int gi, wave;
    place<L, LPR>(&gi, &wave);
    const int64_t* tb = work_ptr<int64_t>(base, work_layout(base->N, base->n_bins, base->capacity).batch);
    const int64_t sub = (int64_t)(first + blockIdx.x) * GPB + gi;
    const int64_t item = tb[pos0] + sub / LPR;
    if (GPB == 1 && item >= tb[pos1]) return;
    if (MODE != 2) build_bounds(sm.tt, th, threadIdx.x, threads_of(L, LPR));
    if constexpr (GPB > 1) {
        __syncthreads();
        if (item >= tb[pos1]) return;
    }
    const int lo = __builtin_amdgcn_readfirstlane(find_run(tb, pos0, pos1, item));
    const pa_state* st = base + order.run[lo];
    const int64_t r0 = (item - tb[lo]) * 64 + sub % LPR * (64 / LPR);
    if (r0 >= st->R) return;
    sweep_shared<L, MODE, LAYOUT, LPR>(st, r0, wave, sm.g[gi], sm.tt, p, th);
}

// Initial population and energies of runs of one side (grid.y: position in order), written once: drawing
// the rows and then reading them back per bond took 1.3 ms at L = 16, 10^6 replicas, this 0.37 ms.
template <int L, int LAYOUT>
__global__ void __launch_bounds__(threads_of(L, always_split(L) ? 4 : 1)) k_init_group(pa_state* base, uint32_t first,
                                                                                      BatchOrder order)
{
    constexpr int LPR = always_split(L) ? 4 : 1;
    __shared__ BlockSmem<L, LPR> sm;
    const pa_state* st = base + order.run[blockIdx.y];
    int gi, wave;
    place<L, LPR>(&gi, &wave);
    const int64_t r0 = ((int64_t)(first + blockIdx.x) * groups_of(L, LPR) + gi) * (64 / LPR);
    // (a wave that leaves alone is a whole group and meets no barrier)
    if (r0 >= (LAYOUT == PA_U8 ? st->R : st->capacity)) return;
    sweep_shared<L, 2, LAYOUT, LPR, true>(st, r0, wave, sm.g[gi], sm.tt, SweepParams{}, Thr{});
}

template <int L>
static void launch_init(pa_state* base, const BatchOrder& order, int n, int64_t cap, int layout, hipStream_t s)
{
    constexpr int LPR = always_split(L) ? 4 : 1;
    const int64_t per_block = 64 / LPR * groups_of(L, LPR);
    const dim3 b(threads_of(L, LPR));
    launch_parts((cap + per_block - 1) / per_block, (int)b.x, [&](uint32_t first, unsigned blocks) {
        const dim3 g(blocks, (unsigned)n);
        if (layout == PA_U8) hipLaunchKernelGGL((k_init_group<L, PA_U8>), g, b, 0, s, base, first, order);
        else hipLaunchKernelGGL((k_init_group<L, PA_BITS64>), g, b, 0, s, base, first, order);
    });
}

struct Launch {
    const pa_run* run;   // one run, or
    pa_state* base;      // the states of a batch with positions pos0 .. pos1 - 1 of order
    int pos0, pos1;
    const BatchOrder* order;
    int64_t items;       // 64-replica groups of the capacity (the grid)
    int64_t groups;      // and of the target population (the split)
};

template <int L, int LAYOUT, int LPR>
static void launch(const Launch& a, const SweepParams& p, const Thr& th, hipStream_t s)
{
    constexpr int GPB = groups_of(L, LPR);
    const dim3 b(threads_of(L, LPR));
    const bool z = all_tops_zero(th);
    launch_parts((a.items * LPR + GPB - 1) / GPB, (int)b.x, [&](uint32_t first, unsigned blocks) {
        const dim3 g(blocks);
        if (a.run) {
            if (z) hipLaunchKernelGGL((k_sweep_group<L, 2, LAYOUT, LPR>), g, b, 0, s, a.run->state, first, p, th);
            else hipLaunchKernelGGL((k_sweep_group<L, 0, LAYOUT, LPR>), g, b, 0, s, a.run->state, first, p, th);
        } else {
            if (z)
                hipLaunchKernelGGL((k_sweep_group_batch<L, 2, LAYOUT, LPR>), g, b, 0, s, a.base, first, a.pos0, a.pos1, *a.order,
                                   p, th);
            else
                hipLaunchKernelGGL((k_sweep_group_batch<L, 0, LAYOUT, LPR>), g, b, 0, s, a.base, first, a.pos0, a.pos1, *a.order,
                                   p, th);
        }
    });
}

template <int L, int LAYOUT>
static void launch(const Launch& a, const SweepParams& p, const Thr& th, hipStream_t s)
{
    // (L = 4: one word per colour, nothing to split)
    if constexpr (L > 4) {
        if (always_split(L) || a.groups < (L > 6 && p.n_sweeps <= kShortSweeps ? kShortGroups : kSplitGroups)) {
            launch<L, LAYOUT, 4>(a, p, th, s);
            return;
        }
    }
    if constexpr (!always_split(L)) launch<L, LAYOUT, 1>(a, p, th, s);
}

static int dispatch(int L, int layout, const Launch& a, const SweepParams& p, hipStream_t s)
{
    if (!fast_sweep_thresholds_ok(p)) return PA_ERR_ARG;
    const Thr th = make_thr(p);
#define PA_GROUP_L(LL) \
    case LL: \
        if (layout == PA_U8) launch<LL, PA_U8>(a, p, th, s); \
        else launch<LL, PA_BITS64>(a, p, th, s); \
        return PA_OK;
    switch (L) {
        PA_GROUP_L(4) PA_GROUP_L(6) PA_GROUP_L(8) PA_GROUP_L(10) PA_GROUP_L(12) PA_GROUP_L(14) PA_GROUP_L(16)
        PA_GROUP_L(18) PA_GROUP_L(20) PA_GROUP_L(24)
        default: return PA_ERR_ARG;
    }
#undef PA_GROUP_L
}

}  // namespace group

// initial spins and energies of the n runs order.run[0 ..] of side L (cap: their largest capacity)
int launch_init_group(int L, int layout, pa_state* base, const BatchOrder& order, int n, int64_t cap, hipStream_t s)
{
#define PA_INIT_L(LL) \
    case LL: group::launch_init<LL>(base, order, n, cap, layout, s); return PA_OK;
    switch (L) {
        PA_INIT_L(4) PA_INIT_L(6) PA_INIT_L(8) PA_INIT_L(10) PA_INIT_L(12) PA_INIT_L(14) PA_INIT_L(16) PA_INIT_L(18)
        PA_INIT_L(20) PA_INIT_L(24)
        default: return PA_ERR_ARG;
    }
#undef PA_INIT_L
}

int launch_sweep_group(const pa_run& run, const SweepParams& p, hipStream_t s)
{
    const group::Launch a = {&run, nullptr, 0, 0, nullptr, (run.capacity + 63) / 64, (run.R0 + 63) / 64};
    return group::dispatch(run.L, run.layout, a, p, s);
}

int launch_sweep_group_batch(int L, int layout, pa_state* base, int pos0, int pos1, const BatchOrder& order,
                             const SweepParams& p, int64_t items, int64_t groups, hipStream_t s)
{
    if (items <= 0) return PA_OK;
    const group::Launch a = {nullptr, base, pos0, pos1, &order, items, groups};
    return group::dispatch(L, layout, a, p, s);
}

// ------------------------------------------------------------------ a batch of runs
// The runs' states are contiguous (state r at base + r).  Work items are (run, 64-replica group);
// k_batch_tiles lays them out in the order given by the host (position p holds run order[p]).
__global__ void __launch_bounds__(256) k_batch_tiles(pa_state* base, int n_runs, BatchOrder order)
{
    int64_t* tb = work_ptr<int64_t>(base, work_layout(base->N, base->n_bins, base->capacity).batch);
    __shared__ int64_t cnt[kMaxBatch];
    for (int pos = threadIdx.x; pos < n_runs; pos += blockDim.x) {
        pa_state* st = base + order.run[pos];
        cnt[pos] = st->status ? 0 : (st->R + 63) / 64;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t acc = 0;
        for (int pos = 0; pos < n_runs; ++pos) {
            tb[pos] = acc;
            acc += cnt[pos];
        }
        tb[n_runs] = acc;
    }
}

static int g_batch_order = 1;  // 0: as given, 1: larger lattices first

bool group_sweep_supported(int dim, int L)
{
    return dim == 3 && L % 2 == 0 && ((L >= 4 && L <= 20) || L == 24);
}

// Sweep of n_runs contiguous runs (3D, sides of group_sweep_supported, one layout): the runs are
// grouped by lattice size (groups ordered by the cost of a tile, larger first, or by first
// appearance), one work list over all groups, one launch per group.
int launch_sweep_batch(const pa_run* runs, int n_runs, const SweepParams& p, hipStream_t s)
{
    if (n_runs > kMaxBatch || !fast_sweep_thresholds_ok(p)) return PA_ERR_ARG;
    // distinct sizes in order of first appearance, then (order 1) by tile cost, larger first
    int sizes[kMaxBatch], n_sizes = 0;
    for (int r = 0; r < n_runs; ++r) {
        bool seen = false;
        for (int g = 0; g < n_sizes; ++g) seen = seen || sizes[g] == runs[r].L;
        if (!seen) sizes[n_sizes++] = runs[r].L;
    }
    auto tile_cost = [](int L) { return (double)L * L * L * 64; };
    if (g_batch_order == 1)
        std::stable_sort(sizes, sizes + n_sizes, [&](int a, int b) { return tile_cost(a) > tile_cost(b); });
    BatchOrder order;
    int group_end[kMaxBatch];
    int64_t group_items[kMaxBatch], group_R0[kMaxBatch];  // 64-replica items of the capacities, of the targets
    int pos = 0;
    for (int g = 0; g < n_sizes; ++g) {
        group_items[g] = group_R0[g] = 0;
        for (int r = 0; r < n_runs; ++r) {
            if (runs[r].L != sizes[g]) continue;
            order.run[pos++] = (uint16_t)r;
            group_items[g] += (runs[r].capacity + 63) / 64;
            group_R0[g] += (runs[r].R0 + 63) / 64;
        }
        group_end[g] = pos;
    }
    pa_state* base = runs[0].state;
    hipLaunchKernelGGL(k_batch_tiles, dim3(1), dim3(256), 0, s, base, n_runs, order);
    for (int g = 0, pos0 = 0; g < n_sizes; pos0 = group_end[g], ++g) {
        const int L = sizes[g], pos1 = group_end[g];
        const int st = launch_sweep_group_batch(L, runs[0].layout, base, pos0, pos1, order, p, group_items[g], group_R0[g], s);
        if (st != PA_OK) return st;
    }
    return PA_OK;
}

}  // namespace pa

// batch schedule for the autotuner: order of the size groups (0: first appearance, 1: larger lattices
// first); the blocks per CU and the launch form of a persistent sweep are checked and have no effect,
// as every size takes one block per item; (0, 0, 0) restores the defaults
extern "C" int pa_set_batch_config(int blocks_per_cu, int order, int launch)
{
    if (blocks_per_cu == 0 && order == 0 && launch == 0) {
        pa::g_batch_order = 1;
        return PA_OK;
    }
    if (blocks_per_cu < 1 || blocks_per_cu > 32 || order < 0 || order > 1 || launch < 0 || launch > 2)
        return PA_ERR_ARG;
    pa::g_batch_order = order;
    return PA_OK;
}

// Colour strings of a cube: the sites of one colour of a replica as one bit string, and how the
// neighbours of its words are formed.  Shared by the sweep kernels that keep a replica this way.
//
// Colour string.  Half-site b = m + (L/2) (y + L z) (m = 0 .. L/2 - 1) holds the sites x = 2 m and
// 2 m + 1 of row (y, z); exactly one of them has colour c, x = 2 m + sigma with sigma = (c + y + z)
// mod 2.  Bit b of the colour-c string is that site, so the string has L^3 / 2 bits, its Metropolis
// field is field b mod 8 of Philox call b / 8, and a 32-bit word is four whole calls.  The
// neighbours of bit b are bits of the other colour's string:
//  - x: bit b itself on one side; bit b + 1 (x + 1, sigma = 1) or b - 1 (x - 1, sigma = 0) on the
//    other, wrapping within the row (b - (L/2 - 1) and b + (L/2 - 1));
//  - y: bits b + L/2 and b - L/2, wrapping within the plane (b -+ (L - 1) L / 2);
//  - z: bits b + L^2/2 and b - L^2/2, wrapping around the string.
// So every neighbour word is a funnel shift of two words of the other string by a constant, and
// the in-row and in-plane wraps are bit selects by per-word masks.  The strings are kept in LDS
// with a few ghost words on both sides holding the string's periodic continuation (refreshed after
// each colour phase), so the z wraps need no selects and no funnel leaves the buffer.
#pragma once

#include "pa_common.h"
#include "pa_sweep_words.h"

namespace pa {

namespace strings {

using namespace words;

template <int L>
struct Geo {
    static constexpr int H2 = L / 2;              // colour sites per row
    static constexpr int NP = L * L / 2;          // bits per plane
    static constexpr int NH = L * NP;             // bits per string
    static constexpr int NW = (NH + 31) / 32;     // words per string
    static constexpr int G = NP / 32 + 1;         // ghost words on each side: a funnel by up to
                                                  // NP bits reads words k - G .. k + G
    static constexpr int EW = NW + 2 * G;         // words of an extended string
    static constexpr int NR = L * L;              // lattice rows per replica
    static constexpr int WB = L <= 8 ? 1 : (L <= 16 ? 2 : 4);  // bytes of a bit-packed row
    static constexpr int STRIDE = (L * L * L + 15) / 16 * 16;  // bytes of a byte row
    static constexpr int TW = 12;                 // table dwords per (colour, word)
    static constexpr uint32_t LAST = NH % 32 ? (1u << (NH % 32)) - 1u : 0xFFFFFFFFu;  // valid bits of the last word
};

// offset of extended-string word e (0 .. EW - 1) inside the string: 32 (e - G) mod NH, taken
// non-negative; a ghost word holds the 32 string bits from there on
template <int L>
__host__ __device__ constexpr int ghost_origin(int e)
{
    using Gm = Geo<L>;
    return ((32 * (e - Gm::G)) % Gm::NH + Gm::NH) % Gm::NH;
}

// every ghost word is a funnel of string words that exist (so the refresh reads no ghost)
template <int L>
constexpr bool ghosts_in_string()
{
    using Gm = Geo<L>;
    for (int e = 0; e < Gm::EW; ++e) {
        if (e >= Gm::G && e < Gm::G + Gm::NW) continue;
        const int o = ghost_origin<L>(e);
        if (o % 32 == 0 ? o / 32 >= Gm::NW : o / 32 + 1 >= Gm::NW) return false;
    }
    return true;
}

// word q of the other string relative to word k, shifted by off bits (funnel of two words); S: dwords
// from a word to the next in LDS (the replicas side by side)
template <int OFF, int S>
__device__ __forceinline__ uint32_t funnel(const uint32_t* Ok)
{
    constexpr int q = OFF >= 0 ? OFF / 32 : -((-OFF + 31) / 32);  // floor(OFF / 32)
    constexpr int r = OFF - 32 * q;
    const uint32_t lo = Ok[q * S];
    if constexpr (r == 0) {
        return lo;
    } else {
        const uint32_t hi = Ok[(q + 1) * S];
        return __builtin_amdgcn_alignbit(hi, lo, r);
    }
}

// The geometry masks of a side's words, known when it is compiled: per (colour, word) 0 the sites with x even
// (sigma = 0), 1 and 2 the first and last site of a row (m = 0, m = L/2 - 1), 3 and 4 the first and last row of a
// plane (y = 0, y = L - 1), 5 the bits that are sites (b < L^3 / 2).
template <int L>
struct Masks {
    uint32_t w[2 * Geo<L>::NW][6];
};

template <int L>
constexpr Masks<L> make_masks()
{
    using Gm = Geo<L>;
    Masks<L> t = {};
    for (int b = 0; b < Gm::NH; ++b) {
        const int m = b % Gm::H2, r = b / Gm::H2, y = r % L, z = r / L;
        const uint32_t bit = 1u << (b & 31);
        for (int c = 0; c < 2; ++c) {
            uint32_t* w = t.w[c * Gm::NW + (b >> 5)];
            w[0] |= (c + y + z) & 1 ? 0u : bit;
            w[1] |= m == 0 ? bit : 0u;
            w[2] |= m == Gm::H2 - 1 ? bit : 0u;
            w[3] |= y == 0 ? bit : 0u;
            w[4] |= y == L - 1 ? bit : 0u;
            w[5] |= bit;
        }
    }
    return t;
}

template <int L>
__device__ constexpr Masks<L> g_masks = make_masks<L>();

// The per-word tables, by waves first, first + step, .. of step.  Entries: 0..5
// the coupling masks (bit set where J = -1) of the +x, -x, +y, -y, +z, -z bonds (without COUPLINGS, J unused,
// left as they are), 6..11 the geometry masks.  Lanes 0..31 take bit t of word k of colour 0, lanes 32..63 the
// same bit of colour 1, and a ballot of each bond's sign gives the two words at once.  (The geometry masks
// by ballots too: one sweep of L = 16, 3 10^5 replicas 332 us, so 325; 5 10^4, whose blocks have 16 replicas, 94 and 86.)
template <int L, bool COUPLINGS = true>
__device__ void build_tables(const int8_t* J, uint32_t* tab, int lane, int first = 0, int step = 1)
{
    using Gm = Geo<L>;
    for (int e = 64 * first + lane; e < 12 * Gm::NW; e += 64 * step) tab[e / 6 * Gm::TW + 6 + e % 6] = (&g_masks<L>.w[0][0])[e];
    if constexpr (!COUPLINGS) return;
    const int c = lane >> 5, t = lane & 31;
    for (int k = first; k < Gm::NW; k += step) {
        const int b = 32 * k + t;
        bool f[6] = {false, false, false, false, false, false};
        if (b < Gm::NH) {
            const int m = b % Gm::H2, r = b / Gm::H2, y = r % L, z = r / L;
            const int x = 2 * m + ((c + y + z) & 1);
            const int xm = (x + L - 1) % L, ym = (y + L - 1) % L, zm = (z + L - 1) % L;
            const int i = x + L * (y + L * z);
            f[0] = J[3 * i + 0] < 0;
            f[1] = J[3 * (xm + L * (y + L * z)) + 0] < 0;
            f[2] = J[3 * i + 1] < 0;
            f[3] = J[3 * (x + L * (ym + L * z)) + 1] < 0;
            f[4] = J[3 * i + 2] < 0;
            f[5] = J[3 * (x + L * (y + L * zm)) + 2] < 0;
        }
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            const uint64_t v = __ballot(f[e]);
            if (lane == 0) {
                tab[(0 * Gm::NW + k) * Gm::TW + e] = (uint32_t)v;
                tab[(1 * Gm::NW + k) * Gm::TW + e] = (uint32_t)(v >> 32);
            }
        }
    }
}

// the six neighbour words of word k of a colour (Ok: word k of the other string, T: the word's
// table entry)
template <int L, int S>
__device__ __forceinline__ void neighbours(const uint32_t* Ok, const uint32_t* T, uint32_t nb[6])
{
    using Gm = Geo<L>;
    constexpr int H2 = Gm::H2, NP = Gm::NP;
    const uint32_t a0 = Ok[0];
    const uint32_t sig0 = T[6], rf = T[7], rl = T[8], yf = T[9], yl = T[10];
    nb[0] = select_bits(sig0, a0, select_bits(rl, funnel<-(H2 - 1), S>(Ok), funnel<1, S>(Ok)));
    nb[1] = select_bits(sig0, select_bits(rf, funnel<H2 - 1, S>(Ok), funnel<-1, S>(Ok)), a0);
    nb[2] = select_bits(yl, funnel<H2 - NP, S>(Ok), funnel<H2, S>(Ok));
    nb[3] = select_bits(yf, funnel<NP - H2, S>(Ok), funnel<-H2, S>(Ok));
    nb[4] = funnel<NP, S>(Ok);
    nb[5] = funnel<-NP, S>(Ok);
}

// Sites 2 h (ev) and 2 h + 1 (od) of the 32 half-sites h of word k, from the byte rows: 64 bytes of
// the replica's row as 16-byte pieces (the row has stride bytes, a multiple of 16; pieces past it are
// zero)
__device__ __forceinline__ void load_word_u8(const uint8_t* row, int stride, int k, uint32_t* ev, uint32_t* od)
{
    uint32_t e = 0, o = 0;
    uint4 q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        q[i] = 64 * k + 16 * i < stride ? *reinterpret_cast<const uint4*>(row + 64 * k + 16 * i) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t d[4] = {q[i].x, q[i].y, q[i].z, q[i].w};
#pragma unroll
        for (int t = 0; t < 2; ++t) {  // eight sites: even ones in bytes 0, 2 of two dwords
            e |= pack4(__builtin_amdgcn_perm(d[2 * t + 1], d[2 * t], 0x06040200u)) << (8 * i + 4 * t);
            o |= pack4(__builtin_amdgcn_perm(d[2 * t + 1], d[2 * t], 0x07050301u)) << (8 * i + 4 * t);
        }
    }
    *ev = e;
    *od = o;
}

__device__ __forceinline__ void store_word_u8(uint8_t* row, int stride, int k, uint32_t ev, uint32_t od)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (64 * k + 16 * i >= stride) break;
        uint32_t d[4];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t e = unpack4(ev >> (8 * i + 4 * t)), o = unpack4(od >> (8 * i + 4 * t));
            d[2 * t] = __builtin_amdgcn_perm(o, e, 0x05010400u);
            d[2 * t + 1] = __builtin_amdgcn_perm(o, e, 0x07030602u);
        }
        *reinterpret_cast<uint4*>(row + 64 * k + 16 * i) = make_uint4(d[0], d[1], d[2], d[3]);
    }
}

// The ghost words (and the unused bits of a partial last word) of a string whose length is not a
// whole number of words (S at the replica's column, Q dwords from word to word), ghost i taken by unit
// i mod units.  Unit 0 fills the last word before it forms the one ghost word that reads it; no other
// ghost reads a word that another unit writes, as all come from words of the string.
template <int L, int Q>
__device__ __forceinline__ void refresh_ghosts(uint32_t* S, int unit, int units)
{
    using Gm = Geo<L>;
    static_assert(ghosts_in_string<L>(), "ghost words must come from string words");
    constexpr int G = Gm::G, NW = Gm::NW, last = G + NW - 1;
    if (unit == 0) {
        S[last * Q] = select_bits(Gm::LAST, S[last * Q], S[G * Q] << (Gm::NH % 32));
        constexpr int o = ghost_origin<L>(G - 1), q = G + o / 32;
        S[(G - 1) * Q] = __builtin_amdgcn_alignbit(S[(q + 1) * Q], S[q * Q], o % 32);
    }
    for (int i = unit; i < 2 * G - 1; i += units) {
        // ghosts 0 .. G - 2 before the string, then those after it
        const int e = i < G - 1 ? i : NW + i + 1;
        const int o = i < G - 1 ? Gm::NH - 32 * (G - e) : 32 * (e - G) - Gm::NH;
        const uint32_t* a = S + (G + (o >> 5)) * Q;
        S[e * Q] = __builtin_amdgcn_alignbit(a[Q], a[0], o & 31);
    }
}

// even and odd bits of a row word of up to 32 bits, as 16-bit numbers
__device__ __forceinline__ uint32_t split_row(uint32_t v, uint32_t* odd)
{
    uint32_t o;
    const uint32_t e = split_colours(v, &o);
    *odd = (o | (o >> 8)) & 0xFFFFu;
    return (e | (e >> 8)) & 0xFFFFu;
}

__device__ __forceinline__ uint32_t merge_row(uint32_t e, uint32_t o)
{
    return merge_colours((e | (e << 8)) & 0x00FF00FFu, (o | (o << 8)) & 0x00FF00FFu);
}

// lattice row (y, z) of a replica (bit x: the site) from its strings (E0, E1 at word 0 of the string; S
// dwords from word to word); the word after a string's last one is a ghost word, so it exists
template <int L, int S>
__device__ __forceinline__ uint32_t string_row(int y, int z, const uint32_t* E0, const uint32_t* E1)
{
    constexpr int H2 = Geo<L>::H2;
    constexpr uint32_t HM = (1u << H2) - 1u;
    const int b0 = H2 * (y + L * z), k = b0 >> 5, sh = b0 & 31;
    const uint32_t c0 = __builtin_amdgcn_alignbit(E0[(k + 1) * S], E0[k * S], sh) & HM;
    const uint32_t c1 = __builtin_amdgcn_alignbit(E1[(k + 1) * S], E1[k * S], sh) & HM;
    const bool odd = (y + z) & 1;  // colour 0 takes x = 2 m + (y + z) mod 2
    return merge_row(odd ? c1 : c0, odd ? c0 : c1);
}

// the position of a batch's work list that item belongs to
__device__ __forceinline__ int find_run(const int64_t* tb, int pos0, int pos1, int64_t item)
{
    int lo = pos0, hi = pos1;  // tb[lo] <= item < tb[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tb[mid] <= item) lo = mid;
        else hi = mid;
    }
    return lo;
}

}  // namespace strings
}  // namespace pa

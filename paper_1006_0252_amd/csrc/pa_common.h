// Internal header of libpa: device Philox, work-buffer layout, shared constants.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pa.h"

namespace pa {

// stream tags: fourth Philox counter word of each kind of draw
constexpr uint32_t kTagInit = 1;
constexpr uint32_t kTagMet = 2;
constexpr uint32_t kTagTie = 3;
constexpr uint32_t kTagPoisson = 4;
constexpr uint32_t kTagCoupling = 5;

// Poisson ladder: levels 2^m, m in [kLadderMin, kLadderMax]; Poisson(64) blocks above 64
constexpr int kLadderMin = -20;
constexpr int kLadderMax = 6;
constexpr int kLadderLevels = kLadderMax - kLadderMin + 1;
constexpr int kLadderCap = 256;  // entries per level (the largest level, 2^6, needs < 200)

// scan tile: replicas per block of the copy numbers and of their device-wide exclusive scan
constexpr int kScanTile = 256;

struct uint4v { uint32_t x, y, z, w; };

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each two 32x32->64
// products of counter words 0 and 2, Weyl key schedule between rounds.  The three-way xor
// of each round is one v_bitop3 (truth table 0x96 = a ^ b ^ c) on gfx950.
__device__ inline uint4v philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return {c0, c1, c2, c3};
}

__host__ __device__ inline uint32_t word_of(const uint4v& v, int w)
{
    return w == 0 ? v.x : (w == 1 ? v.y : (w == 2 ? v.z : v.w));
}

// byte offsets of the scratch arrays inside pa_run.work
struct WorkLayout {
    size_t hist;      // int64 [n_bins]   replicas per energy bin
    size_t bin_q;     // int64 [n_bins]   Poisson(64) blocks of the bin's mean copy number
    size_t bin_keep;  // uint64 [n_bins]  thinning threshold floor(rem 2^(32-m))
    size_t bin_m;     // int32 [n_bins]   ladder level m
    size_t scan;      // int64 [n_scan + 1] block sums of the copy-number scan
    size_t src;       // int32 [capacity] source replica of each new replica
    size_t qhist;     // int64 [N + 1]    overlap histogram (Hamming distance)
    size_t misc;      // int64 [64]       small reductions (E min/max, pending ln Q)
    size_t batch;     // int64 [1025]     work-list offsets of a batched sweep (first run of a batch)
    size_t total;
};

__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

__host__ __device__ inline WorkLayout work_layout(int64_t N, int64_t n_bins, int64_t capacity)
{
    WorkLayout w;
    size_t o = 0;
    w.hist = o;     o = align256(o + 8 * (size_t)n_bins);
    w.bin_q = o;    o = align256(o + 8 * (size_t)n_bins);
    w.bin_keep = o; o = align256(o + 8 * (size_t)n_bins);
    w.bin_m = o;    o = align256(o + 4 * (size_t)n_bins);
    const int64_t n_scan = (capacity + kScanTile - 1) / kScanTile;
    w.scan = o;     o = align256(o + 8 * (size_t)(n_scan + 1));
    w.src = o;      o = align256(o + 4 * (size_t)capacity);
    w.qhist = o;    o = align256(o + 8 * (size_t)(N + 1));
    w.misc = o;     o = align256(o + 8 * 64);
    w.batch = o;    o = align256(o + 8 * 1025);
    w.total = o;    // Gaussian couplings only: the sweep's threshold table starts here
    return w;
}

// bytes of the Gaussian sweep tables after WorkLayout::total: the sites of each colour (rounded up to
// whole calls of eight) times 64 neighbour patterns (cube; 4 for the chain, sized for the cube), a u16
// first-look table and then a u64 table of the full thresholds
__host__ __device__ inline size_t gauss_table_bytes(int64_t N) { return (2 + 8) * 64 * 16 * (size_t)((N / 2 + 7) / 8); }

template <typename T>
__device__ inline T* work_ptr(const pa_state* st, size_t off)
{
    return reinterpret_cast<T*>(st->work + off);
}

// sweep parameters passed by value
struct SweepParams {
    uint32_t thi[8];     // top 16 bits of T64 per class c (0x10000 = always accept)
    uint64_t T64[8];     // full thresholds per class c
    int64_t t0;          // first global sweep index
    int32_t n_sweeps;
    int32_t rpb;         // replicas (u8) or 64-replica groups (bits64) per block
};

// a batched sweep's run order: position p of the work list holds run order.run[p] (at most
// kMaxBatch runs)
constexpr int kMaxBatch = 1024;
struct BatchOrder {
    uint16_t run[kMaxBatch];
};

inline int hip_status(hipError_t e) { return e == hipSuccess ? PA_OK : PA_ERR_HIP; }

// exp written out for the Gaussian-coupling path, so that host and device reach the same bits:
// x = k ln 2 + r, k = floor(x / ln 2 + 1/2), r by a two-part ln 2 (the high part has 32
// significant bits, so k ln2_hi is exact), e^r by its Taylor series to r^13 in Horner form,
// scaled by 2^k; 0 below -745.  Products and sums are rounded one by one.
__device__ inline double expd(double x)
{
#pragma clang fp contract(off)
    if (x < -745.0) return 0.0;
    const double k = floor(x * 1.4426950408889634 + 0.5);
    const double r = (x - k * 0.6931471803691238) - k * 1.9082149292705877e-10;
    double p = 1.6059043836821613e-10;
    p = p * r + 2.08767569878681e-09;
    p = p * r + 2.505210838544172e-08;
    p = p * r + 2.755731922398589e-07;
    p = p * r + 2.7557319223985893e-06;
    p = p * r + 2.48015873015873e-05;
    p = p * r + 0.0001984126984126984;
    p = p * r + 0.001388888888888889;
    p = p * r + 0.008333333333333333;
    p = p * r + 0.041666666666666664;
    p = p * r + 0.16666666666666666;
    p = p * r + 0.5;
    p = p * r + 1.0;
    p = p * r + 1.0;
    return ldexp(p, (int)k);
}

}  // namespace pa

// Run initialisation (Sec. II: R0 replicas at beta = 0, each uniform over the 2^N
// microstates; couplings +-1 from the disorder seed; energies E = + sum J s s).
#include <math.h>
#include <stddef.h>
#include <string.h>

#include <algorithm>

#include "pa_common.h"
#include "pa_host.h"
#include "pa_lattice.h"

namespace pa {

// All kernels here take runs with consecutive states (grid.y = run), so a batch is initialised by a few
// launches: one per kernel and run took 5 to 10 us each, the runs one after the other (256 runs of the
// mixed batch: 26 ms of 128; 200 rings: 5 ms of a 10 ms pass).

// the host's states by value, as many as fit a kernel's arguments
constexpr int kStatesPerLaunch = 12;
struct StateChunk {
    pa_state s[kStatesPerLaunch];
};

__global__ void __launch_bounds__(64) k_write_states(pa_state* base, StateChunk c)
{
    const uint32_t* src = reinterpret_cast<const uint32_t*>(&c.s[blockIdx.x]);
    reinterpret_cast<uint32_t*>(base + blockIdx.x)[threadIdx.x] = src[threadIdx.x];
}

// J_b = -1 iff bit (b mod 128) of Philox(ctr (b/128, 0, 0, 5), key disorder seed) is set
__global__ void __launch_bounds__(256) k_couplings(const pa_state* __restrict__ base)
{
    const pa_state* st = base + blockIdx.y;
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= st->n_bonds) return;
    const uint4v v = philox10((uint32_t)(b >> 7), 0u, 0u, kTagCoupling, (uint32_t)st->disorder_seed,
                              (uint32_t)(st->disorder_seed >> 32));
    const uint32_t bit = (word_of(v, (b & 127) >> 5) >> (b & 31)) & 1u;
    st->J[b] = bit ? (int8_t)-1 : (int8_t)1;
}

// u8: thread per (replica, 16 consecutive sites); spin i of replica r is bit (i mod 128)
// of Philox(ctr (i/128, r, 0, 1), key seed); first: the first block of this part of the grid
__global__ void __launch_bounds__(256) k_init_u8(const pa_state* __restrict__ base, uint32_t first)
{
    const pa_state* st = base + blockIdx.y;
    const uint32_t k0 = (uint32_t)st->seed, k1 = (uint32_t)(st->seed >> 32);
    const int N = st->N, stride = st->row_stride;
    const int per_row = stride / 16;
    const int64_t t = (int64_t)(first + blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t r = t / per_row;
    const int q = (int)(t - r * per_row);
    if (r >= st->R0) return;
    const int i0 = q * 16;
    const uint4v v = philox10((uint32_t)(i0 >> 7), (uint32_t)r, 0u, kTagInit, k0, k1);
    const uint32_t word = word_of(v, (i0 & 127) >> 5) >> (i0 & 31);  // 16 spins in bits 0..15
    uint8_t b[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) b[j] = (i0 + j < N) ? (uint8_t)((word >> j) & 1u) : (uint8_t)0;
    uint8_t* dst = (uint8_t*)st->spins[0] + r * stride + i0;
    *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<uint4*>(b);
}

// bit-packed rows: thread per replica; row word (g, row, l) of replica 64 g + l at
// (g * n_rows + row) * 64 + l, bit x = site x + L row (cube) or 32 row + x (chain)
__device__ inline int row_len(const pa_state* st, int row) { return st->dim == 1 ? min(32, st->N - 32 * row) : st->L; }
__device__ inline int n_rows_of(const pa_state* st) { return st->dim == 1 ? (st->N + 31) / 32 : st->L * st->L; }
__device__ inline int row_bytes(const pa_state* st) { return st->dim == 1 ? 4 : (st->L <= 8 ? 1 : (st->L <= 16 ? 2 : 4)); }

__device__ inline uint32_t load_row(const pa_state* st, int buf, int64_t r, int row)
{
    const int WB = row_bytes(st);
    const int64_t idx = ((r >> 6) * n_rows_of(st) + row) * 64 + (r & 63);
    const uint8_t* base = (const uint8_t*)st->spins[buf];
    if (WB == 1) return base[idx];
    if (WB == 2) return ((const uint16_t*)base)[idx];
    return ((const uint32_t*)base)[idx];
}

__global__ void __launch_bounds__(256) k_init_bits64(const pa_state* __restrict__ states)
{
    const pa_state* st = states + blockIdx.y;
    const uint32_t k0 = (uint32_t)st->seed, k1 = (uint32_t)(st->seed >> 32);
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= st->capacity) return;
    const bool valid = r < st->R0;
    const int NR = n_rows_of(st), WB = row_bytes(st);
    const int rowsites = st->dim == 1 ? 32 : st->L;
    uint8_t* base = (uint8_t*)st->spins[0];
    int blk = -1;
    uint4v v = {0, 0, 0, 0};
    // word q of the replica's stream (spins 32 q .. 32 q + 31), the calls made in increasing order
    auto word_at = [&](int q) -> uint32_t {
        if ((q >> 2) != blk) {
            blk = q >> 2;
            v = philox10((uint32_t)blk, (uint32_t)r, 0u, kTagInit, k0, k1);
        }
        return word_of(v, q & 3);
    };
    for (int row = 0; row < NR; ++row) {
        // the row's spins are the len consecutive stream bits from i0: one word, or the top of one
        // and the bottom of the next
        const int len = row_len(st, row);
        const int i0 = rowsites * row;
        const int q0 = i0 >> 5, q1 = (i0 + len - 1) >> 5;
        const uint32_t lo = word_at(q0);
        const uint32_t hi = q1 != q0 ? word_at(q1) : 0u;
        const uint32_t lm = len == 32 ? 0xFFFFFFFFu : (1u << len) - 1u;
        uint32_t w = (uint32_t)(((((uint64_t)hi) << 32) | lo) >> (i0 & 31)) & lm;
        if (!valid) w = 0;
        const int64_t idx = ((r >> 6) * NR + row) * 64 + (r & 63);
        if (WB == 1) base[idx] = (uint8_t)w;
        else if (WB == 2) ((uint16_t*)base)[idx] = (uint16_t)w;
        else ((uint32_t*)base)[idx] = w;
    }
}

// u8 energies: one wave per replica, lanes over sites, each site owns its + bonds
__global__ void __launch_bounds__(256) k_energy_u8(const pa_state* __restrict__ base, uint32_t first, int buf)
{
    const pa_state* st = base + blockIdx.y;
    const int N = st->N, L = st->L, dim = st->dim, stride = st->row_stride;
    const int64_t r = (int64_t)(first + blockIdx.x) * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= st->R) return;
    const uint8_t* s = (const uint8_t*)st->spins[buf] + r * stride;
    const int8_t* J = st->J;
    int e = 0;
    for (int i = lane; i < N; i += 64) {
        const int si = s[i];
        if (dim == 1) {
            const int j = (i + 1 == N) ? 0 : i + 1;
            e += (int)J[i] * (1 - 2 * (si ^ s[j]));
        } else {
            int nb[3];
            plus_neighbours3(i, L, nb);
#pragma unroll
            for (int a = 0; a < 3; ++a) e += (int)J[3 * i + a] * (1 - 2 * (si ^ s[nb[a]]));
        }
    }
    for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
    if (lane == 0) st->energy[buf][r] = e;
}

// bit-packed energies: thread per replica, E = n_bonds - 2 * (bonds with J s s = -1)
__global__ void __launch_bounds__(256) k_energy_bits64(const pa_state* __restrict__ base, int buf)
{
    const pa_state* st = base + blockIdx.y;
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int L = st->L;
    const int NR = n_rows_of(st);
    const int8_t* J = st->J;
    int neg = 0;
    if (st->dim == 3) {
        // the block first turns the couplings into sign masks per row and axis (bit x: J < 0 on the
        // bond from site x + L row towards +axis), then each replica counts its unsatisfied bonds a
        // row word at a time
        __shared__ uint32_t jmask[3 * 32 * 32];
        for (int e = threadIdx.x; e < 3 * NR; e += blockDim.x) {
            const int row = e / 3, a = e - 3 * row;
            uint32_t m = 0;
            for (int x = 0; x < L; ++x) m |= (uint32_t)(J[3 * (x + L * row) + a] < 0) << x;
            jmask[e] = m;
        }
        __syncthreads();
        if (r >= st->R) return;
        const uint32_t lm = L == 32 ? 0xFFFFFFFFu : (1u << L) - 1u;
        for (int row = 0; row < NR; ++row) {
            const int y = row % L, z = row / L;
            const uint32_t own = load_row(st, buf, r, row) & lm;
            const uint32_t yp = load_row(st, buf, r, (y + 1) % L + L * z) & lm;
            const uint32_t zp = load_row(st, buf, r, y + L * ((z + 1) % L)) & lm;
            const uint32_t sx = ((own >> 1) | (own << (L - 1))) & lm;  // bit x: site x + 1 (periodic)
            neg += __popc(own ^ sx ^ jmask[3 * row]);
            neg += __popc((own ^ yp ^ jmask[3 * row + 1]) & lm);
            neg += __popc((own ^ zp ^ jmask[3 * row + 2]) & lm);
        }
    } else {
        if (r >= st->R) return;
        for (int row = 0; row < NR; ++row) {
            const int len = row_len(st, row);
            const uint32_t own = load_row(st, buf, r, row);
            const int nrow = row + 1 == NR ? 0 : row + 1;
            const uint32_t nxt = load_row(st, buf, r, nrow);
            for (int x = 0; x < len; ++x) {
                const uint32_t si = (own >> x) & 1u;
                const uint32_t sj = x + 1 < len ? (own >> (x + 1)) & 1u : nxt & 1u;
                neg += (int)(si ^ sj ^ (uint32_t)(J[32 * row + x] < 0));
            }
        }
    }
    st->energy[buf][r] = st->n_bonds - 2 * neg;
}

// record[0] and the energy base E_base = -n_bonds + ((E_0 + n_bonds) mod 4): every energy
// of a +-1 realisation has the residue of E_0 mod 4 (each flip changes E by 4c - 2z)
__global__ void __launch_bounds__(256) k_init_finish(pa_state* base)
{
    pa_state* st = base + blockIdx.y;
    // record[0] is the first 16 doubles
    const int64_t n = (int64_t)st->n_records * (int)(sizeof(pa_record) / sizeof(double));
    double* d = reinterpret_cast<double*>(st->record);
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
        double v = 0.0;
        if (i == offsetof(pa_record, minus_betaF) / sizeof(double)) v = st->ln_omega;
        if (i == offsetof(pa_record, R) / sizeof(double)) v = (double)st->R;
        d[i] = v;
    }
    if (threadIdx.x != 0) return;
    const int B = st->n_bonds;
    if (st->couplings != PA_GAUSS) {
        const int E0 = st->energy[0][0];
        st->E_base = -B + (((E0 + B) % 4) + 4) % 4;
    }
    st->initialised = 1;
}

static pa_state host_state(const pa_run& run, const pa_sizes& sz)
{
    pa_state h;
    memset(&h, 0, sizeof(h));
    h.dim = run.dim;
    h.L = run.L;
    h.N = (int32_t)sz.N;
    h.z = 2 * run.dim;
    h.n_bonds = (int32_t)sz.n_bonds;
    h.layout = run.layout;
    h.n_bins = (int32_t)sz.n_bins;
    h.row_stride = (int32_t)sz.row_stride;
    h.capacity = run.capacity;
    h.R0 = run.R0;
    h.seed = run.seed;
    h.disorder_seed = run.disorder_seed;
    h.J = run.J;
    h.spins[0] = run.spins[0];
    h.spins[1] = run.spins[1];
    h.energy[0] = run.energy[0];
    h.energy[1] = run.energy[1];
    h.counts = run.counts;
    h.offsets = run.offsets;
    h.work = (uint8_t*)run.work;
    h.record = run.record;
    h.n_records = run.n_records;
    h.R = run.R0;
    h.R_new = run.R0;
    h.ln_omega = (double)sz.N * log(2.0);
    h.couplings = run.couplings;
    return h;
}

int launch_init(const pa_run* runs, int n, const int8_t* const* J_host, hipStream_t s)
{
    pa_state* base = runs[0].state;
    const bool gauss = runs[0].couplings == PA_GAUSS;
    const int layout = runs[0].layout;
    // one launch covers the largest run of the call
    int64_t cap = 0, R0 = 0, bonds = 0, pieces = 0;  // pieces: 16 bytes of a run's byte rows
    bool all_given = J_host != nullptr;
    for (int r = 0; r < n; ++r) {
        pa_sizes sz;
        const int rc = pa_buffer_sizes(runs[r].dim, runs[r].L, layout, runs[r].couplings, runs[r].capacity, runs[r].n_records, &sz);
        if (rc != PA_OK) return rc;
        cap = std::max(cap, runs[r].capacity);
        R0 = std::max(R0, runs[r].R0);
        bonds = std::max(bonds, sz.n_bonds);
        pieces = std::max(pieces, runs[r].R0 * (sz.row_stride / 16));
        const int8_t* J = J_host ? J_host[r] : nullptr;
        all_given = all_given && J;
        if (J) {
            if (gauss) return PA_ERR_ARG;
            for (int64_t b = 0; b < sz.n_bonds; ++b)
                if (J[b] != 1 && J[b] != -1) return PA_ERR_ARG;
        }
    }
    for (int r0 = 0; r0 < n; r0 += kStatesPerLaunch) {
        StateChunk c;
        const int m = std::min(kStatesPerLaunch, n - r0);
        memset(&c, 0, sizeof(c));
        for (int i = 0; i < m; ++i) {
            pa_sizes sz;
            const pa_run& run = runs[r0 + i];
            pa_buffer_sizes(run.dim, run.L, layout, run.couplings, run.capacity, run.n_records, &sz);
            c.s[i] = host_state(run, sz);
        }
        hipLaunchKernelGGL(k_write_states, dim3((unsigned)m), dim3(64), 0, s, base + r0, c);
    }
    const unsigned ny = (unsigned)n;
    auto init_u8 = [&] {
        launch_parts((pieces + 255) / 256, 256, [&](uint32_t first, unsigned blocks) {
            hipLaunchKernelGGL(k_init_u8, dim3(blocks, ny), dim3(256), 0, s, base, first);
        });
    };
    if (gauss) {
        // couplings from the host (libm), then spins as for +-1 couplings and FP64 energies
        int rc = gauss_couplings_upload(runs, n, s);
        if (rc != PA_OK) return rc;
        init_u8();
        rc = launch_energy_gauss(runs, n, s);
        if (rc != PA_OK) return rc;
        hipLaunchKernelGGL(k_init_finish, dim3(1, ny), dim3(256), 0, s, base);
        return hip_status(hipGetLastError());
    }
    if (!all_given) hipLaunchKernelGGL(k_couplings, dim3((unsigned)((bonds + 255) / 256), ny), dim3(256), 0, s, base);
    for (int r = 0; J_host && r < n; ++r) {
        if (!J_host[r]) continue;
        const int64_t B = runs[r].dim == 1 ? runs[r].L : 3 * (int64_t)runs[r].L * runs[r].L * runs[r].L;
        if (hipMemcpyAsync(runs[r].J, J_host[r], (size_t)B, hipMemcpyHostToDevice, s) != hipSuccess) return PA_ERR_HIP;
    }
    // cubes the group kernel takes: spins and energies in one pass, one launch per side; when the call
    // holds any other run, every run draws its spins and then sums its energies from them
    bool group = n <= kMaxBatch;
    for (int r = 0; r < n; ++r) group = group && group_sweep_supported(runs[r].dim, runs[r].L);
    if (group) {
        bool done[33] = {};
        for (int r = 0; r < n; ++r) {
            const int L = runs[r].L;
            if (done[L]) continue;
            done[L] = true;
            BatchOrder order;
            int m = 0;
            int64_t capL = 0;
            for (int q = r; q < n; ++q) {
                if (runs[q].L != L) continue;
                order.run[m++] = (uint16_t)q;
                capL = std::max(capL, runs[q].capacity);
            }
            const int rc = launch_init_group(L, layout, base, order, m, capL, s);
            if (rc != PA_OK) return rc;
        }
    } else if (layout == PA_U8) {
        init_u8();
        launch_parts((R0 + 3) / 4, 256, [&](uint32_t first, unsigned blocks) {
            hipLaunchKernelGGL(k_energy_u8, dim3(blocks, ny), dim3(256), 0, s, base, first, 0);
        });
    } else {
        const dim3 g((unsigned)((cap + 255) / 256), ny);
        hipLaunchKernelGGL(k_init_bits64, g, dim3(256), 0, s, base);
        hipLaunchKernelGGL(k_energy_bits64, g, dim3(256), 0, s, base, 0);
    }
    hipLaunchKernelGGL(k_init_finish, dim3(1, ny), dim3(256), 0, s, base);
    return hip_status(hipGetLastError());
}

}  // namespace pa

"""Runs and batches whose launches hold 2^32 threads or a few more: a launch cut short to the few is seen in
the first thousand replicas, so the capacities are far above the populations."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


def room(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip(f"needs {gib} GiB of device memory")


# threads per replica of capacity: side 8 four (initialisation) and eight (few replicas), chains four
@pytest.mark.parametrize("dim,L,cap,gib,n", [(3, 8, (1 << 30) + 64, 190, 1), (3, 8, (1 << 28) + 64, 120, 2),
                                             (1, 130, (1 << 30) + 64, 90, 1)])
def test_large_capacity(dim, L, cap, gib, n):
    print(f"[case] large capacity dim={dim} L={L} cap={cap} n={n}", flush=True)
    room(gib)
    R = 1000
    J = o.couplings(dim, L, 3)
    if n == 1:
        obj = pa.Run(dim, L, R, 5, 3, 2, capacity=cap, layout="bits64", device=DEV).init()
        runs = [obj]
    else:
        specs = [dict(dim=dim, L=L, R0=R, seed=5 + i, disorder_seed=3) for i in range(n)]
        obj = pa.Batch(specs, 2, layout="bits64", device=DEV, capacity_factor=cap / R).init()
        runs = obj.runs
    st = pa.Schedule([0.0, 0.5], 2, runs[0].n_bins, device=DEV).step(1)
    want = []
    for i, run in enumerate(runs):
        s, E = o.init_population(dim, L, J, 5 + i, R)
        got = first_replicas(run, R)
        assert np.array_equal(got[0], s) and np.array_equal(got[1], E)
        o.sweep(dim, L, J, 5 + i, 0.5, R, s, E, st.t0, st.n_sweeps)
        want.append((s, E))
    obj.sweep(st)
    for run, (s, E) in zip(runs, want):
        got = first_replicas(run, R)
        assert np.array_equal(got[0], s) and np.array_equal(got[1], E)


def first_replicas(run, R):
    """spins and energies of the population of R replicas (its buffers are too long to copy whole)"""
    info = run.query()
    assert info.R == R
    row = int(run.sizes.spins_bytes) // run.capacity
    raw = run.spins[info.cur][: (R + 63) // 64 * 64 * row].cpu().numpy()
    return (pa.unpack_spins(raw, run.dim, run.L, run.layout, R, int(run.sizes.row_stride)),
            run.energy[info.cur][: 4 * R].cpu().numpy().view(np.int32))


def test_uneven_gaussian_batch():
    """1100 runs take the blocks of the largest one each"""
    print("[case] uneven Gaussian batch", flush=True)
    specs = [dict(dim=3, L=6, R0=1_000_000 if r == 700 else 40, seed=r + 1, disorder_seed=3, couplings="gauss")
             for r in range(1100)]
    batch = pa.Batch(specs, 2, layout="u8", device=DEV).init()
    st = pa.Schedule([0.4, 0.5], 1, batch.runs[0].n_bins, device=DEV).step(1)
    J = o.couplings_gauss(3, 6, 3)
    batch.sweep(st)
    for r in (0, 1, 699, 700, 701, 1099):
        s, E = o.init_replicas_gauss(3, 6, J, r + 1, 0, 40)
        o.sweep_replicas_gauss(3, 6, J, r + 1, 0.5, 0, s, E, st.t0, st.n_sweeps)
        got = batch.runs[r].population()
        assert np.array_equal(got[0][:40], s) and np.array_equal(got[1][:40], E)


def test_mixed_chains_initialised():
    """a run of many short chains beside one of few long ones: the most replicas times the longest rows are 2^32
    pieces of 16 bytes and 1.6 10^6 more"""
    print("[case] mixed chains", flush=True)
    sizes = [(16, (1 << 24) + 6400), (4096, 70)]
    specs = [dict(dim=1, L=N, R0=R, seed=i + 1, disorder_seed=3) for i, (N, R) in enumerate(sizes)]
    batch = pa.Batch(specs, 2, layout="u8", device=DEV).init()
    for i, (N, R) in enumerate(sizes):
        J = o.couplings(1, N, 3)
        run = batch.runs[i]
        E = run.energies()
        for first in (0, R // 2 // 64 * 64, R - 64):
            n = min(64, R - first)
            s_o, E_o = o.init_replicas(1, N, J, i + 1, first, n)
            raw = run.spins[0][first * N: (first + n) * N].cpu().numpy().reshape(n, N)
            assert np.array_equal(raw, s_o) and np.array_equal(E[first: first + n], E_o)

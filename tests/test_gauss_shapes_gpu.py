"""The tabled Gaussian sweep against the oracle, bit for bit, over the shapes its kernels split
differently: chains whose strings fill one register, two, or LDS words with and without a remainder,
cubes of every tabled side, shapes past the tables, and a step whose thresholds sit at the top of the
16-bit bound (where first looks of 0xFFFE and 0xFFFF are decided from the 64-bit threshold)."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


def check(dim, L, R, beta, ns=2, seed=6, ds=8):
    print(f"[case] gauss shape dim={dim} L={L} R={R} beta={beta}", flush=True)
    run = pa.Run(dim, L, R, seed, ds, 2, capacity=(R + 63) // 64 * 64, layout="u8", device=DEV, couplings="gauss").init()
    run.sweep(pa.Schedule([0.0, beta], ns, run.n_bins, device=DEV).step(1))
    assert run.status()[0] == pa.PA_OK
    s, E = run.population()
    J = o.couplings_gauss(dim, L, ds)
    s_o, E_o = o.init_replicas_gauss(dim, L, J, seed, 0, R)
    o.sweep_replicas_gauss(dim, L, J, seed, beta, 0, s_o, E_o, 0, ns)
    assert np.array_equal(s, s_o), np.nonzero((s != s_o).any(axis=1))[0][:10]
    assert np.array_equal(E, E_o)
    return run


# calls per colour 1 .. 8 (registers), then words: whole, with a remainder, and past the tables (4096)
@pytest.mark.parametrize("N", [4, 6, 14, 16, 18, 32, 34, 62, 64, 66, 80, 98, 114, 126, 128, 130, 192, 250, 256, 258,
                               1026, 4096, 4098])
def test_chains(N):
    check(1, N, 65 if N > 1000 else 130, 0.9)
    check(1, N, 1, 2.0)


@pytest.mark.parametrize("L", [2, 4, 6, 8, 10, 12, 14, 16, 18])
def test_cubes(L):
    check(3, L, 65, 0.6)
    check(3, L, 1, 3.0)


@pytest.mark.parametrize("dim,L,R", [(3, 8, 1500), (3, 6, 1500), (1, 64, 6000), (1, 256, 2000)])
def test_thresholds_at_the_top_of_the_bound(dim, L, R):
    # dE of a few units at this beta: T16 from 0xFFFA to 0xFFFF; 10^7 attempts, so some 300 first looks
    # of 0xFFFE and 0xFFFF
    check(dim, L, R, 6e-6, ns=12)


def test_many_runs_and_mixed_sides():
    """ten runs (an XCD range each holds parts of runs) and a batch of different sides"""
    specs = [dict(dim=3, L=6, R0=100 + 7 * i, seed=i + 1, disorder_seed=2, couplings="gauss") for i in range(10)]
    mixed = [dict(dim=3, L=L, R0=90, seed=L, disorder_seed=L, couplings="gauss") for L in (4, 6, 10)]
    for sp in (specs, mixed):
        batch = pa.Batch(sp, 2, layout="u8", device=DEV).init()
        step = pa.Schedule([0.0, 1.1], 3, max(r.n_bins for r in batch.runs), device=DEV).step(1)
        batch.sweep(step)
        assert batch.status()[0] == pa.PA_OK
        for q, run in zip(sp, batch.runs):
            J = o.couplings_gauss(3, q["L"], q["disorder_seed"])
            s_o, E_o = o.init_replicas_gauss(3, q["L"], J, q["seed"], 0, q["R0"])
            o.sweep_replicas_gauss(3, q["L"], J, q["seed"], 1.1, 0, s_o, E_o, 0, 3)
            s, E = run.population()
            assert np.array_equal(s, s_o) and np.array_equal(E, E_o)

"""The group sweep kernel (cubes, the waves of a block sharing its replicas) against the oracle, bit for
bit: both forms (64 replicas per block; 16 with four lanes each, for fewer than 1024 64-replica
groups and from L = 20 on), every side, both layouts, the edges of the blocks, and batches that mix
sides the forms treat differently."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"
SIDES = [4, 6, 8, 10, 12, 14, 16, 18, 20, 24]


def sampled_sweep(L, layout, R, beta, groups, ns=2):
    """ns sweeps of a fresh population; the replicas [a, b) of every group against the oracle's."""
    run = pa.Run(3, L, R, 13, 4, 2, capacity=(R + 63) // 64 * 64, layout=layout, device=DEV).init()
    run.sweep(pa.Schedule([0.0, beta], ns, run.n_bins, device=DEV).step(1))
    assert run.status()[0] == pa.PA_OK
    J = o.couplings(3, L, 4)
    E = run.energies()
    for a, b in groups:
        s_o, E_o = o.init_replicas(3, L, J, 13, a, b - a)
        o.sweep_replicas(3, L, J, 13, beta, a, s_o, E_o, 0, ns)
        assert np.array_equal(run.replica_spins(np.arange(a, b)), s_o), (L, layout, R, beta, a)
        assert np.array_equal(E[a:b], E_o), (L, layout, R, beta, a)


@pytest.mark.parametrize("layout", ["u8", "bits64"])
@pytest.mark.parametrize("L", SIDES)
def test_small_populations(L, layout):
    print(f"[case] group sweep L={L} {layout}", flush=True)
    for R, beta in ((1, 0.5), (17, 1.4), (64, 3.5), (81, 0.8)):
        sampled_sweep(L, layout, R, beta, [(0, R)])


@pytest.mark.parametrize("layout", ["u8", "bits64"])
@pytest.mark.parametrize("L", [s for s in SIDES if s < 20])
def test_large_populations(L, layout):
    """64 replicas per block: 1024 groups and a ragged one; the first, a middle and the last replicas"""
    print(f"[case] group sweep, many groups, L={L} {layout}", flush=True)
    R = 65536 + 37
    for beta in (0.6, 3.2):
        sampled_sweep(L, layout, R, beta, [(0, 3), (32767, 32770), (R - 3, R)])


@pytest.mark.parametrize("layout", ["u8", "bits64"])
def test_batch_of_every_form(layout):
    """runs of sides 4, 14, 18 and 20 in one batch equal the same runs alone"""
    print(f"[case] group sweep batch {layout}", flush=True)
    specs = [dict(dim=3, L=L, R0=R0, seed=i + 1, disorder_seed=i // 2 + 1)
             for i, (L, R0) in enumerate([(4, 100), (14, 65), (18, 33), (14, 200), (20, 16), (4, 1)])]
    batch = pa.Batch(specs, 2, layout=layout, device=DEV).init()
    step = pa.Schedule([0.0, 0.9], 3, max(r.n_bins for r in batch.runs), device=DEV).step(1)
    batch.sweep(step)
    assert batch.status()[0] == pa.PA_OK
    for sp, b in zip(specs, batch.runs):
        solo = pa.Run(3, sp["L"], sp["R0"], sp["seed"], sp["disorder_seed"], 2, layout=layout, device=DEV).init()
        solo.sweep(step)
        assert np.array_equal(b.energies(), solo.energies())
        assert np.array_equal(b.population()[0], solo.population()[0])


@pytest.mark.parametrize("layout", ["u8", "bits64"])
@pytest.mark.parametrize("shapes", [[(3, 4, 70), (3, 18, 20), (3, 4, 1), (3, 20, 17)], [(3, 2, 70), (3, 6, 65)],
                                    [(1, 40, 70), (1, 64, 3)]])
def test_batch_initial_populations(shapes, layout):
    """couplings, spins, energies and records of a batch initialised at once: sides of the group kernel,
    a call that holds another side, and chains; one run's couplings given"""
    print(f"[case] batch init {shapes} {layout}", flush=True)
    specs = [dict(dim=d, L=L, R0=R0, seed=50 + i, disorder_seed=i) for i, (d, L, R0) in enumerate(shapes)]
    batch = pa.Batch(specs, 3, layout=layout, device=DEV)
    J_given = 1 - 2 * (np.arange(batch.runs[1].n_bonds) % 3 == 0).astype(np.int8)
    for given in (False, True):
        J_list = [np.ascontiguousarray(o.couplings(sp["dim"], sp["L"], sp["disorder_seed"]), np.int8) for sp in specs]
        J_list[1] = J_given if given else J_list[1]
        batch.init(J_list if given else None)
        for sp, J, run in zip(specs, J_list, batch.runs):
            assert np.array_equal(run.couplings(), J)
            s, E = run.population()
            s_o, E_o = o.init_replicas(sp["dim"], sp["L"], J, sp["seed"], 0, sp["R0"])
            assert np.array_equal(s, s_o) and np.array_equal(E, E_o)
            rec = run.records()
            assert rec[0, 4] == sp["R0"] and rec[0, 2] == run.N * np.log(2.0) and not rec[1:].any()

"""One to four sweeps around 384 groups of 64 replicas, where a call's lanes per replica change with its number
of sweeps, against the oracle on the first, the last and some replicas between: rows moved whole (sides 4, 6),
word by word (8, 16) and row by row."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("ns", [1, 3, 4])
@pytest.mark.parametrize("groups", [383, 384])
@pytest.mark.parametrize("layout", ["bits64", "u8"])
@pytest.mark.parametrize("L", [4, 6, 8, 10, 16, 18])
def test_few_sweeps(L, layout, groups, ns):
    print(f"[case] short sweeps L={L} {layout} groups={groups} ns={ns}", flush=True)
    R = 64 * groups - 11
    run = pa.Run(3, L, R, 6, 3, 2, capacity=64 * groups, layout=layout, device=DEV).init()
    J = o.couplings(3, L, 3)
    st = pa.Schedule([0.0, 0.6], ns, run.n_bins, device=DEV).step(1)
    ranges = [(0, 70), (64 * 200 + 30, 40), (R - 60, 60)]
    want = [o.init_replicas(3, L, J, 6, first, n) for first, n in ranges]

    def check():
        E = run.energies()
        for (first, n), (s_o, E_o) in zip(ranges, want):
            assert np.array_equal(run.replica_spins(np.arange(first, first + n)), s_o)
            assert np.array_equal(E[first: first + n], E_o)

    check()
    run.sweep(st)
    for (first, _), (s_o, E_o) in zip(ranges, want):
        o.sweep_replicas(3, L, J, 6, 0.6, first, s_o, E_o, st.t0, ns)
    check()
    if layout == "bits64":  # the words of the replicas past R stay zero
        row = int(run.sizes.spins_bytes) // run.capacity
        last = run.spins[0][: 64 * groups * row].cpu().numpy()[-64 * row:]
        W = 1 if L <= 8 else (2 if L <= 16 else 4)
        assert not last.reshape(-1, 64, W)[:, -11:].any()

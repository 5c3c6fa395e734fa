"""Gaussian cubes of sides 8 and 10 in batches small enough for a thread per call, with as many runs as take the
blocks' interleaved order (eight) and more, against the oracle."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("L,n,R", [(8, 8, 300), (8, 9, 70), (8, 20, 129), (10, 8, 200), (10, 11, 65)])
def test_runs_of_a_batch(L, n, R):
    print(f"[case] gauss split batch L={L} n={n} R={R}", flush=True)
    specs = [dict(dim=3, L=L, R0=R, seed=i + 1, disorder_seed=3 + i % 3, couplings="gauss") for i in range(n)]
    batch = pa.Batch(specs, 2, layout="u8", device=DEV).init()
    st = pa.Schedule([0.5, 0.6], 2, batch.runs[0].n_bins, device=DEV).step(1)
    batch.sweep(st)
    for sp, run in zip(specs, batch.runs):
        J = o.couplings_gauss(3, L, sp["disorder_seed"])
        s, E = o.init_replicas_gauss(3, L, J, sp["seed"], 0, R)
        o.sweep_replicas_gauss(3, L, J, sp["seed"], 0.6, 0, s, E, st.t0, st.n_sweeps)
        got = run.population()
        assert np.array_equal(got[0], s) and np.array_equal(got[1], E)

"""The +-1 chain sweep against the oracle, bit for bit: every number of calls held in registers, words in
LDS with and without a remainder, past the kernels' length, both layouts, both first-look regimes, a
step below the bounds' range, ragged groups, and a batch."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


def check(run, N, seed, ds, R, beta, ns, t0=0):
    J = o.couplings(1, N, ds)
    s_o, E_o = o.init_replicas(1, N, J, seed, 0, R)
    o.sweep_replicas(1, N, J, seed, beta, 0, s_o, E_o, t0, ns)
    s, E = run.population()
    assert np.array_equal(s, s_o), (N, R, beta)
    assert np.array_equal(E, E_o), (N, R, beta)


@pytest.mark.parametrize("layout", ["u8", "bits64"])
@pytest.mark.parametrize("N", [4, 6, 14, 16, 18, 30, 32, 34, 48, 62, 64, 66, 80, 98, 126, 128, 130, 160, 192, 250, 256,
                               514, 4096, 4098])
def test_lengths(N, layout):
    print(f"[case] chain sweep N={N} {layout}", flush=True)
    for R, beta, ns in ((1, 0.7, 2), (130, 0.3, 3), (300, 3.5, 3), (65, 2e-6, 1)):
        run = pa.Run(1, N, R, 3, 5, 2, layout=layout, device=DEV).init()
        run.sweep(pa.Schedule([0.0, beta], ns, run.n_bins, device=DEV).step(1))
        assert run.status()[0] == pa.PA_OK
        check(run, N, 3, 5, R, beta, ns)


@pytest.mark.parametrize("N", [64, 200])
def test_ties_and_batch(N):
    """enough attempts for hundreds of first-look ties, over the runs of a batch of uneven populations"""
    print(f"[case] chain batch N={N}", flush=True)
    specs = [dict(dim=1, L=N, R0=R0, seed=i + 1, disorder_seed=i // 2) for i, R0 in enumerate((2000, 1, 64, 1500))]
    batch = pa.Batch(specs, 2, layout="u8", device=DEV).init()
    batch.sweep(pa.Schedule([0.0, 1.3], 60, batch.runs[0].n_bins, device=DEV).step(1))
    assert batch.status()[0] == pa.PA_OK
    for sp, run in zip(specs, batch.runs):
        check(run, N, sp["seed"], sp["disorder_seed"], sp["R0"], 1.3, 60)

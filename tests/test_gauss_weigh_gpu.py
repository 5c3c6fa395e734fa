"""Gaussian weights and their sum in one block per run (capacity up to 8192) and by separate kernels (above),
against the oracle: the same populations under both capacities, at the edges of the block's loads and
chunks, with copy numbers in the hundreds, and moments and overlaps measured twice."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("R", [1, 256, 257, 2048, 2049, 5000])
def test_copy_numbers(R):
    print(f"[case] gauss weights R={R}", flush=True)
    J = o.couplings_gauss(1, 32, 4)
    s_o, E_o = o.init_replicas_gauss(1, 32, J, 3, 0, R)
    for b1 in (0.1, 0.9):
        st, c_o, S_o, lnQ_o, E_lo_o = o.copy_numbers_gauss(3, 1, 0.0, b1, float(R), E_o)
        for cap in (8192, 8256):
            run = pa.Run(1, 32, R, 3, 4, 2, capacity=cap, layout="u8", device=DEV, couplings="gauss").init()
            run.resample(pa.Schedule([0.0, b1], 1, run.n_bins, device=DEV).step(1))
            if c_o.sum() == 0:
                assert run.status()[1] == pa.PA_FLAG_EXTINCT
                continue
            assert st == 0 and run.status()[0] == pa.PA_OK
            assert np.array_equal(run.counts_offsets(R)[0], c_o)
            rec = run.records()[1]
            assert rec[3] == S_o and rec[5] == E_lo_o and rec[4] == c_o.sum()
            assert abs(rec[1] - lnQ_o) <= 1e-12 * max(1.0, abs(lnQ_o))
            assert np.array_equal(run.population()[1], np.repeat(E_o, c_o))


@pytest.mark.parametrize("couplings,R", [("gauss", 300), ("pm1", 300), ("pm1", 9000)])
def test_overlaps_measured_twice(couplings, R):
    """the overlap histogram starts from zero at every measurement"""
    print(f"[case] overlaps twice {couplings} R={R}", flush=True)
    specs = [dict(dim=3, L=4, R0=R, seed=i + 1, disorder_seed=2, couplings=couplings) for i in range(2)]
    batch = pa.Batch(specs, 2, layout="u8", device=DEV).init()
    batch.measure(True)
    first = [run.records()[0].copy() for run in batch.runs]
    batch.measure(True)
    for a, run in zip(first, batch.runs):
        assert np.array_equal(a, run.records()[0]) and a[12] == R
    pops = [run.population()[0] for run in batch.runs]
    h, P = o.overlap_hist(64, pops[0], pops[1])
    q = 1.0 - 2.0 * np.arange(65) / 64.0
    assert P == R and abs(first[0][9] - (h * q**2).sum() / P) < 1e-12

"""The energy histogram is zero between calls: moments, resampled fractions and steps taken after one
another in any order, repeated, after a refused step and after a new initialisation, against the oracle."""
import ctypes

import numpy as np
import pytest

from oracle import learned as ol
from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


# bins in LDS, one wave's worth of energies, and more bins than the LDS copy takes (L = 28: 32929)
@pytest.mark.parametrize("dim,L,R,cap,layout", [(3, 6, 9000, 12800, "bits64"), (1, 200, 70, 8256, "u8"), (3, 28, 200, 8256, "bits64")])
def test_histogram_between_calls(dim, L, R, cap, layout):
    print(f"[case] histogram between calls dim={dim} L={L}", flush=True)
    J = o.couplings(dim, L, 3)
    run = pa.Run(dim, L, R, 8, 3, 3, capacity=cap, layout=layout, device=DEV)

    def moments(k, E):
        pa.measure([run])
        for got, want, tol in zip(run.records()[k][6:9], o.energy_moments(E), (1e-12, 1e-12, 1e-9)):
            assert abs(got - want) <= tol * max(1.0, abs(want))

    def fraction(E):
        dbs, out = np.array([0.01, 0.1], np.float64), torch.empty(2, dtype=torch.float64, device=DEV)
        pa.check(pa.lib().pa_resampled_fraction(ctypes.byref(run.desc), 1, pa._np(dbs), 2, out.data_ptr()), "fraction")
        want = np.array([ol.rho(*ol.histogram(E), d) for d in dbs])
        torch.cuda.synchronize()
        assert np.allclose(out.cpu().numpy(), want, rtol=1e-12, atol=1e-14)

    db = 0.3 / np.sqrt(L ** dim)
    for _ in range(2):  # a new initialisation after a refused step
        run.init()
        s_o, E_o = o.init_population(dim, L, J, 8, R, capacity=cap)
        for call in (fraction, lambda E: moments(0, E), lambda E: moments(0, E), fraction):
            call(E_o[:R])
        run.resample(pa.Schedule([0.0, db], 1, run.n_bins, device=DEV).step(1))
        r = o.resample(dim, L, 8, 1, 0.0, db, R, R, s_o, E_o, cap)
        assert r["status"] == 0 and run.status()[0] == pa.PA_OK
        assert run.records()[1][3] == r["S"] and run.records()[1][4] == r["R_new"] and run.records()[1][5] == r["E_lo"]
        E = r["E"][: r["R_new"]]
        assert np.array_equal(run.population()[1], E)
        moments(1, E)
        fraction(E)
        run.resample(pa.Schedule([db, 2 * db], 1, run.n_bins, device=DEV, R_targets=[0, 4 * cap]).step(1))
        assert run.status()[1] == pa.PA_FLAG_CAPACITY

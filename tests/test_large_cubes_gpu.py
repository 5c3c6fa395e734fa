"""Cold sweeps of cubes past side 18 in small and large launches (by the capacity) against the oracle, bit for
bit, with enough attempts for dozens of zero draws."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("layout", ["u8", "bits64"])
@pytest.mark.parametrize("L", [20, 24])
def test_cold_sweeps(L, layout):
    print(f"[case] cold sweeps L={L} {layout}", flush=True)
    J = o.couplings(3, L, 5)
    R, ns = 130, 4
    s_o, E_o = o.init_replicas(3, L, J, 3, 0, R)
    o.sweep_replicas(3, L, J, 3, 3.2, 0, s_o, E_o, 0, ns)
    for cap in (192, 8192, 8256):
        run = pa.Run(3, L, R, 3, 5, 2, capacity=cap, layout=layout, device=DEV).init()
        run.sweep(pa.Schedule([0.0, 3.2], ns, run.n_bins, device=DEV).step(1))
        assert run.status()[0] == pa.PA_OK
        s, E = run.population()
        assert np.array_equal(s, s_o) and np.array_equal(E, E_o), (L, cap)

"""The tabled Gaussian sweep with a call per thread or wave (few groups) and with a word per wave (many)
against the oracle, bit for bit: the same populations under a small and a large capacity, which alone
chooses the kernel, at the edges of calls, words and blocks, with first looks at the top of the bound."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("dim,L", [(3, 8), (3, 10)] + [(1, N) for N in (32, 34, 48, 50, 64, 126, 130, 192, 250, 258, 1024)])
def test_both_splits(dim, L):
    print(f"[case] gauss split dim={dim} L={L}", flush=True)
    J = o.couplings_gauss(dim, L, 8)
    for R, beta, ns in ((1, 2.0, 2), (17, 0.8, 3), (130, 0.5, 2), (300 if dim == 3 else 1500, 6e-6, 6)):
        s_o, E_o = o.init_replicas_gauss(dim, L, J, 6, 0, R)
        o.sweep_replicas_gauss(dim, L, J, 6, beta, 0, s_o, E_o, 0, ns)
        for cap in (64 * -(-R // 64), 64 * 400):
            run = pa.Run(dim, L, R, 6, 8, 2, capacity=cap, layout="u8", device=DEV, couplings="gauss").init()
            run.sweep(pa.Schedule([0.0, beta], ns, run.n_bins, device=DEV).step(1))
            assert run.status()[0] == pa.PA_OK
            s, E = run.population()
            assert np.array_equal(s, s_o) and np.array_equal(E, E_o), (dim, L, R, cap)

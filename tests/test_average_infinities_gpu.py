"""Infinite and NaN values through the device's weighted average: the same as plain sums give."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("M,at", [(1, 0), (64, 63), (130, 7)])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_infinite_observable_and_run(M, at, value):
    print(f"[case] average M={M} value={value}", flush=True)
    g = np.random.default_rng(M)
    x, A = 900.0 + g.standard_normal(M), g.standard_normal((M, 2))
    A[at, 0] = value
    s = torch.cuda.current_stream(DEV).cuda_stream

    def average(x):
        xd, Ad = torch.from_numpy(x).to(DEV), torch.from_numpy(A).to(DEV)
        out = torch.zeros(5, dtype=torch.float64, device=DEV)
        pa.check(pa.lib().pa_weighted_average_dev(1, M, xd.data_ptr(), None, Ad.data_ptr(), 2, out.data_ptr(), s), "average")
        return out.cpu().numpy()

    out = average(x)
    assert out[0] == value or (np.isnan(value) and np.isnan(out[0]))
    w = np.exp(x - x.max())
    assert abs(out[1] - (w * A[:, 1]).sum() / w.sum()) < 1e-12 and abs(out[4] - x.mean()) < 1e-9
    if M > 1 and value == -np.inf:  # a run of weight zero
        x[(at + 1) % M] = -np.inf
        out = average(x)
        w[(at + 1) % M] = 0.0
        assert abs(out[1] - (w * A[:, 1]).sum() / w.sum()) < 1e-12 and out[4] == -np.inf

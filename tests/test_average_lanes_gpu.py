"""Many averages of few terms, which take 1, 4 or 16 lanes each instead of a wave: every average of the call
against numpy, at the edges of the lanes and of the rule.  Tolerance 1e-12 relative: FP64 sums of at most 129
terms in another order."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def close(a, b):
    return np.all(np.abs(a - b) <= 1e-12 * np.maximum(1.0, np.abs(b)))


def weighted(x, R, A):
    """[.., M], [.., M] or None, [.., M, n_obs] -> [.., n_obs + 3]"""
    xr = x + (0.0 if R is None else np.log(R))
    top = xr.max(-1, keepdims=True)
    w = np.exp(xr - top)
    Z, M = w.sum(-1), x.shape[-1]
    bF = top[..., 0] + np.log(Z) - np.log(float(M) if R is None else R.sum(-1))
    var = x.var(-1, ddof=1) if M > 1 else np.zeros(x.shape[:-1])
    return np.concatenate([((w / Z[..., None])[..., None] * A).sum(-2), np.stack([bF, var, x.mean(-1)], -1)], -1)


def stream():
    return torch.cuda.current_stream(DEV).cuda_stream


@pytest.mark.parametrize("n", [1, 4095, 4096, 32769, 65535, 65536])
@pytest.mark.parametrize("M", [1, 4, 5, 16, 17, 64, 65, 128, 129])
def test_weighted_and_overlap_averages(n, M):
    print(f"[case] average lanes n={n} M={M}", flush=True)
    if n * M > 5_000_000:
        n = 5_000_000 // M
    g = np.random.default_rng(n + M)
    x, A = 900.0 + 2.0 * g.standard_normal((n, M)), g.standard_normal((n, M, 5))
    R = g.uniform(1e3, 1e5, (n, M)) if M % 2 else None
    xd, Ad, Rd = dev(x), dev(A), dev(R if R is not None else np.zeros(1))
    Rp = Rd.data_ptr() if R is not None else None
    out = torch.full((n, 8), np.nan, dtype=torch.float64, device=DEV)
    pa.check(pa.lib().pa_weighted_average_dev(n, M, xd.data_ptr(), Rp, Ad.data_ptr(), 5, out.data_ptr(), stream()), "average")
    assert close(out.cpu().numpy(), weighted(x, R, A))
    x2, Q = g.standard_normal((n, M, 2)), g.uniform(0.1, 1.0, (n, M, 3))
    R2 = g.uniform(1.0, 9.0, (n, M, 2))
    d = [dev(a) for a in (x2, R2, Q)]
    out = torch.full((n, 4), np.nan, dtype=torch.float64, device=DEV)
    pa.check(pa.lib().pa_overlap_average_dev(n, M, d[0].data_ptr(), d[1].data_ptr(), d[2].data_ptr(), out.data_ptr(),
                                             stream()), "overlap")
    q = weighted(x2.sum(-1), R2.prod(-1), Q)[:, :3]
    assert close(out.cpu().numpy(), np.concatenate([q, 0.5 * (3.0 - q[:, 1:2] / q[:, :1] ** 2)], -1))


@pytest.mark.parametrize("sets,M,n_boot", [(40, 8, 2000), (40, 9, 2000), (30, 3, 3), (20000, 5, 6), (90, 64, 400), (50, 100, 100)])
def test_bootstrap(sets, M, n_boot):
    print(f"[case] bootstrap lanes sets={sets} M={M} n_boot={n_boot}", flush=True)
    g = np.random.default_rng(sets + M)
    x, A = 900.0 + 2.0 * g.standard_normal((sets, M)), g.standard_normal((sets, M, 1))
    idx = g.integers(0, M, (n_boot, M)).astype(np.int32)
    idx[1, M - 1] = M if sets % 20 else -1  # outside the set: this replicate alone is NaN
    xd, Ad, idd = dev(x), dev(A), dev(idx)
    rep = torch.zeros((sets, n_boot, 4), dtype=torch.float64, device=DEV)
    err = torch.zeros((sets, 4), dtype=torch.float64, device=DEV)

    def call(n):
        pa.check(pa.lib().pa_bootstrap_dev(sets, M, xd.data_ptr(), None, Ad.data_ptr(), 1, n, idd.data_ptr(), rep.data_ptr(),
                                           err.data_ptr(), stream()), "bootstrap")
        return rep.cpu().numpy().reshape(-1)[: sets * n * 4].reshape(sets, n, 4), err.cpu().numpy()

    got, e = call(n_boot)
    good = np.arange(n_boot) != 1
    pick = idx[good]
    assert np.all(np.isnan(got[:, 1])) and np.all(np.isnan(e))
    assert close(got[:, good], weighted(x[:, pick], None, A[:, pick]))
    idx[1] = idx[0]
    idd.copy_(dev(idx))
    got, e = call(n_boot)
    want = got.std(axis=1, ddof=1)
    assert np.all(np.abs(e - want) <= 1e-10 * np.maximum(np.abs(want), 1e-6))

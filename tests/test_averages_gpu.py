"""Device averages over runs (weighted, bootstrap, overlap pairs), a wave per average, against the oracle at
the edges of the wave and of the observables taken at once.  Tolerance 1e-12 relative: FP64 sums of at most
a few hundred terms in another order."""
import numpy as np
import pytest

import inputs
from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def close(a, b):
    return np.all(np.abs(np.asarray(a) - np.asarray(b)) <= 1e-12 * np.maximum(1.0, np.abs(b)))


@pytest.mark.parametrize("sets,M,n_obs,n_boot,weighted", [(1, 1, 1, 1, False), (3, 2, 0, 2, True), (2, 63, 1, 65, True),
                                                           (5, 64, 4, 64, False), (4, 65, 5, 3, True),
                                                           (2, 200, 9, 40, True)])
def test_weighted_and_bootstrap(sets, M, n_obs, n_boot, weighted):
    print(f"[case] averages sets={sets} M={M} n_obs={n_obs} n_boot={n_boot}", flush=True)
    g = np.random.default_rng(70 + M)
    x = 900.0 + 2.0 * g.standard_normal((sets, M))
    R = g.uniform(1e3, 1e5, (sets, M)) if weighted else None
    A = g.standard_normal((sets, M, n_obs))
    idx = g.integers(0, M, (n_boot, M)).astype(np.int32)
    s = torch.cuda.current_stream(DEV).cuda_stream
    xd, Ad, idd = dev(x), dev(A), dev(idx)
    Rd = dev(R) if weighted else None
    out = torch.full((sets, n_obs + 3), np.nan, dtype=torch.float64, device=DEV)
    rep = torch.full((sets, n_boot, n_obs + 3), np.nan, dtype=torch.float64, device=DEV)
    err = torch.full((sets, n_obs + 3), np.nan, dtype=torch.float64, device=DEV)
    Rp = Rd.data_ptr() if weighted else None
    Ap = Ad.data_ptr() if n_obs else None
    pa.check(pa.lib().pa_weighted_average_dev(sets, M, xd.data_ptr(), Rp, Ap, n_obs, out.data_ptr(), s), "average")
    pa.check(pa.lib().pa_bootstrap_dev(sets, M, xd.data_ptr(), Rp, Ap, n_obs, n_boot, idd.data_ptr(), rep.data_ptr(),
                                       err.data_ptr(), s), "bootstrap")
    out, rep, err = (t.cpu().numpy() for t in (out, rep, err))
    for i in range(sets):
        w = o.weighted_average(x[i], A[i], None if R is None else R[i])
        assert close(out[i], np.concatenate([w["A_bar"], [w["minus_betaF_bar"], w["var"], w["mean"]]]))
        for b in range(n_boot):
            w = o.weighted_average(x[i][idx[b]], A[i][idx[b]], None if R is None else R[i][idx[b]])
            assert close(rep[i, b], np.concatenate([w["A_bar"], [w["minus_betaF_bar"], w["var"], w["mean"]]]))
        want = rep[i].std(axis=0, ddof=1) if n_boot > 1 else np.zeros(n_obs + 3)
        assert np.all(np.abs(err[i] - want) <= 1e-10 * np.maximum(np.abs(want), 1e-6))


@pytest.mark.parametrize("sets,pairs", [(1, 1), (3, 63), (2, 64), (5, 65), (2, 150)])
def test_overlap_average(sets, pairs):
    print(f"[case] overlap average sets={sets} pairs={pairs}", flush=True)
    x, R, Q = inputs.overlap_pair_sets(80 + pairs, sets, pairs)
    out = torch.full((sets, 4), np.nan, dtype=torch.float64, device=DEV)
    xd, Rd, Qd = dev(x), dev(R), dev(Q)
    pa.check(pa.lib().pa_overlap_average_dev(sets, pairs, xd.data_ptr(), Rd.data_ptr(), Qd.data_ptr(), out.data_ptr(),
                                             torch.cuda.current_stream(DEV).cuda_stream), "overlap")
    out = out.cpu().numpy()
    for i in range(sets):
        w = o.overlap_average(x[i], Q[i], R[i])
        assert close(out[i], w)

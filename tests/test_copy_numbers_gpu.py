"""Copy numbers against the oracle, bit for bit, where a lane's draws change hands: means from 1e-4 to
hundreds (the table's first entries, its binary search, Poisson(64) blocks, thinning by the lane and by
the wave), energies that span more bins than the small kernel keeps weights of, in the kernel for small
populations and in the one for large ones."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"


# steps in beta over energies between -12288 and -12288 + 4 bins: the mean falls by exp(-4 db) a bin
@pytest.mark.parametrize("cap", [4096, 4160])
@pytest.mark.parametrize("R,bins,db,layout", [(1500, 3000, 1e-5, "bits64"), (1100, 2000, 1e-3, "u8"),
                                              (1030, 1025, 2.5e-3, "bits64"), (1024, 40, 2e-2, "u8"),
                                              (900, 400, 3e-2, "bits64"), (1500, 200, 0.2, "u8"),
                                              (1300, 2500, 0.3, "bits64"), (65, 30, 0.05, "bits64")])
def test_copy_numbers(R, bins, db, layout, cap):
    print(f"[case] copy numbers R={R} bins={bins} db={db} cap={cap}", flush=True)
    L = 16
    run = pa.Run(3, L, R, 12, 3, 2, capacity=cap, layout=layout, device=DEV).init()
    g = np.random.default_rng(R + bins)
    E = (-3 * L**3 + 4 * g.integers(0, bins, R)).astype(np.int32)
    E[0], E[-1] = -3 * L**3, -3 * L**3 + 4 * (bins - 1)
    run.energy[0][: 4 * R].view(torch.int32).copy_(torch.from_numpy(E))
    torch.cuda.synchronize()
    run.resample(pa.Schedule([0.5, 0.5 + db], 1, run.n_bins, device=DEV).step(1))
    assert run.status()[0] == pa.PA_OK
    _, c_o, S_o, _, E_lo_o = o.copy_numbers(12, 1, 0.5, 0.5 + db, float(R), E)
    c, off = run.counts_offsets(R)
    assert np.array_equal(c, c_o) and np.array_equal(off, np.concatenate([[0], np.cumsum(c_o)]))
    rec = run.records()[1]
    assert rec[3] == S_o and rec[4] == c_o.sum() and rec[5] == E_lo_o
    assert np.array_equal(run.population()[1], np.repeat(E, c_o))

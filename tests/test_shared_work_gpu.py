"""The work buffer is scratch: runs of different shapes share one on a stream, and it is overwritten before
every call, against the same runs with work buffers of their own."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"
# dim, L, R, layout, couplings: histograms in LDS and in global memory (L = 28), populations of several
# blocks and of one, chains and cubes, both coupling kinds
SHAPES = [(3, 6, 9000, "bits64", "pm1"), (1, 200, 12000, "u8", "pm1"), (3, 28, 9000, "bits64", "pm1"),
          (3, 4, 300, "u8", "pm1"), (3, 4, 9000, "u8", "gauss"), (1, 50, 9000, "u8", "gauss")]


def fractions(run):
    dbs, out = np.array([0.01, 0.1], np.float64), torch.zeros(2, dtype=torch.float64, device=DEV)
    if run.couplings_kind == pa.PA_PM1:
        pa.check(pa.lib().pa_resampled_fraction(ctypes.byref(run.desc), 1, pa._np(dbs), 2, out.data_ptr()), "fraction")
    return out


def steps(runs, before_call):
    """two steps of every run in turn, call by call, with overlaps of the pairs (a run and its own copy)"""
    got = [[] for _ in runs]
    scheds = [pa.Schedule([0.0, *(np.array([1, 2]) * 0.3 / np.sqrt(r.N))], 1, r.n_bins, device=DEV) for r, _ in runs]
    for pair in runs:
        for r in pair:
            before_call()
            r.init()
    for k in (1, 2):
        for call in ("fraction", "resample", "sweep", "measure"):
            for i, pair in enumerate(runs):
                st = scheds[i].step(k)
                if call == "measure":
                    before_call()
                    pa.measure(list(pair), [1, -1])
                    continue
                for r in pair:
                    if r.L == 28 and call == "sweep":
                        continue  # (a side that no sweep takes)
                    before_call()
                    if call == "fraction":
                        got[i].append(fractions(r))
                    else:
                        getattr(r, call)(st)
    return [[*(t.cpu().numpy() for t in g), *(x for r in pair for x in (r.records(), *r.population()))]
            for g, pair in zip(got, runs)]


@pytest.mark.parametrize("seed", [1, 2])
def test_shared_and_overwritten_work(seed):
    print(f"[case] shared work seed={seed}", flush=True)
    make = lambda: [tuple(pa.Run(d, L, R, s, 3, 3, layout=lay, device=DEV, couplings=c) for s in (seed, seed + 10))  # noqa: E731
                    for d, L, R, lay, c in SHAPES]
    want = steps(make(), lambda: None)
    runs = make()
    work = torch.empty(max(int(r.sizes.work_bytes) for p in runs for r in p), dtype=torch.uint8, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    for p in runs:
        for r in p:
            r.desc.work = work.data_ptr()
    got = steps(runs, lambda: work.random_(0, 256, generator=gen))
    for shape, a, b in zip(SHAPES, want, got):
        assert len(a) == len(b) and all(np.array_equal(x, y, equal_nan=True) for x, y in zip(a, b)), shape

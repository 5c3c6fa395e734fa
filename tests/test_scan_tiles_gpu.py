"""Offsets and sources of populations whose tile sums are added by every block or scanned first: around
2048 tiles of 256 replicas of capacity, around whole rounds of the scan (8192 tiles), and a batch of both."""
import numpy as np
import pytest

from oracle import oracle as o

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"
TILE = 256


def check(run, E0, seed, target):
    c = o.copy_numbers(seed, 1, 0.0, 0.3, target, E0)[1]
    counts, offsets = run.counts_offsets(len(E0))
    assert np.array_equal(counts, c) and np.array_equal(offsets, np.concatenate([[0], np.cumsum(c, dtype=np.int64)]))
    assert run.status()[1] == 0 and np.array_equal(run.energies(), np.repeat(E0, c))


@pytest.mark.parametrize("R,cap", [(500_000, 2048 * TILE), (500_000, 2048 * TILE + 64), (8192 * TILE - 1, 8300 * TILE),
                                   (8192 * TILE + 1, 8300 * TILE), (3 * 8192 * TILE, 25000 * TILE), (300, 8300 * TILE)])
def test_offsets_and_sources(R, cap):
    print(f"[case] scan of tiles R={R} cap={cap}", flush=True)
    run = pa.Run(1, 16, R, 4, 3, 2, capacity=cap, layout="bits64", device=DEV).init()
    E0 = run.energies()
    run.resample(pa.Schedule([0.0, 0.3], 1, run.n_bins, device=DEV).step(1))
    check(run, E0, 4, float(R))


def test_batch_of_uneven_runs():
    print("[case] scan of tiles in a batch", flush=True)
    sizes = [700, 600_000, 256, 2_200_000]
    specs = [dict(dim=1, L=16, R0=R, seed=i + 1, disorder_seed=3) for i, R in enumerate(sizes)]
    batch = pa.Batch(specs, 2, layout="bits64", device=DEV, capacity_factor=1.3).init()
    E0 = [r.energies() for r in batch.runs]
    batch.resample(pa.Schedule([0.0, 0.3], 1, batch.runs[0].n_bins, device=DEV).step(1))
    for i, (r, E) in enumerate(zip(batch.runs, E0)):
        check(r, E, i + 1, float(sizes[i]))

"""More averages in a call than a launch has waves (2^26): every one is formed."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import pa  # noqa: E402

DEV = "cuda:0"
N = (1 << 26) + 1001


def stream():
    return torch.cuda.current_stream(DEV).cuda_stream


def test_weighted_averages_of_one_run():
    print("[case] many weighted averages", flush=True)
    x = torch.arange(N, dtype=torch.float64, device=DEV) * 0.25
    out = torch.full((N, 3), -1.0, dtype=torch.float64, device=DEV)
    pa.check(pa.lib().pa_weighted_average_dev(N, 1, x.data_ptr(), None, None, 0, out.data_ptr(), stream()), "averages")
    assert torch.equal(out[:, 0], x) and torch.equal(out[:, 2], x) and not out[:, 1].any()


def test_overlap_averages_of_one_pair():
    print("[case] many overlap averages", flush=True)
    x = torch.zeros((N, 2), dtype=torch.float64, device=DEV)
    Q = torch.rand((N, 3), dtype=torch.float64, device=DEV, generator=torch.Generator(DEV).manual_seed(1)) + 0.5
    out = torch.full((N, 4), -1.0, dtype=torch.float64, device=DEV)
    pa.check(pa.lib().pa_overlap_average_dev(N, 1, x.data_ptr(), None, Q.data_ptr(), out.data_ptr(), stream()), "overlaps")
    assert torch.equal(out[:, :3], Q)
    assert torch.equal(out[:, 3], 0.5 * (3.0 - Q[:, 1] / (Q[:, 0] * Q[:, 0])))


def test_bootstrap_replicates_of_two_runs():
    print("[case] many bootstrap replicates", flush=True)
    x = torch.tensor([[0.3, -0.4]], dtype=torch.float64, device=DEV)

    def call(idx):
        rep = torch.full((len(idx), 3), -7.0, dtype=torch.float64, device=DEV)
        err = torch.empty(3, dtype=torch.float64, device=DEV)
        pa.check(pa.lib().pa_bootstrap_dev(1, 2, x.data_ptr(), None, None, 0, len(idx), idx.data_ptr(), rep.data_ptr(),
                                           err.data_ptr(), stream()), "bootstrap")
        return rep, err

    four = torch.tensor([[0, 0], [0, 1], [1, 0], [1, 1]], dtype=torch.int32, device=DEV)
    which = torch.randint(0, 4, (N,), device=DEV, generator=torch.Generator(DEV).manual_seed(2))
    rep, err = call(four[which].contiguous())
    assert torch.equal(rep, call(four)[0][which])
    # a lane adds N / 64 terms of one sign: relative error below N / 64 2^-53 each for mean and squares
    assert torch.allclose(err, rep.std(dim=0), rtol=4 * (N / 64) * 2.0 ** -53, atol=0.0)

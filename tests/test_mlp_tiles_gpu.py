"""The network's forward and gradient at the edges of the 32-sample tiles and past one tile per block (512
blocks), against the FP64 oracle.  Tolerances: FP32 sums of 64 terms per layer through three layers, a few
1e-6 of each sample's output, and sums over the batch in blocks, well inside 1e-4 of a parameter block's
largest entry."""
import ctypes

import numpy as np
import pytest

import inputs
from oracle import learned as ol

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1006_0252_amd import learned, pa  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("B", [1, 31, 32, 33, 64, 95, 16384, 16421])
def test_forward_and_gradient(B):
    print(f"[case] mlp tiles B={B}", flush=True)
    s = torch.cuda.current_stream(DEV).cuda_stream
    theta = inputs.mlp_theta(61, scale=1.5)
    th = torch.from_numpy(theta).to(DEV)
    w = torch.empty(learned.N_PARAMS, dtype=torch.int16, device=DEV)
    pa.check(pa.lib().pa_bf16_round(th.data_ptr(), w.data_ptr(), learned.N_PARAMS, s), "round")
    X = inputs.mlp_features(62 + B, B, zero_var_every=29 if B > 30 else 0)
    t = inputs.mlp_targets(63 + B, B, bad_every=23 if B > 30 else 0)
    Xd, td = torch.from_numpy(X).to(DEV), torch.from_numpy(t).to(DEV)
    w64 = ol.bf16_values(ol.bf16_bits(theta))
    out = torch.full((B,), np.nan, dtype=torch.float32, device=DEV)
    pa.check(pa.lib().pa_mlp_forward(w.data_ptr(), Xd.data_ptr(), B, 1e-4, 0.25, out.data_ptr(), s), "forward")
    want = ol.forward(w64, X.astype(np.float64), np.float32(1e-4), np.float32(0.25))
    assert np.allclose(out.cpu().numpy().astype(np.float64), want, rtol=1e-5, atol=0)
    nb = ctypes.c_int64()
    pa.check(pa.lib().pa_mlp_work_bytes(B, ctypes.byref(nb)), "work")
    # garbage that must not be read, and a guard behind the work memory that must not be written
    work = torch.full((int(nb.value) + 4096,), 0x7F, dtype=torch.uint8, device=DEV)
    grad = torch.full((learned.N_PARAMS,), np.nan, dtype=torch.float32, device=DEV)
    loss = torch.full((1,), np.nan, dtype=torch.float32, device=DEV)
    pa.check(pa.lib().pa_mlp_grad(w.data_ptr(), Xd.data_ptr(), td.data_ptr(), B, work.data_ptr(), grad.data_ptr(),
                                  loss.data_ptr(), s), "grad")
    assert bool((work[int(nb.value):] == 0x7F).all())
    L_o, g_o = ol.loss_and_grad(w64, X.astype(np.float64), t)
    assert abs(float(loss.item()) - L_o) <= 1e-5 * L_o
    g = grad.cpu().numpy().astype(np.float64)
    sizes = {"W1": 384, "b1": 64, "W2": 4096, "b2": 64, "W3": 4096, "b3": 64, "w4": 64, "b4": 1}
    for name, lo in ol.OFF.items():
        a, b = g[lo:lo + sizes[name]], g_o[lo:lo + sizes[name]]
        assert np.abs(a - b).max() <= 1e-4 * np.abs(b).max(), name

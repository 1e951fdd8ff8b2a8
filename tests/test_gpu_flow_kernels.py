"""The flow head's embedding and readout kernels against fp64."""
import ctypes as C

import numpy as np
import pytest

from paper_2508_10259_amd import workload as W
from gpu_util import log
from test_gpu_kernels import _ptr, _stream, probe  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_tok,a,d", [(1, 1, 128), (8, 7, 640), (13, 32, 4096), (17, 256, 384)])
@pytest.mark.parametrize("shift", [0, 1])  # weights off the 16-byte grid: element by element
def test_flow_kernels(probe, dtype, n_tok, a, d, shift):  # noqa: F811
    import torch
    log(f"flow kernels {dtype} n_tok={n_tok} a={a} d={d} shift={shift}")
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    ct = 1 if dtype == "bf16" else 0

    def dev(x):
        t = torch.empty(x.size + shift, dtype=td, device="cuda")
        t[shift:].copy_(torch.from_numpy(x.reshape(-1)))
        return t[shift:].view(x.shape)

    x = W.random_gaussian((n_tok, a), 121, n_tok, a, dtype="f32")
    w_in = dev(W.random_gaussian((d, a), 122, d, a, dtype="f32"))
    w_t = dev(W.random_gaussian((d,), 123, d, dtype="f32"))
    w_out = dev(W.random_gaussian((a, d), 124, a, d, dtype="f32", std=0.02))
    f64 = lambda t: t.double().cpu().numpy()  # noqa: E731
    xd = torch.from_numpy(x.copy()).cuda()
    h = torch.full((n_tok, d), float("nan"), device="cuda")
    tau, dt, eps = 0.3, 0.25, 1e-5
    assert probe.ams_probe_flow(ct, _ptr(xd), _ptr(w_in), _ptr(w_t), _ptr(w_out), C.c_float(tau), C.c_float(eps),
                                C.c_float(dt), n_tok, a, d, _ptr(h), _stream()) == 0
    torch.cuda.synchronize()
    ref = x.astype(np.float64) @ f64(w_in).T + np.float64(np.float32(tau)) * f64(w_t)
    got = f64(h)
    assert np.max(np.abs(got - ref)) <= 2e-6 * np.max(np.abs(ref)) * np.sqrt(a)  # fp32 sums of a products
    r = 1.0 / np.sqrt(np.mean(got * got, -1, keepdims=True) + eps)
    out = x + dt * r * (got @ f64(w_out).T)
    assert np.max(np.abs(f64(xd) - out)) <= 2e-6 * max(1.0, np.max(np.abs(out)))

"""The feed's sums of squares for the next projection's RMSNorm, and its vectorised copies."""
import numpy as np
import pytest

from paper_2508_10259_amd import workload as W
from gpu_util import log
from test_gpu_kernels import _dev, _ptr, _rand, _stream, probe  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,n_bins", [(1, 128, 3), (3, 640, 100), (17, 4096, 256)])
def test_argmax_feed_ss(probe, B, d, n_bins):  # noqa: F811
    import torch
    log(f"argmax_feed ss B={B} d={d} n_bins={n_bins}")
    lg = W.random_gaussian((B, n_bins), 131, B, dtype="f32")
    E = _rand((n_bins, d), 132, n_bins, d)
    tok = torch.zeros(B, dtype=torch.int32, device="cuda")
    h = torch.full((B, d), float("nan"), device="cuda")
    h16, lo = (torch.full((B, d), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    ss = torch.full((B, d // 128), float("nan"), device="cuda")
    lgd, Ed = _dev(lg, "f32"), _dev(E, "f16")
    assert probe.ams_probe_argmax_feed_ss(_ptr(lgd), n_bins, _ptr(Ed), B, d, n_bins, _ptr(tok), _ptr(h), _ptr(h16),
                                          _ptr(lo), _ptr(ss), _stream()) == 0
    torch.cuda.synchronize()
    t = lg.argmax(1)
    assert np.array_equal(tok.cpu().numpy(), t)
    rows = E[t]
    assert np.array_equal(h16.cpu().numpy(), rows) and np.array_equal(h.cpu().numpy(), rows.astype(np.float32))
    assert float(lo.abs().max()) == 0.0
    ref = (rows.astype(np.float64) ** 2).reshape(B, d // 128, 128).sum(-1)
    assert np.max(np.abs(ss.cpu().numpy() - ref) / ref) <= 2e-6  # fp32 sums of 128 squares

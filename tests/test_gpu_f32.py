"""The kernels of fp32 models through the probe library, against their plain definitions in fp64."""
import ctypes as C

import numpy as np
import pytest

from paper_2508_10259_amd import workload as W
from gpu_util import log
from test_gpu_kernels import (EPI_RESID, EPI_STORE, EPI_SWIGLU, _dev, _ptr, _rope_tab, _silu, _stream, _to_pages,
                              _unpack_gu, probe)  # noqa: F401

pytestmark = pytest.mark.gpu


def _epilogue(epi, y, h0):
    if epi == EPI_STORE:
        return y
    if epi == EPI_RESID:
        return h0 + y
    g, up = _unpack_gu(y.T, y.shape[1] // 2)
    return (_silu(g) * up).T


def _check(got, ref, K):
    # fp32 products and sums: an error of 2^-24 per addition, random in sign over K of them
    tol = 1e-5 * max(1.0, float(np.max(np.abs(ref)))) * np.sqrt(K / 128)
    err = float(np.max(np.abs(got - ref)))
    assert err <= tol, f"max abs err {err:.3e} > {tol:.3e}"


@pytest.mark.parametrize("epi,norm,splits", [(EPI_STORE, True, 1), (EPI_SWIGLU, True, 1), (EPI_RESID, False, 1),
                                             (EPI_RESID, False, 3), (EPI_RESID, False, 4)])
@pytest.mark.parametrize("M", [1, 15, 17, 32, 33, 64])
@pytest.mark.parametrize("N,K", [(256, 256), (96, 1088), (512, 4096)])
def test_gemv_f32(probe, epi, norm, splits, M, N, K):  # noqa: F811
    import torch
    log(f"gemv_f32 epi={epi} norm={norm} splits={splits} M={M} N={N} K={K}")
    eps = 1e-5
    x = W.random_gaussian((M, K), 101, M, K, dtype="f32") * np.float32(3.0)
    Wt = W.random_gaussian((N, K), 102, N, K, dtype="f32", std=0.05)
    h0 = W.random_gaussian((M, N), 103, M, dtype="f32")
    x64 = x.astype(np.float64)
    rs = 1.0 / np.sqrt(np.mean(x64 * x64, axis=-1, keepdims=True) + eps) if norm else 1.0
    ref = _epilogue(epi, (x64 * rs) @ Wt.astype(np.float64).T, h0.astype(np.float64))
    ldo = N // 2 if epi == EPI_SWIGLU else N
    xd, wd = _dev(x, "f32"), _dev(Wt, "f32")
    part = torch.full((splits, M, N), float("nan"), device="cuda")
    cnt = torch.zeros(N // 16, dtype=torch.int32, device="cuda")
    for _ in range(2):  # the counters are zero again after a launch
        out = torch.from_numpy(h0.copy()).cuda() if epi == EPI_RESID else torch.zeros((M, ldo), device="cuda")
        rc = probe.ams_probe_gemv_f32(epi, _ptr(xd), int(norm), C.c_float(eps), _ptr(wd), M, N, K, _ptr(out), ldo,
                                      splits, _ptr(part), _ptr(cnt), _stream())
        assert rc == 0
        torch.cuda.synchronize()
        _check(out.cpu().numpy().astype(np.float64), ref, K)
        assert int(cnt.abs().sum()) == 0


@pytest.mark.parametrize("epi", [EPI_STORE, EPI_RESID, EPI_SWIGLU])
@pytest.mark.parametrize("M,N,K", [(65, 192, 128), (200, 256, 1088), (1100, 3072, 128)])  # 64- and 128-wide tiles
def test_gemm_f32(probe, epi, M, N, K):  # noqa: F811
    import torch
    log(f"gemm_f32 epi={epi} M={M} N={N} K={K}")
    x = W.random_gaussian((M, K), 104, M, K, dtype="f32")
    Wt = W.random_gaussian((N, K), 105, N, K, dtype="f32", std=0.05)
    h0 = W.random_gaussian((M, N), 106, M, dtype="f32")
    ref = _epilogue(epi, x.astype(np.float64) @ Wt.astype(np.float64).T, h0.astype(np.float64))
    ldo = N // 2 if epi == EPI_SWIGLU else N
    out = torch.from_numpy(h0.copy()).cuda() if epi == EPI_RESID else torch.zeros((M, ldo), device="cuda")
    xd, wd, null = _dev(x, "f32"), _dev(Wt, "f32"), C.c_void_p(None)
    assert probe.ams_probe_gemm(0, epi, _ptr(xd), null, _ptr(wd), M, N, K, _ptr(out), ldo, null, null, _stream()) == 0
    torch.cuda.synchronize()
    _check(out.cpu().numpy().astype(np.float64), ref, K)


@pytest.mark.parametrize("dh,segs", [
    (64, [(0, 280, 16), (1, 0, 1), (2, 129, 3), (3, 63, 17)]),
    (128, [(0, 300, 16), (1, 0, 5), (2, 470, 1), (3, 37, 33)]),
    (64, [(1, 0, 130), (0, 15, 2)]),
    (128, [(2, 200, 70)]),
])
def test_attn_f32(probe, dh, segs):  # noqa: F811
    """Causal attention of packed segments over fp32 pages whose slots past each row's last key hold NaN."""
    import torch
    B, H, cap = 4, 2, 512
    d, half = H * dh, dh // 2
    log(f"attn_f32 dh={dh} segs={segs}")
    n_tok = sum(n for _, _, n in segs)
    qkv = W.random_gaussian((n_tok, 3 * d), 107, dh, n_tok, dtype="f32")
    K = W.random_gaussian((B, H, cap, dh), 108, dh, dtype="f32")
    V = W.random_gaussian((B, H, cap, dh), 109, dh, dtype="f32")
    for b, p0, n in segs:
        K[b, :, p0 + n:] = np.nan
        V[b, :, p0 + n:] = np.nan
    tab = _rope_tab(cap, dh)
    off = np.cumsum([0] + [n for _, _, n in segs]).astype(np.int32)
    perm = np.random.default_rng(dh + n_tok).permutation(B * (cap // 64)).astype(np.int32)
    pt_d, offd = torch.from_numpy(perm).cuda(), torch.from_numpy(off).cuda()
    rows = torch.tensor([b for b, _, _ in segs], dtype=torch.int32, device="cuda")
    pos = torch.tensor([p for _, p, _ in segs], dtype=torch.int32, device="cuda")
    qkv_d, tab_d = _dev(qkv, "f32"), _dev(tab, "f32")
    K_d, V_d = _dev(_to_pages(K, perm), "f32"), _dev(_to_pages(V, perm), "f32")
    o = torch.full((n_tok, d), float("nan"), device="cuda")
    rc = probe.ams_probe_attn_prefill(0, _ptr(qkv_d), _ptr(rows), _ptr(pos), _ptr(offd), len(segs), n_tok,
                                      max(n for _, _, n in segs), max(p + n for _, p, n in segs), H, dh, cap,
                                      _ptr(pt_d), _ptr(tab_d), _ptr(K_d), _ptr(V_d), _ptr(o), _stream())
    assert rc == 0
    torch.cuda.synchronize()
    got = o.cpu().numpy().astype(np.float64)
    for si, (b, p0, n) in enumerate(segs):
        for i in range(n):
            t, p = off[si] + i, p0 + i
            cs = tab[p].astype(np.float64)
            for h in range(H):
                q = qkv[t, h * dh:(h + 1) * dh].astype(np.float64)
                qr = np.concatenate([q[:half] * cs[:, 0] - q[half:] * cs[:, 1],
                                     q[:half] * cs[:, 1] + q[half:] * cs[:, 0]]) / np.sqrt(dh)
                s_ = K[b, h, :p + 1].astype(np.float64) @ qr
                w = np.exp(s_ - s_.max())
                ref = (w / w.sum()) @ V[b, h, :p + 1].astype(np.float64)
                # __expf is within a few 2^-22 of exp over scores of a few units
                err = float(np.max(np.abs(got[t, h * dh:(h + 1) * dh] - ref)))
                assert err <= 1e-5 * np.max(np.abs(V[b, h, :p + 1])), (si, i, h, err)

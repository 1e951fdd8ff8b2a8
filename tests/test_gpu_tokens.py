"""The tile shapes of the token passes' fp16 GEMMs against the exact products of their inputs."""
import ctypes as C

import numpy as np
import pytest

from paper_2508_10259_amd import workload as W
from gpu_util import log
from test_gpu_kernels import EPI_RESID, EPI_STORE, EPI_SWIGLU, _dev, _f, _ptr, _rand, _silu, _stream, _unpack_gu, probe  # noqa: F401,E501

pytestmark = pytest.mark.gpu
EPI_PART = 3
TILES = ((256, 256), (128, 256), (256, 128), (128, 128), (128, 128), (64, 128), (128, 64), (64, 256))


def _frag32(Wt):
    """MFMA fragment order of W [N][K] for any K a multiple of 32."""
    N, K = Wt.shape
    return np.ascontiguousarray(Wt.reshape(N // 16, 16, K // 32, 4, 8).transpose(0, 2, 3, 1, 4)).reshape(N, K)


@pytest.mark.parametrize("tile", range(len(TILES)))
@pytest.mark.parametrize("epi,splits", [(EPI_STORE, 1), (EPI_RESID, 1), (EPI_SWIGLU, 1), (EPI_PART, 1), (EPI_PART, 3)])
def test_gemm_tokens_tile(probe, tile, epi, splits):  # noqa: F811
    """Token counts around the tile's edges, fewer K steps than the kernels' slots and stages (64,
    128, 192) and more (576), splits of unequal lengths."""
    import torch
    bm, bn = TILES[tile]
    N = 3 * bn
    for M, K in ((1, 64), (bm - 1, 128), (bm, 192), (bm + 1, 576), (2 * bm + 17, 448), (9 * bm + 5, 256)):
        if splits > K // 64:
            continue
        log(f"gemm_tokens tile={TILES[tile]} epi={epi} splits={splits} M={M} N={N} K={K}")
        u, Wt = _rand((M, K), 111, M, K), _rand((N, K), 112, N, K, std=0.05)
        h0 = W.random_gaussian((M, N), 113, M, dtype="f32")
        y = _f(u, "f16") @ _f(Wt, "f16").T
        ldo = N // 2 if epi == EPI_SWIGLU else N
        if epi == EPI_SWIGLU:
            g, up = _unpack_gu(y.T, N // 2)
            ref = (_silu(g) * up).T
            out = torch.full((M, ldo), float("nan"), dtype=torch.float16, device="cuda")
        elif epi == EPI_RESID:
            ref, out = h0 + y, torch.from_numpy(h0.copy()).cuda()
        else:
            ref, out = y, torch.full((splits, M, N), float("nan"), device="cuda")
        ud, wd = _dev(u, "f16"), _dev(_frag32(Wt), "f16")
        assert probe.ams_probe_gemm_tokens(tile, epi, _ptr(ud), _ptr(wd), M, N, K, _ptr(out), ldo, splits,
                                           _stream()) == 0
        torch.cuda.synchronize()
        got = out.float().cpu().numpy().astype(np.float64)
        if epi == EPI_PART:
            for s in range(splits):  # a split holds its own range of K steps
                k0, k1 = s * (K // 64) // splits * 64, (s + 1) * (K // 64) // splits * 64
                part = _f(u[:, k0:k1], "f16") @ _f(Wt[:, k0:k1], "f16").T
                assert np.max(np.abs(got[s] - part)) <= 2e-5 * max(1.0, np.max(np.abs(part))) * np.sqrt(K / 64), s
            continue
        got = got.reshape(ref.shape)
        scale = max(1.0, float(np.max(np.abs(ref))))
        tol = 2e-5 * scale * np.sqrt(K / 64)  # fp16 products are exact in the fp32 accumulator
        if epi == EPI_SWIGLU:
            tol = max(tol, 2 ** -11 * scale)  # the fp16 output
        assert float(np.max(np.abs(got - ref))) <= tol


def test_gemm_tokens_refusals(probe):  # noqa: F811
    import torch
    x = torch.zeros(1 << 20, dtype=torch.float16, device="cuda")
    out = torch.zeros(1 << 20, device="cuda")

    def call(tile, epi, M, N, K, splits):
        return probe.ams_probe_gemm_tokens(tile, epi, _ptr(x), _ptr(x), M, N, K, _ptr(out), N, splits, _stream())

    assert call(0, EPI_STORE, 8, 128, 64, 1) != 0   # N not a multiple of the tile width
    assert call(5, EPI_STORE, 8, 128, 96, 1) != 0   # K not a multiple of 64
    assert call(5, EPI_STORE, 8, 128, 128, 2) != 0  # splits without partial sums
    assert call(5, EPI_PART, 8, 128, 128, 3) != 0   # more splits than K steps
    assert call(len(TILES), EPI_STORE, 8, 128, 128, 1) != 0


@pytest.mark.parametrize("M,K,segs", [(65, 1024, 3), (130, 64, 1), (300, 1984, 8), (513, 4096, 5)])
def test_tiles_same_bits(probe, M, K, segs):  # noqa: F811
    """Every tile shape gives the same bits, and so do a residual projection whose K ranges one
    workgroup adds and the reduction of the same ranges' partial sums."""
    import torch
    N = 768
    log(f"same bits M={M} K={K} segs={segs}")
    ud, wd = _dev(_rand((M, K), 114, M, K), "f16"), _dev(_frag32(_rand((N, K), 115, N, K, std=0.05)), "f16")
    h0 = torch.from_numpy(W.random_gaussian((M, N), 116, M, dtype="f32")).cuda()
    y0 = hp = None
    for tile in range(len(TILES)):
        y, h, part = torch.empty_like(h0), h0.clone(), torch.empty((segs, M, N), device="cuda")
        assert probe.ams_probe_gemm_tokens(tile, EPI_STORE, _ptr(ud), _ptr(wd), M, N, K, _ptr(y), N, 1, _stream()) == 0
        assert probe.ams_probe_gemm_tokens(tile, EPI_PART, _ptr(ud), _ptr(wd), M, N, K, _ptr(part), N, segs,
                                           _stream()) == 0
        assert probe.ams_probe_part_resid(_ptr(part), segs, M, N, _ptr(h), None, None, _stream()) == 0
        y0, hp = (y, h) if y0 is None else (y0, hp)
        assert torch.equal(y, y0) and torch.equal(h, hp), TILES[tile]
        h = h0.clone()
        rc = probe.ams_probe_gemm_tokens_segs(tile, _ptr(ud), _ptr(wd), M, N, K, _ptr(h), segs, _stream())
        if tile == 0 and segs > 1:  # no registers for the second accumulator
            assert rc != 0
        else:
            assert rc == 0 and torch.equal(h, hp), TILES[tile]
    assert probe.ams_probe_gemm_tokens_segs(4, _ptr(ud), _ptr(wd), M, N, K, _ptr(h), K // 64 + 1, _stream()) != 0


@pytest.mark.parametrize("d,splits", [(1024, 2), (1152, 5), (2048, 8), (4096, 1), (4096, 16), (5120, 4)])
def test_norms_same_bits(probe, d, splits):  # noqa: F811
    """A row's norm has the same bits in a pass of any length, alone and after the residual reduction."""
    import torch
    log(f"norms d={d} splits={splits}")
    part = torch.from_numpy(W.random_gaussian((splits, 400, d), 117, d, dtype="f32")).cuda()
    h0 = torch.from_numpy(W.random_gaussian((400, d), 118, d, dtype="f32")).cuda()
    out = {}
    for M in (400, 256, 65, 3):
        h, p = h0[:M].clone(), part[:, :M].contiguous()
        un, ur = (torch.empty((M, d), dtype=torch.float16, device="cuda") for _ in range(2))
        eps = C.c_float(1e-5)
        assert probe.ams_probe_rmsnorm(2, _ptr(h), M, d, eps, _ptr(un), None, _stream()) == 0
        assert probe.ams_probe_resid_norm(_ptr(p), splits, M, d, _ptr(h), eps, _ptr(ur), _stream()) == 0
        out[M] = (un, ur, h)
        assert all(torch.equal(a, b[:M]) for a, b in zip(out[M], out[400])), M


@pytest.mark.parametrize("M", [1, 8, 9, 16, 17, 32, 33, 48, 64])
@pytest.mark.parametrize("N,K", [(96, 128), (416, 1152), (1024, 4096)])
@pytest.mark.parametrize("epi", [EPI_STORE, EPI_RESID, EPI_SWIGLU])
def test_tokens_short(probe, M, N, K, epi):  # noqa: F811
    """Passes of up to 64 tokens against the exact product, and bit for bit the GEMV on row-major weights."""
    import torch
    log(f"tokens_short epi={epi} M={M} N={N} K={K}")
    u, Wt = _rand((M, K), 121, M, K), _rand((N, K), 122, N, K, std=0.05)
    ldo = N // 2 if epi == EPI_SWIGLU else N
    h0 = W.random_gaussian((M, N), 123, M, dtype="f32")
    dt = torch.float16 if epi == EPI_SWIGLU else torch.float32
    a = torch.zeros((M, ldo), dtype=dt, device="cuda") if epi == EPI_SWIGLU else torch.from_numpy(h0.copy()).cuda()
    b = a.clone()
    ud = _dev(u, "f16")
    wd, wf = _dev(Wt, "f16"), _dev(_frag32(Wt), "f16")
    assert probe.ams_probe_gemm_tokens_short(epi, _ptr(ud), _ptr(wf), M, N, K, _ptr(a), ldo, _stream()) == 0
    assert probe.ams_probe_gemm(2, epi, _ptr(ud), None, _ptr(wd), M, N, K, _ptr(b), ldo, None, None,
                                _stream()) == 0
    assert torch.equal(a, b)
    y = _f(u, "f16") @ _f(Wt, "f16").T
    if epi == EPI_SWIGLU:
        g, up = _unpack_gu(y.T, N // 2)
        y = (_silu(g) * up).T
    elif epi == EPI_RESID:
        y = y + h0
    scale = max(1.0, float(np.max(np.abs(y))))
    tol = max(2e-5 * scale * np.sqrt(K / 64), 2 ** -11 * scale if epi == EPI_SWIGLU else 0.0)
    assert float(np.max(np.abs(a.double().cpu().numpy() - y))) <= tol
    assert probe.ams_probe_gemm_tokens_short(epi, _ptr(ud), _ptr(wf), 65, N, K, _ptr(a), ldo, _stream()) != 0
    assert probe.ams_probe_gemm_tokens_short(epi, _ptr(ud), _ptr(wf), M, N, K - 64, _ptr(a), ldo, _stream()) != 0

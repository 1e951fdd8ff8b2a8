"""Contexts whose workspace does not hold the partial sums of the preferred split counts, against the
fp64 reference: an fp32 residual projection that uses the scratch of u and qkv, wide decode GEMMs
with fewer splits, and a pass of 40 tokens that stays off the wide GEMM."""
import pytest

from paper_2508_10259_amd import workload as W
from gpu_util import ForcedRef, Pair, compare, gpu_new_tokens, log, small_spec
from test_gpu_rows import TOL_BF16, TOL_F32, _gpu, _prefix  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,H,F,lens,cap", [
    ("f32", 640, 10, 8192, (40,), 128),
    ("bf16", 640, 10, 1024, tuple(range(5, 17)), 64),
    ("bf16", 2048, 16, 2560, (40,), 64),
])
def test_small_workspace(dtype, d, H, F, lens, cap):
    from paper_2508_10259_amd.runtime import DeviceContext
    tol = TOL_F32 if dtype == "f32" else TOL_BF16
    spec = small_spec(dtype, 2, d, H, F)
    pair = Pair(spec, seed=41)
    B, A = len(lens), 3
    pre = [_prefix(spec, 41, 0, b, n) for b, n in enumerate(lens)]
    ctx = DeviceContext(pair.dev, B, cap)
    refs = [ForcedRef(pair.p, x) for x in pair.prefixes_f64(pre)]
    ctx.build(*pair.dev.pack_prefixes(pre))
    for s, n in enumerate((0, 18, 1)):
        new = [W.make_observation(spec, 41, 10 + s, b, n) for b in range(B)] if n else [None] * B
        t, nl = gpu_new_tokens(spec, new)
        if n:
            ctx.append(t, nl)
        tok, z = ctx.step(A)
        tok, z = tok.cpu().numpy(), z.cpu().numpy()
        for b in range(B):
            c = compare(refs[b].step(None if new[b] is None else pair.obs_f64(new[b]), tok[b]), z[b], tok[b], tol)
            log(f"{dtype} d={d} step {s} row {b}: max abs {c.max_abs:.2e}")
            assert c.max_abs <= tol and c.band == 1.0
    ctx.close()

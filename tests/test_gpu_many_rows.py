"""Contexts of more than 64 rows (the fp16 decode runs them in groups of at most 64), against the
fp64 reference: forced and free-running steps over ragged prefixes, with observation tokens between."""
import numpy as np
import pytest

from paper_2508_10259_amd import workload as W
from gpu_util import ForcedRef, Pair, compare, gpu_new_tokens, log, small_spec
from test_gpu_rows import TOL_BF16, TOL_F32, _gpu, _prefix  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,d,H,F", [
    ("bf16", 65, 256, 4, 512),    # two groups on the wide GEMMs
    ("bf16", 130, 512, 4, 1536),  # three groups, heads of 128
    ("bf16", 70, 384, 6, 1024),   # no workspace for the wide GEMMs' partial sums
    ("f32", 66, 256, 4, 512),     # one group
])
def test_many_rows(dtype, B, d, H, F):
    import torch
    from paper_2508_10259_amd.runtime import DeviceContext
    tol = TOL_F32 if dtype == "f32" else TOL_BF16
    spec = small_spec(dtype, 2, d, H, F)
    pair = Pair(spec, seed=51)
    A, lens = 3, [2 + (11 * b) % 29 for b in range(B)]
    pre = [_prefix(spec, 51, 0, b, n) for b, n in enumerate(lens)]
    ctx = DeviceContext(pair.dev, B, 64)
    refs = [ForcedRef(pair.p, x) for x in pair.prefixes_f64(pre)]
    ctx.build(*pair.dev.pack_prefixes(pre))
    for s in range(2):
        new = [W.make_observation(spec, 51, 10 + s, b, (b + s) % 3) if (b + s) % 3 else None for b in range(B)]
        t, nl = gpu_new_tokens(spec, new)
        fed = np.random.default_rng(s).integers(0, spec.n_bins, (B, A)).astype(np.int32) if s else None
        forced = torch.from_numpy(fed).cuda() if s else None
        tok, z = ctx.step(A, t, nl, forced=forced)
        tok, z = tok.cpu().numpy(), z.cpu().numpy()
        worst = 0.0
        for b in range(B):
            zr = refs[b].step(None if new[b] is None else pair.obs_f64(new[b]), tok[b] if fed is None else fed[b])
            c = compare(zr, z[b], tok[b], tol)
            worst = max(worst, c.max_abs)
            assert c.max_abs <= tol and c.band == 1.0, (s, b, c)
        log(f"{dtype} B={B} d={d} step {s}: max abs {worst:.2e}")
    ctx.close()

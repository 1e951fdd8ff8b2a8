"""fp16 token passes of at most 64 tokens on weights large enough for the wide GEMM (33 to 64
tokens; QKV and gate|up from 10 M weights, residual projections from 4 M), against the fp64
reference: builds and appends on both sides of its 32-token switch, and with a gate|up projection of
one split (SwiGLU from registers) and of two."""
import pytest

from paper_2508_10259_amd import workload as W
from gpu_util import ForcedRef, Pair, compare, gpu_new_tokens, log, small_spec
from test_gpu_rows import TOL_BF16, _gpu, _prefix  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [2560, 16384])
@pytest.mark.parametrize("lens,news", [((16,), (1, 13)), ((20, 44), (3, 8)), ((7, 9, 1), (5, 17))])
def test_short_passes(F, lens, news):
    from paper_2508_10259_amd.runtime import DeviceContext
    spec = small_spec("bf16", 1, 2048, 16, F)
    pair = Pair(spec, seed=31)
    B, A = len(lens), 3
    pre = [_prefix(spec, 31, 0, b, n) if n > 1 else
           W.Prefix(W.make_observation(spec, 31, 0, b, 1), W.np.zeros(0, W.np.int32)) for b, n in enumerate(lens)]
    prefix, plens = pair.dev.pack_prefixes(pre)
    ctx = DeviceContext(pair.dev, B, 128)
    refs = [ForcedRef(pair.p, x) for x in pair.prefixes_f64(pre)]
    ctx.build(prefix, plens)
    for s, n in enumerate((0,) + tuple(news)):
        new = [W.make_observation(spec, 31, 10 + s, b, n) for b in range(B)] if n else [None] * B
        t, nl = gpu_new_tokens(spec, new)
        if n:
            ctx.append(t, nl)
        tok, z = ctx.step(A)
        tok, z = tok.cpu().numpy(), z.cpu().numpy()
        for b in range(B):
            zr = refs[b].step(None if new[b] is None else pair.obs_f64(new[b]), tok[b])
            c = compare(zr, z[b], tok[b], TOL_BF16)
            log(f"F={F} lens={lens} step {s} row {b}: max abs {c.max_abs:.2e}")
            assert c.max_abs <= TOL_BF16 and c.band == 1.0


@pytest.mark.parametrize("d,H,F", [(4096, 32, 4224), (4224, 33, 256)])
def test_persistent_decode_widths(d, H, F):
    """The persistent decode on both sides of the width up to which it keeps a phase's activations
    in LDS, with one to three units of a phase per workgroup."""
    from paper_2508_10259_amd.runtime import DeviceContext
    spec = small_spec("bf16", 1, d, H, F)
    pair = Pair(spec, seed=33)
    B, A, lens = 3, 4, (9, 70, 33)
    pre = [_prefix(spec, 33, 0, b, n) for b, n in enumerate(lens)]
    prefix, plens = pair.dev.pack_prefixes(pre)
    ctx = DeviceContext(pair.dev, B, 128)
    assert ctx.persistent_decode
    refs = [ForcedRef(pair.p, x) for x in pair.prefixes_f64(pre)]
    ctx.build(prefix, plens)
    tok, z = ctx.step(A)
    tok, z = tok.cpu().numpy(), z.cpu().numpy()
    for b in range(B):
        c = compare(refs[b].step(None, tok[b]), z[b], tok[b], TOL_BF16)
        log(f"d={d} row {b}: max abs {c.max_abs:.2e}")
        assert c.max_abs <= TOL_BF16 and c.band == 1.0

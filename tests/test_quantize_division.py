"""The quantizer divides a weight by its group's scale as weight * (1 / scale) with two fused corrections.  For fp16 operands
the quotient must be the correctly rounded one: checked here for every pair of significands (powers of two only shift the
exponents, and neither quotient nor remainder leaves the normal range of binary32)."""
import numpy as np
import pytest


def _fma32(a, b, c):
    """float32 fused multiply-add of float32 arrays: the product of a 24-bit and an 11-bit (or 24-bit) significand and the
    sum below are formed in extended precision and rounded once."""
    wide = a.astype(np.longdouble) * b.astype(np.longdouble) + c.astype(np.longdouble)
    return wide.astype(np.float32)


def test_corrected_quotient_is_correctly_rounded():
    sig = np.arange(1024, 2048, dtype=np.float32)
    for s in sig:
        rcp = np.float32(1.0) / s
        a = sig
        q = (a * rcp).astype(np.float32)
        for _ in range(2):
            q = _fma32(_fma32(-q, np.full_like(a, s), a), np.full_like(a, rcp), q)
        assert np.array_equal(q, a / s), s


@pytest.mark.gpu
@pytest.mark.parametrize("bits,group,d,f", [(2, 64, 512, 1), (3, 32, 1024, 5), (4, 128, 512, 33), (8, 256, 1536, 3), (1, 32, 512, 7)])
def test_quantizer_over_the_range_of_fp16(bits, group, d, f):
    """Groups of every magnitude, some with infinities, ends of the matrix that fill no workgroup."""
    import floe_synth as S
    import gpu_common as G
    import oracle as O
    import paper_2505_05950_amd as F
    w = S.normal(S.stream_key(96, 50, S.KIND_MISC, bits), f * d).reshape(f, d // group, group)
    with np.errstate(over="ignore"):
        w = (w * np.exp2(np.arange(f * (d // group)) % 34 - 18.0).reshape(f, -1, 1)).reshape(f, d).astype(np.float16)
    codes, scale, zero = O.quantize(w, bits, group)
    gc, gs, gz = F.floe_quantize_expert(G.dev(w), bits, group)
    assert np.array_equal(G.host_u32(gc), codes)
    assert np.array_equal(gs.cpu().numpy().view(np.uint16), scale.view(np.uint16))
    assert np.array_equal(gz.cpu().numpy().view(np.uint16), zero.view(np.uint16))

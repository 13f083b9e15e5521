"""The rounding of the RoPE rotation, bit for bit, in every kernel family that
applies it.  With equal key and value weights the cache holds each rotated
pair (k) beside its inputs (v): exactly in fp32 models, and in bf16 ones whose
weight rows pick one normed element each, so that a projection is a bf16
value.  The rotation is then recomputed on the CPU:
lo = fma(x0, cos, -(x1 sin)), hi = fma(x1, cos, x0 sin); the integer kernels
of one weight tile per wave fuse the other product of hi."""
import math

import numpy as np
import pytest

from paper_2510_26843_amd import cas, synth

pytestmark = pytest.mark.gpu

S = synth.ModelShape
SHAPES = {
    # QKV rows below 8192 (K split over four waves), and above (one wave per K range: four tiles per workgroup)
    "f32": S("f32", 1, 64, 4, 4, 64, 64, 512, 1e4, 1e-6, "f32"),
    "f32_tall": S("f32_tall", 1, 64, 64, 64, 64, 64, 512, 1e4, 1e-6, "f32"),
    # 1044 tiles of 16 rows: six per workgroup, two per wave
    "f32_two": S("f32_two", 1, 64, 87, 87, 64, 64, 512, 1e4, 1e-6, "f32"),
    # 1216 tiles: eight per workgroup, or (int8) split evenly over workgroups of six one-tile waves
    "f32_even": S("f32_even", 1, 64, 152, 76, 64, 64, 512, 1e4, 1e-6, "f32"),
    "bf16": S("bf16", 1, 256, 20, 20, 128, 128, 512, 1e4, 1e-6, "bf16"),
    "bf16_tall": S("bf16_tall", 1, 256, 24, 24, 128, 128, 512, 1e4, 1e-6, "bf16"),
}


def _model(shape, max_ctx):
    w = synth.gen_weights(shape, seed=4)
    lw = w["layers"][0]
    if shape.dtype == "bf16":
        pick = np.zeros(shape.tensor_shape("wk"), dtype=np.uint16)
        pick[np.arange(len(pick)), np.random.default_rng(5).integers(0, shape.d_model, len(pick))] = 0x3f80
        lw["wk"] = lw["wv"] = pick
    else:
        lw["wv"] = lw["wk"]
    m = cas.Model(shape, max_ctx=max_ctx, max_tree=128)
    m.load_weights(w)
    return m


def _f32(a):
    return (a.astype(np.uint32) << 16).view(np.float32) if a.dtype == np.uint16 else a


def _fma(a, b, c):
    # the product of two floats is exact in 64 bits, the sum rounds once there and once here
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


def _check(shape, k, v, other, must_differ):
    """k, v [heads][slots][hd] of the cache; other: the other product of hi is fused."""
    half, n = shape.head_dim // 2, k.shape[1]
    inv = [math.pow(shape.rope_theta, -2.0 * i / shape.head_dim) for i in range(half)]
    ang = np.arange(n, dtype=np.float64)[:, None] * np.array(inv)
    cs, sn = np.cos(ang).astype(np.float32), np.sin(ang).astype(np.float32)
    x0, x1 = _f32(v)[..., :half], _f32(v)[..., half:]
    rnd = synth.f32_to_bf16_bits if shape.dtype == "bf16" else (lambda a: a)
    hi = [rnd(_fma(x1, cs, x0 * sn)), rnd(_fma(x0, sn, x1 * cs))]
    assert np.array_equal(k[..., :half], rnd(_fma(x0, cs, -(x1 * sn))))
    bad = np.argwhere(k[..., half:] != hi[other])
    assert len(bad) == 0, (len(bad), bad[:4])
    if must_differ:
        assert not np.array_equal(hi[0], hi[1])  # (the inputs tell the two apart)


def _fill(m, shape, n, T, quant):
    """KV of n slots from calls of T rows."""
    toks = [int(t) for t in synth.gen_prompt(shape.vocab, n, seed=6)]
    for i in range(0, n, T):
        part = toks[i:i + T]
        m.forward(part, synth.chain_parents(len(part)), act_quant=quant, logits=False)
        m.set_committed(i + len(part))
    return m.kv_read(0, n)


@pytest.mark.parametrize("name", ["f32", "f32_tall", "f32_two", "f32_even"])
@pytest.mark.parametrize("T,quant,gemv", [(T, q, False) for T in (1, 7, 33, 128) for q in (0, 1, 2)] + [(1, 1, True)])
def test_rotation_rounding_f32(name, T, quant, gemv):
    shape = SHAPES[name]
    m = _model(shape, 256)
    m.set_gemv(gemv)
    if quant == 1:
        m.build_int8()
    elif quant == 2:
        m.build_int4()
    k, v = _fill(m, shape, max(T, 9), T, quant)
    # two tiles per wave: the 1044 tiles; of 1216, int4's and the GEMV-style ones (no even split)
    two = name == "f32_two" or (name == "f32_even" and (quant == 2 or gemv))
    _check(shape, k, v, other=int(quant > 0 and not two), must_differ=True)
    m.close()


# (a bf16 element tells the two forms apart once in some 100 000)
@pytest.mark.parametrize("name", ["bf16", "bf16_tall"])
@pytest.mark.parametrize("T,n", [(1, 200), (16, 800), (32, 1600), (64, 1600), (128, 1600)])
def test_rotation_rounding_bf16(name, T, n):
    shape = SHAPES[name]
    m = _model(shape, n)
    k, v = _fill(m, shape, n, T, 0)
    _check(shape, k, v, other=0, must_differ=n == 1600)
    m.close()

"""Prefill of prompts longer than a tree against the same tokens committed
chunk by chunk through the verify forward (a chain of up to 128 nodes): the
committed KV of every layer, the logits the prefill leaves behind and the
next forward's logits hold the same bits, whatever the block and tile edges."""
import dataclasses
import gc

import numpy as np
import pytest
import torch  # (before the library: both then share one HIP runtime)

from paper_2510_26843_amd import cas, synth

S = synth.ModelShape
SHAPES = {
    # fp32; head width 64
    "f32": S("f32", 2, 256, 4, 4, 64, 688, 512, 1e4, 1e-6, "f32"),
    # bf16 grouped query, every matrix short: four K ranges (QKV, gate/up), 2 and 5 split-K sums, pad columns
    "gqa": S("gqa", 2, 512, 8, 2, 64, 1376, 512, 5e5, 1e-6, "bf16"),
    # head width 128; gate/up tall (one K range) with a tile count off the block edges; fewer chunks than ranges
    "tall": S("tall", 2, 256, 4, 2, 128, 4416, 512, 1e4, 1e-6, "bf16"),
    # tall QKV, rows of more than one block's tiles
    "mha": S("mha", 1, 1024, 24, 24, 128, 4448, 512, 1e4, 1e-6, "bf16"),
    # rows of more than 4096 elements in the norms
    "wide": S("wide", 1, 4608, 2, 2, 128, 512, 512, 1e4, 1e-6, "bf16"),
    # the matrices of the large models, narrow: short and tall QKV, gate/up and residual projections
    "big": S("big", 1, 256, 32, 8, 128, 14336, 512, 5e5, 1e-6, "bf16"),
    "bigq": S("bigq", 1, 256, 40, 40, 128, 13824, 512, 1e4, 1e-6, "bf16"),
    "bigd": S("bigd", 1, 8192, 2, 2, 64, 256, 512, 1e4, 1e-6, "bf16"),
    "mid": S("mid", 1, 1024, 12, 12, 128, 2752, 512, 1e4, 1e-6, "bf16"),
    # groups of query heads that do not divide the attention's four tiles
    "g3": S("g3", 1, 256, 6, 2, 128, 512, 512, 1e4, 1e-6, "bf16"),
    "g5": S("g5", 1, 256, 10, 2, 64, 512, 512, 1e4, 1e-6, "bf16"),
}
SHAPES.update({k + "_f32": dataclasses.replace(SHAPES[k], name=k + "_f32", dtype="f32")
               for k in ("big", "bigq", "bigd", "mid", "wide")})
LENGTHS = [(0, 129), (0, 256), (37, 411), (0, 1025), (100, 2300)]
# beside these, the lengths at which the large matrices take each block form
CASES = [(s, h, n) for s in ("f32", "gqa", "tall", "mha", "wide") for h, n in LENGTHS] + [
    (s + t, h, n) for t in ("", "_f32") for s, h, n in
    (("big", 37, 411), ("big", 0, 1025), ("bigq", 5, 411), ("bigq", 0, 1000), ("bigq", 0, 129), ("bigd", 0, 129),
     ("bigd", 0, 600), ("bigd", 3, 2048), ("mid", 0, 1025), ("mid", 0, 411))] + [
    ("wide_f32", 0, 1025), ("g3", 37, 411), ("g5", 37, 411), ("g5", 0, 1025)]


def _forms(shape, T):
    """(type, epilogue, block, K ranges, ranges apart) of a layer's linear layers over T rows."""
    wt = cas.W_BF16 if shape.dtype == "bf16" else cas.W_F32
    q, kv, d, f = shape.n_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim, shape.d_model, shape.ffn_dim
    for epi, N, K in (("qkv", q + 2 * kv, d), ("resid", d, q), ("gate/up", 2 * f, d), ("resid", d, f)):
        bn, bt, ranges, apart = cas.op_prefill_block(wt, N, K, T, epi == "resid")
        yield shape.dtype, epi, bn, bt, ranges > 1, bool(apart)


def test_cases_take_every_block_form():
    """Every form that k_gemm_rows is built in is among the cases compared below."""
    got = {f for s, _, n in CASES for b in range((n + 2047) // 2048)
           for f in _forms(SHAPES[s], n * (b + 1) // ((n + 2047) // 2048) - n * b // ((n + 2047) // 2048))}
    want = {(t, e, bn, bt, r, False) for t in ("bf16", "f32") for e in ("qkv", "gate/up", "resid")
            for bn, bt, r in ((64, 64, True), (128, 128, True), (128, 256, True), (128, 128, False), (128, 256, False),
                              (256, 256, False))}
    want |= {(t, "resid", 128, 128, True, True) for t in ("bf16", "f32")}
    assert got == want, (sorted(want - got), sorted(got - want))


def _model(shape, w, max_ctx):
    m = cas.Model(shape, max_ctx=max_ctx, max_tree=128)
    m.load_weights(w)
    return m


def _chunks(m, toks):
    for i in range(0, len(toks), 128):
        part = toks[i:i + 128]
        lg = m.forward(part, list(range(-1, len(part) - 1)))
        m.compact(list(range(len(part))))
    return lg


@pytest.mark.gpu
@pytest.mark.parametrize("name,head,n", CASES)
def test_long_prefill_matches_tree_chunks(name, head, n):
    shape = SHAPES[name]
    w = synth.gen_weights(shape, seed=3)
    toks = [int(x) for x in synth.gen_prompt(shape.vocab, head + n, seed=n)]
    ref, got = _model(shape, w, head + n + 128), _model(shape, w, head + n + 128)
    for m in (ref, got):
        if head:
            m.prefill(toks[:head])
    lg = _chunks(ref, toks[head:])
    got.prefill(toks[head:])
    assert got.committed == ref.committed == head + n
    ids, probs = got.topk(4, len(lg))  # the last chunk's logits stay readable
    order = np.argsort(-lg, axis=1, kind="stable")[:, :4]
    assert np.array_equal(ids, order)
    for l in range(shape.n_layers):
        for a, b in zip(got.kv_read(l, head + n), ref.kv_read(l, head + n)):
            assert np.array_equal(a, b), (l, np.argwhere(a != b)[:4])
    tree = synth.tree_from_branching(*synth.TREE_TINY)
    tt = synth.gen_tree_tokens(tree, shape.vocab, seed=9)
    assert np.array_equal(got.forward(tt, tree), ref.forward(tt, tree))
    ref.close()
    got.close()


def _free():
    gc.collect()  # (contexts that other tests left open)
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.gpu
def test_prefill_buffers_are_taken_by_the_first_long_prompt():
    # the blocks' buffers of this shape are 105 MB (2048 rows, widths 1024 and
    # 16384, eight split-K sums of 512 rows); the context's weights, their
    # staging, the KV cache of 4096 slots and the trees' buffers 180 MB
    shape = S("mem", 1, 1024, 8, 8, 128, 16384, 512, 1e4, 1e-6, "bf16")
    w = synth.gen_weights(shape, seed=3)
    prompt = synth.gen_prompt(shape.vocab, 2300, seed=1)
    m = _model(shape, w, 4096)
    m.prefill(prompt[:300])
    m.close()  # (the code is loaded, and the loads' staging is gone)
    free = _free()
    m = _model(shape, w, 4096)
    m.prefill(prompt[:128])
    held = _free()
    assert free - held < 240e6
    m.prefill(prompt[128:300])
    blocks = _free()
    assert 90e6 < held - blocks < 150e6
    m.set_committed(0)
    m.prefill(prompt)
    assert _free() == blocks  # kept, not taken again
    m.close()
    assert _free() >= held


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["f32", "gqa"])
@pytest.mark.parametrize("rows", [0, 511, 700, 1024])
def test_long_prefill_where_the_device_has_no_room(name, rows):
    """Smaller blocks, or tree chunks where not even those fit: the same bits."""
    shape = SHAPES[name]
    w = synth.gen_weights(shape, seed=3)
    prompt = synth.gen_prompt(shape.vocab, 2300, seed=1)
    ms = []
    for limit in (-1, rows):
        m = cas.Model(shape, max_ctx=2500, max_tree=128, debug=True)
        m.load_weights(w)
        m.debug_limit_prefill(limit)
        m.prefill(prompt)
        assert m.committed == 2300 and m.debug_check() == 0
        ms.append(m)
    a, b = ms
    for l in range(shape.n_layers):
        for x, y in zip(a.kv_read(l, 2300), b.kv_read(l, 2300)):
            assert np.array_equal(x, y)
    n = (2300 - 1) % 128 + 1
    for x, y in zip(a.topk(4, n), b.topk(4, n)):
        assert np.array_equal(x, y)
    a.close()
    b.close()


@pytest.mark.gpu
def test_long_prefill_refuses_what_it_refused():
    shape = SHAPES["f32"]
    m = cas.Model(shape, max_ctx=512, max_tree=64)
    with pytest.raises(cas.CasError):
        m.prefill([1] * 300)  # nothing loaded
    m.load_weights(synth.gen_weights(shape, seed=3))
    for bad in ([1] * 513, [1] * 200 + [shape.vocab], [-1] + [1] * 200):
        with pytest.raises(cas.CasError):
            m.prefill(bad)
        assert m.committed == 0
    m.prefill([1] * 300)
    assert m.committed == 300
    m.close()

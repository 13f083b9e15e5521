"""Timed workloads of the token-tree decoder through its Python binding.

A case is one of the calls that a decoding program makes again and again, on a
decoder of a few layers of one of the repository's shapes (every layer costs
the same, so two to eight of them stand for the whole depth):

- "forward": one forward over a token tree against a committed KV cache.  Full
  depth it is a verify call (T = 1: plain decoding); with odd layers skipped,
  quantised activations or an attention window it is a draft call, followed as
  in the decoding loops by the top-4 candidates of its rows.
- "ttft": time to first token: the prefill of a prompt into an empty cache and
  the first forward over T nodes after it.
- "round": one round of speculative decoding: the one-row skip draft of the
  root and its candidates, the verify of the tree, greedy acceptance, the KV
  commit and the rollback, as the benchmark's step.

Tokens, weights and the committed KV are random with the scales that the
repository's own synthetic inputs have (weights N(0, 0.02^2), k and v
N(0, 1.28^2)).
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2510_26843_amd import cas, synth

K_TOP = 4  # candidates a draft call asks for
MAX_TREE = 128

# Shapes of the tests beside the model shapes: a small grouped-query decoder
# with ragged widths (head width 64) and a small multi-head one.
SHAPES = dict(synth.SHAPES)
SHAPES["gqa_small"] = synth.ModelShape("gqa_small", 2, 512, 8, 2, 64, 1376, 1024, 5e5, 1e-6, "bf16")
SHAPES["mha_small"] = synth.ModelShape("mha_small", 2, 1024, 8, 8, 128, 2752, 4096, 1e4, 1e-6, "bf16")


def _case(kind, shape, layers, T, ctx, name=None, quant=0, skip=0, sink=0, window=0):
    c = {"kind": kind, "shape": shape, "layers": layers, "T": T, "ctx": ctx, "quant": quant, "skip": skip,
         "sink": sink, "window": window}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest calls: a round of the fp32 decoder of the static cascade,
        # where launches, small kernels and host work count
        _case("round", "tiny", 4, 15, 700, "tiny fp32 round"),
        # plain greedy decoding on the grouped-query shape, and as the
        # baseline step of every speculative run
        _case("forward", "llama3_8b", 4, 1, 4096, "8b decode"),
        # the benchmark's tree verify
        _case("forward", "llama2_7b", 4, 32, 1024, "7b verify 32"),
        # the largest tree of the latency sweep
        _case("forward", "llama2_7b", 4, 128, 2048, "7b verify 128"),
        # the grouped-query verify of the DyTC runs, at an odd tree size and context
        _case("forward", "llama3_8b", 4, 61, 4095, "8b verify 61"),
        # the 13B tree
        _case("forward", "llama2_13b", 2, 64, 2048, "13b verify 64"),
        # draft levels: int8 over a leaf with its siblings, int4 one node, and
        # a sink + window draft of a long context
        _case("forward", "llama2_13b", 4, 7, 2048, "13b draft int8", quant=1, skip=1),
        _case("forward", "llama2_13b", 4, 1, 2048, "13b draft int4", quant=2, skip=1),
        _case("forward", "llama2_7b", 4, 3, 8190, "7b draft window", skip=1, sink=4, window=1024),
        # prompts: the benchmark's 1024 tokens and a longer odd one
        _case("ttft", "llama2_7b", 4, 1, 1024, "7b first token 1024"),
        _case("ttft", "llama3_8b", 4, 16, 3001, "8b first token 3001"),
        # a whole round of the benchmark (8 of its 32 layers)
        _case("round", "llama2_7b", 8, 32, 1024, "7b round"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    shape = rng.choice(["tiny", "gqa_small", "mha_small", "llama2_7b", "llama2_7b", "llama2_13b", "llama3_8b",
                        "llama3_8b"])
    small = shape in ("tiny", "gqa_small", "mha_small")
    layers = {"tiny": 4, "gqa_small": 2, "mha_small": 2, "llama2_13b": 2}.get(shape, 4)
    kind = rng.choice(["forward", "forward", "draft", "draft", "ttft", "ttft", "round"])
    T = _log_int(rng, 1, 128)
    ctx = _log_int(rng, 33, 3001 if small else 8190)
    if kind == "ttft":
        return _case("ttft", shape, layers, min(T, 16), _log_int(rng, 17, 2999))
    if kind == "round":
        return _case("round", shape, layers, T, ctx)
    if kind == "forward":
        return _case("forward", shape, layers, T, ctx)
    T = _log_int(rng, 1, 16)  # a leaf with its siblings, or a tree level
    quant = rng.choice([0, 1, 2])
    window = rng.choice([0, 0, 256, 1024])
    return _case("forward", shape, layers, T, ctx, quant=quant, skip=1, sink=4 if window else 0, window=window)


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

def _shape(case):
    return SHAPES[case["shape"]].with_layers(case["layers"])


def _is_draft(case):
    return bool(case["quant"] or case["skip"] or case["window"])


def _skip(case):
    return [l % 2 for l in range(case["layers"])]


def _gen(seed, *what):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(np.random.SeedSequence([seed, *what]).generate_state(1, np.uint64)[0] >> 1))
    return g


def _normal(shape, rows_cols, std, g):
    x = torch.randn(rows_cols, generator=g, device="cuda", dtype=torch.float32) * std
    return x.to(torch.bfloat16) if shape.dtype == "bf16" else x


_CODES = {n: i for i, n in enumerate(("embed", "lm_head") + synth.LAYER_TENSORS)}


def _weight(shape, name, layer, seed):
    return _normal(shape, shape.tensor_shape(name), 0.02, _gen(seed, 1, layer + 1, _CODES[name]))


def _kv(shape, layer, n, seed):
    g = _gen(seed, 2, layer)
    dims = (shape.n_kv_heads, n, shape.head_dim)
    return _normal(shape, dims, 1.28, g), _normal(shape, dims, 1.28, g)


def _host(t):
    t = t.contiguous().cpu()
    return t.view(torch.int16).numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.numpy()


def _tree(case):
    if case["T"] == 15:
        return synth.tree_from_branching(*synth.TREE_TINY)
    if case["T"] == 32:
        return synth.tree_from_branching(*synth.TREE_7B)
    if case["T"] == 64:
        return synth.tree_from_branching(*synth.TREE_13B)
    if _is_draft(case) or case["T"] == 1:
        return [-1] + [0] * (case["T"] - 1)  # the root, or a leaf with its siblings
    return synth.balanced_tree(case["T"])


def _tokens(case, seed):
    shape, par = _shape(case), _tree(case)
    return synth.gen_tree_tokens(par, shape.vocab, seed=seed + 2), synth.gen_prompt(shape.vocab, case["ctx"], seed=seed + 1)


class _Logits:
    """A model's logits buffer as an array that torch can view.  The view's
    storage holds this object, and it the model, so the buffer outlives every
    tensor that shows it."""

    def __init__(self, model, rows, cols):
        self.model = model
        self.__cuda_array_interface__ = {"shape": (rows, cols), "typestr": "<f4",
                                         "data": (model.logits_device()[0], False), "version": 2}


_stream = None


def _one_stream():
    """One stream for every model, as a program has that decodes one sequence at a time."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def prepare(case, seed):
    shape = _shape(case)
    m = cas.Model(shape, max_ctx=case["ctx"] + MAX_TREE, max_tree=MAX_TREE, stream=_one_stream().cuda_stream)
    ones = np.ones(shape.d_model, dtype=np.float32)
    for n in ("embed", "lm_head"):
        m.load_tensor(n, 0, _host(_weight(shape, n, -1, seed)))
    m.load_tensor("final_norm", 0, ones)
    for l in range(shape.n_layers):
        for n in synth.LAYER_TENSORS:
            m.load_tensor(n, l, _host(_weight(shape, n, l, seed)))
        m.load_tensor("attn_norm", l, ones)
        m.load_tensor("ffn_norm", l, ones)
    if case["quant"] == 1:
        m.build_int8()
    elif case["quant"] == 2:
        m.build_int4()
    if case["kind"] != "ttft":
        for l in range(shape.n_layers):
            k, v = _kv(shape, l, case["ctx"], seed)
            m.kv_load(l, _host(k), _host(v))
        m.set_committed(case["ctx"])
    toks, prompt = _tokens(case, seed)
    logits = torch.as_tensor(_Logits(m, MAX_TREE, shape.vocab), device="cuda")
    return {"model": m, "case": case, "toks": toks, "par": np.asarray(_tree(case), dtype=np.int32), "prompt": prompt,
            "root": np.asarray([-1], dtype=np.int32), "skip": np.asarray(_skip(case), dtype=np.uint8), "logits": logits}


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------

def run(state):
    m, c, T = state["model"], state["case"], state["case"]["T"]
    if c["kind"] == "ttft":
        m.set_committed(0)
        m.prefill(state["prompt"])
        m.forward(state["toks"], state["par"], logits=False)
        return {"logits": state["logits"][:T]}
    if c["kind"] == "round":
        m.forward(state["toks"][:1], state["root"], skip=state["skip"], logits=False)
        _, probs = m.topk(K_TOP, 1)
        m.forward(state["toks"], state["par"], logits=False)
        path, _ = m.accept()
        m.compact(path)
        m.set_committed(c["ctx"])
        # (the accepted tokens follow the logits' argmax, and a near-tie among
        # random logits may fall either way: the logits stand for them)
        return {"logits": state["logits"][:T], "draft_probs": probs}
    if not _is_draft(c):
        m.forward(state["toks"], state["par"], logits=False)
        return {"logits": state["logits"][:T]}
    m.forward(state["toks"], state["par"], skip=state["skip"] if c["skip"] else None, act_quant=c["quant"],
              attn_window=(c["sink"], c["window"]) if c["window"] else None, logits=False)
    _, probs = m.topk(K_TOP, T)
    return {"logits": state["logits"][:T], "probs": probs}


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------

def _forward_work(case, T, ctx, layers, quant=0, window=None, head_rows=None):
    s = _shape(case)
    es = 2 if s.dtype == "bf16" else 4
    head_rows = T if head_rows is None else head_rows
    kv = s.n_kv_heads * s.head_dim
    q = s.n_heads * s.head_dim
    seen = min(ctx, window[0] + window[1]) if window and window[1] else ctx
    wbytes = s.layer_params() * es
    if quant:
        wbytes = s.layer_params() // (2 if quant == 2 else 1) + 4 * (q + 2 * kv + 2 * s.d_model + 2 * s.ffn_dim)
    b = layers * (wbytes + 2 * kv * es * (seen + T)) + T * s.d_model * es
    b += s.vocab * s.d_model * es + head_rows * s.vocab * 4
    flops = 2.0 * T * layers * s.layer_params() + 2.0 * head_rows * s.vocab * s.d_model
    flops += 4.0 * T * layers * q * (seen + (T + 1) / 2)
    return b, flops


def work(case):
    T, ctx, L = case["T"], case["ctx"], case["layers"]
    run_layers = L - sum(_skip(case)) if case["skip"] else L
    if case["kind"] == "ttft":
        parts = [_forward_work(case, ctx, 0, L, head_rows=0), _forward_work(case, T, ctx, L)]
    elif case["kind"] == "round":
        parts = [_forward_work(case, 1, ctx, L - sum(_skip(case))), _forward_work(case, T, ctx, L)]
    else:
        parts = [_forward_work(case, T, ctx, run_layers, case["quant"], (case["sink"], case["window"]))]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    # measured against exact(): fp32 up to 8e-7 of the logits' norm; bf16
    # 0.9e-2 to 1.1e-2 over two to four layers, 1.5e-2 where the KV cache comes
    # from a prefill of the same model or over eight layers.  Two roundings of
    # one sum are that far apart; the quantised drafts move in steps of a code
    if case["shape"] == "tiny":
        return {"rel": 1e-2 if case["quant"] else 4e-6}
    return {"rel": 3e-2 if case["kind"] != "forward" or case["quant"] else 2e-2}


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------

def _quant(x, qmax):
    s = x.abs().amax(dim=-1, keepdim=True) / qmax
    return torch.where(s > 0, torch.clamp(torch.round(x / s), -qmax, qmax), torch.zeros_like(x)) * s


class _Exact:
    def __init__(self, case, seed):
        self.case, self.seed, self.s = case, seed, _shape(case)
        self.kv = [None] * self.s.n_layers

    def weight(self, name, layer, qmax=0):
        w = _weight(self.s, name, layer, self.seed).double()
        return _quant(w, qmax) if qmax else w

    def norm(self, h):
        return h / torch.sqrt((h * h).mean(-1, keepdim=True) + self.s.rms_eps)

    def rope(self, x, pos):  # x [T][heads][hd]
        half = self.s.head_dim // 2
        inv = self.s.rope_theta ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / self.s.head_dim)
        a = pos.double()[:, None, None] * inv
        x0, x1 = x[..., :half], x[..., half:]
        return torch.cat([x0 * a.cos() - x1 * a.sin(), x0 * a.sin() + x1 * a.cos()], dim=-1)

    def forward(self, toks, pos, vis, skip=None, quant=0, head=True, keep=False):
        """toks [T]; pos [T]; vis [T][slots + T] bool over the committed slots and the call's rows."""
        s, T = self.s, len(toks)
        qmax = {0: 0, 1: 127, 2: 7}[quant]
        lin = lambda x, n, l: (_quant(x, qmax) if qmax else x) @ self.weight(n, l, qmax).T  # noqa: E731
        h = self.weight("embed", -1)[torch.as_tensor(np.asarray(toks), device="cuda").long()]
        for l in range(s.n_layers):
            if skip is not None and skip[l]:
                continue
            x = self.norm(h)
            q = self.rope(lin(x, "wq", l).view(T, s.n_heads, s.head_dim), pos)
            k = self.rope(lin(x, "wk", l).view(T, s.n_kv_heads, s.head_dim), pos).transpose(0, 1)
            v = lin(x, "wv", l).view(T, s.n_kv_heads, s.head_dim).transpose(0, 1)
            if self.kv[l] is not None:
                k, v = torch.cat([self.kv[l][0], k], 1), torch.cat([self.kv[l][1], v], 1)
            out = torch.empty(T, s.n_heads, s.head_dim, device="cuda", dtype=torch.float64)
            G = s.n_heads // s.n_kv_heads
            for hh in range(s.n_heads):
                sc = q[:, hh] @ k[hh // G].T / math.sqrt(s.head_dim)
                out[:, hh] = torch.softmax(sc.masked_fill(~vis, -math.inf), dim=-1) @ v[hh // G]
            if keep:
                self.kv[l] = (k, v)
            h = h + lin(out.reshape(T, -1), "wo", l)
            x = self.norm(h)
            h = h + lin(torch.nn.functional.silu(lin(x, "w_gate", l)) * lin(x, "w_up", l), "w_down", l)
        return self.norm(h) @ self.weight("lm_head", -1).T if head else None


def exact(case, seed):
    if case["quant"] == 2:
        # one code of the 4-bit grid is a seventh of a row's largest value, so
        # the last bit of an activation decides over much of an output: no
        # value in more bits is nearer than another
        return None
    shape, T, ctx = _shape(case), case["T"], case["ctx"]
    toks, prompt = _tokens(case, seed)
    par = _tree(case)
    e = _Exact(case, seed)
    if case["kind"] == "ttft":
        tri = torch.ones(ctx, ctx, dtype=torch.bool, device="cuda").tril()
        e.forward(prompt, torch.arange(ctx, device="cuda"), tri, head=False, keep=True)
    else:
        e.kv = [tuple(x.double() for x in _kv(shape, l, ctx, seed)) for l in range(shape.n_layers)]
    depth, anc = np.zeros(T, dtype=np.int64), np.zeros((T, T), dtype=bool)
    for i, p in enumerate(par):
        if p >= 0:
            depth[i], anc[i] = depth[p] + 1, anc[p]
        anc[i, i] = True
    seen = np.ones(ctx, dtype=bool)
    if case["window"]:
        seen = (np.arange(ctx) < case["sink"]) | (np.arange(ctx) >= ctx - case["window"])
    vis = torch.as_tensor(np.concatenate([np.broadcast_to(seen, (T, ctx)), anc], axis=1), device="cuda")
    pos = torch.as_tensor(ctx + depth, device="cuda")
    top = lambda lg: torch.softmax(lg, -1).topk(K_TOP, -1).values  # noqa: E731
    if case["kind"] == "round":
        draft = e.forward(toks[:1], pos[:1], vis[:1, :ctx + 1], skip=_skip(case))
        return {"logits": e.forward(toks, pos, vis), "draft_probs": top(draft)}
    if case["kind"] == "ttft" or not _is_draft(case):
        return {"logits": e.forward(toks, pos, vis)}
    lg = e.forward(toks, pos, vis, skip=_skip(case) if case["skip"] else None, quant=case["quant"])
    return {"logits": lg, "probs": top(lg)}

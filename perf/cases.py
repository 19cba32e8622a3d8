"""Performance cases of the draft-tree verification library: what a serving or training program has it do.

Every case is one call pattern through the public entry points (`paper_2605_11186_amd`), at shapes that the
benchmark and the tests of this repository use: whole verify steps from the smallest to the largest tree and
context, plain decoding, the stage-1 draft loop, a staged cascaded cycle, tree attention alone, weights
streamed from host memory, and the adapter-training loss.  `draw` gives more cases of the same ranges.

Weights are N(0, 0.02), gains 1 + N(0, 0.02), committed K/V rows N(0, 1), token ids uniform with distinct
siblings: the distributions of the benchmark's inputs.
"""
import math
import random

import numpy as np
import torch

import paper_2605_11186_amd as cats

# layers, hidden, heads, head_dim, ffn, vocab
SHAPES = {
    "tiny": (2, 256, 4, 64, 688, 1024),
    "7b": (32, 4096, 32, 128, 11008, 32000),
    "13b": (40, 5120, 40, 128, 13824, 32000),
}
RMS_EPS, ROPE_BASE = 1e-6, 10000.0


def listed():
    return [
        # a small model's whole step, 15-node binary-sized tree: launch latency and host work
        dict(name="tiny_t15_s128", kind="verify", shape="tiny", layers=2, nodes=15, max_depth=3, ctx=128, packed=True),
        # a caller with its own layer code: the tree-masked attention of one 7B layer over a long context
        dict(name="attention_7b_t64_s4096", kind="attention", heads=32, head_dim=128, nodes=64, max_depth=8, ctx=4096),
        # plain greedy decoding (root-only tree), one token with its read-back: the baseline of speculation
        dict(name="decode_7b_s1024", kind="decode", shape="7b", layers=32, ctx=1024, packed=True),
        # stage 1 of the cascaded cycle: five draft tokens through two layers, adapter and shared LM head
        dict(name="draft_7b_g5_s1024", kind="draft", shape="7b", layers=2, gamma=5, ctx=1024, packed=True),
        # stages 2 and 3 of one cycle: chain, then corrections, through 8 shallow layers; the rest on the tree
        dict(name="cascade_7b_g5_s1024", kind="cascade", shape="7b", layers=32, shallow=8, gamma=5, corrections=2, ctx=1024, packed=True),
        # the sweep's smallest tree and context
        dict(name="verify_7b_t16_s512", kind="verify", shape="7b", layers=32, nodes=16, max_depth=8, ctx=512, packed=True),
        # the headline step: 63-node tree behind 1024 tokens
        dict(name="verify_7b_t63_s1024", kind="verify", shape="7b", layers=32, nodes=63, max_depth=6, ctx=1024, packed=True),
        # the sweep's largest tree and context
        dict(name="verify_7b_t128_s4096", kind="verify", shape="7b", layers=32, nodes=128, max_depth=8, ctx=4096, packed=True),
        # the larger model's step
        dict(name="verify_13b_t64_s2048", kind="verify", shape="13b", layers=40, nodes=64, max_depth=7, ctx=2048, packed=True),
        # weights used as the checkpoint holds them (row-major), ragged sizes, typical acceptance that
        # accepts whole paths (so that the cache is rolled back along one)
        dict(name="rowmajor_7b_t33_s1000", kind="verify", shape="7b", layers=8, nodes=33, max_depth=5, ctx=1000, packed=False, typical=True),
        # offload regime: layer weights in pinned host memory, four of the layers
        dict(name="streamed_7b_t128_s1024", kind="streamed", shape="7b", layers=4, nodes=128, max_depth=8, ctx=1024, packed=True),
        # adapter training: loss and gradient of a batch of positions, a tenth of them masked
        dict(name="loss_p4096_v32000_k10", kind="loss", positions=4096, vocab=32000, top_k=10, grad=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "verify", "attention", "decode", "draft", "cascade", "streamed", "loss"])
    if kind == "loss":
        return dict(kind=kind, positions=_log_int(rng, 64, 4096), vocab=4 * _log_int(rng, 250, 8000),
                    top_k=rng.choice([1, 5, 10, 20, 50]), grad=rng.random() < 0.75)
    if kind == "attention":
        d = rng.choice([64, 128])
        return dict(kind=kind, heads=rng.choice([4, 8, 16, 32, 40]), head_dim=d, nodes=_log_int(rng, 1, 128),
                    max_depth=rng.randint(2, 16), ctx=_log_int(rng, 64, 4096))
    shape = rng.choice(["tiny", "7b", "7b", "7b", "13b"])
    packed = rng.random() < 0.75
    ctx = _log_int(rng, 32, 4096)
    if kind == "verify":
        nodes = _log_int(rng, 2, 128)
        most = {"tiny": 2, "7b": 32, "13b": 40 if nodes <= 64 and ctx <= 2048 else 24}[shape]
        c = dict(kind=kind, shape=shape, layers=_log_int(rng, min(4, most), most), nodes=nodes,
                 max_depth=rng.randint(2, 16), ctx=ctx, packed=packed)
        if rng.random() < 0.25:
            c["typical"] = True
        return c
    if kind == "decode":
        return dict(kind=kind, shape=shape, layers=2 if shape == "tiny" else _log_int(rng, 4, 32), ctx=ctx, packed=packed)
    gamma = rng.randint(2, 12)
    if kind == "draft":
        return dict(kind=kind, shape=shape, layers=rng.randint(1, 2 if shape == "tiny" else 4), gamma=gamma, ctx=ctx, packed=packed)
    if kind == "cascade":
        layers = 2 if shape == "tiny" else _log_int(rng, 6, 32)
        return dict(kind=kind, shape=shape, layers=layers, shallow=max(1, layers // 4), gamma=gamma,
                    corrections=rng.randint(1, gamma), ctx=ctx, packed=packed)
    shape = rng.choice(["tiny", "7b"])
    return dict(kind="streamed", shape=shape, layers=2 if shape == "tiny" else rng.randint(2, 4), nodes=_log_int(rng, 2, 128),
                max_depth=rng.randint(2, 16), ctx=ctx, packed=True)


# ---------------------------------------------------------------- inputs
def _normal(gen, shape, std, mean=0.0):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(mean, std, generator=gen)


def _tree(rng, nodes, max_depth):
    """Random parents (uniform over the earlier nodes above the depth cap), as the sweep's trees."""
    parent, depth = [-1], [0]
    for _ in range(1, nodes):
        p = rng.choice([j for j in range(len(parent)) if depth[j] < max_depth])
        parent.append(p)
        depth.append(depth[p] + 1)
    return np.array(parent, np.int32), np.array(depth, np.int32)


def _tokens(rng, parent, vocab):
    used, out = {}, []
    for p in parent:
        seen = used.setdefault(int(p), set())
        t = rng.randrange(vocab)
        while t in seen:
            t = rng.randrange(vocab)
        seen.add(t)
        out.append(t)
    return np.array(out, np.int32)


def _layer(gen, hidden, ffn, packed, adapter=False):
    shapes = {"wq": (hidden, hidden), "wk": (hidden, hidden), "wv": (hidden, hidden), "wo": (hidden, hidden)}
    gains = ["g_attn"]
    if not adapter:
        shapes.update(w_gate=(ffn, hidden), w_up=(ffn, hidden), w_down=(hidden, ffn))
        gains.append("g_ffn")
    w = {k: _normal(gen, s, 0.02) for k, s in shapes.items()}
    w.update({k: _normal(gen, (hidden,), 0.02, 1.0) for k in gains})
    if packed:
        w = {k: cats.cats_pack_matrix(v) if v.dim() == 2 else v for k, v in w.items()}
    return w


def _caches(gen, layers, heads, head_dim, max_ctx, ctx):
    """Keys [layers][heads][max_ctx][head_dim] and transposed values, committed rows N(0, 1), the rest zero."""
    k = torch.zeros(layers, heads, max_ctx, head_dim, dtype=torch.bfloat16, device="cuda")
    v = torch.zeros(layers, heads, head_dim, max_ctx, dtype=torch.bfloat16, device="cuda")
    k[:, :, :ctx] = _normal(gen, (layers, heads, ctx, head_dim), 1.0)
    v[..., :ctx] = _normal(gen, (layers, heads, head_dim, ctx), 1.0)
    return k, v


def _nodes(case):
    if case["kind"] == "decode":
        return 1
    if case["kind"] == "draft":
        return case["gamma"] + 1
    if case["kind"] == "cascade":
        return 1 + case["gamma"] + case["corrections"]
    return case["nodes"]


class State:
    """What the caller's program holds between steps; releases the library's context with itself."""

    ctx = None

    def __del__(self):
        if self.ctx is not None:
            torch.cuda.synchronize()
            cats.cats_destroy(self.ctx)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = random.Random(seed)
    s = State()
    s.case, kind = case, case["kind"]
    if kind == "loss":
        # rows as a language model's head gives them: a normal bulk and a few boosted tokens
        P, V = case["positions"], case["vocab"]
        rows = []
        for _ in range(2):
            z = torch.empty(P, V, device="cuda").normal_(0.0, 2.5, generator=gen)
            boosted = torch.randint(0, V, (P, 8), device="cuda", generator=gen)
            z.scatter_add_(1, boosted, torch.empty(P, 8, device="cuda").uniform_(2.0, 12.0, generator=gen))
            rows.append(z)
        s.target, s.draft = rows
        s.mask = (torch.rand(P, device="cuda", generator=gen) < 0.9).to(torch.uint8)
        s.loss = torch.zeros(1, device="cuda")
        s.per_pos = torch.zeros(P, device="cuda")
        s.topk = torch.zeros(P, case["top_k"], dtype=torch.int32, device="cuda")
        s.grad = torch.zeros(P, V, device="cuda") if case["grad"] else None
        return s

    T, S = _nodes(case), case["ctx"]
    s.max_ctx = (S + T + 63) // 64 * 64
    if kind == "attention":
        nh, d = case["heads"], case["head_dim"]
        s.k, s.v = (c[0] for c in _caches(gen, 1, nh, d, s.max_ctx, S + T))
        s.kv = cats.KVLayer(s.k.data_ptr(), s.v.data_ptr())
        s.q = _normal(gen, (T, nh * d), 1.0)
        s.out = torch.zeros_like(s.q)
        parent, depth = _tree(rng, T, case["max_depth"])
        s.ctx = cats.cats_create(cats.ModelDesc(1, nh * d, nh, d, 64, 64, s.max_ctx, T, RMS_EPS, ROPE_BASE, 0))
        s.tree = np.zeros(T, np.int32), parent, depth   # token ids play no part here
        return s

    _, H, nh, d, F, V = SHAPES[case["shape"]]
    L, packed = case["layers"], case["packed"]
    layers = []
    for _ in range(L):
        w = _layer(gen, H, F, packed)
        if kind == "streamed":   # the weights live in pinned host memory
            host = {n: torch.empty(t.shape, dtype=t.dtype, pin_memory=True) for n, t in w.items()}
            for n, t in w.items():
                host[n].copy_(t)
            w = host
        layers.append(w)
    s.layers, s.layers_arr = layers, cats.layer_array(layers)
    s.embed = _normal(gen, (V, H), 0.02)
    s.g_final = _normal(gen, (H,), 0.02, 1.0)
    w_lm = _normal(gen, (V, H), 0.02)
    s.w_lm = cats.cats_pack_matrix(w_lm) if packed else w_lm
    s.k, s.v = _caches(gen, L, nh, d, s.max_ctx, S)
    s.kv = cats.kv_array(list(s.k), list(s.v))
    desc = cats.ModelDesc(L, H, nh, d, F, V, s.max_ctx, T, RMS_EPS, ROPE_BASE, int(packed))
    s.ctx = cats.cats_create(desc)
    s.result = cats.accept_result_tensor()
    s.logits = torch.zeros(T, V, device="cuda")
    s.argmax = torch.zeros(T, dtype=torch.int32, device="cuda")
    s.hidden = torch.zeros(T, H, device="cuda")
    if kind in ("verify", "streamed"):
        parent, depth = _tree(rng, T, case["max_depth"])
        s.tree = _tokens(rng, parent, V), parent, depth
        if case.get("typical"):
            cats.cats_set_acceptance(s.ctx, 1, 1e-12, 0.3, 1.0)
        if kind == "streamed":
            n = cats.cats_layer_weight_bytes(desc)
            s.staging = [torch.empty(n, dtype=torch.uint8, device="cuda") for _ in range(2)]
    elif kind == "decode":
        s.tree = np.array([rng.randrange(V)], np.int32), np.array([-1], np.int32), np.array([0], np.int32)
        s.host = cats.AcceptResult()
    elif kind == "draft":
        s.adapter = _layer(gen, H, F, packed, adapter=True)
        s.adapter_arr = cats.layer_array([s.adapter])
        s.g_adapter = _normal(gen, (H,), 0.02, 1.0)
        s.ka, s.va = _caches(gen, 1, nh, d, s.max_ctx, S)
        s.kv_adapter = cats.kv_array(list(s.ka), list(s.va))
        s.root = rng.randrange(V)
        s.tokens = torch.zeros(T, dtype=torch.int32, device="cuda")
    else:   # cascade
        g = case["gamma"]
        s.root = rng.randrange(V)
        s.main = [rng.randrange(V) for _ in range(g)]
        s.corr = [-1] * g
        for i in rng.sample(range(g), case["corrections"]):
            s.corr[i] = (s.main[i] + rng.randrange(1, V)) % V
        s.h_shallow = torch.zeros(T, H, device="cuda")
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    case, kind = s.case, s.case["kind"]
    stream = torch.cuda.current_stream()
    if kind == "loss":
        cats.cats_reduced_kl_loss(s.target, s.draft, case["top_k"], s.loss, s.per_pos, mask=s.mask,
                                  topk_idx_out=s.topk, grad_out=s.grad, stream=stream)
        return [s.loss, s.per_pos, s.topk] + ([s.grad] if s.grad is not None else [])
    S = case["ctx"]
    if kind == "attention":
        cats.cats_set_tree(s.ctx, *s.tree, stream)
        cats.cats_tree_attention(s.ctx, s.q, s.kv, S, s.out, stream)
        return [s.out]
    L = case["layers"]
    if kind == "draft":
        cats.cats_draft_chain(s.ctx, s.layers_arr, 0, L, s.adapter_arr, s.g_adapter, s.w_lm, s.embed, s.kv,
                              s.kv_adapter, S, s.root, case["gamma"], s.tokens, hidden_out=s.hidden, stream=stream)
        return [s.tokens, s.hidden, s.k, s.v, s.ka, s.va]
    if kind == "cascade":
        g, sv = case["gamma"], case["shallow"]
        tok, parent, depth, _ = cats.cats_build_tree(s.root, s.main)
        cats.cats_set_tree(s.ctx, tok, parent, depth, stream)
        cats.cats_verify_nodes(s.ctx, s.layers_arr, 0, sv, s.embed, None, s.kv, S, 0, s.h_shallow[: g + 1], stream)
        tok, parent, depth, _ = cats.cats_build_tree(s.root, s.main, s.corr)
        cats.cats_set_tree(s.ctx, tok, parent, depth, stream)
        cats.cats_verify_nodes(s.ctx, s.layers_arr, 0, sv, s.embed, None, s.kv, S, g + 1, s.h_shallow[g + 1:], stream)
        cats.cats_verify_tree(s.ctx, s.layers_arr, sv, L, None, s.h_shallow, s.g_final, s.w_lm, s.kv, S, s.result,
                              hidden_out=s.hidden, logits_out=s.logits, argmax_out=s.argmax, stream=stream)
        cats.cats_accept_and_compact(s.ctx, s.argmax, s.kv, 0, sv, S, s.result, stream=stream)
        return [s.h_shallow, s.hidden, s.logits, s.argmax, s.result, s.k, s.v]
    cats.cats_set_tree(s.ctx, *s.tree, stream)
    if kind == "streamed":
        cats.cats_verify_tree_streamed(s.ctx, s.layers_arr, 0, L, s.staging, s.embed, None, s.g_final, s.w_lm, s.kv, S,
                                       s.result, hidden_out=s.hidden, logits_out=s.logits, argmax_out=s.argmax, stream=stream)
    else:   # a decoding program waits for its token; a verify step's result stays on the device
        cats.cats_verify_tree(s.ctx, s.layers_arr, 0, L, s.embed, None, s.g_final, s.w_lm, s.kv, S, s.result,
                              hidden_out=s.hidden, logits_out=s.logits, argmax_out=s.argmax,
                              out_host=s.host if kind == "decode" else None, stream=stream)
    return [s.hidden, s.logits, s.argmax, s.result, s.k, s.v]


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "loss":
        P, V = case["positions"], case["vocab"]
        return {"bytes": 4 * P * V * (3 if case["grad"] else 2), "flops": 8 * P * V}
    T, S = _nodes(case), case["ctx"]
    if kind == "attention":
        H = case["heads"] * case["head_dim"]
        return {"bytes": 4 * (S + T) * H + 4 * T * H, "flops": 4 * T * (S + T) * H}
    _, H, nh, d, F, V = SHAPES[case["shape"]]
    L = case["layers"]
    layer, attn_only, head = 4 * H * H + 3 * F * H, 4 * H * H, V * H

    def rows(n, k_layers):   # n rows of one pass through k_layers layers: context and own rows read, own rows written
        return (4 * (S + n) * H + 4 * n * H) * k_layers

    def att(n, k_layers):
        return 4 * n * (S + n) * H * k_layers

    if kind == "draft":
        g = case["gamma"]
        w = (g + 1) * L * layer + g * (attn_only + head)
        return {"bytes": 2 * w + (g + 1) * rows(1, L) + g * rows(1, 1) + 4 * (g + 1) * H, "flops": 2 * w + (g + 1) * att(1, L) + g * att(1, 1)}
    if kind == "cascade":
        g, c, sv = case["gamma"], case["corrections"], case["shallow"]
        w_shallow, w_rest = sv * layer, (L - sv) * layer
        flops = 2 * ((g + 1) + c) * w_shallow + 2 * T * (w_rest + head) + att(g + 1, sv) + att(c, sv) + att(T, L - sv)
        return {"bytes": 2 * (2 * w_shallow + w_rest + head) + rows(g + 1, sv) + rows(c, sv) + rows(T, L - sv) + 4 * T * (V + 2 * H), "flops": flops}
    w = L * layer + head
    return {"bytes": 2 * w + rows(T, L) + 4 * T * (V + H) + 2 * T * H, "flops": 2 * T * w + att(T, L)}


def tolerance(case):
    """About four times what another order of the same sums changes, measured by verifying the first half of a
    tree alone (another split of the products): float32 outputs 5e-5, bf16 cache rows 3.5e-4 (one unit in the
    last place, 2^-8 of the value at most, where the two values straddle a rounding boundary).  The attention
    output is one bf16 rounding (1.7e-3 against float32); the loss is float32 sums with hardware exponentials."""
    kind = case["kind"]
    if kind == "loss":
        return {"rel": 1e-5, "differ": 0.001}
    if kind == "attention":
        return {"rel": 4e-3, "max": 0.016}
    return {"rel": 1.4e-3, "max": 0.032, "differ": 0.01}

"""Tree attention where a wave walks several key blocks: enough heads that a chunk is long, contexts that end
inside and on a block, one to four query groups, both head sizes, against float64 attention."""
import numpy as np
import pytest
import torch

import paper_2605_11186_amd as cats
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,d,T,S", [(32, 128, 128, 1025), (40, 128, 33, 2048), (64, 64, 64, 1311), (64, 128, 96, 511),
                                         (64, 64, 2, 2047), (16, 128, 100, 0)])
def test_long_chunks(heads, d, T, S):
    gen = torch.Generator(device="cuda").manual_seed(7 * T + S)
    H, max_ctx = heads * d, (S + T + 63) // 64 * 64
    normal = lambda *s: torch.empty(*s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, k, v = normal(T, H), normal(heads, max_ctx, d), normal(heads, d, max_ctx)
    k[:, S + T:] = float("nan")      # rows past the tree must not be seen
    v[..., S + T:] = float("nan")
    parent, depth = synth.random_tree(T, 8, T)
    ctx = cats.cats_create(cats.ModelDesc(1, H, heads, d, 64, 64, max_ctx, T, 1e-6, 10000.0, 0))
    try:
        out = torch.zeros_like(q)
        cats.cats_set_tree(ctx, np.zeros(T, np.int32), parent, depth, torch.cuda.current_stream())
        cats.cats_tree_attention(ctx, q, cats.KVLayer(k.data_ptr(), v.data_ptr()), S, out, torch.cuda.current_stream())
        got = out.cpu().double()
    finally:
        torch.cuda.synchronize()
        cats.cats_destroy(ctx)
    see = torch.zeros(T, S + T, dtype=torch.bool)
    see[:, :S] = True
    for i in range(T):
        j = i
        while j >= 0:
            see[i, S + j] = True
            j = int(parent[j])
    qd = q.cpu().double().view(T, heads, d).transpose(0, 1)
    kd, vd = k.cpu().double()[:, : S + T], v.cpu().double()[..., : S + T]
    p = (qd @ kd.transpose(1, 2) / d ** 0.5).masked_fill(~see, -np.inf).softmax(-1)
    ref = (p @ vd.transpose(1, 2)).transpose(0, 1).reshape(T, H)
    # one bf16 rounding of the output (2^-9 of each entry), everything before it at 16 bits or more
    assert torch.isfinite(got).all()
    assert float((got - ref).norm() / ref.norm()) <= 2.0 ** -9

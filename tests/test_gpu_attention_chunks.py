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


def _one_head(d, max_ctx, k_rows):
    """One head's zeroed keys and values of which only the first k_rows rows are ever visible."""
    k = torch.empty(1, max_ctx, d, dtype=torch.bfloat16, device="cuda")
    v = torch.empty(1, d, max_ctx, dtype=torch.bfloat16, device="cuda")
    k[:, :k_rows] = 0
    v[..., :k_rows] = 0
    return k, v


def _attend_to_one_row_each(d, max_ctx, S, rows):
    """Query t matches the key of row rows[t] alone (its score is about 8 sqrt(d), all others stay below half
    of it), so that the output is that row's value."""
    T = len(rows)
    gen = torch.Generator(device="cuda").manual_seed(d)
    k, v = _one_head(d, max_ctx, S + T)
    q = torch.empty(T, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    want = torch.empty(T, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    for t, r in enumerate(rows):
        k[0, r] = 8 * q[t]
        v[0, :, r] = want[t]
    ctx = cats.cats_create(cats.ModelDesc(1, d, 1, d, 64, 64, max_ctx, T, 1e-6, 10000.0, 0))
    try:
        out = torch.zeros_like(q)
        parent = np.arange(T, dtype=np.int32) - 1
        cats.cats_set_tree(ctx, np.zeros(T, np.int32), parent, np.arange(T, dtype=np.int32), torch.cuda.current_stream())
        cats.cats_tree_attention(ctx, q, cats.KVLayer(k.data_ptr(), v.data_ptr()), S, out, torch.cuda.current_stream())
        torch.cuda.synchronize()
    finally:
        cats.cats_destroy(ctx)
    assert torch.equal(out, want)


@pytest.mark.parametrize("d", [128, 64])
def test_keys_past_32_bit_element_offsets(d):
    """Rows on both sides of the one whose first element is number 2^32 of its head, and the last one."""
    first = 2 ** 32 // d
    S = first + 100
    _attend_to_one_row_each(d, (S + 4 + 63) // 64 * 64, S, [first - 1, first, first + 1, S - 1])


def test_value_rows_past_32_bit_element_offsets():
    """A cache so wide that dimension 15 of a 16-dimension block starts past element 2^32 of the block."""
    _attend_to_one_row_each(64, (2 ** 32 // 15 + 64) // 64 * 64, 70, [0, 33, 69])


@pytest.mark.parametrize("heads,d,T,S", [(28, 128, 32, 1500), (32, 128, 32, 1500), (8, 128, 64, 700), (8, 128, 65, 700),
                                         (28, 128, 3, 255), (28, 128, 2, 286), (1, 128, 128, 4000),
                                         (8, 128, 16, 1000), (8, 128, 16, 1100), (8, 128, 16, 1500),
                                         (8, 128, 64, 3500), (8, 128, 80, 3140), (8, 128, 80, 3500), (8, 128, 97, 3500)])
def test_both_wave_counts(heads, d, T, S):
    """Either side of the line between four and eight waves (more than eight chunks a head): by heads, by query groups and by
    key blocks.  Eight waves of 16 queries: one head, and 8 heads with 16 nodes; of 32 queries: 8 heads with 80 nodes."""
    test_long_chunks(heads, d, T, S)

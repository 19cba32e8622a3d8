"""Where a call leaves its final rows: the last launch writes them straight into hidden_out when that is 16-byte
aligned and any layer ran, a copy does otherwise.  Both ways, in place on hidden_in too, must give the same bits, in the
draft chain as well; the cache rows after the joint walk-and-roll-back launch must be those of the walk followed by the roll-back."""
import numpy as np
import pytest
import torch

import paper_2605_11186_amd as cats
import synth
from gpu_common import Pair, to_dev_bf16

pytestmark = pytest.mark.gpu
SEED, S = 31, 70


@pytest.fixture(scope="module")
def pair():
    p = Pair(synth.TINY, SEED, max_ctx=192, max_tree=64, packed=True)
    yield p
    p.close()


def rows(pair, T, layers, out, hidden_in, verify):
    kc, vc = pair.oracle_cache_random(SEED, S)
    ks, vs = pair.device_cache_from_oracle(kc, vc, S)
    parent, depth = synth.random_tree(T, 5, 3) if T > 1 else (np.array([-1], np.int32), np.array([0], np.int32))
    cats.cats_set_tree(pair.ctx, synth.distinct_sibling_tokens(parent, synth.TINY.vocab, SEED), parent, depth)
    embed = pair.d_embed if hidden_in is None else None
    if verify:
        cats.cats_verify_tree(pair.ctx, pair.layers_arr, 0, layers, embed, hidden_in, pair.d_final["g_final"],
                              pair.d_final["w_lm"], cats.kv_array(ks, vs), S, pair.res_dev, hidden_out=out)
    else:
        cats.cats_verify_nodes(pair.ctx, pair.layers_arr, 0, layers, embed, hidden_in, cats.kv_array(ks, vs), S, 0, out)
    torch.cuda.synchronize()
    return out.cpu().numpy().copy()


@pytest.mark.parametrize("verify", [False, True], ids=["nodes", "tree"])
@pytest.mark.parametrize("T", [1, 2, 17, 64])
@pytest.mark.parametrize("layers", [0, 1, 2])
def test_hidden_out_anywhere_gives_the_same_rows(pair, T, layers, verify):
    H = pair.dims.hidden
    buf = torch.zeros(T * H + 4, device="cuda")
    aligned, shifted = buf[: T * H].view(T, H), buf[1: T * H + 1].view(T, H)
    want = rows(pair, T, layers, aligned, None, verify)
    assert np.isfinite(want).all() and np.abs(want).max() > 0
    assert np.array_equal(rows(pair, T, layers, shifted, None, verify), want)
    # from the caller's rows, in place: the rows that the embedding table would have given
    rows(pair, T, 0, aligned, None, verify)
    assert np.array_equal(rows(pair, T, layers, aligned, aligned, verify), want)


@pytest.mark.parametrize("layers", [1, 2])
def test_draft_chain_leaves_its_rows_anywhere(pair, layers):
    d, gamma = pair.dims, 5
    ad = synth.adapter_weights(d, SEED, 0)
    adapter = cats.pack_layer({k: to_dev_bf16(v) for k, v in ad.items() if k != "g_out"})
    adapter_arr, g_out = cats.layer_array([adapter]), to_dev_bf16(ad["g_out"])
    got = []
    for shift in (0, 1, 2):
        ks, vs = pair.device_cache_from_oracle(*pair.oracle_cache_random(SEED, S), S)
        ka, va = ks[0].clone(), vs[0].clone()
        buf = torch.full(((gamma + 1) * d.hidden + 4,), float("nan"), device="cuda")
        rows = buf[shift: (gamma + 1) * d.hidden + shift].view(gamma + 1, d.hidden)
        tokens = torch.zeros(gamma + 1, dtype=torch.int32, device="cuda")
        cats.cats_draft_chain(pair.ctx, pair.layers_arr, 0, layers, adapter_arr, g_out, pair.d_final["w_lm"], pair.d_embed,
                              cats.kv_array(ks, vs), cats.kv_array([ka], [va]), S, 3, gamma, tokens, hidden_out=rows)
        torch.cuda.synchronize()
        assert torch.isnan(buf[:shift]).all() and torch.isnan(buf[rows.numel() + shift:]).all()
        got.append((rows.clone(), tokens.clone(), ks[0].view(torch.int16).clone(), vs[0].view(torch.int16).clone()))
    assert torch.isfinite(got[0][0]).all()
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))


@pytest.mark.parametrize("T,layers", [(1, 2), (2, 2), (33, 1), (64, 2)])
def test_walk_with_roll_back_is_the_walk_and_the_roll_back(pair, T, layers):
    rng = np.random.default_rng(T)
    parent, depth = synth.random_tree(T, 6, T) if T > 1 else (np.array([-1], np.int32), np.array([0], np.int32))
    tok = synth.distinct_sibling_tokens(parent, synth.TINY.vocab, SEED)
    amax = rng.integers(0, synth.TINY.vocab, T).astype(np.int32)
    deepest = int(np.argmax(depth))   # accept its whole path
    node = deepest
    while node > 0:
        amax[parent[node]] = tok[node]
        node = parent[node]
    cats.cats_set_tree(pair.ctx, tok, parent, depth)
    d = pair.dims
    gen = torch.Generator(device="cuda").manual_seed(T)
    k0 = torch.randn(layers, d.n_heads, 192, d.head_dim, device="cuda", generator=gen).to(torch.bfloat16)
    v0 = torch.randn(layers, d.n_heads, d.head_dim, 192, device="cuda", generator=gen).to(torch.bfloat16)
    a, dev = torch.from_numpy(amax).cuda(), torch.zeros_like(pair.res_dev)
    ka, va, kb, vb = k0.clone(), v0.clone(), k0.clone(), v0.clone()
    cats.cats_accept_and_compact(pair.ctx, a, cats.kv_array(list(ka), list(va)), 0, layers, S, pair.res_dev)
    cats.cats_accept_and_compact(pair.ctx, a, None, 0, 0, S, dev)
    cats.cats_compact_along(pair.ctx, dev, cats.kv_array(list(kb), list(vb)), 0, layers, S)
    torch.cuda.synchronize()
    assert torch.equal(pair.res_dev, dev)
    res = cats.accept_result_from_tensor(dev)
    assert res == pair.oracle.accept(tok, parent, depth, amax, S)
    path = res["path"][: res["n_accepted"] + 1]
    kw, vw = k0.clone(), v0.clone()
    for i, n in enumerate(path):
        kw[:, :, S + i] = k0[:, :, S + n]
        vw[..., S + i] = v0[..., S + n]
    for got in ((ka, va), (kb, vb)):
        assert torch.equal(got[0], kw) and torch.equal(got[1], vw)

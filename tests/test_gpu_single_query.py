"""Attention of a single query around its tile and chunk edges: no context row, one, full and partly filled tiles of 128
keys, a last chunk of one block (merged where it would only make workgroups share compute units), the query at the root and
at later nodes (keys: the context and its own path alone), both head sizes; whole layer against the oracle."""
import numpy as np
import pytest
import torch

import paper_2605_11186_amd as cats
import synth
from gpu_common import Pair, rel_err

pytestmark = pytest.mark.gpu
TOL = 16 * 2.0 ** -17   # 16 mantissa bits of every operand, float32 sums, four products in a row


@pytest.fixture(scope="module", params=[(4, 64), (2, 128), (64, 64), (24, 128)], ids=lambda p: f"{p[0]}x{p[1]}")
def pair(request):
    heads, d = request.param
    p = Pair(synth.ModelDims(1, heads * d, heads, d, 128, 64), 9, max_ctx=1536, max_tree=16, precision="f32", packed=True)
    yield p
    p.close()


@pytest.mark.parametrize("S", [0, 1, 31, 127, 128, 129, 160, 161, 532, 1024, 1056, 1300])
def test_root_and_later_nodes(pair, S):
    kc, vc = pair.oracle_cache_random(4, S)
    ks, vs = pair.device_cache_from_oracle(kc, vc, S)
    kv = cats.kv_array(ks, vs)
    # node 0 alone, then node 1, then node 3 = child of 1 that must not see node 2: one query each
    parent, depth = np.array([-1, 0, 0, 1], np.int32), np.array([0, 1, 1, 2], np.int32)
    tok = np.array([5, 6, 7, 8], np.int32)
    want = pair.oracle.tree_forward(kc.copy(), vc.copy(), S, parent, depth, tokens=tok, layer_end=1)
    for n in range(1, 5):
        cats.cats_set_tree(pair.ctx, tok[:n], parent[:n], depth[:n])
        out = torch.full((1, pair.dims.hidden), float("nan"), device="cuda")
        cats.cats_verify_nodes(pair.ctx, pair.layers_arr, 0, 1, pair.d_embed, None, kv, S, n - 1, out)
        got = out.cpu().numpy()
        # rows of earlier nodes come back from the bf16 cache, so later queries see them at 2^-9
        assert rel_err(got, want[n - 1: n]) <= (TOL if n == 1 else 2.0 ** -8), (n, S)


@pytest.mark.parametrize("S", [100, 128, 200, 1300])
def test_values_behind_a_zero_weight_do_not_count(pair, S):
    """Two opposite keys so long that one of them takes the whole weight of the first tile (partly filled at 100 rows, full
    beyond), in every head: the other rows of that tile, whose weights underflow to zero, may hold anything."""
    kc, vc = pair.oracle_cache_random(4, S)
    ks, vs = pair.device_cache_from_oracle(kc, vc, S)
    a, b, tile = 5, 77, min(S, 128)
    ks[0][:, a] *= 2.0 ** 20   # (so long that it takes no luck of the head's query)
    ks[0][:, b] = -ks[0][:, a]
    others = [r for r in range(tile) if r not in (a, b)]

    def rows():
        cats.cats_set_tree(pair.ctx, np.array([5], np.int32), np.array([-1], np.int32), np.array([0], np.int32))
        out = torch.full((1, pair.dims.hidden), float("nan"), device="cuda")
        cats.cats_verify_nodes(pair.ctx, pair.layers_arr, 0, 1, pair.d_embed, None, cats.kv_array(ks, vs), S, 0, out)
        return out.cpu()

    want = rows()
    assert torch.isfinite(want).all()
    for anything in (float("inf"), float("-inf"), float("nan")):
        vs[0][:, :, others] = anything
        assert torch.equal(rows(), want), anything

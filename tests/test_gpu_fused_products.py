"""The q|k|v and gate|up products at the sizes where their kernels change: one layer against the oracle, every count
of column groups per workgroup, every number of 16-row blocks at its edges, products that fall back alone or both,
both weight layouts and head sizes."""
import numpy as np
import pytest
import torch

import paper_2605_11186_amd as cats
import synth
from gpu_common import Pair, rel_err

pytestmark = pytest.mark.gpu

# Every operand of the layer's four products keeps 16 mantissa bits or more (2^-17 of its value lost), the sums are
# float32: 4 * 2^-17 on the scale of the largest value if all losses of a sum went one way, four times that granted
# for the attention's own steps.  Cache rows are bf16: one unit in the last place where a boundary lies between the two.
TOL = 16 * 2.0 ** -17
KV_TOL = 2.0 ** -8

# heads, head_dim, ffn, packed, rows                                 column groups: q|k|v, gate|up
CASES = [
    (5, 64, 848, False, (2, 40)), (5, 64, 848, True, (65, 15)),      # 1, 1; hidden 320: half a packed chunk at the end
    (16, 128, 5632, False, (16, 33, 128)), (16, 128, 5632, True, (17, 48, 49, 96, 97)),   # 2, 3
    (8, 128, 8192, False, (65,)), (8, 128, 8192, True, (33, 128)),   # 1, 4
    (16, 64, 10240, False, (96,)), (16, 64, 10240, True, (17, 112)),   # 1, 5
    (4, 64, 4096, True, (16, 64)),                                   # 1, 2
    (40, 128, 13824, False, (80,)), (40, 128, 13824, True, (16, 96, 128)),   # 4 (packed beyond 16 rows: none), 7
    (64, 64, 16384, False, (33,)), (64, 64, 16384, True, (50, 128)),   # 3 (packed: none at 128), 8
    (85, 64, 1040, True, (20,)),                                     # 4 with two row blocks, none
    (48, 128, 16384, True, (33,)),                                   # none, 8
    (16, 64, 16400, False, (33,)), (16, 64, 16400, True, (64,)),     # 1, none: wider than the kernel covers
    (86, 64, 16400, False, (20,)),                                   # none, none
    (24, 128, 1040, True, (128, 16)),                                # none, none; 3, 1
]


@pytest.mark.parametrize("heads,d,ffn,packed,sizes", CASES, ids=[f"{c[0]}x{c[1]}-{c[2]}-{'packed' if c[3] else 'rows'}" for c in CASES])
def test_one_layer_against_the_oracle(heads, d, ffn, packed, sizes):
    dims = synth.ModelDims(1, heads * d, heads, d, ffn, 64)
    S = 45
    pair = Pair(dims, 3, max_ctx=192, max_tree=128, precision="f32", packed=packed)
    try:
        w = cats.layer_weights_struct(pair.d_layers[0])
        kc, vc = pair.oracle_cache_random(5, S)
        # rows of an earlier, larger call stay in the packed activations: they must not reach a smaller call's result
        ks, vs = pair.device_cache_from_oracle(kc, vc, S)
        parent, depth = synth.random_tree(128, 8, 1)
        cats.cats_set_tree(pair.ctx, np.zeros(128, np.int32), parent, depth)
        stale = torch.full((128, dims.hidden), float("nan"), device="cuda")
        cats.cats_verify_layer(pair.ctx, w, stale, cats.KVLayer(ks[0].data_ptr(), vs[0].data_ptr()), S)
        for T in sizes:
            parent, depth = synth.random_tree(T, 8, T)
            x = synth.random_hidden(dims, T, T)
            ks, vs = pair.device_cache_from_oracle(kc, vc, S)
            hidden = torch.from_numpy(x).cuda()
            cats.cats_set_tree(pair.ctx, np.zeros(T, np.int32), parent, depth)
            cats.cats_verify_layer(pair.ctx, w, hidden, cats.KVLayer(ks[0].data_ptr(), vs[0].data_ptr()), S)
            got = hidden.cpu().numpy()
            o_kc, o_vc = kc.copy(), vc.copy()
            ref = pair.oracle.tree_forward(o_kc, o_vc, S, parent, depth, hidden_in=x, layer_end=1)
            gk, gv = pair.device_rows(ks, vs, 0, S + T)
            err = rel_err(got, ref), rel_err(gk, o_kc[0, :S + T]), rel_err(gv, o_vc[0, :S + T])
            print(f"{T} rows: hidden {err[0]:.2e}  k {err[1]:.2e}  v {err[2]:.2e}")
            assert err[0] <= TOL and err[1] <= KV_TOL and err[2] <= KV_TOL
    finally:
        pair.close()

"""How the attention launches are cut into workgroups: the rules of the dispatch, built for the CPU."""
import ctypes as C

import pytest

import host_shim
from test_gpu_attention_variants import CASES

CUS, MAX_CHUNKS = 256, 32


@pytest.fixture(scope="module")
def shim():
    return host_shim.build("""
#include "attn_split.hpp"
extern "C" void tree_split(int heads, int d, int rows, int keys, int cus, int max_chunks, int* out) {
    const AttnSplit s = attn_split(heads, d, rows, keys, cus, max_chunks);
    out[0] = s.queries;
    out[1] = s.chunks;
    out[2] = s.waves;
}
extern "C" void row_split_of(int keys, int* out) {
    const RowSplit s = row_split(keys);
    out[0] = s.chunks;
    out[1] = s.span;
}
""")


def tree(shim, heads, d, rows, ctx, cus=CUS):
    """queries, chunks, waves"""
    out = (C.c_int * 3)()
    shim.tree_split(heads, d, rows, ctx + rows, cus, MAX_CHUNKS, out)
    return tuple(out)


def test_16_query_workgroups_beyond_16_rows_fit_the_compute_units(shim):
    for cus in (CUS, 128, 32):
        for d in (64, 128):
            for heads in [*range(1, 129), 200, 1000]:
                for rows in range(1, 129):
                    for ctx in (0, 40, 300, 700, 2100, 4096):
                        queries, chunks, waves = tree(shim, heads, d, rows, ctx, cus)
                        groups, blocks = -(-rows // queries), -(-(ctx + rows) // 32)
                        assert (d, queries, waves) in CASES and 1 <= chunks <= min(MAX_CHUNKS, blocks)
                        if rows <= 16:
                            assert queries == 16
                        elif queries == 16:
                            assert heads * groups * chunks <= cus
                        if chunks > 1:
                            assert heads * groups * chunks <= cus


def test_every_variant_has_a_size_of_several_chunks(shim):
    for (d, queries, waves), sizes in CASES.items():
        for heads, rows, ctx in sizes:
            q, chunks, w = tree(shim, heads, d, rows, ctx)
            assert (q, w) == (queries, waves) and chunks > 1, (heads, d, rows, ctx, q, chunks, w)


@pytest.mark.parametrize("heads,d,rows,ctx", [(64, 64, 65, 300), (64, 64, 128, 40), (40, 128, 97, 8), (40, 128, 128, 300), (64, 128, 96, 128),
                                              (128, 64, 33, 128), (32, 128, 64, 2048), (40, 128, 30, 1500)])
def test_32_queries_where_16_were_slower(shim, heads, d, rows, ctx):
    assert tree(shim, heads, d, rows, ctx)[0] == 32


@pytest.mark.parametrize("heads,d,rows,ctx", [(32, 128, 128, 300), (32, 128, 20, 300), (32, 128, 32, 1024), (32, 128, 63, 512), (8, 128, 64, 4096),
                                              (64, 64, 64, 128), (40, 128, 96, 128), (128, 64, 32, 128)])
def test_16_queries_where_32_were_slower(shim, heads, d, rows, ctx):
    assert tree(shim, heads, d, rows, ctx)[0] == 16


def test_a_single_query_has_chunks_of_one_pass(shim):
    out = (C.c_int * 2)()
    for keys in [*range(0, 10000), 40000, 2 ** 25]:
        shim.row_split_of(keys, out)
        chunks, span = out
        assert 1 <= chunks <= MAX_CHUNKS and span % 32 == 0
        assert (chunks - 1) * span < max(keys, 1) <= chunks * span   # every chunk has keys, none more than the span
        if keys <= 128 * MAX_CHUNKS:
            assert span == 128

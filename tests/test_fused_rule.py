"""Which kernel takes the q|k|v and the gate|up product: the rules of the dispatch, called in the library itself."""
import ctypes as C

import pytest

import paper_2605_11186_amd as cats


class FusedRule(C.Structure):
    _fields_ = [("groups", C.c_int), ("K", C.c_int), ("rows", C.c_int), ("n_cus", C.c_int), ("packed", C.c_bool)]


def column_groups(name, groups, hidden, rows, packed, n_cus=256):
    lib = C.CDLL(str(cats.library_path()))
    rule = getattr(lib, f"_Z{len(name)}{name}RK9FusedRule")
    rule.argtypes, rule.restype = [C.POINTER(FusedRule)], C.c_int
    return rule(C.byref(FusedRule(groups, hidden, rows, n_cus, packed)))


def qkv(hidden, rows, packed=True, n_cus=256):
    return column_groups("fused_qkv_groups", 3 * hidden // 16, hidden, rows, packed, n_cus)


def swiglu(hidden, ffn, rows, packed=True, n_cus=256):
    return column_groups("fused_swiglu_groups", ffn // 8, hidden, rows, packed, n_cus)


@pytest.mark.parametrize("rows", [2, 16, 17, 32, 33, 64, 65, 96, 97, 128])
@pytest.mark.parametrize("packed", [False, True])
def test_a_fused_product_has_one_workgroup_per_compute_unit(rows, packed):
    for n_cus in (256, 128, 32):
        for hidden in range(64, 8193, 64):
            R = qkv(hidden, rows, packed, n_cus)
            fewest = -(-3 * hidden // 16 // n_cus)
            assert R in (0, fewest) and R <= 4
            assert packed or R or fewest > 4
        for ffn in range(16, 20001, 16):
            R = swiglu(1024, ffn, rows, packed, n_cus)
            assert R in (0, -(-ffn // 8 // n_cus)) and R <= 8
    assert qkv(1024, 1, packed) == 0 and swiglu(1024, 4096, 1, packed) == 0   # single rows have their own kernels


@pytest.mark.parametrize("hidden,rows", [(5120, 32), (5120, 64), (4352, 64), (4864, 96), (3584, 128), (3072, 64)])
def test_qkv_stays_with_partial_tiles_where_fused_was_slower(hidden, rows):
    assert qkv(hidden, rows) == 0


@pytest.mark.parametrize("hidden,ffn,rows", [(5120, 4112, 64), (5120, 1408, 32), (5120, 2816, 128), (5120, 5632, 96),
                                             (4096, 4112, 128), (4096, 688, 96), (8192, 2064, 64), (8192, 8208, 96)])
def test_gate_up_stays_with_partial_tiles_where_fused_was_slower(hidden, ffn, rows):
    assert swiglu(hidden, ffn, rows) == 0


@pytest.mark.parametrize("hidden,ffn,rows,R_qkv,R_swiglu", [
    (256, 688, 15, 1, 1), (2048, 5632, 128, 2, 3), (4096, 11008, 16, 3, 6), (4096, 11008, 63, 3, 6),
    (4096, 11008, 96, 3, 6), (4096, 11008, 128, 0, 6), (5120, 13824, 16, 4, 7), (5120, 13824, 64, 0, 7), (5120, 13824, 128, 0, 7)])
def test_common_layer_shapes(hidden, ffn, rows, R_qkv, R_swiglu):
    assert qkv(hidden, rows) == R_qkv and swiglu(hidden, ffn, rows) == R_swiglu

// The q|k|v product with norm factor, rotation and cache append (kernel and split: fused.hpp).
#include "fused.hpp"

// The partial-tile product deals its work out evenly; here the launch lasts as long as one workgroup, which streams
// 16 R rows of weights whether or not the units cover the chip, and whose work per k grows with R times the row blocks
// (so does its register need: from R = 4 on the ring is one step deep at 48 rows and more).  What is saved is a launch and the
// partial tiles.  Measured as fused minus partial-tile, one layer, packed weights (us): hidden 2048 (R = 2)
// -3.3 at 63 rows, -7.4 at 96, -4.5 at 128; hidden 4096 (R = 3) -4.4 at 16, -2.0 at 63, -7.9 at 96, +1.2 at 128; hidden 5120 (R = 4)
// -3.2 at 16, +1.3 at 32, +3.4 at 63, +2.5 at 128; hidden 3072 (192 units of R = 3) +2.9 at 64, +4.4 at 128.  From 65 to 96 rows
// the partial-tile product holds three accumulator blocks a wave and is at its worst.  The line follows 110
// widths from 256 to 8192 at 13 row counts: on its wrong side are at most 2.5 % of a layer.  Row-major weights: the
// partial-tile product is so much slower that fused won at all but 2 % of the points, and lost 1.9 % at most there.
// More than four groups (hidden beyond 5461 on 256 units) are not built yet. Measured there, packed (us): hidden 8192 with six
// -7.7 of 154 at 16 rows, -4.4 at 64, -5.8 at 128; hidden 6144 with five -2.2 at 16, +0.4 at 64, +7.3 at 128.
int fused_qkv_groups(const FusedRule& p) {
    if (p.rows < 2) return 0;   // a single row has kernels of its own
    for (int R : {1, 2, 3, 4}) {
        if ((p.groups + R - 1) / R > p.n_cus) continue;
        if (!p.packed) return R;
        const float k = p.K / 4096.f, uneven = R - static_cast<float>(p.groups) / p.n_cus;
        const int m = fused_row_blocks(p.rows);
        return k * ((m == 1 ? 0.86f : 1.87f) * uneven + 0.063f * R * m) < (m == 6 ? 2.f : 1.f) ? R : 0;
    }
    return 0;
}

void launch_fused_qkv(const FusedArgs& a, int R, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    if (R == 1) return launch_r<1, EPI_QKV>(a, st, e0, e1);
    if (R == 2) return launch_r<2, EPI_QKV>(a, st, e0, e1);
    if (R == 3) return launch_r<3, EPI_QKV>(a, st, e0, e1);
    return launch_r<4, EPI_QKV>(a, st, e0, e1);
}

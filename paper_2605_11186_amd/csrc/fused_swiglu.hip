// The gate|up product with norm factor and SwiGLU (kernel and split: fused.hpp).
#include "fused.hpp"

// Where the line lies (see also fused_qkv.hip): a workgroup's time grows with K, with the rows of weights that it streams beyond
// an even share and with the row blocks of X that it reads; what is saved grows with the partial tiles, rows times columns.
// The partial-tile product is at its best from 17 to 32 rows (small tiles; this one is then no better placed than at 48)
// and at its worst from 65 to 96 (three accumulator blocks a wave).
// Measured as fused minus partial-tile, one layer, packed weights (us): hidden 4096 / ffn 11008 -4.7 at 16
// rows, -5.2 at 63, -4.7 at 128; 5120 / 13824 -8.5, -6.1, -8.0; 2048 / 5632 -3.5, -5.6, -2.1; but 5120 / 4112 (172 units
// of R = 3) -1.3 at 16 rows, +5.0 at 64, +15 at 128, and 8192 / 2064 +1.5, +13, +25.  Over 150 pairs of widths at 13 row
// counts, on the wrong side are 4 % of a layer at most, 2 % or more at 2 % of the points.
int fused_swiglu_groups(const FusedRule& p) {
    if (p.rows < 2) return 0;   // a single row has kernels of its own
    for (int R : {1, 2, 3, 4, 5, 6, 7, 8}) {
        if ((p.groups + R - 1) / R > p.n_cus) continue;
        const float k = p.K / 4096.f, uneven = R - static_cast<float>(p.groups) / p.n_cus;
        const float tiles = 1e-4f * p.rows * p.groups;
        const int m = fused_row_blocks(p.rows);
        const bool pays = p.packed ? k * (m == 2 ? 2.87f : m) * (0.23f * uneven + 0.52f) < (m == 6 ? 1.6f : 1.f) + 0.38f * tiles
                                   : k * m * (0.2f * uneven + 0.3f) < 1.f + 0.42f * tiles;
        return pays ? R : 0;
    }
    return 0;
}

void launch_fused_swiglu(const FusedArgs& a, int R, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    if (R == 1) return launch_r<1, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 2) return launch_r<2, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 3) return launch_r<3, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 4) return launch_r<4, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 5) return launch_r<5, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 6) return launch_r<6, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 7) return launch_r<7, EPI_SWIGLU>(a, st, e0, e1);
    return launch_r<8, EPI_SWIGLU>(a, st, e0, e1);
}

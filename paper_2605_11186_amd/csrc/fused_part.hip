// Products that end with partial tiles: output and down projections, LM head (kernel and split: fused.hpp).
#include "fused.hpp"

namespace {
constexpr int SPLIT_MAX_ROWS = 48;
}

FusedSplit fused_split(int N, int K, int n_cus, int rows) {
    // A single row has kernels of its own.  Beyond 48 rows the products of gemm.hip are faster: their tiles
    // are four times as wide, and every workgroup here reads 64 columns' worth of all rows of X.
    if (rows < 2 || rows > SPLIT_MAX_ROWS) return {0, 0};
    if (N % 16 != 0 || K % 32 != 0) return {0, 0};
    FusedSplit best{0, 0};
    int most = 0;
    for (int R : {4, 5, 2, 1, 8}) {
        const int units = (N / 16 + R - 1) / R;
        if (units > n_cus) continue;
        // at least two k steps for each of the eight waves, at most eight ranges
        const int ksplit = std::max(1, std::min({n_cus / units, K / 32 / 16, 8}));
        if (units * ksplit > most) {
            most = units * ksplit;
            best = {R, ksplit};
        }
    }
    return best;
}

void launch_fused_part(const FusedArgs& a, int R, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    if (R == 1) return launch_r<1, EPI_PART>(a, st, e0, e1);
    if (R == 2) return launch_r<2, EPI_PART>(a, st, e0, e1);
    if (R == 4) return launch_r<4, EPI_PART>(a, st, e0, e1);
    if (R == 5) return launch_r<5, EPI_PART>(a, st, e0, e1);
    return launch_r<8, EPI_PART>(a, st, e0, e1);
}

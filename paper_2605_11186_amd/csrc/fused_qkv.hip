// The q|k|v product with norm factor, rotation and cache append (kernel and split: fused.hpp).
#include "fused.hpp"

int fused_qkv_groups(int groups, int n_cus, int rows) {
    if (rows < 2) return 0;   // a single row has kernels of its own
    for (int R : {1, 2, 3, 4})
        if ((groups + R - 1) / R <= n_cus) return R;
    return 0;
}

void launch_fused_qkv(const FusedArgs& a, int R, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    if (R == 1) return launch_r<1, EPI_QKV>(a, st, e0, e1);
    if (R == 2) return launch_r<2, EPI_QKV>(a, st, e0, e1);
    if (R == 3) return launch_r<3, EPI_QKV>(a, st, e0, e1);
    return launch_r<4, EPI_QKV>(a, st, e0, e1);
}

// The gate|up product with norm factor and SwiGLU (kernel and split: fused.hpp).
#include "fused.hpp"

int fused_swiglu_groups(int groups, int n_cus, int rows) {
    if (rows < 2) return 0;   // a single row has kernels of its own
    for (int R : {2, 4, 6, 7, 8})
        if ((groups + R - 1) / R <= n_cus) return R;
    return 0;
}

void launch_fused_swiglu(const FusedArgs& a, int R, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    if (R == 2) return launch_r<2, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 4) return launch_r<4, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 6) return launch_r<6, EPI_SWIGLU>(a, st, e0, e1);
    if (R == 7) return launch_r<7, EPI_SWIGLU>(a, st, e0, e1);
    return launch_r<8, EPI_SWIGLU>(a, st, e0, e1);
}

// Instantiations of the implicit-GEMM kernel for backward passes that read the forward pass's weights (FWD_WT in
// igemm_kernel.h): the tiles that stride-1 and 1x1 backward passes run on, in a translation unit of their own so that
// they compile beside the others.  A plan whose tile is not here has its weights transformed by a launch of its own.
//
// Measured against the transform launch and the same tiles (three sets of tensors in turn): bf16 1024 -> 256 1x1 at 14x14,
// N = 8 8.6 -> 5.1 us, 2048 -> 384 at 8x8, N = 24, 11.2 -> 6.5 (the small tile in the register-operand kernel's place), 395 passes
// at N = 2 ... 192 on average 0.83 of the time; fp32 0.97 (377 passes; 0.78 under 10 us, 0.99 beyond 90: the operand is
// four 4-byte reads there for one of 16, next to 256 clocks of MFMAs).
#include "igemm_kernel.h"

namespace convmi {

#define WT(DT, WK, WM, FK, FM, NPL, R, S, PPT) IGEMM_ENTRY_WT(DT, WK, WM, FK, FM, NPL, R, S, PPT, 2, 0)
#define WT_SMALL(DT, NPL, R, S, PPT) WT(DT, 2, 2, 1, 2, NPL, R, S, PPT), WT(DT, 2, 2, 2, 2, NPL, R, S, PPT)
#define WT_NT(DT, WK, WM, FK, FM, NPL, PPT, NB) \
    IGEMM_ENTRY_WT(DT, WK, WM, FK, FM, NPL, 1, 1, PPT, NB, 0), IGEMM_ENTRY_WT(DT, WK, WM, FK, FM, NPL, 1, 1, PPT, NB, 1)
static IgemmEntry g_fwd_wt[] = {
    // 64 x 128 and 128 x 128 tiles
    WT_SMALL(CONV_BF16, 4, 1, 1, 0), WT_SMALL(CONV_BF16, 8, 1, 1, 0), WT_SMALL(CONV_BF16, 2, 3, 3, 1),
    WT_SMALL(CONV_BF16, 2, 3, 3, 2), WT_SMALL(CONV_BF16, 2, 3, 3, 3), WT_SMALL(CONV_BF16, 2, 1, 7, 1),
    WT_SMALL(CONV_BF16, 2, 7, 1, 1), WT_SMALL(CONV_BF16, 2, 7, 1, 2),
    WT_SMALL(CONV_F32, 4, 1, 1, 0), WT_SMALL(CONV_F32, 8, 1, 1, 0), WT_SMALL(CONV_F32, 2, 3, 3, 1),
    WT_SMALL(CONV_F32, 2, 3, 3, 2), WT_SMALL(CONV_F32, 2, 3, 3, 3), WT_SMALL(CONV_F32, 2, 1, 7, 1),
    WT_SMALL(CONV_F32, 2, 7, 1, 1), WT_SMALL(CONV_F32, 2, 7, 1, 2),
    // larger ones, 1x1
    WT_NT(CONV_BF16, 4, 1, 1, 7, 4, 1, 2), WT_NT(CONV_BF16, 4, 1, 1, 7, 4, 1, 3), WT_NT(CONV_BF16, 2, 2, 1, 7, 4, 2, 2),
    WT_NT(CONV_BF16, 2, 2, 1, 7, 4, 2, 3), WT_NT(CONV_BF16, 4, 2, 2, 4, 8, 1, 2), WT(CONV_BF16, 2, 2, 2, 4, 4, 1, 1, 1),
    WT(CONV_BF16, 4, 1, 1, 7, 8, 1, 1, 1),
    WT_NT(CONV_F32, 4, 1, 1, 7, 4, 1, 2), WT_NT(CONV_F32, 2, 2, 1, 7, 4, 2, 2),
    // ... and of several taps
    WT(CONV_BF16, 1, 4, 2, 4, 2, 3, 3, 3), WT(CONV_BF16, 1, 4, 2, 4, 2, 3, 3, 4), WT(CONV_BF16, 2, 4, 2, 4, 2, 3, 3, 3),
    WT(CONV_BF16, 2, 4, 2, 4, 2, 3, 3, 4), WT(CONV_BF16, 1, 4, 2, 4, 2, 1, 7, 3), WT(CONV_BF16, 1, 4, 2, 4, 2, 7, 1, 3),
    WT(CONV_F32, 4, 1, 1, 7, 2, 3, 3, 2), WT(CONV_F32, 2, 2, 1, 7, 2, 3, 3, 3), WT(CONV_F32, 1, 4, 1, 7, 2, 3, 3, 5),
    WT(CONV_F32, 1, 4, 1, 7, 2, 3, 3, 6),
};

IgemmEntry *igemm_fwd_wt_entries(int *count)
{
    *count = (int)(sizeof(g_fwd_wt) / sizeof(g_fwd_wt[0]));
    return g_fwd_wt;
}

}  // namespace convmi

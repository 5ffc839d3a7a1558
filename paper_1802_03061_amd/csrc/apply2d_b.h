// Per-L entry points of pass B (one translation unit per L, see apply2d_b.hip).
#pragma once
#include "apply2d.h"

namespace rte {
#define RTE_DECL_PASSB(L) \
    template <typename T> int pass_b_L##L(const Apply2DArgs<T>& a, int nbatch);
RTE_DECL_PASSB(0) RTE_DECL_PASSB(1) RTE_DECL_PASSB(2) RTE_DECL_PASSB(3) RTE_DECL_PASSB(4)
RTE_DECL_PASSB(5) RTE_DECL_PASSB(6) RTE_DECL_PASSB(7) RTE_DECL_PASSB(8)
RTE_DECL_PASSB(9) RTE_DECL_PASSB(10) RTE_DECL_PASSB(11) RTE_DECL_PASSB(12)     // FP32 only
RTE_DECL_PASSB(13) RTE_DECL_PASSB(14) RTE_DECL_PASSB(15) RTE_DECL_PASSB(16)
#undef RTE_DECL_PASSB

// Pass B in split form (apply2d_split, apply2d_few_columns: unpacked work buffer, work2 required;
// apply2d_bm.hip).  More than 17 modes: variant 0 couples the modes by an FFT along the mode axis (twm:
// twiddles of length mode_fft_len(L)), variant 1 by the direct Toeplitz sum.  Up to 17: k_couple_regs.
constexpr int PASSB_FUSED_MAX_L = 8;      // in both precisions at every size
constexpr int PASSB_FUSED_MAX_L_F32 = 16;  // in FP32 up to padded y = PASSB_FUSED_MAX_PY
constexpr int PASSB_FUSED_MAX_PY = 512;
constexpr int PASSB_FEW_COLUMNS = 64;      // FP64, 11 to 17 modes, padded y = 1024: apply2d_few_columns
inline int mode_fft_len(int L) { int p = 1; while (p < 4 * L + 1) p <<= 1; return p; }
template <typename T> int pass_b_large(const Apply2DArgs<T>& a, int nbatch);
}  // namespace rte

// Pass B of the 2D apply for one value of L (this file is compiled once per L = 0..16 with
// -DRTE_PASSB_L=<L>): FFT along y of every channel, per-frequency mode coupling with the kernel
// spectra, inverse FFT along y (Sec. 3.3.1: the kernel depends on x - y and on k' - k only, so
// the convolution over y and the sum over k' meet at each frequency).  The kernels are in
// passb_wave.h.
//
// Coupling at frequency (kx, ky), for channels a_0 = u_0, (a_k, b_k) = sqrt2 (Re u_k, Im u_k) and the
// complex modes W_{+-k} = (A_k +- i B_k)/sqrt2, W_0 = A_0:
//   V_k = sum_{k'} Khat_{k'-k} W_{k'},  k = -L..L  -- Toeplitz in the mode index
//   out: A_0 = V_0, A_k = (V_k + V_{-k})/sqrt2, B_k = -i (V_k - V_{-k})/sqrt2
// with Khat read from the quarter table (see apply2d.hip for the symmetries), evaluated in the
// channels (passb_wave.h).
#include "apply2d.h"
#include "apply2d_b.h"
#include "passb_wave.h"

#ifndef RTE_PASSB_L
#error "compile with -DRTE_PASSB_L=<L>"
#endif

namespace rte {

// A block keeps the spectra of its columns in LDS (k_pass_b_wave) wherever they fit 160 KB; FP64
// with L > 4 at padded y = 1024 runs each column in two halves (k_pass_b_half).  L = 9..16 come here in FP32
// up to padded y = 512 (apply2d_split).  Pass B at 512^2,
// L = 8: FP32 38.5 us, where the form it replaces (block-wide FFT stages, complex coupling) took
// 57-60 us; FP64 see k_pass_b_half.
template <typename T, int PY>
static int launch_py(const Apply2DArgs<T>& a, int nbatch) {
    constexpr int L = RTE_PASSB_L;
    if (!a.pack || (a.bcorr.y && (sizeof(T) != 4 || a.single_in || nbatch != 1))) return -6;
    const int nkq = a.PX / 2 + 1, nkx = a.PX / 2;
    if constexpr (L == 0) {
        if (!a.bcorr.y) {   // the correction enters with k_pass_b_wave's loads
            launch_iso<T, PY>(a, nbatch, nkx, nkq);
            return 0;
        }
    }
    if constexpr (wave_fits<T, PY, L>()) {
        launch_wave<T, PY, L>(a, nbatch, nkx, nkq);
        return 0;
    } else if constexpr (L <= 8) {
        if (!a.twyh) return -5;
        launch_half<T, PY, L, 8>(a, nbatch, nkx, nkq);
        return 0;
    } else {
        return -1;   // apply2d_split: not routed here
    }
}

template <typename T>
static int launch_pass_b_impl(const Apply2DArgs<T>& a, int nbatch) {
    switch (a.PY) {
        case 16: return launch_py<T, 16>(a, nbatch);
        case 32: return launch_py<T, 32>(a, nbatch);
        case 64: return launch_py<T, 64>(a, nbatch);
        case 128: return launch_py<T, 128>(a, nbatch);
        case 256: return launch_py<T, 256>(a, nbatch);
        case 512: return launch_py<T, 512>(a, nbatch);
        case 1024: return launch_py<T, 1024>(a, nbatch);
    }
    return -1;
}

#define RTE_CAT2(a, b) a##b
#define RTE_CAT(a, b) RTE_CAT2(a, b)
template <>
int RTE_CAT(pass_b_L, RTE_PASSB_L)<float>(const Apply2DArgs<float>& a, int nbatch) {
    return launch_pass_b_impl<float>(a, nbatch);
}
#if RTE_PASSB_L <= 8
template <>
int RTE_CAT(pass_b_L, RTE_PASSB_L)<double>(const Apply2DArgs<double>& a, int nbatch) {
    return launch_pass_b_impl<double>(a, nbatch);
}
#endif

#if RTE_PASSB_L == 0
// ---- batched isotropic form ----

// Variants (padded y >= 128) = waves per block (the tuner times them).
constexpr int batch_waves(int var) { return var == 1 ? 2 : var == 2 ? 8 : var == 3 ? 1 : 4; }
template <typename T>
constexpr int batch_b_variants(int PY) { return PY < 128 ? 1 : 4; }
template <typename T, int PY, int NW>
static void launch_b_batch_nw(const BatchProb<T>* probs, const int2* items, int nitems, const int* act,
                              hipStream_t st) {
    hipLaunchKernelGGL((k_pass_b_batch<T, PY, NW>), dim3(nitems), dim3(NW * 64), 0, st, probs, items, act);
}
template <typename T, int PY>
static void launch_b_batch(const BatchProb<T>* probs, const int2* items, int nitems, const int* act, int var,
                           hipStream_t st) {
    if constexpr (PY >= 128) {
        if (var == 1) return launch_b_batch_nw<T, PY, 2>(probs, items, nitems, act, st);
        if (var == 2) return launch_b_batch_nw<T, PY, 8>(probs, items, nitems, act, st);
        if (var == 3) return launch_b_batch_nw<T, PY, 1>(probs, items, nitems, act, st);
    }
    launch_b_batch_nw<T, PY, 4>(probs, items, nitems, act, st);
}
template <typename T>
int apply2d_batch_col_variants(int PY) { return batch_b_variants<T>(PY); }
template <typename T>
int apply2d_batch_cols(int PY, int var) {
    if (var < 0 || var >= apply2d_batch_col_variants<T>(PY)) return 0;
    return batch_waves(var) * (64 / wave_lanes(PY));
}
template <typename T>
int apply2d_batch_pass_b(int PY, const BatchProb<T>* probs, const int2* items, int nitems, const int* act, int var,
                         hipStream_t st) {
    if (nitems <= 0) return 0;
    if (var < 0 || var >= apply2d_batch_col_variants<T>(PY)) return -1;
    switch (PY) {
        case 16: launch_b_batch<T, 16>(probs, items, nitems, act, var, st); break;
        case 32: launch_b_batch<T, 32>(probs, items, nitems, act, var, st); break;
        case 64: launch_b_batch<T, 64>(probs, items, nitems, act, var, st); break;
        case 128: launch_b_batch<T, 128>(probs, items, nitems, act, var, st); break;
        case 256: launch_b_batch<T, 256>(probs, items, nitems, act, var, st); break;
        case 512: launch_b_batch<T, 512>(probs, items, nitems, act, var, st); break;
        case 1024: launch_b_batch<T, 1024>(probs, items, nitems, act, var, st); break;
        default: return -1;
    }
    return 0;
}
template int apply2d_batch_col_variants<float>(int);
template int apply2d_batch_col_variants<double>(int);
template int apply2d_batch_cols<float>(int, int);
template int apply2d_batch_cols<double>(int, int);
template int apply2d_batch_pass_b<float>(int, const BatchProb<float>*, const int2*, int, const int*, int,
                                         hipStream_t);
template int apply2d_batch_pass_b<double>(int, const BatchProb<double>*, const int2*, int, const int*, int,
                                          hipStream_t);
#endif

}  // namespace rte

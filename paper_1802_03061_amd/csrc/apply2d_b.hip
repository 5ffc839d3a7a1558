// Pass B of the 2D apply for one value of L (this file is compiled once per L = 0..16 with
// -DRTE_PASSB_L=<L>): FFT along y of every channel, per-frequency mode coupling with the kernel
// spectra, inverse FFT along y (Sec. 3.3.1: the kernel depends on x - y and on k' - k only, so
// the convolution over y and the sum over k' meet at each frequency).  The kernels are in
// passb_wave.h; the batched isotropic pass B is at the end of this file.
//
// Coupling at frequency (kx, ky), for channels a_0 = u_0, (a_k, b_k) = sqrt2 (Re u_k, Im u_k) and the
// complex modes W_{+-k} = (A_k +- i B_k)/sqrt2, W_0 = A_0:
//   V_k = sum_{k'} Khat_{k'-k} W_{k'},  k = -L..L  -- Toeplitz in the mode index
//   out: A_0 = V_0, A_k = (V_k + V_{-k})/sqrt2, B_k = -i (V_k - V_{-k})/sqrt2
// with Khat read from the quarter table (see apply2d.hip for the symmetries), evaluated in the
// channels (passb_wave.h).
#include "apply2d.h"
#include "apply2d_b.h"
#include "fft.h"
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
// ---- batched isotropic form: one block per (problem, group of NCOL columns) ----
//
// The column spectra in LDS, the y-FFTs by the whole block.  The spectrum of the isotropic kernel is
// real.  Column 0 packs x-frequencies 0 and PX/2 (see packed_split in passb_wave.h).
template <typename T, int PY, int NCOL, int NTHR>
__global__ __launch_bounds__(NTHR) void k_pass_b_batch(const BatchProb<T>* __restrict__ probs,
                                                       const int2* __restrict__ items, const int* __restrict__ act) {
    constexpr int LD = padded(PY);
    constexpr int KH = PY / 2 + 1;
    // FFT stages in groups of at most ~3 radix-8 butterflies per thread
    constexpr int G0 = (3 * NTHR * 8) / PY;
    constexpr int G = G0 >= NCOL ? NCOL : (G0 < 1 ? 1 : G0);
    __shared__ cx<T> spec[NCOL * LD];
    __shared__ cx<T> tws[PY];
    const int2 item = items[blockIdx.x];
    const BatchProb<T>& d = probs[item.x];
    if (act && !act[item.x]) return;
    const int tid = threadIdx.x;
    const int ny = d.ny, nkx = d.PX / 2, kx0 = item.y * NCOL;
    cx<T>* base = d.work;
    stage_twiddles<T, PY, NTHR>(tws, d.twy, tid);
    // first stage from the loads: rows y >= ny are zero padding
    using In = PaddedIn<T, PY, NCOL, NTHR>;
    constexpr int R0 = In::R0, NB0 = In::NB0;
    In in;
    fft_padded_load<T, PY, NCOL, NTHR>(in, tid, [&](int f, int y) {   // a clamped index instead of a branch
        return base[(kx0 + f < nkx && y < ny) ? (size_t)(kx0 + f) * ny + y : 0];
    });
#pragma unroll
    for (int it = 0; it < In::IT; ++it) {
        const int idx = tid + it * NTHR;
        const int j = idx % NB0, f = idx / NB0;
#pragma unroll
        for (int r = 0; r < R0 / 2; ++r)
            if (!(kx0 + f < nkx && j + r * NB0 < ny)) in.v[it][r] = mk((T)0, (T)0);
    }
#pragma unroll
    for (int it = 0; it < In::IT; ++it) {
        const int idx = tid + it * NTHR;
        if (In::NBT % NTHR == 0 || idx < In::NBT) {
            const int j = idx % NB0, f = idx / NB0;
            cx<T> v[R0];
#pragma unroll
            for (int r = 0; r < R0; ++r) v[r] = r < R0 / 2 ? in.v[it][r] : mk((T)0, (T)0);
            dft_small<T, R0, false>(v);
#pragma unroll
            for (int r = 0; r < R0; ++r) spec[f * LD + sw(j * R0 + r)] = v[r];
        }
    }
    __syncthreads();
    block_fft_grouped_range<T, PY, NCOL, G, LD, NTHR, false, R0, PY>(spec, tws, tid);
    for (int idx = tid; idx < NCOL * PY; idx += NTHR) {
        const int f = idx % PY, kx = kx0 + idx / PY;
        if (kx >= nkx) continue;
        cx<T>* sp = spec + (idx / PY) * LD;
        if (kx == 0) {
            if (f > PY / 2) continue;
            const int fm = (PY - f) & (PY - 1);
            const T kd = d.Q[f].re, kq = d.Q[(size_t)nkx * KH + f].re;
            const cx<T> z = sp[sw(f)], w = conj(sp[sw(fm)]);
            const cx<T> D = scale(z + w, (T)0.5 * kd), Qv = scale(mul_mi(z - w), (T)0.5 * kq);
            sp[sw(f)] = D + mul_i(Qv);
            if (fm != f) sp[sw(fm)] = conj(D) + mul_i(conj(Qv));
        } else {
            const T k = d.Q[(size_t)kx * KH + (f > PY / 2 ? PY - f : f)].re;
            sp[sw(f)] = scale(sp[sw(f)], k);
        }
    }
    __syncthreads();
    fft_inverse_cropped_grouped<T, PY, NCOL, G, LD, NTHR>(spec, tws, tid, [&](int f, int y, cx<T> v) {
        if (kx0 + f < nkx && y < ny) base[(size_t)(kx0 + f) * ny + y] = v;
    });
}

constexpr int iso_cols() { return 4; }
constexpr int iso_threads(int n) { return n / 8 >= 512 ? 512 : (n / 8 >= 256 ? 256 : (n / 8 >= 128 ? 128 : 64)); }

// Batched pass-B variants (padded y >= 128): 0 = the fused form's columns per block and threads;
// 1 = the same columns with half the threads; 2 = twice the columns; 3 = half the columns.
template <typename T, int PY, int NCOL>
constexpr bool batch_b_fits() {
    return ((long)NCOL * padded(PY) + PY + 2) * (long)sizeof(cx<T>) <= 160 * 1024;
}
template <typename T, int PY>
constexpr int batch_b_variants() {
    return PY < 128 ? 1 : (batch_b_fits<T, PY, 2 * iso_cols()>() ? 4 : 2);
}
template <typename T, int PY, int NCOL, int NT>
static void launch_b_batch_nc(const BatchProb<T>* probs, const int2* items, int nitems, const int* act,
                              hipStream_t st) {
    static_assert(batch_b_fits<T, PY, NCOL>(), "batched pass-B columns exceed the LDS budget");
    hipLaunchKernelGGL((k_pass_b_batch<T, PY, NCOL, NT>), dim3(nitems), dim3(NT), 0, st, probs, items, act);
}
template <typename T, int PY>
static void launch_b_batch(const BatchProb<T>* probs, const int2* items, int nitems, const int* act, int var,
                           hipStream_t st) {
    constexpr int NCOL = iso_cols();
    constexpr int NT = iso_threads(NCOL * PY);
    if constexpr (batch_b_variants<T, PY>() >= 2) {
        if (var == 1) return launch_b_batch_nc<T, PY, NCOL, (NT / 2 > 64 ? NT / 2 : 64)>(probs, items, nitems, act, st);
    }
    if constexpr (batch_b_variants<T, PY>() >= 4) {
        if (var == 2) return launch_b_batch_nc<T, PY, 2 * NCOL, iso_threads(2 * NCOL * PY)>(probs, items, nitems,
                                                                                            act, st);
        if (var == 3) return launch_b_batch_nc<T, PY, NCOL / 2, iso_threads(NCOL / 2 * PY)>(probs, items, nitems,
                                                                                            act, st);
    }
    launch_b_batch_nc<T, PY, NCOL, NT>(probs, items, nitems, act, st);
}
template <typename T>
int apply2d_batch_col_variants(int PY) {
    switch (PY) {
        case 128: return batch_b_variants<T, 128>();
        case 256: return batch_b_variants<T, 256>();
        case 512: return batch_b_variants<T, 512>();
        case 1024: return batch_b_variants<T, 1024>();
        default: return 1;
    }
}
template <typename T>
int apply2d_batch_cols(int PY, int var) {
    constexpr int NCOL = iso_cols();   // the same for every PY when C = 1
    if (var < 0 || var >= apply2d_batch_col_variants<T>(PY)) return 0;
    return var == 2 ? 2 * NCOL : var == 3 ? NCOL / 2 : NCOL;
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

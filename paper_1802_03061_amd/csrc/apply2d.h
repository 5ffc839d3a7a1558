// Host-side interface of the 2D FFT apply kernels.
#pragma once
#include "../../include/rte.h"
#include "common.h"
#include "krylov.h"

namespace rte {

// APPLY_K: K = K~ D alone (pass C as APPLY_KT, with the factors of APPLY_A)
enum { APPLY_A = 0, APPLY_KT = 1, APPLY_RESID = 2, APPLY_K = 3 };

struct ChanScale {
    double s[2 * RTE_MAX_L + 1];   // per-channel factor applied in pass A (D for operator A, 1 for K~)
};

// The coarse correction added in pass B instead of pass A (FP32, L <= 8).  Pass A
// has transformed the vector alone; pass B adds, to every column before its y-FFT, the
// x-spectrum of the correction cs P y scaled as pass A scales its input.  P is separable (an
// x- then a y-interpolation), so the x-spectrum of row yy of P y_c is (1 - a) G_c[r0] + a G_c[r1],
// with (r0, r1, a) the y-interpolation of row yy and G_c[R](kx) = sum_X y_c[R][X] phi[X][kx],
// phi[X] being the x-spectrum of the fine row of interpolation weights of coarse column X (its
// column 0 holds (phi(0), phi(PX/2)) when the work buffer is packed).
struct CorrB {
    const float* y = nullptr;       // coarse field [C][Hc][Wc], 16-byte aligned, Wc a multiple of 4
    const void* phi = nullptr;      // cx<float> [Wc][nkx], nkx = columns of the work buffer
    const float* coef = nullptr;    // [C] in device memory: pass A's factor of channel c times cs
    int Hc = 0, Wc = 0, F = 1;
};

template <typename T>
struct Apply2DArgs {
    int nx, ny, PX, PY, L, C;
    cx<T>* work;               // work buffer [nbatch][C][NKS][ny], NKS = pack ? PX/2 : PX/2+1
    cx<T>* work2;              // split form only: [nbatch][C][NKS][PY] (may be null otherwise)
    const cx<T>* Q;            // quarter spectra [2L+1][PX/2+1][PY/2+1], scaled by 1/(PX PY); for pass B
                               // in two halves each column's even frequencies before its odd ones
    const cx<T>* twx;          // exp(-2 pi i q/PX), q < PX
    const cx<T>* twy;          // exp(-2 pi i q/PY), q < PY
    hipStream_t stream;
    const cx<T>* twm = nullptr;   // L > 8: stage twiddles of the mode-axis FFT (length mode_fft_len(L))
    const cx<T>* twyh = nullptr;  // pass B in two halves: see half_twiddles
    int pack = 0;              // 1: x-frequencies 0 and PX/2 share column 0 of the work buffer
    int var[3] = {0, 0, 0};    // kernel variant of passes A, B, C (see apply2d_variant_count)
    // The input's channels other than channel 0 are zero and pass A ran for channel 0 alone, so
    // pass B takes channel 0 only (the other channels' spectra are zero).  The right-hand side K~ f.
    int single_in = 0;
    // Optional coarse correction (operator A, one batch entry): the input of the apply is taken as
    // x + cs P y, y = corr[C][ny/cF][nx/cF] (FP32), P = bilinear interpolation from the coarse
    // cell centres, clamped -- the flexible-GMRES vector z = v + s P N(R v / s) formed on the fly.
    const float* corr = nullptr;
    int cF = 1;
    double cs = 0.0;
    // Set (bcorr.y non-null): pass B adds the correction's x-spectrum (see CorrB); pass A is not
    // run by apply2d_from_b.
    CorrB bcorr;
};

// Kernel variants (same arithmetic, different tiling; results agree up to rounding):
//   passes A and C (PX >= 128): row tiles of 16, 8, 32 or 4 rows (FP32) / 8, 4, 16 or 2 rows (FP64)
//   pass B: one form per shape (passb_wave.h).  The variant numbers of the forms it replaced stay
//   valid and select it.
//   pass B in split form: the coupling as a mode-axis FFT or as a register-blocked direct sum
// Number of variants of `pass` (0 = A, 1 = B, 2 = C) for this shape and precision, and how many of
// them are kernels of their own (the tuner times those).
template <typename T>
int apply2d_variant_count(int pass, int L, int PX, int PY);
template <typename T>
int apply2d_tuned_variants(int pass, int L, int PX, int PY);

// One isotropic problem (C = 1) of a batched apply.  Pass A reads in (+ j * stride when jin is
// set, j read from the device), pass C writes out (+ (j + 1) * stride when jout is set) and reads
// in again (operator A, residual) and bvec (residual).  The x-frequencies 0 and PX/2 are always
// packed into column 0 of the work buffer.
template <typename T>
struct BatchProb {
    int nx, ny, PX, PY;
    double s;                  // pass-A factor: mu_s sigma_0 for A and the residual, 1 for K~
    cx<T>* work;               // [PX/2][ny]
    const cx<T>* Q;            // quarter spectrum [PX/2+1][PY/2+1], scaled by 1/(PX PY)
    const cx<T>* twx;
    const cx<T>* twy;
    const double* in;
    double* out;
    const double* bvec;
    size_t stride;
    int jin, jout;
    const double* scale;       // factor of in per Krylov column (entry j), or null
};

// Batched passes over a list of (problem index, tile) items whose problems all have this PX
// (passes A, C: tiles of apply2d_batch_rows(var) rows) or this PY (pass B: groups of
// apply2d_batch_cols(PY, var) columns).  act[p] == 0 skips problem p (act may be NULL); dj (may be
// NULL) points to the Krylov column index j.  Variants (same arithmetic, different tiling; -1 when
// var is out of range): passes A and C share the row tile (the single-problem row tiles, padded
// x >= 128); pass B takes 4, 2, 8 or 1 waves per block (padded y >= 128; a wave transforms 64 / (PY / 8)
// columns side by side, at least one).
template <typename T>
int apply2d_batch_row_variants(int PX);
template <typename T>
int apply2d_batch_rows(int var);
template <typename T>
int apply2d_batch_col_variants(int PY);
template <typename T>
int apply2d_batch_cols(int PY, int var);
template <typename T>
int apply2d_batch_pass_a(int PX, const BatchProb<T>* probs, const int2* items, int nitems, const int* act,
                         const int* dj, int var, hipStream_t st);
template <typename T>
int apply2d_batch_pass_b(int PY, const BatchProb<T>* probs, const int2* items, int nitems, const int* act, int var,
                         hipStream_t st);
template <typename T>
int apply2d_batch_pass_c(int PX, const BatchProb<T>* probs, const int2* items, int nitems, const int* act,
                         const int* dj, int mode, int var, hipStream_t st);

// y = x - K~ D x (APPLY_A), K~ x (APPLY_KT) or b - (x - K~ D x) (APPLY_RESID) on nbatch channel
// vectors [nbatch][C][ny][nx] stored as TV (float64, or float32 with T = float; b is float64),
// computed with FFTs in precision T.
template <typename T, typename TV>
int apply2d(const Apply2DArgs<T>& a, const TV* x, const double* b, TV* y, int mode,
            const ChanScale& sc, int nbatch);
template <typename T, typename TV>
int apply2d_pass_a(const Apply2DArgs<T>& a, const TV* x, const ChanScale& sc, int nbatch);
// The Gram-Schmidt update of Krylov vector w = K u_j against u_0 .. u_j (rows of V, pitch ld) and pass A
// of the next apply, whose input it is, in one launch (k_update_a); t: the column's Arnoldi state.
// partial takes one partial sum of |u_{j+1}|^2 per block, at most one per grid row; *nblk: their number.
template <typename T, typename TV>
int apply2d_update_a(const Apply2DArgs<T>& a, TV* w, const TV* V, size_t ld, const ArnoldiArgs& t, double* partial,
                     const ChanScale& sc, int nbatch, int* nblk);
template <typename T>
int apply2d_pass_b(const Apply2DArgs<T>& a, int nbatch);
// Whether pass B runs in split form (a full-length buffer, work2, between its transforms and its
// coupling, and the work buffer unpacked: x-frequencies 0 and PX/2 in columns of their own instead
// of sharing column 0): more than 17 modes, except in FP32 up to 33 modes at padded y <= 512, whose
// column spectra fit LDS.  At 256^2, L = 16 in FP32 the split form took 83 us, the other 31 us.
template <typename T>
bool apply2d_split(int L, int PY);
// Whether pass B runs the y-transforms in two halves (twyh needed).
template <typename T>
bool apply2d_b_halves(int L, int PY);
// Where pass B would run in halves, but on so few columns (over nbatch batch entries) that a block per
// column leaves most CUs idle: it takes the split form too (pack = 0, work2; not for single_in, whose
// halves are faster).  FP64 applies in halves and in split form, us: L = 5, 8x512 (8 columns) 37.1 and 23.5,
// 16x512 (16) 34.8 and 22.9, 32x512 (32) 36.0 and 28.0, 64x512 (64) 39.9 and 37.1, 128x512 (128) 46.4 and 48.5;
// L = 8 55.2 and 29.0, 50.3 and 27.0, 52.6 and 36.6, 58.0 and 43.0, 64.8 and 67.6.
template <typename T>
bool apply2d_few_columns(int L, int PX, int PY, int nbatch);
template <typename T, typename TV>
int apply2d_pass_c(const Apply2DArgs<T>& a, const TV* x, const double* b, TV* y, int mode,
                   int nbatch);
// Pass A (pass 0) or C (pass 2) of v = A u or K~ u on general complex mode vectors u, v
// [2L+1][ny][nx] (complex double), as two batch entries of the work buffer (apply2d_modes.hip).  singles > 0:
// on so many [ny][nx] slabs instead, each a channel of its own (3D).
template <typename T>
int apply2d_modes_pass(const Apply2DArgs<T>& a, int pass, const void* u, void* v, int mode, const ChanScale& sc,
                       int singles);
// Passes B and C of y = A (x + cs P y) for one batch entry, pass A having already written the
// x-spectrum of the scaled x alone into a.work; a.bcorr and a.corr describe the correction.
template <typename T, typename TV>
int apply2d_from_b(const Apply2DArgs<T>& a, const TV* x, TV* y);

}  // namespace rte

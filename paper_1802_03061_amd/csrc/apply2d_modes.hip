// The x-passes (2D: A and C, 3D: the first and the last) on general complex mode vectors, in 2D
// u[2L+1][ny][nx] (mode k at row k + L).
//
// Such a vector is two real fields p + i q, whose channels the apply handles as two batch entries
// (channels as in apply2d.hip).  Channel by channel the two are the real and imaginary part of
//     z_0 = u_0,   z_{2k-1} = (u_k + u_-k)/sqrt2,   z_{2k} = -i (u_k - u_-k)/sqrt2.
// Inverse: u_{+-k} = (z_{2k-1} +- i z_{2k})/sqrt2.  The modes are read and written once, in the passes
// themselves; separate conversions to channels and back were two launches and 4 (2L+1) real vectors of
// traffic.
//
// A complex x-transform carries two rows y, y + 1 of one real field, as in the channel form, never p
// and q together: each keeps its own accuracy however far apart they are, and a real flux
// (conjugate-symmetric modes, q = 0) comes back exactly real.  The modes hold p and q of a row side by
// side, so neighbouring lanes take the rows y and y + 1 and exchange halves (swap_pair): the even lane
// goes on with both rows of p, the odd one with both rows of q, and back on the way out.
//
// A block takes R rows (even) of one mode pair (k, -k), 2R transforms (k = 0: R); without PAIR (3D, where every
// mode is a channel) R rows of one slab.  Bound: latency at small grids, HBM at large ones.  Applies
// with conversions and with these passes, us: FP32 200x150, L = 2 33.0 and 24.5; 16^2, L = 7 25.3 and 14.7;
// 512^2, L = 2 63.6 and 50.3; FP64 512^2, L = 0 40.4 and 28.2; 3D FP32 isotropic 32^3 35.8 and 31.9, 128^3
// 154 and 119, 64^3 to degree 2 181 and 157.  (Without the exchange, p and q in one transform: 512^2, L = 2
// 48.8, 128^3 117.)
#include "apply2d.h"
#include "apply2d_tile.h"
#include "fft.h"

namespace rte {

constexpr double kHalfSqrt2 = 0.70710678118654752440084436210485;

// The value of the neighbouring lane (2i <-> 2i + 1); both must be active.
__device__ __forceinline__ int swap_pair(int v) { return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true); }
__device__ __forceinline__ float swap_pair(float v) { return __int_as_float(swap_pair(__float_as_int(v))); }
__device__ __forceinline__ double swap_pair(double v) {
    return __hiloint2double(swap_pair(__double2hiint(v)), swap_pair(__double2loint(v)));
}
template <typename T>
__device__ __forceinline__ cx<T> swap_pair(cx<T> v) { return mk(swap_pair(v.re), swap_pair(v.im)); }
// (za + zb)/sqrt2, or u minus it (of_a).  No fused multiply-adds: modes k and -k then round alike, and
// conjugate inputs give exactly conjugate outputs.
__device__ __forceinline__ cx<double> join_pair(cx<double> za, cx<double> zb, bool of_a, cx<double> u) {
#pragma clang fp contract(off)
    const double re = kHalfSqrt2 * (za.re + zb.re), im = kHalfSqrt2 * (za.im + zb.im);
    return of_a ? mk(u.re - re, u.im - im) : mk(re, im);
}
// Own (p, q) of the lane's row to (row y, row y + 1) of its part, and the reverse (the same exchange).
template <typename E>
__device__ __forceinline__ void exchange(E& first, E& second, int part) {
    const E got = swap_pair(part ? first : second);
    if (part) first = got;
    else second = got;
}

template <typename T, int PX, int R, int NTHR, bool PAIR>
__global__ __launch_bounds__(NTHR) void k_pass_a_modes(const cx<double>* __restrict__ u, cx<T>* __restrict__ Tb,
                                                       const cx<T>* __restrict__ tw, int nx, int ny, int L,
                                                       ChanScale sc, int pack) {
    constexpr int LD = padded(PX) + 1, H = PX / 2;
    constexpr int R0 = fft_radix(PX, 1), NB0 = PX / R0, NBT = R * NB0, IT = (NBT + NTHR - 1) / NTHR;
    __shared__ cx<T> buf[(PAIR ? 2 : 1) * R * LD];
    __shared__ cx<T> tws[PX];
    const int tid = threadIdx.x, k = PAIR ? blockIdx.y : 0;
    const int y0 = xcd_tile(blockIdx.x, gridDim.x) * R;
    const size_t N = (size_t)nx * ny;
    const cx<double>* up = u + (size_t)(PAIR ? L + k : blockIdx.y) * N;
    const cx<double>* um = u + (size_t)(PAIR ? L - k : blockIdx.y) * N;
    stage_twiddles<T, PX, NTHR>(tws, tw, tid);
    cx<double> p[IT][R0 / 2], m[IT][R0 / 2];   // every load before the first use, clamped instead of guarded
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int idx = tid + it * NTHR, j = (idx >> 1) % NB0, y = y0 + 2 * ((idx >> 1) / NB0) + (idx & 1);
#pragma unroll
        for (int r = 0; r < R0 / 2; ++r) {
            const int x = j + r * NB0;
            const size_t o = ((NBT % NTHR == 0 || idx < NBT) && x < nx && y < ny) ? (size_t)y * nx + x : 0;
            p[it][r] = up[o];
            m[it][r] = PAIR ? um[o] : p[it][r];
        }
    }
    const double s = sc.s[k ? 2 * k : 0] * (k ? kHalfSqrt2 : 1.0);
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int idx = tid + it * NTHR, part = idx & 1, j = (idx >> 1) % NB0, rp = (idx >> 1) / NB0;
        const int y = y0 + 2 * rp + part, row = part * (R / 2) + rp;   // row: of the transforms in buf
        if (NBT % NTHR == 0 || idx < NBT) {
            cx<T> a[R0], b[R0];
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                const bool ok = r < R0 / 2 && j + r * NB0 < nx && y < ny;
                const cx<double> vp = p[it][r < R0 / 2 ? r : 0], vm = m[it][r < R0 / 2 ? r : 0];
                const cx<double> za = k ? vp + vm : vp, zb = mul_mi(vp - vm);
                a[r] = ok ? mk((T)(s * za.re), (T)(s * za.im)) : mk((T)0, (T)0);
                b[r] = ok ? mk((T)(s * zb.re), (T)(s * zb.im)) : mk((T)0, (T)0);
                if (r < R0 / 2) {
                    exchange(a[r].re, a[r].im, part);
                    if (PAIR) exchange(b[r].re, b[r].im, part);
                }
            }
            dft_small<T, R0, false>(a);
            if (PAIR) dft_small<T, R0, false>(b);
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                buf[row * LD + sw(j * R0 + r)] = a[r];
                if (PAIR) buf[(R + row) * LD + sw(j * R0 + r)] = b[r];
            }
        }
    }
    __syncthreads();
    if (PAIR && k) fft_stages_range<T, PX, 2 * R, LD, NTHR, false, R0, PX>(buf, tws, tid);
    else fft_stages_range<T, PX, R, LD, NTHR, false, R0, PX>(buf, tws, tid);
    // spectra of the real parts (batch entry 0) and the imaginary parts (entry 1) of each channel
    const int NKS = pack ? H : H + 1, C = PAIR ? 2 * L + 1 : gridDim.y;
    const size_t chan = (size_t)NKS * ny, entry = C * chan;
    const int nf = NKS * R;
    for (int idx = tid; idx < (k ? 2 * nf : nf); idx += NTHR) {
        const int row = idx % R, half = idx >= nf ? 1 : 0, kx = (idx - half * nf) / R, y = y0 + row;
        const int part = row & 1;
        const cx<T>* b = buf + (half * R + part * (R / 2) + row / 2) * LD;
        cx<T> P, Q;   // rows y and y + 1 of the part, then p and q of the row
        if (pack && kx == 0) {   // (X[0], X[PX/2])
            const cx<T> z0 = b[sw(0)], zh = b[sw(H)];
            P = mk(z0.re, zh.re);
            Q = mk(z0.im, zh.im);
        } else {
            const cx<T> z = b[sw(kx)], zc = conj(b[sw((PX - kx) & (PX - 1))]);
            P = scale(z + zc, (T)0.5);
            Q = scale(mul_mi(z - zc), (T)0.5);
        }
        exchange(P, Q, part);
        if (y >= ny) continue;
        cx<T>* out = Tb + (size_t)(PAIR ? (k ? 2 * k - 1 + half : 0) : blockIdx.y) * chan + (size_t)kx * ny + y;
        out[0] = P;
        out[entry] = Q;
    }
}

template <typename T, int PX, int R, int NTHR, bool PAIR>
__global__ __launch_bounds__(NTHR) void k_pass_c_modes(const cx<T>* __restrict__ Tb, const cx<double>* __restrict__ u,
                                                       cx<double>* __restrict__ v, const cx<T>* __restrict__ tw, int nx,
                                                       int ny, int L, int mode, int pack) {
    constexpr int LD = padded(PX) + 1, H = PX / 2;
    __shared__ cx<T> buf[(PAIR ? 2 : 1) * R * LD];
    __shared__ cx<T> tws[PX];
    const int tid = threadIdx.x, k = PAIR ? blockIdx.y : 0;
    const int y0 = xcd_tile(blockIdx.x, gridDim.x) * R;
    const int NKS = pack ? H : H + 1, C = PAIR ? 2 * L + 1 : gridDim.y;
    const size_t N = (size_t)nx * ny, chan = (size_t)NKS * ny, entry = C * chan;
    const cx<T>* src = Tb + (size_t)(PAIR ? (k ? 2 * k - 1 : 0) : blockIdx.y) * chan;
    stage_twiddles<T, PX, NTHR>(tws, tw, tid);
    constexpr int U = 4;   // spectrum entries per thread at a time, loads first
    const int nf = NKS * R, nl = k ? 2 * nf : nf;
    for (int i0 = tid; i0 < nl; i0 += U * NTHR) {
        cx<T> xa[U], xb[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int idx = i0 + q * NTHR, row = idx % R, half = idx >= nf ? 1 : 0, kx = (idx - half * nf) / R;
            const size_t o = idx < nl && y0 + row < ny ? half * chan + (size_t)kx * ny + y0 + row : 0;
            xa[q] = src[o];
            xb[q] = src[o + entry];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int idx = i0 + q * NTHR, row = idx % R, half = idx >= nf ? 1 : 0, kx = (idx - half * nf) / R;
            if (idx >= nl) continue;
            const bool in = y0 + row < ny;
            const int part = row & 1;
            cx<T> P = in ? xa[q] : mk((T)0, (T)0), Q = in ? xb[q] : mk((T)0, (T)0);
            exchange(P, Q, part);
            cx<T>* b = buf + (half * R + part * (R / 2) + row / 2) * LD;
            if (pack && kx == 0) {
                b[sw(0)] = mk(P.re, Q.re);
                b[sw(H)] = mk(P.im, Q.im);
            } else {
                if (kx == 0 || kx == H) { P.im = 0; Q.im = 0; }
                b[sw(kx)] = P + mul_i(Q);
                if (kx > 0 && kx < H) b[sw(PX - kx)] = conj(P) + mul_i(conj(Q));
            }
        }
    }
    __syncthreads();
    // the last stage in registers, both channels of a mode pair by one thread (see pass_c_tile)
    constexpr int NSL = fft_last_ns(PX), RL = PX / NSL, TWL = stage_tw_offset(PX, NSL);
    if (PAIR && k) fft_stages_range<T, PX, 2 * R, LD, NTHR, true, 1, NSL>(buf, tws, tid);
    else fft_stages_range<T, PX, R, LD, NTHR, true, 1, NSL>(buf, tws, tid);
    const cx<double>* up = u + (size_t)(PAIR ? L + k : blockIdx.y) * N;
    const cx<double>* um = u + (size_t)(PAIR ? L - k : blockIdx.y) * N;
    cx<double>* vp = v + (size_t)(PAIR ? L + k : blockIdx.y) * N;
    cx<double>* vm = v + (size_t)(PAIR ? L - k : blockIdx.y) * N;
    for (int idx = tid; idx < R * NSL; idx += NTHR) {
        const int part = idx & 1, j = (idx >> 1) % NSL, rp = (idx >> 1) / NSL;
        const int y = y0 + 2 * rp + part, row = part * (R / 2) + rp;
        cx<double> p[RL / 2], m[RL / 2];
        if (mode == APPLY_A) {
#pragma unroll
            for (int r = 0; r < RL / 2; ++r) {
                const size_t o = (j + r * NSL < nx && y < ny) ? (size_t)y * nx + j + r * NSL : 0;
                p[r] = up[o];
                m[r] = PAIR ? um[o] : p[r];
            }
        }
        cx<T> a[RL], b[RL];
#pragma unroll
        for (int r = 0; r < RL; ++r) {
            a[r] = buf[row * LD + sw(j + r * NSL)];
            b[r] = k ? buf[(R + row) * LD + sw(j + r * NSL)] : mk((T)0, (T)0);
        }
        if constexpr (NSL > 1) {
#pragma unroll
            for (int r = 1; r < RL; ++r) {
                cx<T> w = tws[TWL + j * (RL - 1) + (r - 1)];
                w.im = -w.im;
                a[r] = a[r] * w;
                b[r] = b[r] * w;
            }
        }
        dft_small<T, RL, true>(a);
        if (k) dft_small<T, RL, true>(b);
#pragma unroll
        for (int r = 0; r < RL / 2; ++r) {
            exchange(a[r].re, a[r].im, part);
            if (k) exchange(b[r].re, b[r].im, part);
        }
        if (y >= ny) continue;
#pragma unroll
        for (int r = 0; r < RL / 2; ++r) {
            const int x = j + r * NSL;
            if (x >= nx) continue;
            const size_t o = (size_t)y * nx + x;
            const cx<double> za = cvt<double>(a[r]), zb = mul_i(cvt<double>(b[r]));
            const bool of_a = mode == APPLY_A;
            if (k) {
                vp[o] = join_pair(za, zb, of_a, p[r]);
                vm[o] = join_pair(za, mk(-zb.re, -zb.im), of_a, m[r]);
            } else {
                vp[o] = of_a ? p[r] - za : za;
            }
        }
    }
}

// ---------------------------------------------------------------------------- dispatch -------
// Rows per block (pairs): 2R transforms in at most 70 KB (two blocks per CU), at most 8 rows (64 bytes of a
// spectrum column in FP32), and half of that where the grid would not give every CU a block.  Whole
// applies in FP32 with R and R/2 rows: 200x150, L = 2 (57 blocks of R) 31.6 and 24.4 us; 512^2, L = 0 (128)
// 24.2 and 21.1; 256^2, L = 4 (160) 35.7 and 30.0; 300x257, L = 3 (260) 59.9 and 65.7; 400x300, L = 8 (675)
// 133 and 163.
// FP64 at padded x = 1024: one block per CU either way (two rows and the twiddles take 86 KB), so four rows
// (156 KB, whole 64-byte pieces of a spectrum column) by 512 threads, and two only where their blocks
// still run at once.  Two rows by 256 threads, four by 256 and by 512, us: 512^2, L = 8 316, 301, 283; 300^2,
// L = 16 1326, 1249, 1236 (separate conversions 1262); 512x16, L = 4 (two rows by either) 25.5 and 24.2.
template <typename T, int PX>
constexpr bool modes_wide() { return sizeof(T) == 8 && PX == 1024; }
template <typename T, int PX>
constexpr int mode_rows() {
    int r = modes_wide<T, PX>() ? 4 : 8;
    while (!modes_wide<T, PX>() && r > 2 && 2L * r * (padded(PX) + 1) * (long)sizeof(cx<T>) > 70 * 1024) r /= 2;
    return r;
}
template <typename T, int PX, int R, bool PAIR>
static void launch_modes_r(const Apply2DArgs<T>& a, int pass, const cx<double>* u, cx<double>* v, int mode,
                           const ChanScale& sc, int ngroups) {
    constexpr int NT = modes_wide<T, PX>() ? 512 : 256;
    dim3 grid((a.ny + R - 1) / R, ngroups);
    if (pass == 0)
        hipLaunchKernelGGL((k_pass_a_modes<T, PX, R, NT, PAIR>), grid, dim3(NT), 0, a.stream, u, a.work, a.twx, a.nx, a.ny,
                           a.L, sc, a.pack);
    else
        hipLaunchKernelGGL((k_pass_c_modes<T, PX, R, NT, PAIR>), grid, dim3(NT), 0, a.stream, a.work, u, v, a.twx, a.nx,
                           a.ny, a.L, mode, a.pack);
}
template <typename T, int PX>
static int launch_modes(const Apply2DArgs<T>& a, int pass, const cx<double>* u, cx<double>* v, int mode,
                        const ChanScale& sc, int singles) {
    constexpr int R = mode_rows<T, PX>(), RH = R > 2 ? R / 2 : 2;
    const int ngroups = singles ? singles : a.L + 1;
    const long most = modes_wide<T, PX>() ? 256 : 512;   // blocks of RH rows
    const bool few = (long)((a.ny + R - 1) / R) * ngroups < 256 && (long)((a.ny + RH - 1) / RH) * ngroups <= most;
    if (singles) {
        if (few) launch_modes_r<T, PX, RH, false>(a, pass, u, v, mode, sc, ngroups);
        else launch_modes_r<T, PX, R, false>(a, pass, u, v, mode, sc, ngroups);
    } else {
        if (few) launch_modes_r<T, PX, RH, true>(a, pass, u, v, mode, sc, ngroups);
        else launch_modes_r<T, PX, R, true>(a, pass, u, v, mode, sc, ngroups);
    }
    return 0;
}
template <typename T>
int apply2d_modes_pass(const Apply2DArgs<T>& a, int pass, const void* u, void* v, int mode, const ChanScale& sc,
                       int singles) {
    const auto* x = (const cx<double>*)u;
    auto* y = (cx<double>*)v;
    switch (a.PX) {
        case 16: return launch_modes<T, 16>(a, pass, x, y, mode, sc, singles);
        case 32: return launch_modes<T, 32>(a, pass, x, y, mode, sc, singles);
        case 64: return launch_modes<T, 64>(a, pass, x, y, mode, sc, singles);
        case 128: return launch_modes<T, 128>(a, pass, x, y, mode, sc, singles);
        case 256: return launch_modes<T, 256>(a, pass, x, y, mode, sc, singles);
        case 512: return launch_modes<T, 512>(a, pass, x, y, mode, sc, singles);
        case 1024: return launch_modes<T, 1024>(a, pass, x, y, mode, sc, singles);
    }
    return -1;
}
template int apply2d_modes_pass<float>(const Apply2DArgs<float>&, int, const void*, void*, int, const ChanScale&,
                                       int);
template int apply2d_modes_pass<double>(const Apply2DArgs<double>&, int, const void*, void*, int, const ChanScale&,
                                       int);

}  // namespace rte

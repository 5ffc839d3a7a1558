// 3D FFT apply (Sec. 2.3.1 with d = 3; Sec. 3.1.2 for the spherical-harmonic modes).
//
// u is C real fields [C][nz][ny][nx] (C = 1: isotropic; C = (L+1)^2: the real spherical-harmonic
// modes of sh3d.h).  Isotropic: the kernel h^3 exp(-mu_t r)/(4 pi r^2) has a real, even spectrum,
// stored as the octant Q3[kx][ky][kz] (scaled by 1/(PX PY PZ)).  Modes: the (a, b) block of the
// kernel, kappa(r) Y_a(w) Y_b(w), has a spectrum F_ab = i^(l_b - l_a) R_ab with R_ab real, stored as
// one octant per pair a <= b, and reflecting ky or kz multiplies it by the parities of Y_a and Y_b.
// Five passes per channel:
//   A  x-FFT (real-to-complex) of every row, per z-slab, stored T1[c][z][kx][y]   (2D pass A)
//   B  y-FFT of every (c, z, kx) column times the channel's factor of D, stored T2[c][kx][ky][z]
//   C  z-FFT of every (kx, ky) column of every channel, multiply by the spectrum (C > 1: the
//      mode coupling y_a = sum_b F_ab w_b per frequency), inverse z-FFT, in place
//   D  inverse y-FFT, stored back to T1[c][z][kx][y]
//   E  inverse x-FFT (complex-to-real), crop, y = u - v / v / residual           (2D pass C)
// Each pass reads and writes HBM in 128-byte runs: B and D move tiles of TZ consecutive z.
#include "apply3d.h"
#include "fft_wave.h"
#include "sh3d.h"

#include <algorithm>

namespace rte {

template <typename T, int PY, int TZ, int NTHR>
__global__ __launch_bounds__(NTHR) void k_pass3_b(const cx<T>* __restrict__ T1, cx<T>* __restrict__ T2,
                                                  const cx<T>* __restrict__ tw, int ny, int nz, int nkx, size_t t1sz,
                                                  size_t t2sz, ChanScale3 sc) {
    constexpr int LD = padded(PY) + 1;   // odd row pitch: the TZ transforms start on different banks
    __shared__ cx<T> buf[TZ * LD];
    __shared__ cx<T> tws[PY];
    const int tid = threadIdx.x;
    const int kx = blockIdx.x, z0 = blockIdx.y * TZ, ch = blockIdx.z;
    const T s = (T)sc.s[ch];
    T1 += ch * t1sz;
    T2 += ch * t2sz;
    stage_twiddles<T, PY, NTHR>(tws, tw, tid);
    __syncthreads();
    // rows y >= ny are zero padding: the first stage is computed from the loads
    fft_forward_padded<T, PY, TZ, LD, NTHR>(buf, tws, tid, [&](int zl, int y) {
        const int z = z0 + zl;
        return (z < nz && y < ny) ? scale(T1[((size_t)z * nkx + kx) * ny + y], s) : mk((T)0, (T)0);
    });
    for (int idx = tid; idx < TZ * PY; idx += NTHR) {
        const int zl = idx % TZ, ky = idx / TZ;
        const int z = z0 + zl;
        if (z < nz) T2[((size_t)kx * PY + ky) * nz + z] = buf[zl * LD + sw(ky)];
    }
}

// Isotropic pass C.  Every column is transformed by part of one wave, from its loads to its stores,
// in an LDS row of its own: no block barrier anywhere.  The spectrum multiplies the last forward
// stage's registers; its values and the wave's next columns are loaded ahead of the transforms.
// Bound: HBM.  Between events in FP32 it takes 23.2 us at 128^3 (76 MB) and 121 us at 200^3, where
// block-wide stages over 8 columns with the multiply between two barriers took 28.2 and 168 us.  (The
// same transforms in the spherical-harmonic z-pass below, whose coupling needs the barriers anyway,
// did not change its time.)
template <typename T, int PZ>
__global__ __launch_bounds__(384) void k_pass3_c(cx<T>* __restrict__ T2, const T* __restrict__ Q3,
                                                 const cx<T>* __restrict__ tw, int nz, int PY, int ncol) {
    constexpr int LN = wave_lanes(PZ);
    constexpr int SPW = 64 / LN;            // columns a wave runs side by side
    constexpr int LD = padded(PZ);
    constexpr int NSL = fft_last_ns(PZ), RL = PZ / NSL, R0 = fft_radix(PZ, 1);
    using Last = WaveStage<T, PZ, LN, RL, NSL, false>;
    extern __shared__ __align__(16) double smem_c[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = (threadIdx.x & 63) % LN, sub = (threadIdx.x & 63) / LN;
    cx<T>* buf = reinterpret_cast<cx<T>*>(smem_c) + (wave * SPW + sub) * LD;
    const int HY = PY / 2 + 1, HZ = PZ / 2 + 1;
    const int step = gridDim.x * (blockDim.x / 64) * SPW;
    int col = (blockIdx.x * (blockDim.x / 64) + wave) * SPW + sub;
    WaveIn<T, PZ, LN> in;
    in.load(T2 + (size_t)min(col, ncol - 1) * nz, nz, l);
    // every lane of a wave runs the same number of rounds: columns past the last are not stored
    for (int base = col - sub; base < ncol; base += step, col += step) {
        const int cc = min(col, ncol - 1), kx = cc / PY, ky = cc % PY;
        const T* q = Q3 + ((size_t)kx * HY + (ky <= PY / 2 ? ky : PY - ky)) * HZ;
        T qv[Last::ITEMS][RL];
#pragma unroll
        for (int it = 0; it < Last::ITEMS; ++it)
#pragma unroll
            for (int r = 0; r < RL; ++r) {
                const int kz = (l + it * LN + r * NSL) & (PZ - 1);
                qv[it][r] = q[kz <= PZ / 2 ? kz : PZ - kz];
            }
        in.first_stage(buf, nz, true, l);
        wave_sync();
        if constexpr (NSL > 1) {
            wave_stages<T, PZ, LN, false, R0, NSL>(buf, tw, l);
            cx<T> v[Last::ITEMS][RL];
            Last::compute(v, buf, tw, l);
            wave_sync();
#pragma unroll
            for (int it = 0; it < Last::ITEMS; ++it)
#pragma unroll
                for (int r = 0; r < RL; ++r) v[it][r] = scale(v[it][r], qv[it][r]);
            Last::store(v, buf, l);
        } else if (l == 0) {   // a single stage: lane 0 holds the whole spectrum
#pragma unroll
            for (int r = 0; r < RL; ++r) buf[r] = scale(buf[r], qv[0][r]);
        }
        wave_sync();
        if (base + step < ncol) in.load(T2 + (size_t)min(col + step, ncol - 1) * nz, nz, l);
        wave_inverse<T, PZ, LN>(buf, tw, T2 + (size_t)cc * nz, nz, col < ncol, l);
        wave_sync();
    }
}

// Degree and reflection parities of the first 16 modes, as compile-time tables (sh3d.h).
constexpr int kShDeg[16] = {0, 1, 1, 1, 2, 2, 2, 2, 2, 3, 3, 3, 3, 3, 3, 3};
constexpr int kShNegY[16] = {0, 1, 0, 0, 1, 1, 0, 0, 0, 1, 1, 1, 0, 0, 0, 0};   // m < 0
constexpr int kShNegZ[16] = {0, 0, 1, 0, 0, 1, 0, 1, 0, 0, 1, 0, 1, 0, 1, 0};   // l - |m| odd

template <typename T>
__device__ __forceinline__ cx<T> times_i_pow(cx<T> v, int q) {   // v i^q, q in 0..3
    return q == 0 ? v : q == 1 ? mul_i(v) : q == 2 ? mk(-v.re, -v.im) : mul_mi(v);
}

// Pass C with the mode coupling.  A block takes the column pair (kx, fy) and (kx, PY - fy), which
// read the same octant entries (fy = 0 and PY/2 are single columns): the z-FFT of all CH channels of
// both columns in LDS, then per frequency kz (one thread each, both columns)
//     w'_b = i^(l_b) s_b w_b,   y'_a = sum_b R_ab w'_b,   y_a = i^(-l_a) s_a y'_a,
// s_a = the parities of Y_a for the reflections that map (ky, kz) into the stored octant, which
// equals y_a = sum_b F_ab w_b; R_ba = (-1)^(l_a + l_b) R_ab supplies the lower triangle, and every
// R value read serves both columns.  Then the inverse z-FFT of every channel of both columns.
template <typename T, int PZ, int CH, int NTHR>
__global__ __launch_bounds__(NTHR) void k_pass3_c_sh(cx<T>* __restrict__ T2, const T* __restrict__ Q,
                                                     const cx<T>* __restrict__ tw, int nz, int PY, size_t t2sz,
                                                     size_t noct) {
    constexpr int LD = padded(PZ) + 1;
    __shared__ cx<T> buf[2 * CH * LD];
    __shared__ cx<T> tws[PZ];
    const int tid = threadIdx.x;
    const int HY = PY / 2 + 1, HZ = PZ / 2 + 1;
    const int kx = blockIdx.x / HY, fy = blockIdx.x % HY;
    const bool pair = fy > 0 && fy < PY / 2;
    const size_t col0 = (size_t)kx * PY + fy, col1 = (size_t)kx * PY + (PY - fy);
    stage_twiddles<T, PZ, NTHR>(tws, tw, tid);
    __syncthreads();
    // transforms 0..CH-1: column (kx, fy); CH..2CH-1: column (kx, PY - fy), zero when single
    fft_forward_padded<T, PZ, 2 * CH, LD, NTHR>(buf, tws, tid, [&](int t, int z) {
        const int c = t % CH;
        const bool second = t >= CH;
        return (z < nz && (!second || pair)) ? T2[c * t2sz + (second ? col1 : col0) * nz + z] : mk((T)0, (T)0);
    });
    const T* Qc = Q + ((size_t)kx * HY + fy) * HZ;
    for (int kz = tid; kz < PZ; kz += NTHR) {
        const bool negz = kz > PZ / 2;
        const int fz = negz ? PZ - kz : kz;
        cx<T> w0[CH], y0[CH], w1[CH], y1[CH];
#pragma unroll
        for (int b = 0; b < CH; ++b) {
            // first column: ky = fy <= PY/2 (no y reflection); second: ky = PY - fy (reflected)
            cx<T> v = buf[b * LD + sw(kz)];
            if (kShNegZ[b] && negz) v = mk(-v.re, -v.im);
            w0[b] = times_i_pow(v, kShDeg[b] & 3);
            cx<T> u = buf[(CH + b) * LD + sw(kz)];
            if (kShNegY[b] != (kShNegZ[b] && negz)) u = mk(-u.re, -u.im);
            w1[b] = times_i_pow(u, kShDeg[b] & 3);
            y0[b] = mk((T)0, (T)0);
            y1[b] = mk((T)0, (T)0);
        }
#pragma unroll
        for (int a = 0; a < CH; ++a) {
#pragma unroll
            for (int b = a; b < CH; ++b) {
                const T r = Qc[(size_t)(a * CH - a * (a - 1) / 2 + (b - a)) * noct + fz];
                y0[a].re = fma(r, w0[b].re, y0[a].re);
                y0[a].im = fma(r, w0[b].im, y0[a].im);
                y1[a].re = fma(r, w1[b].re, y1[a].re);
                y1[a].im = fma(r, w1[b].im, y1[a].im);
                if (b != a) {
                    const T rb = ((kShDeg[a] + kShDeg[b]) & 1) ? -r : r;
                    y0[b].re = fma(rb, w0[a].re, y0[b].re);
                    y0[b].im = fma(rb, w0[a].im, y0[b].im);
                    y1[b].re = fma(rb, w1[a].re, y1[b].re);
                    y1[b].im = fma(rb, w1[a].im, y1[b].im);
                }
            }
        }
#pragma unroll
        for (int a = 0; a < CH; ++a) {
            cx<T> v = times_i_pow(y0[a], (4 - (kShDeg[a] & 3)) & 3);
            if (kShNegZ[a] && negz) v = mk(-v.re, -v.im);
            buf[a * LD + sw(kz)] = v;
            cx<T> u = times_i_pow(y1[a], (4 - (kShDeg[a] & 3)) & 3);
            if (kShNegY[a] != (kShNegZ[a] && negz)) u = mk(-u.re, -u.im);
            buf[(CH + a) * LD + sw(kz)] = u;
        }
    }
    __syncthreads();
    fft_inverse_cropped<T, PZ, 2 * CH, LD, NTHR>(buf, tws, tid, [&](int t, int z, cx<T> v) {
        const int c = t % CH;
        const bool second = t >= CH;
        if (z < nz && (!second || pair)) T2[c * t2sz + (second ? col1 : col0) * nz + z] = v;
    });
}

template <typename T, int PY, int TZ, int NTHR>
__global__ __launch_bounds__(NTHR) void k_pass3_d(cx<T>* __restrict__ T1, const cx<T>* __restrict__ T2,
                                                  const cx<T>* __restrict__ tw, int ny, int nz, int nkx, size_t t1sz,
                                                  size_t t2sz) {
    constexpr int LD = padded(PY) + 1;   // odd row pitch: the TZ transforms start on different banks
    __shared__ cx<T> buf[TZ * LD];
    __shared__ cx<T> tws[PY];
    const int tid = threadIdx.x;
    const int kx = blockIdx.x, z0 = blockIdx.y * TZ, ch = blockIdx.z;
    T1 += ch * t1sz;
    T2 += ch * t2sz;
    stage_twiddles<T, PY, NTHR>(tws, tw, tid);
    // every load of the tile is issued before the first LDS store, so their latencies overlap
    constexpr int PER = (TZ * PY + NTHR - 1) / NTHR;
    cx<T> v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int idx = tid + u * NTHR;
        const int zl = idx % TZ, ky = idx / TZ;
        const int z = z0 + zl;
        v[u] = ((TZ * PY) % NTHR == 0 || idx < TZ * PY) && z < nz ? T2[((size_t)kx * PY + ky) * nz + z]
                                                                   : mk((T)0, (T)0);
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int idx = tid + u * NTHR;
        if ((TZ * PY) % NTHR == 0 || idx < TZ * PY) buf[(idx % TZ) * LD + sw(idx / TZ)] = v[u];
    }
    __syncthreads();
    // only rows y < ny are kept: the last inverse stage writes them directly
    fft_inverse_cropped<T, PY, TZ, LD, NTHR>(buf, tws, tid, [&](int zl, int y, cx<T> v) {
        const int z = z0 + zl;
        if (z < nz && y < ny) T1[((size_t)z * nkx + kx) * ny + y] = v;
    });
}

// z-rows per block of the y-passes: 8 (variant 0), 4 or 16 (variants 1, 2).  At 128^3 in FP32, 16
// and 4 rows were slower than 8: 15.1 / 22.3 and 19.4 / 27.0 us for the forward / inverse pass
// against 13.4 / 21.1.
template <typename T, int PY, int TZ>
static void launch3_bd_tz(const Apply3DArgs<T>& a, bool inverse) {
    const int nkx = a.PX / 2 + 1;
    const size_t t1sz = (size_t)a.nz * nkx * a.ny, t2sz = (size_t)nkx * a.PY * a.nz;
    dim3 grid(nkx, (a.nz + TZ - 1) / TZ, a.C);
    if (!inverse)
        hipLaunchKernelGGL((k_pass3_b<T, PY, TZ, 256>), grid, dim3(256), 0, a.stream, a.T1, a.T2, a.twy, a.ny, a.nz,
                           nkx, t1sz, t2sz, a.sc);
    else
        hipLaunchKernelGGL((k_pass3_d<T, PY, TZ, 256>), grid, dim3(256), 0, a.stream, a.T1, a.T2, a.twy, a.ny, a.nz,
                           nkx, t1sz, t2sz);
}

template <typename T, int PY>
static void launch3_bd(const Apply3DArgs<T>& a, bool inverse) {
    const int v = a.var[inverse ? 2 : 0];
    if (v == 1) launch3_bd_tz<T, PY, 4>(a, inverse);
    else if (v == 2) launch3_bd_tz<T, PY, 16>(a, inverse);
    else launch3_bd_tz<T, PY, 8>(a, inverse);
}

// Isotropic pass C with `waves` (2, 4 or 6) waves per block, as many blocks as the device holds at
// once.
template <typename T, int PZ>
static void launch3_c_iso(const Apply3DArgs<T>& a, int ncol, int waves) {
    constexpr int SPW = 64 / wave_lanes(PZ);
    const size_t lds = (size_t)waves * SPW * padded(PZ) * sizeof(cx<T>);
    static const unsigned cap[3] = {resident_blocks(k_pass3_c<T, PZ>, 256, 4 * (lds / waves)),
                                    resident_blocks(k_pass3_c<T, PZ>, 128, 2 * (lds / waves)),
                                    resident_blocks(k_pass3_c<T, PZ>, 384, 6 * (lds / waves))};
    const unsigned need = (unsigned)((ncol + waves * SPW - 1) / (waves * SPW));
    const unsigned nb = std::min(need, cap[waves == 4 ? 0 : (waves == 2 ? 1 : 2)]);
    hipLaunchKernelGGL((k_pass3_c<T, PZ>), dim3(nb), dim3(64 * waves), lds, a.stream, a.T2, a.Q3, a.twz, a.nz, a.PY, ncol);
}

template <typename T, int PZ>
static int launch3_c(const Apply3DArgs<T>& a) {
    const size_t ncol = (size_t)(a.PX / 2 + 1) * a.PY;
    if (a.C == 1) {
        launch3_c_iso<T, PZ>(a, (int)ncol, a.var[1] == 1 ? 2 : (a.var[1] == 2 ? 6 : 4));
        return 0;
    }
    if constexpr (PZ > 256) {
        return -1;                                       // the mode coupling is built for padded z <= 256
    } else {
    const size_t t2sz = ncol * a.nz;
    const size_t noct = (size_t)(a.PX / 2 + 1) * (a.PY / 2 + 1) * (PZ / 2 + 1);
    const unsigned npairs = (unsigned)((a.PX / 2 + 1) * (a.PY / 2 + 1));   // blocks: (kx, fy) column pairs
    constexpr int NT = PZ >= 256 ? 256 : (PZ < 64 ? 64 : PZ);
    switch (a.C) {
#define RTE_CSH(CHN)                                                                                              \
    case CHN:                                                                                                     \
        hipLaunchKernelGGL((k_pass3_c_sh<T, PZ, CHN, NT>), dim3(npairs), dim3(NT), 0, a.stream, a.T2, a.Q3, a.twz,   \
                           a.nz, a.PY, t2sz, noct);                                                               \
        return 0;
        RTE_CSH(4) RTE_CSH(9) RTE_CSH(16)
#undef RTE_CSH
    }
    return -1;
    }
}

template <typename T>
int apply3d_pass(const Apply3DArgs<T>& a, int which) {
    const int P = which == 2 ? a.PZ : a.PY;
    switch (P) {
#define RTE_C3(PP)                                              \
    case PP:                                                    \
        if (which == 1) launch3_bd<T, PP>(a, false);            \
        else if (which == 3) launch3_bd<T, PP>(a, true);        \
        else return launch3_c<T, PP>(a);                        \
        return 0;
        RTE_C3(16) RTE_C3(32) RTE_C3(64) RTE_C3(128) RTE_C3(256) RTE_C3(512)
#undef RTE_C3
    }
    return -1;
}

template <typename T>
int apply3d_variant_count(int which, int C, int PZ) {
    (void)PZ;
    if (which == 1 || which == 3) return 3;
    if (which == 2) return C == 1 ? 3 : 1;
    return 0;
}
template int apply3d_variant_count<float>(int, int, int);
template int apply3d_variant_count<double>(int, int, int);

template int apply3d_pass<float>(const Apply3DArgs<float>&, int);
template int apply3d_pass<double>(const Apply3DArgs<double>&, int);

}  // namespace rte

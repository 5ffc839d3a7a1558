// Pass B with wave-private y-FFTs and the mode coupling in real arithmetic.
//
// A block holds the spectra of NCOL columns x C channels in LDS, and every sequence is transformed by
// one wave (or part of one) from its loads to its spectrum and back, so a transform's stages are ordered
// by the wave alone and the block meets at two barriers per column group: before and after the
// coupling.  Waves drift apart between them, and one wave's LDS latency hides behind another's
// arithmetic.
//
// Coupling.  In the real-channel basis the operator's (c, c') kernel is kappa(r) times a product of
// cos k theta, sin k theta: with Khat_m = C_m + i S_m (the spectra of kappa cos m theta and kappa
// sin m theta), d = k' - k and e = k' + k,
//     A'_k = sum_k' (C_d + C_e) A_k' - (S_d + S_e) B_k',    B'_k = sum_k' (S_d - S_e) A_k' + (C_d - C_e) B_k'
// (k' = 0: sqrt2 C_k A_0 and -sqrt2 S_k A_0).  The kernel of order m has the parity (-1)^m, so C_m and
// S_m are real for even m and imaginary for odd m: with the channels of odd k multiplied by -i the
// matrix is real, and a complex value times an entry takes two multiply-adds instead of four.  At the
// mirror frequency PY - f only the sign of S changes.
//
// Bound and measured (512^2, L = 8, FP32, MI355X): vector arithmetic.  The form this replaces (stages
// by the whole block, complex coupling) took 57-60 us with 21.3M vector instructions and its vector
// units busy 58 % of the time; this one takes 39 us with 16.4M (the column traffic alone: 14 us).
// Without the coupling it takes 29.6 us, without the transforms but for their first and last stages
// 29.5, without both 19.8.  Twiddles are read from memory (L1-resident): staging them in LDS cost each
// block a memory latency and took 0.5 us longer at 256^2.  At 256^2, L = 8 the FP64 apply went from 72 to
// 42 us.  With 33 modes at 256^2 in FP32 pass B takes 31 us, where forward transforms, a register-blocked
// complex coupling and inverse transforms through a full-length buffer took 83 us.
#pragma once
#include "apply2d.h"
#include "fft_wave.h"
#include "spectra.h"

namespace rte {

// Adds the coarse correction's x-spectrum (CorrB) to the loaded rows of the sequence of channel c
// in column kx: G[R] = coef_c sum_X y_c[R][X] phi[X][kx], one coarse row R per lane at a time, goes
// through the transform's own LDS row (not in use yet), then interpolates in y onto every row.
template <typename T, int P, int LN>
__device__ __forceinline__ void wave_corr(WaveIn<T, P, LN>& in, cx<T>* buf, const CorrB& cb, int c, int kx, int nkx,
                                          int ny, int l) {
    const cx<T>* phi = reinterpret_cast<const cx<T>*>(cb.phi) + kx;
    const int Hc = cb.Hc, Wc = cb.Wc;
    const T k = (T)cb.coef[c];
    for (int R = l; R < Hc; R += LN) {
        const float4* y4 = reinterpret_cast<const float4*>(cb.y + ((size_t)c * Hc + R) * Wc);
        T gr = 0, gi = 0;
        for (int X = 0; X < Wc; X += 4) {   // whole float4s, see CorrB
            const float4 t = y4[X / 4];
            const float yv[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const cx<T> ph = phi[(size_t)(X + u) * nkx];
                gr += (T)yv[u] * ph.re;
                gi += (T)yv[u] * ph.im;
            }
        }
        buf[R] = mk(k * gr, k * gi);
    }
    wave_sync();
    const float invF = 1.f / (float)cb.F;
    using W = WaveIn<T, P, LN>;
#pragma unroll
    for (int it = 0; it < W::ITEMS; ++it)
#pragma unroll
        for (int r = 0; r < W::R0 / 2; ++r) {
            const float yi = ((float)(l + it * LN + r * W::NB) + 0.5f) * invF - 0.5f;
            const float f0 = floorf(yi);
            const int i0 = (int)f0;
            const int lo = min(max(i0, 0), Hc - 1);
            const T wt = (i0 < 0 || i0 >= Hc - 1) ? (T)0 : (T)(yi - f0);
            const cx<T> g0 = buf[lo], g1 = buf[min(lo + 1, Hc - 1)];
            in.v[it][r].re += g0.re + wt * (g1.re - g0.re);
            in.v[it][r].im += g0.im + wt * (g1.im - g0.im);
        }
    wave_sync();
}

// The real form of Khat_m: (c, s) with C_m = c, S_m = s for even m and C_m = i c, S_m = i s for odd m.
template <typename T>
__device__ __forceinline__ void khat_real(cx<T> K, int m, T& c, T& s) {
    c = (m & 1) ? K.im : K.re;
    s = (m & 1) ? -K.re : K.im;
}

// Channels of odd k times -i on the way in, times i on the way out.
template <typename T>
__device__ __forceinline__ cx<T> phase_in(cx<T> z, int k) { return (k & 1) ? mul_mi(z) : z; }
template <typename T>
__device__ __forceinline__ cx<T> phase_out(cx<T> z, int k) { return (k & 1) ? mul_i(z) : z; }

// The entry sums of modes k and q (both >= 1), with the sign that the phases leave: A'_k takes aa A_q +
// ab B_q, B'_k takes ba A_q + bb B_q.
template <typename T, int L>
struct PairSums {
    T p, m, sp, sm;   // C_d + C_e, C_d - C_e, S_d + S_e, S_d - S_e with d = q - k, e = q + k
    __device__ __forceinline__ PairSums(const T (&c)[2 * L + 1], const T (&s)[2 * L + 1], int k, int q) {
        const int d = q > k ? q - k : k - q, e = q + k;
        const T sd = q > k ? s[d] : (q < k ? -s[d] : (T)0);
        p = c[d] + c[e];
        m = c[d] - c[e];
        sp = sd + s[e];
        sm = sd - s[e];
    }
};
template <typename T>
__device__ __forceinline__ void rmac(cx<T>& o, T r, cx<T> z) {
    o.re = fma(r, z.re, o.re);
    o.im = fma(r, z.im, o.im);
}
// modes of opposite parity: -1 into an even mode, +1 into an odd one
constexpr bool pair_neg(int k, int q) { return ((k ^ q) & 1) && !(k & 1); }

// Row k = 0: A'_0 = C_0 A_0 + sqrt2 sum_q (C_q A_q - S_q B_q).
template <typename T, int L>
__device__ __forceinline__ cx<T> couple_row0(const cx<T> (&a)[L + 1], const cx<T> (&b)[L + 1],
                                             const T (&c)[2 * L + 1], const T (&s)[2 * L + 1]) {
    cx<T> t = mk((T)0, (T)0);
#pragma unroll
    for (int q = 1; q <= L; ++q) {
        rmac(t, (q & 1) ? -c[q] : c[q], a[q]);
        rmac(t, (q & 1) ? s[q] : -s[q], b[q]);
    }
    const T r2 = (T)1.41421356237309504880168872420970;
    return mk(fma(c[0], a[0].re, r2 * t.re), fma(c[0], a[0].im, r2 * t.im));
}

// The channels (a: A_k, b: B_k, phases taken out) coupled with the real entries c[m], s[m], m = 0..2L,
// one output mode after another; st(channel, value) takes the outputs.
template <typename T, int L, typename ST>
__device__ __forceinline__ void couple_rows(const cx<T> (&a)[L + 1], const cx<T> (&b)[L + 1], T (&c)[2 * L + 1],
                                            T (&s)[2 * L + 1], ST st) {
    st(0, couple_row0<T, L>(a, b, c, s));
    const cx<T> a0 = scale(a[0], (T)1.41421356237309504880168872420970);
#pragma unroll
    for (int k = 1; k <= L; ++k) {
        // The entry sums of row k also appear in other rows, and the compiler would keep them all
        // live for that (spilling); hiding where c and s come from makes each row form its own.
#pragma unroll
        for (int m = 0; m <= 2 * L; ++m) asm volatile("" : "+v"(c[m]), "+v"(s[m]));
        __builtin_amdgcn_sched_barrier(0);
        cx<T> oa = scale(a0, c[k]), ob = scale(a0, -s[k]);
#pragma unroll
        for (int q = 1; q <= L; ++q) {
            const PairSums<T, L> e(c, s, k, q);
            const bool n = pair_neg(k, q);
            rmac(oa, n ? -e.p : e.p, a[q]);
            rmac(ob, n ? -e.sm : e.sm, a[q]);
            rmac(oa, n ? e.sp : -e.sp, b[q]);
            rmac(ob, n ? -e.m : e.m, b[q]);
        }
        st(2 * k - 1, phase_out(oa, k));
        st(2 * k, phase_out(ob, k));
    }
}

// The same with every output accumulating at once: the four sums of an unordered pair of modes serve
// both of its rows (half the additions, 2 (2L+1) more live values: 41.0 -> 38.6 us at 512^2, L = 8 in
// FP32; FP64 in halves has no registers left for it).
template <typename T, int L, typename ST>
__device__ __forceinline__ void couple_all(const cx<T> (&a)[L + 1], const cx<T> (&b)[L + 1], T (&c)[2 * L + 1],
                                           T (&s)[2 * L + 1], ST st) {
    st(0, couple_row0<T, L>(a, b, c, s));
    const T r2 = (T)1.41421356237309504880168872420970;
    const cx<T> a0 = scale(a[0], r2);
    cx<T> oa[L + 1], ob[L + 1];
#pragma unroll
    for (int k = 1; k <= L; ++k) {
        oa[k] = scale(a0, c[k]);
        ob[k] = scale(a0, -s[k]);
    }
#pragma unroll
    for (int k = 1; k <= L; ++k) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = k; q <= L; ++q) {
            const PairSums<T, L> e(c, s, k, q);
            const bool n = pair_neg(k, q), nq = pair_neg(q, k);
            rmac(oa[k], n ? -e.p : e.p, a[q]);
            rmac(ob[k], n ? -e.sm : e.sm, a[q]);
            rmac(oa[k], n ? e.sp : -e.sp, b[q]);
            rmac(ob[k], n ? -e.m : e.m, b[q]);
            if (q > k) {   // row q, column k: d changes sign
                rmac(oa[q], nq ? -e.p : e.p, a[k]);
                rmac(ob[q], nq ? e.sp : -e.sp, a[k]);
                rmac(oa[q], nq ? -e.sm : e.sm, b[k]);
                rmac(ob[q], nq ? -e.m : e.m, b[k]);
            }
        }
        st(2 * k - 1, phase_out(oa[k], k));
        st(2 * k, phase_out(ob[k], k));
    }
}

// The 2L+1 kernel entries of one column at frequency f (0 <= f <= PY/2); q: the column in the table
// of m = 0, the same for all lanes where the block holds one column.
template <typename T, int L>
__device__ __forceinline__ void load_entries(const cx<T>* __restrict__ q, size_t qs, unsigned f, T (&c)[2 * L + 1],
                                             T (&s)[2 * L + 1]) {
#pragma unroll
    for (int m = 0; m <= 2 * L; ++m) khat_real((q + m * qs)[f], m, c[m], s[m]);
}

// Channel row pitch in LDS: at least two pad slots (index 16 and 17 or 33, which sw() never yields).
constexpr int wave_ld(int P) { return padded(P) < 18 ? 18 : padded(P); }
// A pad slot for each of the two self-mirrored frequencies 0 and PY/2.
constexpr int self_slot(int P, int f) { return f == 0 ? 16 : (P == 16 ? 17 : 33); }

// The slots of one frequency in every channel row of a column.  LDS instructions carry a 64 KB
// immediate offset, so a few byte offsets, PER channels apart, reach all rows; they are hidden from
// the compiler, which would otherwise keep one address register per row beyond the first 64 KB.
template <typename T, int C, int LD>
struct Slots {
    static constexpr int PITCH = LD * (int)sizeof(cx<T>);
    static constexpr int PER = 65535 / PITCH < C ? 65535 / PITCH : C;
    static constexpr int N = (C + PER - 1) / PER;
    char* base;
    unsigned o[N];
    __device__ __forceinline__ Slots(cx<T>* sp, int slot) : base(reinterpret_cast<char*>(sp)) {
        o[0] = (unsigned)slot * (unsigned)sizeof(cx<T>);
#pragma unroll
        for (int i = 1; i < N; ++i) {
            o[i] = o[i - 1] + PER * PITCH;
            asm volatile("" : "+v"(o[i]));
        }
    }
    __device__ __forceinline__ cx<T>& operator[](int ch) const {
        return *reinterpret_cast<cx<T>*>(base + o[ch / PER] + (ch % PER) * PITCH);
    }
};

// The coupling of one slot of every channel row, in place, with the entries at frequency f of
// kernel column q (flip: the slot is the mirror frequency's).
template <typename T, int L, int LD, bool ALL>
__device__ __forceinline__ void couple_single(cx<T>* sp, int slot, const cx<T>* __restrict__ q, size_t qs, int f,
                                              bool flip) {
    constexpr int C = 2 * L + 1;
    T c[2 * L + 1], s[2 * L + 1];
    load_entries<T, L>(q, qs, f, c, s);
    const T sg = flip ? (T)-1 : (T)1;
#pragma unroll
    for (int m = 0; m <= 2 * L; ++m) s[m] *= sg;
    const Slots<T, C, LD> p(sp, slot);
    cx<T> a[L + 1], b[L + 1];
    a[0] = p[0];
#pragma unroll
    for (int k = 1; k <= L; ++k) {
        a[k] = phase_in(p[2 * k - 1], k);
        b[k] = phase_in(p[2 * k], k);
    }
    if constexpr (ALL) couple_all<T, L>(a, b, c, s, [&](int ch, cx<T> z) { p[ch] = z; });
    else couple_rows<T, L>(a, b, c, s, [&](int ch, cx<T> z) { p[ch] = z; });
}

// The same when only channel 0 of the input is non-zero (its slot alone is read).
template <typename T, int L, int LD>
__device__ __forceinline__ void couple_first(cx<T>* sp, int slot, const cx<T>* __restrict__ q, size_t qs, int f,
                                             bool flip) {
    const Slots<T, 2 * L + 1, LD> p(sp, slot);
    const T r2 = (T)1.41421356237309504880168872420970, sg = flip ? -r2 : r2;
    const cx<T> a0 = p[0];
#pragma unroll
    for (int k = 0; k <= L; ++k) {
        T c, s;
        khat_real((q + k * qs)[f], k, c, s);
        if (k == 0) {
            p[0] = scale(a0, c);
        } else {
            p[2 * k - 1] = phase_out(scale(a0, r2 * c), k);
            p[2 * k] = phase_out(scale(a0, -sg * s), k);
        }
    }
}

// Column 0 of a packed work buffer holds z = d + i q with d, q the real x-frequency-0 and PX/2
// sequences.  Their spectra D = (Z(f) + conj Z(-f))/2 and Q = (Z(f) - conj Z(-f))/(2i), moved into the
// Z(f) and Z(-f) slots (at f = 0 and PY/2 a pad slot for Q), are coupled with kernel columns of
// their own and joined again (D' and Q' are spectra of real sequences too).  f in 0 .. PY/2.
template <int PY>
__device__ __forceinline__ int packed_q_slot(int f) {
    const int fm = (PY - f) & (PY - 1);
    return fm == f ? self_slot(PY, f) : sw(fm);
}
template <typename T, int PY, int C, int LD>
__device__ __forceinline__ void packed_split(cx<T>* sp, int f) {
    const Slots<T, C, LD> p0(sp, sw(f)), p1(sp, sw((PY - f) & (PY - 1))), w1(sp, packed_q_slot<PY>(f));
#pragma unroll
    for (int ch = 0; ch < C; ++ch) {
        const cx<T> z = p0[ch], w = conj(p1[ch]);
        p0[ch] = scale(z + w, (T)0.5);
        w1[ch] = scale(mul_mi(z - w), (T)0.5);
    }
}
template <typename T, int PY, int C, int LD>
__device__ __forceinline__ void packed_join(cx<T>* sp, int f) {
    const Slots<T, C, LD> p0(sp, sw(f)), w1(sp, packed_q_slot<PY>(f));
#pragma unroll
    for (int ch = 0; ch < C; ++ch) {
        const cx<T> d = p0[ch], q = w1[ch];
        p0[ch] = d + mul_i(q);
        w1[ch] = conj(d) + mul_i(conj(q));
    }
}

// The coupling phase of one column group: every frequency of its columns, between two barriers.
// Items: the D and Q spectra of a packed column 0 (they share the block's threads), then the other
// columns' frequencies.
template <typename T, int PY, int L, int NCOL, int NTHR>
__device__ __forceinline__ void couple_phase(cx<T>* spec, const cx<T>* __restrict__ Q, size_t qs, int nkq, int kx0,
                                             int nkx, bool packed, bool single, int tid) {
    constexpr int C = 2 * L + 1;
    constexpr int LD = wave_ld(PY);
    constexpr int KH = PY / 2 + 1;
    const int npk = packed ? 2 * KH : 0, ncol = min(NCOL, nkx - kx0) - (packed ? 1 : 0);
    __syncthreads();
    if (packed) {
        for (int f = tid; f < KH; f += NTHR) packed_split<T, PY, C, LD>(spec, f);
        __syncthreads();
    }
#pragma unroll 1
    for (int idx = hide(tid); idx < npk + ncol * PY; idx += NTHR) {
        const int i = idx - npk;
        const int col = NCOL == 1 ? 0 : (packed ? 1 : 0) + i / PY;
        int f = NCOL == 1 ? i : i % PY, kx = kx0 + col, slot = sw(f);
        cx<T>* sp = spec + col * C * LD;
        const bool flip = i >= 0 && f > PY / 2;
        if (i < 0) {
            const bool isq = idx >= KH;
            f = isq ? idx - KH : idx;
            slot = isq ? packed_q_slot<PY>(f) : sw(f);
            kx = isq ? nkq - 1 : 0;
            sp = spec;
        } else if (flip) {
            f = PY - f;
        }
        if (single) couple_first<T, L, LD>(sp, slot, Q + (size_t)kx * KH, qs, f, flip);
        else couple_single<T, L, LD, true>(sp, slot, Q + (size_t)kx * KH, qs, f, flip);
    }
    __syncthreads();
    if (packed) {
        for (int f = tid; f < KH; f += NTHR) packed_join<T, PY, C, LD>(spec, f);
        __syncthreads();
    }
}

// Blocks loop over the (batch entry, column group) items blockIdx.x, blockIdx.x + gridDim.x, ...; the
// next item's column loads are issued before the current inverse transforms, so their latency
// and the stores' drain hide behind arithmetic.  A wave with more than one sequence runs them two
// at a time.
template <typename T, int PY, int L, int NCOL, int NW, bool CORR>
__global__ __launch_bounds__(NW * 64) void k_pass_b_wave(cx<T>* __restrict__ Tb, const cx<T>* __restrict__ Q,
                                                         const cx<T>* __restrict__ tw, int ny, int nkx, int nkq,
                                                         int pack, int single, int ngrp, int nitems, CorrB cb) {
    constexpr int C = 2 * L + 1;
    constexpr int NSEQ = NCOL * C;
    constexpr int LD = wave_ld(PY);
    constexpr int LN = wave_lanes(PY);
    constexpr int SPW = 64 / LN;                       // transforms a wave runs side by side
    constexpr int NP = (NSEQ + NW * SPW - 1) / (NW * SPW);   // rounds
    __shared__ cx<T> spec[NSEQ * LD];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l0 = (tid & 63) % LN, sub = (tid & 63) / LN;
    const size_t cstride = (size_t)nkx * ny;
    const size_t qs = (size_t)nkq * (PY / 2 + 1);
    auto seq_of = [&](int p) { return (p * NW + wave) * SPW + sub; };
    auto seq_ptr = [&](int item, int s) {   // sequence s of an item (clamped into the buffer)
        const int b = item / ngrp, kx = min((item % ngrp) * NCOL + s / C, nkx - 1);
        return Tb + ((size_t)b * C + s % C) * cstride + (size_t)kx * ny;
    };
    using In = WaveIn<T, PY, LN>;
    In cur;
    int item = blockIdx.x;
    if (seq_of(0) < NSEQ) cur.load(seq_ptr(item, seq_of(0)), ny, l0);
    for (; item < nitems; item += gridDim.x) {
        const int kx0 = (item % ngrp) * NCOL;
        // first stage of sequence s from its loads
        auto first = [&](In& in, int s, int l) {
            cx<T>* buf = spec + s * LD;
            const int kx = kx0 + s / C;
            if constexpr (CORR) wave_corr<T, PY, LN>(in, buf, cb, s % C, min(kx, nkx - 1), nkx, ny, l);
            in.first_stage(buf, ny, kx < nkx && (!single || s % C == 0), l);
        };
#pragma unroll
        for (int p = 0; p < NP; p += 2) {
            const int s = seq_of(p), s1 = seq_of(p + 1), s2 = seq_of(p + 2);
            const int l = hide(l0);
            if (p + 1 < NP && s1 < NSEQ) {
                In nxt;
                nxt.load(seq_ptr(item, s1), ny, l);
                first(cur, s, l);
                if (p + 2 < NP && s2 < NSEQ) cur.load(seq_ptr(item, s2), ny, l);
                first(nxt, s1, l);
                wave_sync();
                wave_stages2<T, PY, LN, false, fft_radix(PY, 1), PY>(spec + s * LD, spec + s1 * LD, tw, l);
            } else if (s < NSEQ) {
                first(cur, s, l);
                wave_sync();
                wave_stages<T, PY, LN, false, fft_radix(PY, 1), PY>(spec + s * LD, tw, l);
            }
        }
        couple_phase<T, PY, L, NCOL, NW * 64>(spec, Q, qs, nkq, kx0, nkx, pack && kx0 == 0, single != 0,
                                                         tid);
        const int next = item + gridDim.x;
        if (next < nitems && seq_of(0) < NSEQ) cur.load(seq_ptr(next, seq_of(0)), ny, hide(l0));
#pragma unroll
        for (int p = 0; p < NP; p += 2) {
            const int s = seq_of(p), s1 = seq_of(p + 1);
            const int l = hide(l0);
            const bool two = p + 1 < NP && s1 < NSEQ;
            if (two) wave_stages2<T, PY, LN, true, 1, fft_last_ns(PY)>(spec + s * LD, spec + s1 * LD, tw, l);
            if (s < NSEQ) wave_inverse<T, PY, LN>(spec + s * LD, tw, seq_ptr(item, s), ny, kx0 + s / C < nkx, l, two);
            if (two) wave_inverse<T, PY, LN>(spec + s1 * LD, tw, seq_ptr(item, s1), ny, kx0 + s1 / C < nkx, l, true);
        }
    }
}

// ---- columns whose spectra exceed LDS: the y-transform in two halves --------------------------
//
// The first decimation-in-frequency step splits the length-PY transform into its even and odd
// frequencies: the length-PH = PY/2 transforms of x[n] and of x[n] W^n (W = exp(-2 pi i / PY); x is
// zero past ny <= PH).  A block takes one column and runs the halves one after the other, half the
// spectra of every channel in LDS at a time; the inverse is e[n] + W^-n o[n] of the halves' inverses,
// with e kept in registers (a third round's in a spare LDS row) while the odd half runs.  The column
// is read twice (the second time from the caches; up to L = 6 there are registers to hold one of a
// wave's rows) and written once; no full-length buffer.  The quarter spectra are kept even frequencies
// first (half_entry), so that each half reads whole lines of its own: with frequencies in order both
// halves fetched every line.  At 512^2 in FP64 this took pass B from 98 to 88 us for L = 8 and from 73
// to 66 for L = 6 (holding rows at L = 8 spills: 94 and 101 us for one and two); forward transforms,
// coupling and inverse transforms through a full-length buffer (785 MB, at the HBM rate) took 150 us.

// All PH inputs of a transform's first stage.
template <typename T, int P, int LN>
struct WaveFull {
    static constexpr int R0 = fft_radix(P, 1);
    static constexpr int NB = P / R0;
    static constexpr int ITEMS = NB > LN ? NB / LN : 1;
    static_assert(NB >= LN, "every lane has a butterfly");
    cx<T> v[ITEMS][R0];
    __device__ __forceinline__ void load(const cx<T>* __restrict__ src, int ny, int l) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                const int n = l + it * LN + r * NB;
                v[it][r] = src[n < ny ? n : 0];
            }
    }
    // w != nullptr: inputs times w[n]
    __device__ __forceinline__ void first_stage(cx<T>* buf, const cx<T>* __restrict__ w, int ny, int l) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int j = l + it * LN;
            cx<T> z[R0];
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                z[r] = j + r * NB < ny ? v[it][r] : mk((T)0, (T)0);
                if (w) z[r] = z[r] * w[j + r * NB];
            }
            dft_small<T, R0, false>(z);
            cx<T>* dst = buf + sw(j * R0);
#pragma unroll
            for (int r = 0; r < R0; ++r) dst[sw_step(r, 1)] = z[r];
        }
    }
};

// Slot (index in the half) of the mirror of slot k of half h: f = 2k + h.
template <int PH>
__device__ __forceinline__ int half_mirror(int k, int h) { return (PH - k - h) & (PH - 1); }
// Where the packed column's Q at slot k is kept (see packed_q_slot).
template <int PH>
__device__ __forceinline__ int half_q_slot(int k, int h) {
    const int km = half_mirror<PH>(k, h);
    return km == k ? (k == 0 ? 16 : 33) : sw(km);
}

template <typename T, int PY, int L, int NW>
__global__ __launch_bounds__(NW * 64) void k_pass_b_half(cx<T>* __restrict__ Tb, const cx<T>* __restrict__ Q,
                                                         const cx<T>* __restrict__ twh, int ny, int nkx, int nkq,
                                                         int pack, int single, int nitems) {
    constexpr int C = 2 * L + 1;
    constexpr int PH = PY / 2;
    constexpr int KH = PH + 1;
    constexpr int LN = wave_lanes(PH);
    static_assert(LN == 64, "one transform per wave");
    constexpr int NP = (C + NW - 1) / NW;
    constexpr int HOLD = L <= 6 ? 1 : 0;   // input rows kept from the even half to the odd one
    constexpr int NTHR = NW * 64;
    constexpr int LD = wave_ld(PH);
    constexpr int NSL = fft_last_ns(PH), RL = PH / NSL;
    using Last = WaveStage<T, PH, LN, RL, NSL, true>;
    __shared__ cx<T> spec[(C + (NP > 2 ? C - 2 * NW : 0)) * LD];
    const cx<T>* wn = twh + PH;   // W^n after the stage twiddles
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l0 = tid & 63;
    const size_t cstride = (size_t)nkx * ny;
    const size_t qs = (size_t)nkq * KH;
#pragma unroll 1
    for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
        const int kx = item % nkx;
        const bool packed = pack && kx == 0;
        cx<T>* col = Tb + (size_t)(item / nkx) * C * cstride + (size_t)kx * ny;
        cx<T> e[NP < 2 ? NP : 2][Last::ITEMS][RL];
        WaveFull<T, PH, LN> held[HOLD < 1 ? 1 : HOLD];
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int s = p * NW + wave, l = hide(l0);
                if (s < C && (!single || s == 0)) {
                    WaveFull<T, PH, LN> again;
                    WaveFull<T, PH, LN>& in = p < HOLD ? held[p < HOLD ? p : 0] : again;
                    if (p >= HOLD || h == 0) in.load(col + s * cstride, ny, l);
                    in.first_stage(spec + s * LD, h ? wn : nullptr, ny, l);
                    wave_sync();
                    wave_stages<T, PH, LN, false, fft_radix(PH, 1), PH>(spec + s * LD, twh, l);
                }
            }
            __syncthreads();
            const int npk = packed ? (h ? PH / 2 : PH / 2 + 1) : 0;   // mirror pairs of the half
            if (packed) {
                for (int k = tid; k < npk; k += NTHR) {
                    const Slots<T, C, LD> p0(spec, sw(k)), p1(spec, sw(half_mirror<PH>(k, h))),
                        w1(spec, half_q_slot<PH>(k, h));
#pragma unroll
                    for (int ch = 0; ch < C; ++ch) {
                        if (single && ch > 0) continue;
                        const cx<T> z = p0[ch], w = conj(p1[ch]);
                        p0[ch] = scale(z + w, (T)0.5);
                        w1[ch] = scale(mul_mi(z - w), (T)0.5);
                    }
                }
                __syncthreads();
            }
#pragma unroll 1
            for (int idx = hide(tid); idx < (packed ? 2 * npk : PH); idx += NTHR) {
                int k = idx, slot = sw(idx), kq = kx;
                if (packed) {
                    const bool isq = idx >= npk;
                    k = isq ? idx - npk : idx;
                    slot = isq ? half_q_slot<PH>(k, h) : sw(k);
                    kq = isq ? nkq - 1 : 0;
                }
                const int f = 2 * k + h;
                const bool flip = f > PH;
                const cx<T>* q = Q + (size_t)kq * KH;
                const int fe = half_entry(flip ? PY - f : f, PY);
                if (single) couple_first<T, L, LD>(spec, slot, q, qs, fe, flip);
                else couple_single<T, L, LD, false>(spec, slot, q, qs, fe, flip);
            }
            __syncthreads();
            if (packed) {
                for (int k = tid; k < npk; k += NTHR) {
                    const Slots<T, C, LD> p0(spec, sw(k)), w1(spec, half_q_slot<PH>(k, h));
#pragma unroll
                    for (int ch = 0; ch < C; ++ch) {
                        const cx<T> d = p0[ch], q = w1[ch];
                        p0[ch] = d + mul_i(q);
                        w1[ch] = conj(d) + mul_i(conj(q));
                    }
                }
                __syncthreads();
            }
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int s = p * NW + wave, l = hide(l0);
                if (s < C) {
                    cx<T>* buf = spec + s * LD;
                    cx<T>* park = spec + (s + C - 2 * NW) * LD;   // p >= 2 only
                    wave_stages<T, PH, LN, true, 1, NSL>(buf, twh, l);
                    cx<T> v[Last::ITEMS][RL];
                    Last::compute(v, buf, twh, l);
                    wave_sync();
#pragma unroll
                    for (int it = 0; it < Last::ITEMS; ++it)
#pragma unroll
                        for (int r = 0; r < RL; ++r) {
                            const int n = l + it * LN + r * NSL;
                            if (h == 0) {
                                if (p < 2) e[p < 2 ? p : 0][it][r] = v[it][r];
                                else park[n] = v[it][r];
                            } else if (n < ny) {
                                const cx<T> ev = p < 2 ? e[p < 2 ? p : 0][it][r] : park[n];
                                col[s * cstride + n] = ev + v[it][r] * conj(wn[n]);
                            }
                        }
                }
            }
        }
    }
}

// ---- isotropic media: nothing couples the columns ---------------------------------------------
//
// Each column is transformed by one wave or part of one, from its loads to its stores, in an LDS row
// of its own: no block barrier.  The spectrum is real and multiplies the last forward stage's
// registers, except in a packed column 0, whose frequencies f and -f mix (packed_split) and are
// multiplied in LDS.  in: the column's rows, loaded; q: its kernel column, KH = PY/2 + 1 entries; nkq
// columns of them.  with_packed (the same for the whole wave): one of the wave's columns may be packed.
template <typename T, int PY>
__device__ __forceinline__ void iso_column(const WaveIn<T, PY, wave_lanes(PY)>& in, cx<T>* __restrict__ col,
                                           const cx<T>* __restrict__ Q, const cx<T>* __restrict__ tw, int kx, int ny,
                                           int nkq, bool live, bool with_packed, bool pack, cx<T>* buf, int l) {
    constexpr int LN = wave_lanes(PY), KH = PY / 2 + 1;
    constexpr int NSL = fft_last_ns(PY), RL = PY / NSL, R0 = fft_radix(PY, 1);
    using Last = WaveStage<T, PY, LN, RL, NSL, false>;
    const cx<T>* q = Q + (size_t)kx * KH;
    const bool packed = pack && kx == 0;
    T qv[Last::ITEMS][RL];
#pragma unroll
    for (int it = 0; it < Last::ITEMS; ++it)
#pragma unroll
        for (int r = 0; r < RL; ++r) {
            const int f = (l + it * LN + r * NSL) & (PY - 1);
            qv[it][r] = q[f <= PY / 2 ? f : PY - f].re;
        }
    if constexpr (NSL == 1) {
        // padded y = 16: one lane holds the whole column, and the spectrum stays in its registers (through LDS the
        // launch took 4.0 us in FP64 and 3.5 in FP32, now 3.1; 512x8 15.4 -> 14.2 us per apply)
        if (l != 0 || !live) return;
        cx<T> w[PY];
#pragma unroll
        for (int r = 0; r < PY; ++r) w[r] = r < PY / 2 && r < ny ? in.v[0][r < PY / 2 ? r : 0] : mk((T)0, (T)0);
        dft_small<T, PY, false>(w);
        if (packed) {
            const cx<T>* qn = Q + (size_t)(nkq - 1) * KH;
#pragma unroll
            for (int f = 0; f <= PY / 2; ++f) {
                const int fm = (PY - f) & (PY - 1);
                const cx<T> z = w[f], c = conj(w[fm]);
                const cx<T> D = scale(z + c, (T)0.5 * qv[0][f]), E = scale(mul_mi(z - c), (T)0.5 * qn[f].re);
                w[f] = D + mul_i(E);
                if (fm != f) w[fm] = conj(D) + mul_i(conj(E));
            }
        } else {
#pragma unroll
            for (int r = 0; r < PY; ++r) w[r] = scale(w[r], qv[0][r]);
        }
        dft_small<T, PY, true>(w);
#pragma unroll
        for (int r = 0; r < PY / 2; ++r)
            if (r < ny) col[r] = w[r];
        return;
    }
    in.first_stage(buf, ny, live, l);
    wave_sync();
    wave_stages<T, PY, LN, false, R0, NSL>(buf, tw, l);
    cx<T> v[Last::ITEMS][RL];
    Last::compute(v, buf, tw, l);
    wave_sync();
#pragma unroll
    for (int it = 0; it < Last::ITEMS; ++it)
#pragma unroll
        for (int r = 0; r < RL; ++r) v[it][r] = scale(v[it][r], packed ? (T)1 : qv[it][r]);
    Last::store(v, buf, l);
    wave_sync();
    if (with_packed) {
        if (packed) {
            const cx<T>* qn = Q + (size_t)(nkq - 1) * KH;
            for (int f = l; f <= PY / 2; f += LN) {
                const int fm = (PY - f) & (PY - 1);
                const cx<T> z = buf[sw(f)], w = conj(buf[sw(fm)]);
                const cx<T> D = scale(z + w, (T)0.5 * q[f].re), E = scale(mul_mi(z - w), (T)0.5 * qn[f].re);
                buf[sw(f)] = D + mul_i(E);
                if (fm != f) buf[sw(fm)] = conj(D) + mul_i(conj(E));
            }
        }
        wave_sync();
    }
    wave_inverse<T, PY, LN>(buf, tw, col, ny, live, l);
}

// Columns (batch entry, kx) by turns, a wave per block, the next ones' loads issued ahead (as in the
// 3D z-pass).  Bound: launches and latency at these sizes.  One 512^2 medium: FP32 11.3 -> 9.1 us, FP64
// 14.1 -> 10.4 us (event to event, the launch included) against k_pass_b_wave's four columns per block
// with barriers round the multiply; four waves per block 9.4 and 11.9 us.
template <typename T, int PY>
__global__ __launch_bounds__(64) void k_pass_b_iso(cx<T>* __restrict__ Tb, const cx<T>* __restrict__ Q,
                                                   const cx<T>* __restrict__ tw, int ny, int nkx, int nkq, int pack,
                                                   int ncol) {
    constexpr int LN = wave_lanes(PY), SPW = 64 / LN, LD = padded(PY);
    __shared__ cx<T> rows[SPW * LD];
    const int l = threadIdx.x % LN, sub = threadIdx.x / LN;
    cx<T>* buf = rows + sub * LD;
    const int step = gridDim.x * SPW;
    WaveIn<T, PY, LN> in;
    in.load(Tb + (size_t)min((int)blockIdx.x * SPW + sub, ncol - 1) * ny, ny, l);
    for (int base = blockIdx.x * SPW; base < ncol; base += step) {
        const int c = min(base + sub, ncol - 1);
        const WaveIn<T, PY, LN> cur = in;
        if (base + step < ncol) in.load(Tb + (size_t)min(base + step + sub, ncol - 1) * ny, ny, l);
        iso_column<T, PY>(cur, Tb + (size_t)c * ny, Q, tw, c % nkx, ny, nkq, base + sub < ncol, true, pack != 0, buf, l);
        wave_sync();
    }
}

// Batched form: a block takes the NW * SPW columns of one item.  Bound: HBM.  32 media of 512^2 in
// FP32 (201 MB) take 51 us, in FP64 103 us, 32 of 256^2 in FP32 18 us; with four columns per block in
// block-wide stages 75, 212 and 24 us.
template <typename T, int PY, int NW>
__global__ __launch_bounds__(NW * 64) void k_pass_b_batch(const BatchProb<T>* __restrict__ probs,
                                                          const int2* __restrict__ items, const int* __restrict__ act) {
    constexpr int LN = wave_lanes(PY), SPW = 64 / LN, LD = padded(PY);
    __shared__ cx<T> rows[NW * SPW * LD];
    const int2 item = items[blockIdx.x];
    const BatchProb<T>& d = probs[item.x];
    if (act && !act[item.x]) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = (threadIdx.x & 63) % LN, sub = (threadIdx.x & 63) / LN;
    const int nkx = d.PX / 2, ny = d.ny, kx0 = (item.y * NW + wave) * SPW, kx = min(kx0 + sub, nkx - 1);
    cx<T>* col = d.work + (size_t)kx * ny;
    WaveIn<T, PY, LN> in;
    in.load(col, ny, l);
    iso_column<T, PY>(in, col, d.Q, d.twy, kx, ny, nkx + 1, kx0 + sub < nkx, kx0 == 0, true,
                      rows + (wave * SPW + sub) * LD, l);
}

// ---- launch ---------------------------------------------------------------------------------

// Columns per block: enough sequences for a few waves.
template <int L>
constexpr int wave_ncol() { return 2 * L + 1 >= 4 ? 1 : (L == 1 ? 2 : 4); }
template <typename T, int PY, int L>
constexpr bool wave_fits() {
    return (long)wave_ncol<L>() * (2 * L + 1) * wave_ld(PY) * (long)sizeof(cx<T>) <= 160 * 1024;
}
// Waves per block: one per sequence, and enough (up to 8) that a thread couples one frequency: at
// 32^2, L = 0 in FP64 the launch with one wave took 3 us longer than with four, each of a thread's
// four frequencies waiting for its kernel entry.  At most 16; the coupling's live values set lower
// limits: 17 to 21 channels in FP32 take 137 to 150 registers (12 waves leave 168), more up to 230, and
// 11 and more in FP64 up to 244 (8 waves leave 256).
template <typename T, int PY, int L>
constexpr int wave_count() {
    constexpr int SPW = 64 / wave_lanes(PY);
    constexpr int W = (wave_ncol<L>() * (2 * L + 1) + SPW - 1) / SPW;
    constexpr int F = wave_ncol<L>() * PY / 64, F8 = F > 8 ? 8 : (F < 1 ? 1 : F);
    constexpr int N = W > F8 ? W : F8;
    constexpr int top = (sizeof(T) == 8 && L > 4) || L > 10 ? 8 : (L >= 8 ? 12 : 16);
    return N > top ? top : N;
}

template <typename T, int PY, int L, int NW, bool CORR>
inline void launch_wave_nw(const Apply2DArgs<T>& a, int nbatch, int nkx, int nkq) {
    constexpr int NCOL = wave_ncol<L>();
    auto* k = k_pass_b_wave<T, PY, L, NCOL, NW, CORR>;
    static const unsigned cap = resident_blocks(k, NW * 64);   // one value on every device of a kind
    const int ngrp = (nkx + NCOL - 1) / NCOL, nitems = ngrp * nbatch;
    const unsigned nb = (unsigned)nitems < cap ? (unsigned)nitems : cap;
    hipLaunchKernelGGL(k, dim3(nb), dim3(NW * 64), 0, a.stream, a.work, a.Q, a.twy, a.ny, nkx, nkq, a.pack,
                       a.single_in, ngrp, nitems, a.bcorr);
}
template <typename T, int PY, int L>
inline void launch_wave(const Apply2DArgs<T>& a, int nbatch, int nkx, int nkq) {
    constexpr int NW = wave_count<T, PY, L>();
    if constexpr (sizeof(T) == 4 && L <= 8) {   // the preconditioner takes up to 17 modes
        if (a.bcorr.y) return launch_wave_nw<T, PY, L, NW, true>(a, nbatch, nkx, nkq);
    }
    if constexpr (L > 0) launch_wave_nw<T, PY, L, NW, false>(a, nbatch, nkx, nkq);   // L = 0: launch_iso
}

// One wave per block: the columns of a small grid spread over the CUs (see k_pass_b_iso).
template <typename T, int PY>
inline void launch_iso(const Apply2DArgs<T>& a, int nbatch, int nkx, int nkq) {
    auto* k = k_pass_b_iso<T, PY>;
    static const unsigned cap = resident_blocks(k, 64);
    const int ncol = nkx * nbatch, per = 64 / wave_lanes(PY);
    const unsigned want = (unsigned)((ncol + per - 1) / per), nb = want < cap ? want : cap;
    hipLaunchKernelGGL(k, dim3(nb), dim3(64), 0, a.stream, a.work, a.Q, a.twy, a.ny, nkx, nkq, a.pack, ncol);
}

template <typename T, int PY, int L, int NW>
inline void launch_half(const Apply2DArgs<T>& a, int nbatch, int nkx, int nkq) {
    auto* k = k_pass_b_half<T, PY, L, NW>;
    static const unsigned cap = resident_blocks(k, NW * 64);
    const int nitems = nkx * nbatch;
    const unsigned nb = (unsigned)nitems < cap ? (unsigned)nitems : cap;
    hipLaunchKernelGGL(k, dim3(nb), dim3(NW * 64), 0, a.stream, a.work, a.Q, a.twyh, a.ny, nkx, nkq, a.pack,
                       a.single_in, nitems);
}

}  // namespace rte

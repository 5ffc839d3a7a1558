// FFTs of one wave or part of one, staged through an LDS row of their own (gfx950, 64-wide waves).
//
// The stages and tables are those of fft.h; a transform's lanes belong to one wave, whose LDS
// accesses complete in order, so its stages need no block barrier.
#pragma once
#include "fft.h"

namespace rte {

// Orders a wave's LDS writes before its own later reads by other lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v, computed anew where it is used: addresses derived from it are not carried across the phases of
// the item loop (they are cheap, and the coupling needs the registers).
__device__ __forceinline__ int hide(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Lanes per transform: 8 points per lane (16 at length 1024), at most a wave.
constexpr int wave_lanes(int P) { return P / 8 > 64 ? 64 : (P / 8 < 1 ? 1 : P / 8); }

// Swizzled distance of r steps of st from an index whose low four bits leave room for it (sw()).
constexpr int sw_step(int r, int st) { return r * st + (r * st) / 16; }

// One Stockham stage of a transform of length P at buf (swizzled), by LN lanes, lane l of them: the
// butterflies j = l, l + LN, ... are read into v, twiddled and transformed.
template <typename T, int P, int LN, int R, int NS, bool INV>
struct WaveStage {
    static constexpr int NB = P / R;
    static constexpr int ITEMS = NB > LN ? NB / LN : 1;
    static constexpr bool FULL = NB >= LN;
    static constexpr int TWOFF = stage_tw_offset(P, NS);
    static __device__ __forceinline__ void compute(cx<T> (&v)[ITEMS][R], const cx<T>* buf, const cx<T>* tw, int l) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int j = l + it * LN;
            if (FULL || j < NB) {
                const cx<T>* src = buf + sw(j);
#pragma unroll
                for (int r = 0; r < R; ++r) v[it][r] = src[sw_step(r, NB)];
                if constexpr (NS > 1) {
                    const cx<T>* w0 = tw + TWOFF + (j % NS) * (R - 1);
#pragma unroll
                    for (int r = 1; r < R; ++r) {
                        cx<T> w = w0[r - 1];
                        if (INV) w.im = -w.im;
                        v[it][r] = v[it][r] * w;
                    }
                }
                dft_small<T, R, INV>(v[it]);
            }
        }
    }
    static __device__ __forceinline__ void store(const cx<T> (&v)[ITEMS][R], cx<T>* buf, int l) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int j = l + it * LN;
            if (FULL || j < NB) {
                cx<T>* dst = buf + sw((j / NS) * (NS * R) + j % NS);
#pragma unroll
                for (int r = 0; r < R; ++r) dst[sw_step(r, NS)] = v[it][r];
            }
        }
    }
};

// The stages with sub-transform length in [NS, NSEND), in place.
template <typename T, int P, int LN, bool INV, int NS, int NSEND>
__device__ __forceinline__ void wave_stages(cx<T>* buf, const cx<T>* tw, int l) {
    if constexpr (NS < NSEND) {
        constexpr int R = fft_radix(P, NS);
        using S = WaveStage<T, P, LN, R, NS, INV>;
        cx<T> v[S::ITEMS][R];
        S::compute(v, buf, tw, l);
        wave_sync();
        S::store(v, buf, l);
        wave_sync();
        wave_stages<T, P, LN, INV, NS * R, NSEND>(buf, tw, l);
    }
}

// Two transforms side by side in one wave: the second one's instructions fill the first one's
// latencies.
template <typename T, int P, int LN, bool INV, int NS, int NSEND>
__device__ __forceinline__ void wave_stages2(cx<T>* b0, cx<T>* b1, const cx<T>* tw, int l) {
    if constexpr (NS < NSEND) {
        constexpr int R = fft_radix(P, NS);
        using S = WaveStage<T, P, LN, R, NS, INV>;
        cx<T> v0[S::ITEMS][R], v1[S::ITEMS][R];
        S::compute(v0, b0, tw, l);
        S::compute(v1, b1, tw, l);
        wave_sync();
        S::store(v0, b0, l);
        S::store(v1, b1, l);
        wave_sync();
        wave_stages2<T, P, LN, INV, NS * R, NSEND>(b0, b1, tw, l);
    }
}

// The inputs of a transform's first stage: rows y < P/2 of one sequence (the others are zero).
template <typename T, int P, int LN>
struct WaveIn {
    static constexpr int R0 = fft_radix(P, 1);
    static constexpr int NB = P / R0;
    static constexpr int ITEMS = NB > LN ? NB / LN : 1;
    static constexpr bool FULL = NB >= LN;
    cx<T> v[ITEMS][R0 / 2];
    // rows y < ny of src; every load takes a clamped index instead of a branch
    __device__ __forceinline__ void load(const cx<T>* __restrict__ src, int ny, int l) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
#pragma unroll
            for (int r = 0; r < R0 / 2; ++r) {
                const int y = l + it * LN + r * NB;
                v[it][r] = src[y < ny ? y : 0];
            }
    }
    // the first stage (radix R0, no twiddles) into buf
    __device__ __forceinline__ void first_stage(cx<T>* buf, int ny, bool live, int l) const {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int j = l + it * LN;
            if (FULL || j < NB) {
                cx<T> w[R0];
#pragma unroll
                for (int r = 0; r < R0; ++r)
                    w[r] = (r < R0 / 2 && live && j + r * NB < ny) ? v[it][r < R0 / 2 ? r : 0] : mk((T)0, (T)0);
                dft_small<T, R0, false>(w);
                cx<T>* dst = buf + sw(j * R0);
#pragma unroll
                for (int r = 0; r < R0; ++r) dst[sw_step(r, 1)] = w[r];
            }
        }
    }
};

// All inverse stages of the transform at buf; the last one writes the rows y < ny of dst only (done:
// the stages before it have run).
template <typename T, int P, int LN>
__device__ __forceinline__ void wave_inverse(cx<T>* buf, const cx<T>* tw, cx<T>* __restrict__ dst, int ny, bool live,
                                             int l, bool done = false) {
    constexpr int NSL = fft_last_ns(P);
    constexpr int RL = P / NSL;
    if (!done) wave_stages<T, P, LN, true, 1, NSL>(buf, tw, l);
    using S = WaveStage<T, P, LN, RL, NSL, true>;
    cx<T> v[S::ITEMS][RL];
    S::compute(v, buf, tw, l);
    wave_sync();
#pragma unroll
    for (int it = 0; it < S::ITEMS; ++it) {
        const int j = l + it * LN;
        if ((S::FULL || j < S::NB) && live) {
#pragma unroll
            for (int r = 0; r < (RL > 1 ? RL / 2 : 1); ++r) {
                const int y = j + r * NSL;
                if (y < ny) dst[y] = v[it][r];
            }
        }
    }
}

// Grid of a looping kernel: as many blocks as the device holds at once (lds: bytes of
// dynamic LDS per block).
template <typename K>
inline unsigned resident_blocks(K kernel, int nthr, size_t lds = 0) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, reinterpret_cast<const void*>(kernel), nthr, lds) != hipSuccess ||
        cus < 1 || per < 1)
        return 256;
    return (unsigned)(cus * per);
}

}  // namespace rte

// Batched complex FP32 FFT whose first and last stages work from and to the caller's registers: only the exchanges
// between stages go through LDS.  Stockham autosort over a list of radices R...; before a stage the sub-transform
// length is Ns = the product of the radices before it.  Butterfly j in [0, n/R) takes x[j + r n/R] (r < R), multiplies
// by tw[r k n/(R Ns)] with k = j mod Ns, takes an R-point DFT and gives positions (j - k) R + k + s Ns (s < R).  So the
// first stage reads positions j + r n/R and the last one writes positions j + s n/R: both are consecutive over the
// lanes, and a transform whose inputs (or outputs) are needed only in the central half takes r (or s) in [R/4, 3R/4).
//
// Why these radices: an exchange costs an LDS write, a barrier and an LDS read, a twiddle a scattered table read at about
// one a clock and CU; with up to 16 values a thread, 4096 points take two exchanges and 12 table reads per 16 values
// (radix 8: three, and 42, besides the first store and the last load of a transform that lives in LDS).
#pragma once

#include "common.h"

namespace fftr {

template <bool INV>
__device__ __forceinline__ float2 rot4(float2 a) {          // times -i (forward) or +i
    return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}
// Products are kept apart from the sums that use them: fused into those, a butterfly's two outputs round at the sum's
// size instead of the product's, and the rounding error grows.
__device__ __forceinline__ float2 times(float2 a, float2 w) {
#pragma clang fp contract(off)
    const float p = a.y * w.y, q = a.y * w.x;
    return make_float2(__builtin_fmaf(a.x, w.x, -p), __builtin_fmaf(a.x, w.y, q));
}
// times exp(-+ i t) for a compile-time angle, c = cos, s = sin.  Their distance from float (up to 3e-8, the same for every
// value) is put back: with it radix 16 is as exact as radix 8 with its fewer constants.
template <bool INV>
__device__ __forceinline__ float2 turn(float2 a, double c, double s) {
#pragma clang fp contract(off)
    if (INV) s = -s;
    const float ch = (float)c, cl = (float)(c - (double)ch), sh = (float)s, sl = (float)(s - (double)sh);
    const float p = __builtin_fmaf(a.x, cl, a.y * sl), q = __builtin_fmaf(a.y, cl, -(a.x * sl));
    return make_float2(__builtin_fmaf(a.x, ch, __builtin_fmaf(a.y, sh, p)),
                       __builtin_fmaf(a.y, ch, __builtin_fmaf(-a.x, sh, q)));
}

template <bool INV>
__device__ __forceinline__ void dft2(float2 &a, float2 &b) {
    const float2 t = a;
    a = cadd(t, b);
    b = csub(t, b);
}

template <bool INV>
__device__ __forceinline__ void dft4(float2 &a0, float2 &a1, float2 &a2, float2 &a3) {
    const float2 s02 = cadd(a0, a2), d02 = csub(a0, a2), s13 = cadd(a1, a3), d13 = rot4<INV>(csub(a1, a3));
    a0 = cadd(s02, s13);
    a1 = cadd(d02, d13);
    a2 = csub(s02, s13);
    a3 = csub(d02, d13);
}

template <int R, bool INV>
__device__ __forceinline__ void dft(float2 *a) {
    constexpr double H = 0.70710678118654752440, C1 = 0.92387953251128675613, S1 = 0.38268343236508977173;
    if constexpr (R == 2) {
        dft2<INV>(a[0], a[1]);
    } else if constexpr (R == 4) {
        dft4<INV>(a[0], a[1], a[2], a[3]);
    } else if constexpr (R == 8) {
        // n = n0 + 2 n1, k = k1 + 4 k0
        dft4<INV>(a[0], a[2], a[4], a[6]);
        dft4<INV>(a[1], a[3], a[5], a[7]);
        a[3] = turn<INV>(a[3], H, H);
        a[5] = rot4<INV>(a[5]);
        a[7] = turn<INV>(a[7], -H, H);
        float2 o[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            o[k] = cadd(a[2 * k], a[2 * k + 1]);
            o[k + 4] = csub(a[2 * k], a[2 * k + 1]);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = o[k];
    } else {
        static_assert(R == 16, "radix");
        // n = n0 + 4 n1, k = k1 + 4 k0: a[n0 + 4 k1] after the first four
#pragma unroll
        for (int i = 0; i < 4; ++i) dft4<INV>(a[i], a[i + 4], a[i + 8], a[i + 12]);
        a[5] = turn<INV>(a[5], C1, S1);
        a[6] = turn<INV>(a[6], H, H);
        a[7] = turn<INV>(a[7], S1, C1);
        a[9] = turn<INV>(a[9], H, H);
        a[10] = rot4<INV>(a[10]);
        a[11] = turn<INV>(a[11], -H, H);
        a[13] = turn<INV>(a[13], S1, C1);
        a[14] = turn<INV>(a[14], -H, H);
        a[15] = turn<INV>(a[15], -C1, -S1);
        float2 o[16];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            dft4<INV>(a[4 * k], a[4 * k + 1], a[4 * k + 2], a[4 * k + 3]);
#pragma unroll
            for (int q = 0; q < 4; ++q) o[k + 4 * q] = a[4 * k + q];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) a[k] = o[k];
    }
}

// Radices by log2 of the length.  128 points have few threads to spread over, so 16 values a thread are a long serial chain
// and 8 with one exchange more are not: the four passes 11.1 us (8 x 16: 12.9; radix 8 and 2 in LDS: 12.6).
template <int LOGN> struct Plan;
template <> struct Plan<6> { static constexpr int S = 2, R[3] = {8, 8, 1}; };
template <> struct Plan<7> { static constexpr int S = 3, R[3] = {8, 4, 4}; };
template <> struct Plan<8> { static constexpr int S = 2, R[3] = {16, 16, 1}; };
template <> struct Plan<9> { static constexpr int S = 3, R[3] = {8, 8, 8}; };
template <> struct Plan<10> { static constexpr int S = 3, R[3] = {8, 16, 8}; };
template <> struct Plan<11> { static constexpr int S = 3, R[3] = {16, 8, 16}; };
template <> struct Plan<12> { static constexpr int S = 3, R[3] = {16, 16, 16}; };

// One transform of 2^LOGN points over NT = n / E threads, E values each, C transforms interleaved in LDS (position p of
// transform c at C pad(p) + c).
template <int LOGN, int C, bool INV>
struct Fft {
    using P = Plan<LOGN>;
    static constexpr int n = 1 << LOGN, R0 = P::R[0], R1 = P::R[1], R2 = P::R[2], RL = P::R[P::S - 1];
    static constexpr int E = R0 > R1 ? (R0 > R2 ? R0 : R2) : (R1 > R2 ? R1 : R2), NT = n / E;
    // One slot in R0 is left free: a first stage's stores go out R0 apart, and would meet in few banks.
    static constexpr int PAD = R0 == 16 ? 4 : 3, LDS = C * (n + (n >> PAD));
    static constexpr int Q0 = n / R0, QL = n / RL;      // first and last stage: position j + r Q0, j + s QL

    static __device__ __forceinline__ int slot(int p, int c) { return C * (p + (p >> PAD)) + c; }

    // Radix 16 loads the twiddles of r = 1, 2, 3, 4, 8, 12 and forms the others as products of two: table reads are
    // what a stage waits for.  The products' extra rounding (16 x 16 x 16 points: 1.19e-7 against 1.14e-7 relative error
    // of a transform; 1.22e-7 for 8 x 8 x 8 x 8 with table reads only) is less than the fewer stages save.
    template <int R, int Ns>
    struct Tw {
        static constexpr int L = R == 16 ? 6 : R - 1;
        float2 t[E / R][L];
        __device__ __forceinline__ void load(const float2 *__restrict__ tw, int j0) {
            constexpr int step = n / (R * Ns);
#pragma unroll
            for (int i = 0; i < E / R; ++i) {
                const int k = ((j0 + i * NT) & (Ns - 1)) * step;
#pragma unroll
                for (int l = 0; l < L; ++l) t[i][l] = tw[(l < 3 || R < 16 ? l + 1 : 4 * (l - 2)) * k];
            }
        }
        __device__ __forceinline__ void apply(float2 *a) const {
#pragma unroll
            for (int i = 0; i < E / R; ++i)
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    float2 w;
                    if constexpr (R < 16) w = t[i][r - 1];
                    else if (r < 4) w = t[i][r - 1];
                    else if (r % 4 == 0) w = t[i][r / 4 + 2];
                    else w = times(t[i][r % 4 - 1], t[i][r / 4 + 2]);
                    a[i * R + r] = times(a[i * R + r], make_float2(w.x, INV ? -w.y : w.y));
                }
        }
    };
    template <int R>
    static __device__ __forceinline__ void dfts(float2 *a) {
#pragma unroll
        for (int i = 0; i < E / R; ++i) dft<R, INV>(a + i * R);
    }
    template <int R, int Ns>
    static __device__ __forceinline__ void put(const float2 *a, float2 *lds, int j0, int c) {
#pragma unroll
        for (int i = 0; i < E / R; ++i) {
            const int j = j0 + i * NT, k = j & (Ns - 1), base = (j - k) * R + k;
#pragma unroll
            for (int s = 0; s < R; ++s) lds[slot(base + s * Ns, c)] = a[i * R + s];
        }
    }
    template <int R>
    static __device__ __forceinline__ void get(float2 *a, const float2 *lds, int j0, int c) {
#pragma unroll
        for (int i = 0; i < E / R; ++i)
#pragma unroll
            for (int r = 0; r < R; ++r) a[i * R + r] = lds[slot(j0 + i * NT + r * (n / R), c)];
    }

    Tw<R1, R0> t1;
    Tw<P::S == 3 ? R2 : 2, P::S == 3 ? R0 * R1 : 1> t2;

    // asked for after the caller's data loads and before they are used, so that the waits overlap
    __device__ __forceinline__ void twiddles(const float2 *__restrict__ tw, int j0) {
        t1.load(tw, j0);
        if constexpr (P::S == 3) t2.load(tw, j0);
    }

    // a[i R0 + r] = x[j0 + i NT + r Q0] in, a[i RL + s] = X[j0 + i NT + s QL] out; every thread of the block calls it
    __device__ __forceinline__ void run(float2 *a, float2 *lds, int j0, int c) const {
        dfts<R0>(a);
        put<R0, 1>(a, lds, j0, c);
        __syncthreads();
        get<R1>(a, lds, j0, c);
        t1.apply(a);
        dfts<R1>(a);
        if constexpr (P::S == 3) {
            __syncthreads();
            put<R1, R0>(a, lds, j0, c);
            __syncthreads();
            get<R2>(a, lds, j0, c);
            t2.apply(a);
            dfts<R2>(a);
        }
    }
};

}  // namespace fftr

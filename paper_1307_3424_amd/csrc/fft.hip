// A, Z, F and their adjoint: apodise + zero-pad + centred 2-D FFT of the image,
// and the unnormalised inverse + crop + apodise back (Sections 2.2 and 3.1; the
// upsampling U of Eq. 6 is done here in the image domain as zero-padding).
//
// Centring.  With c = Ng/2, the centred DFT
//     X[q] = sum_j z_j exp(-2 pi i (j - c).(q - c) / Ng)
// equals (-1)^(q_u+q_v) FFT((-1)^(j_u+j_v) z)[q] (Ng even), so the signs are
// folded into the first and last pass.
//
// Order of the passes.  The image is non-zero (and wanted back) only in the central N rows and columns of the padded
// grid.  Columns are transformed on the image side: forward, N columns of the image to Ng rows of N values, then all Ng
// rows; adjoint, all Ng rows with N values kept of each, then N columns to the image.  The column passes are the ones
// whose accesses are short pieces (C values), so they should have the fewest bytes: image and half-width rows, not the
// whole grid, which only the row passes touch.
#include "fft_reg.h"

namespace {

// Launch shape per grid size: rows per block of the row passes, columns per block of the column passes.  Measured on
// MI355X, all four passes of a product pair at Ng = 4096: 141 us (310 with in-LDS radix-8 transforms, rows first); with 2
// columns a block instead of 4: 154 us.  Ng = 2048: 50 us (68); 2 or 8 columns: 54, 53.  Ng = 1024: 24.5 us (29); 2 columns: 25.6,
// 8: 28.6.  From Ng = 512 down every pass takes 2 to 4 us, which is a launch, one trip to memory and one to three
// exchanges: Ng = 512, 256, 128 and 64: 13.9 us (15.1), 12.9 (13.1), 11.1 (12.6) and 9.4 (11.6); at 128 8 rows and columns a
// block 11.5, elsewhere blocks of a half to two times the size differ by little.  The row passes at 4096 move
// their 201 MB at 5.3 TB/s; starting each row's values between the passes at another place, against channel conflicts
// of the column passes, changed nothing.
template <int LOGNG> struct Shape;
template <> struct Shape<6> { static constexpr int CR = 8, CC = 8; };
template <> struct Shape<7> { static constexpr int CR = 4, CC = 4; };
template <> struct Shape<8> { static constexpr int CR = 4, CC = 4; };
template <> struct Shape<9> { static constexpr int CR = 1, CC = 2; };
template <> struct Shape<10> { static constexpr int CR = 1, CC = 4; };
template <> struct Shape<11> { static constexpr int CR = 1, CC = 4; };
template <> struct Shape<12> { static constexpr int CR = 1, CC = 4; };

// INVN: the physical apodisation carries the 1/n(l, m) factor.  A template parameter rather than
// a runtime test, so that a kernel's loads are not split by a branch.
template <bool INVN>
__device__ inline float apod_at(const float *__restrict__ apod, int N, float delta, int im, int iu) {
    float a = apod[im] * apod[iu];
    if constexpr (INVN) {
        const float l = (iu - N / 2) * delta, m = (im - N / 2) * delta;
        a *= rsqrtf(1.0f - l * l - m * m);
    }
    return a;
}

__device__ inline float sgn(int k) { return (k & 1) ? -1.0f : 1.0f; }

// Thread layout: j0 is the thread's first butterfly; the transform index c runs fastest in the column passes (a wave
// reads C adjacent values of 64 / C rows) and slowest in the row passes (consecutive values of one row).
template <int LOGNG, int C, bool INV>
struct Pass : fftr::Fft<LOGNG, C, INV> {
    using F = fftr::Fft<LOGNG, C, INV>;
    static constexpr int Ng = F::n, N = Ng / 2, NTH = F::NT * C, LOGC = C == 1 ? 0 : C == 2 ? 1 : C == 4 ? 2 : 3;
    static_assert(1 << LOGC == C && Ng % C == 0, "shape");
};

// Forward, pass 1: columns iu0 .. of the image, apodised, to grid[q_v][N/2 + iu].
template <int LOGNG, int C, bool INVN>
__global__ __launch_bounds__((Pass<LOGNG, C, false>::NTH)) void k_fwd_cols(
    const float2 *__restrict__ x, float2 *__restrict__ grid, const float *__restrict__ apod,
    const float2 *__restrict__ tw, float delta) {
    using P = Pass<LOGNG, C, false>;
    using F = typename P::F;
    constexpr int Ng = P::Ng, N = P::N;
    __shared__ float2 lds[F::LDS];
    const int c = threadIdx.x & (C - 1), j0 = threadIdx.x >> P::LOGC;
    const int iu = (int)xcd_block(blockIdx.x, gridDim.x) * C + c;
    x += (int64_t)blockIdx.y * N * N + iu;
    grid += (int64_t)blockIdx.y * Ng * Ng + N / 2 + iu;
    float2 a[F::E];
    float f[F::E];
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int r = e % F::R0, im = j0 + e / F::R0 * F::NT + r * F::Q0 - N / 2;
        a[e] = make_float2(0.f, 0.f);
        f[e] = 0.f;
        if (r >= F::R0 / 4 && r < 3 * F::R0 / 4) {
            a[e] = x[(int64_t)im * N];
            f[e] = apod_at<INVN>(apod, N, delta, im, iu) * sgn(iu + im);
        }
    }
    F fft;
    fft.twiddles(tw, j0);
#pragma unroll
    for (int e = 0; e < F::E; ++e) a[e] = make_float2(a[e].x * f[e], a[e].y * f[e]);
    fft.run(a, lds, j0, c);
#pragma unroll
    for (int e = 0; e < F::E; ++e) grid[(int64_t)(j0 + e / F::RL * F::NT + e % F::RL * F::QL) * Ng] = a[e];
}

// Forward, pass 2: rows of the grid in place, the central N values in, all out.
template <int LOGNG, int C>
__global__ __launch_bounds__((Pass<LOGNG, C, false>::NTH)) void k_fwd_rows(float2 *__restrict__ grid,
                                                                         const float2 *__restrict__ tw) {
    using P = Pass<LOGNG, C, false>;
    using F = fftr::Fft<LOGNG, 1, false>;
    constexpr int Ng = P::Ng;
    __shared__ float2 lds[C * F::LDS];
    const int c = threadIdx.x / F::NT, j0 = threadIdx.x % F::NT, qv = blockIdx.x * C + c;
    grid += (int64_t)blockIdx.y * Ng * Ng + (int64_t)qv * Ng;
    float2 a[F::E];
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int r = e % F::R0;
        a[e] = make_float2(0.f, 0.f);
        if (r >= F::R0 / 4 && r < 3 * F::R0 / 4) a[e] = grid[j0 + e / F::R0 * F::NT + r * F::Q0];
    }
    F fft;
    fft.twiddles(tw, j0);
    fft.run(a, lds + c * F::LDS, j0, 0);
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int q = j0 + e / F::RL * F::NT + e % F::RL * F::QL;
        const float s = sgn(qv + q);
        grid[q] = make_float2(a[e].x * s, a[e].y * s);
    }
}

// Adjoint, pass 1: rows of the grid in place, inverse, the central N values kept.
template <int LOGNG, int C>
__global__ __launch_bounds__((Pass<LOGNG, C, true>::NTH)) void k_adj_rows(float2 *__restrict__ grid,
                                                                        const float2 *__restrict__ tw) {
    using P = Pass<LOGNG, C, true>;
    using F = fftr::Fft<LOGNG, 1, true>;
    constexpr int Ng = P::Ng;
    __shared__ float2 lds[C * F::LDS];
    const int c = threadIdx.x / F::NT, j0 = threadIdx.x % F::NT, qv = blockIdx.x * C + c;
    grid += (int64_t)blockIdx.y * Ng * Ng + (int64_t)qv * Ng;
    float2 a[F::E];
#pragma unroll
    for (int e = 0; e < F::E; ++e) a[e] = grid[j0 + e / F::R0 * F::NT + e % F::R0 * F::Q0];
    F fft;
    fft.twiddles(tw, j0);
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const float s = sgn(qv + j0 + e / F::R0 * F::NT + e % F::R0 * F::Q0);
        a[e] = make_float2(a[e].x * s, a[e].y * s);
    }
    fft.run(a, lds + c * F::LDS, j0, 0);
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int s = e % F::RL;
        if (s >= F::RL / 4 && s < 3 * F::RL / 4) grid[j0 + e / F::RL * F::NT + s * F::QL] = a[e];
    }
}

// Adjoint, pass 2: columns iu0 .. of the image, inverse, the central N rows apodised.
template <int LOGNG, int C, bool INVN>
__global__ __launch_bounds__((Pass<LOGNG, C, true>::NTH)) void k_adj_cols(
    const float2 *__restrict__ grid, float2 *__restrict__ x, const float *__restrict__ apod,
    const float2 *__restrict__ tw, float delta) {
    using P = Pass<LOGNG, C, true>;
    using F = typename P::F;
    constexpr int Ng = P::Ng, N = P::N;
    __shared__ float2 lds[F::LDS];
    const int c = threadIdx.x & (C - 1), j0 = threadIdx.x >> P::LOGC;
    const int iu = (int)xcd_block(blockIdx.x, gridDim.x) * C + c;
    x += (int64_t)blockIdx.y * N * N + iu;
    grid += (int64_t)blockIdx.y * Ng * Ng + N / 2 + iu;
    float2 a[F::E];
#pragma unroll
    for (int e = 0; e < F::E; ++e) a[e] = grid[(int64_t)(j0 + e / F::R0 * F::NT + e % F::R0 * F::Q0) * Ng];
    F fft;
    fft.twiddles(tw, j0);
    float f[F::E];                                              // output factors
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int s = e % F::RL, im = j0 + e / F::RL * F::NT + s * F::QL - N / 2;
        f[e] = s >= F::RL / 4 && s < 3 * F::RL / 4 ? apod_at<INVN>(apod, N, delta, im, iu) * sgn(iu + im) : 0.f;
    }
    fft.run(a, lds, j0, c);
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int s = e % F::RL, im = j0 + e / F::RL * F::NT + s * F::QL - N / 2;
        if (s >= F::RL / 4 && s < 3 * F::RL / 4) x[(int64_t)im * N] = make_float2(a[e].x * f[e], a[e].y * f[e]);
    }
}

template <int LOGNG>
wp_status fwd(const wp_plan *p, const float2 *x, float2 *grid, int batch, hipStream_t s) {
    constexpr int Ng = 1 << LOGNG, N = Ng / 2;
    using S = Shape<LOGNG>;
    const dim3 gc(N / S::CC, batch), bc(Pass<LOGNG, S::CC, false>::NTH);
    if (p->aphys == WP_APHYS_INV_N)
        hipLaunchKernelGGL((k_fwd_cols<LOGNG, S::CC, true>), gc, bc, 0, s, x, grid, p->apod, p->tw32, (float)p->delta);
    else
        hipLaunchKernelGGL((k_fwd_cols<LOGNG, S::CC, false>), gc, bc, 0, s, x, grid, p->apod, p->tw32, (float)p->delta);
    hipLaunchKernelGGL((k_fwd_rows<LOGNG, S::CR>), dim3(Ng / S::CR, batch), dim3(Pass<LOGNG, S::CR, false>::NTH), 0, s,
                       grid, p->tw32);
    return wp_check_launch("grid_forward");
}

template <int LOGNG>
wp_status adj(const wp_plan *p, float2 *grid, float2 *x, int batch, hipStream_t s) {
    constexpr int Ng = 1 << LOGNG, N = Ng / 2;
    using S = Shape<LOGNG>;
    const dim3 gc(N / S::CC, batch), bc(Pass<LOGNG, S::CC, true>::NTH);
    hipLaunchKernelGGL((k_adj_rows<LOGNG, S::CR>), dim3(Ng / S::CR, batch), dim3(Pass<LOGNG, S::CR, true>::NTH), 0, s,
                       grid, p->tw32);
    if (p->aphys == WP_APHYS_INV_N)
        hipLaunchKernelGGL((k_adj_cols<LOGNG, S::CC, true>), gc, bc, 0, s, grid, x, p->apod, p->tw32, (float)p->delta);
    else
        hipLaunchKernelGGL((k_adj_cols<LOGNG, S::CC, false>), gc, bc, 0, s, grid, x, p->apod, p->tw32, (float)p->delta);
    return wp_check_launch("grid_adjoint");
}

}  // namespace

wp_status launch_grid_forward(const wp_plan *p, const float2 *x, float2 *grid, hipStream_t s, int batch) {
    switch (p->logNg) {
        case 6: return fwd<6>(p, x, grid, batch, s);
        case 7: return fwd<7>(p, x, grid, batch, s);
        case 8: return fwd<8>(p, x, grid, batch, s);
        case 9: return fwd<9>(p, x, grid, batch, s);
        case 10: return fwd<10>(p, x, grid, batch, s);
        case 11: return fwd<11>(p, x, grid, batch, s);
        case 12: return fwd<12>(p, x, grid, batch, s);
    }
    return wp_set_error(WP_EUNSUPPORTED, "grid_forward: Ng = %d", p->Ng);
}

wp_status launch_grid_adjoint(const wp_plan *p, float2 *grid, float2 *x, hipStream_t s, int batch) {
    switch (p->logNg) {
        case 6: return adj<6>(p, grid, x, batch, s);
        case 7: return adj<7>(p, grid, x, batch, s);
        case 8: return adj<8>(p, grid, x, batch, s);
        case 9: return adj<9>(p, grid, x, batch, s);
        case 10: return adj<10>(p, grid, x, batch, s);
        case 11: return adj<11>(p, grid, x, batch, s);
        case 12: return adj<12>(p, grid, x, batch, s);
    }
    return wp_set_error(WP_EUNSUPPORTED, "grid_adjoint: Ng = %d", p->Ng);
}

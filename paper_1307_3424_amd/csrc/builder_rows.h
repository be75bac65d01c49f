// Rows of G for the linear chirp, made from a band of cells around the visibility.
//
// Section 3.1's row is separable, g(q_v, q_u) = g_v(q_v) g_u(q_u), and almost all of it is noise of the
// spectrum's tail: at the workloads' w a row keeps some 15 x 15 of its Ng x Ng entries.  These kernels look
// only at the band of cells the chirp reaches (2 |w| L^2 and a margin on either side of the window, builder_band.h) and
// prove from the spectrum's values that the other cells read that no entry there can be kept:
//     |g(q)|^2 <= (sum_i |KB_i|)^2 max_{d read outside} |h(d)|^2.
// A row whose bound fails, whose band or candidates do not fit, or that keeps all entries (E >= 1) goes to the
// whole-axis kernels of builder.hip (k_row_count, k_row_fill), by way of a list of rows.
//
// Threshold.  K(tau) = sum of the energies >= tau, tau = the largest energy with K(tau) >= E T,
// T = (sum KB_u^2)(sum KB_v^2) (shifted spectra of a unit-modulus chirp are orthonormal).  Energies are
// summed as integers of 2^-62 T (finer than FP64 sums, and independent of the order): one pass adds them
// into a histogram over their leading bits, the histogram's bin that crosses E T is found by a suffix scan,
// and the few energies of that bin are ranked among themselves.  Three passes over the candidates' products
// replace a sort of the axis and 64 bisection steps over it.
//
// What bounds it, from clocks at the phase boundaries (Ng = 4096, two workgroups per CU, 43 k clocks per row): the
// chirp and the FFT 20 k, most of them FP64 issue (about 980 instructions per wavefront), the window's weights and
// their first loads 6-9 k, the band's energies and the bound 5 k, the threshold's passes and their barriers 9 k.
// Times of the launches: see count_rows in builder.hip.
#pragma once

#include "builder_band.h"
#include "builder_util.h"
#include "fft_lds.h"

namespace {

// threads per row: one radix-8 butterfly per thread and stage from Ng = 512 up, one wavefront below
template <int LOGNG>
constexpr int row_threads() { return LOGNG <= 9 ? 64 : 1 << (LOGNG - 3); }

// the spectrum in LDS is padded by one value per eight: the first two stages write with strides of 8 and 64
// values, which would otherwise fall on the same banks
__device__ __forceinline__ int hpad(int i) { return i + (i >> 3); }
template <int LOGNG>
constexpr size_t spectrum_lds() { return (size_t)18 << LOGNG; }

// one radix-R Stockham stage of the padded n-point transform (see fft_lds.h for the indices).  Padded positions
// that are whole multiples of 8 apart are a constant apart, so each side has one computed address per butterfly.
// The twiddles are loaded first: their latency overlaps the LDS reads and the barrier.
template <int LOGN, int NT, int R, int NS>
__device__ __forceinline__ void row_fft_stage(double2 *buf, const double2 *__restrict__ tw, int tid) {
    constexpr int n = 1 << LOGN, nq = n / R, PER = (nq + NT - 1) / NT, step = n / (R * NS);
    static_assert(nq % 8 == 0 && (NS == 1 || NS % 8 == 0), "padded strides");
    double2 reg[PER][R], t[PER][R];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int b = tid + i * NT;
        if (nq % NT == 0 || b < nq) {
            if constexpr (NS > 1) {
                const unsigned k1 = (unsigned)(b & (NS - 1)) * step;
#pragma unroll
                for (int r = 1; r < R; ++r) t[i][r] = tw[r * k1];
            }
            const double2 *src = buf + hpad(b);
#pragma unroll
            for (int r = 0; r < R; ++r) reg[i][r] = src[r * (nq + nq / 8)];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int b = tid + i * NT;
        if (nq % NT == 0 || b < nq) {
            double2 *a = reg[i];
            if constexpr (NS > 1) {
#pragma unroll
                for (int r = 1; r < R; ++r) a[r] = cmul(a[r], t[i][r]);
            }
            if constexpr (R == 8) {
                dft8(a, false);
            } else if constexpr (R == 4) {
                dft4(a, false);
            } else {
                const double2 a0 = a[0];
                a[0] = cadd(a0, a[1]);
                a[1] = csub(a0, a[1]);
            }
            const int k = b & (NS - 1);
            double2 *dst = buf + hpad((b - k) * R + k);       // NS = 1: R = 8, positions 8 b .. 8 b + 7
            constexpr int ds = NS == 1 ? 1 : NS + NS / 8;
#pragma unroll
            for (int s = 0; s < R; ++s) dst[s * ds] = a[s];
        }
    }
    __syncthreads();
}

// h(d) = sum_t exp(i pi w delta^2 t^2) exp(-2 pi i t d / Ng) into the padded LDS buffer; the chirp is even in t,
// so each value is computed once and stored at t and -t.  Ends with a barrier.
template <int LOGNG, int NT = row_threads<LOGNG>()>
__device__ inline void row_spectrum(double2 *h, double wk, double delta, const double2 *__restrict__ tw) {
    constexpr int Ng = 1 << LOGNG;
    const double a = wk * delta * delta;
    for (int i = threadIdx.x; i <= Ng / 2; i += NT) {
        const double t = (double)i;
        double sn, cs;
        sincospi(a * t * t, &sn, &cs);
        const double2 c = make_double2(cs, sn);
        h[hpad(i)] = c;
        if (i > 0) h[hpad(Ng - i)] = c;
    }
    __syncthreads();
    const int tid = threadIdx.x;
    row_fft_stage<LOGNG, NT, 8, 1>(h, tw, tid);
    row_fft_stage<LOGNG, NT, 8, 8>(h, tw, tid);
    if constexpr (LOGNG >= 9) row_fft_stage<LOGNG, NT, 8, 64>(h, tw, tid);
    if constexpr (LOGNG >= 12) row_fft_stage<LOGNG, NT, 8, 512>(h, tw, tid);
    constexpr int NS = 1 << (3 * (LOGNG / 3));
    if constexpr (LOGNG % 3 == 2) row_fft_stage<LOGNG, NT, 4, NS>(h, tw, tid);
    if constexpr (LOGNG % 3 == 1) row_fft_stage<LOGNG, NT, 2, NS>(h, tw, tid);
}

// KB weights of both axes into wt[0..15] (u) and wt[16..31] (v); q0: grid index of the first window cell
// (may lie outside the grid: taken mod Ng)
__device__ inline void row_weights(double ut, double vt, int W, double beta, int Ng, double *wt, int &q0u, int &q0v) {
    const int bu = (int)floor(ut) - W / 2 + 1, bv = (int)floor(vt) - W / 2 + 1;
    q0u = bu + Ng / 2;
    q0v = bv + Ng / 2;
    const int i = threadIdx.x & 15, ax = threadIdx.x >> 4;
    if (ax < 2 && i < W) {
        const double gt = ax ? vt : ut;
        const int base = ax ? bv : bu;
        wt[threadIdx.x] = kb_weight(gt - (double)(base + i), W, beta);
    }
}

// g(q) = Ng^-1 sum_i wt_i h((q0 + i - q) mod Ng)
__device__ __forceinline__ double2 row_value(const double2 *h, int q0, const double *wt, int W, int q, int Ng) {
    double2 g = make_double2(0.0, 0.0);
    for (int i = 0; i < W; ++i) {
        const double2 hv = h[hpad((q0 + i - q) & (Ng - 1))];
        g.x += wt[i] * hv.x;
        g.y += wt[i] * hv.y;
    }
    const double s = 1.0 / Ng;
    return make_double2(g.x * s, g.y * s);
}

// ---------------------------------------------------------------------------- block reductions, NT threads

template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double lane_value(double x, int lane) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// maximum over the wavefront: lane exchanges inside each row of 16, then one lane of each row
__device__ __forceinline__ double wave_max(double x) {
    x = fmax(x, dpp_move<0xB1>(x));      // quad_perm 1,0,3,2
    x = fmax(x, dpp_move<0x4E>(x));      // quad_perm 2,3,0,1
    x = fmax(x, dpp_move<0x141>(x));     // row_half_mirror
    x = fmax(x, dpp_move<0x140>(x));     // row_mirror
    return fmax(fmax(lane_value(x, 0), lane_value(x, 16)), fmax(lane_value(x, 32), lane_value(x, 48)));
}

// maxima of two values over the block
template <int NT>
__device__ __forceinline__ void block_max2(double &a, double &b, double *red) {
    a = wave_max(a);
    b = wave_max(b);
    if constexpr (NT > 64) {
        const int wv = threadIdx.x >> 6;
        __syncthreads();
        if ((threadIdx.x & 63) == 0) {
            red[2 * wv] = a;
            red[2 * wv + 1] = b;
        }
        __syncthreads();
        a = red[0];
        b = red[1];
#pragma unroll
        for (int i = 1; i < NT / 64; ++i) {
            a = fmax(a, red[2 * i]);
            b = fmax(b, red[2 * i + 1]);
        }
    }
}

// ---------------------------------------------------------------------------- the band of a row

// Rows for the whole-axis kernels.  64 lists by row index, their counters on cache lines of their own: one counter is 13 ns
// a row, which on small grids is a tenth of the row itself.
struct RowList {
    static constexpr int N = 64, STEP = 32, COUNTS = N * STEP;
    static int cap(int64_t M) { return (int)((M + N - 1) / N); }
    static int64_t rows(int64_t M) { return N * (int64_t)cap(M); }
    int *row, *count;
    int capacity;

    __device__ __forceinline__ void push(int64_t r) const {
        const int q = (int)r & (N - 1);
        row[(int64_t)q * capacity + atomicAdd(&count[q * STEP], 1)] = (int)r;
    }
    // calls f(row) for every gridDim.x-th row from the blockIdx.x-th on; the same in all wavefronts of a workgroup
    template <class F>
    __device__ __forceinline__ void each(F f) const {
        const int lane = threadIdx.x & 63, n = count[lane * STEP];
        int end = n;                                  // rows of this lane's list and the ones before it
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(end, o);
            if (lane >= o) end += x;
        }
        const int total = __builtin_amdgcn_readlane(end, 63);
        for (int it = blockIdx.x; it < total; it += gridDim.x) {
            const int q = __builtin_popcountll(__ballot(end <= it));
            f((int64_t)row[(int64_t)q * capacity + it - __builtin_amdgcn_readlane(end - n, q)]);
        }
    }
};

constexpr int BAND_CAP = 128;             // candidates per axis
constexpr int BAND_LIST = 256;            // energies of the crossing bin
constexpr int BAND_BINS = 256;

// cells of a band per thread, held in registers: the whole axis up to Ng = 256, else 256 cells (512 with 512
// threads), which is a support of 120 cells
template <int LOGNG>
constexpr int band_groups() {
    constexpr int Ng = 1 << LOGNG, NT = row_threads<LOGNG>();
    return Ng <= 256 ? Ng / NT : (NT >= 256 ? 1 : 256 / NT);
}

// the band of a row; reach: 2 |w| L^2
template <int LOGNG>
__device__ __forceinline__ Band band_of(double wk, double L2, int W, int q0u, int q0v) {
    return row_band(1 << LOGNG, band_groups<LOGNG>() * row_threads<LOGNG>(), 2.0 * fabs(wk) * L2, W, q0u, q0v);
}

// a bound on max |h(d)|^2 over what cells outside the band read (0: none is outside)
template <int LOGNG>
__device__ __forceinline__ double outside_max(const double2 *h, const Band &b, int W, double *red) {
    constexpr int Ng = 1 << LOGNG, NT = row_threads<LOGNG>();
    if (b.cnt == Ng) return 0.0;
    double m = 0.0, z = 0.0;                      // the spectrum is even: one side bounds both
    for (int d = outside_from(b, W) + threadIdx.x; d <= Ng / 2; d += NT) m = fmax(m, energy(h[hpad(d)]));
    block_max2<NT>(m, z, red);
    return m * 1.0001;                            // the two sides differ by rounding
}

// values and 1-D energies of this thread's cells (p = tid + NT j of the band) and the energies' maxima
template <int LOGNG>
__device__ __forceinline__ void band_energies(const double2 *h, const Band &b, int q0u, int q0v, const double *wt, int W,
                                              double2 *ga, double2 *gb, double *A, double *B, double &amax,
                                              double &bmax, double *red) {
    constexpr int Ng = 1 << LOGNG, NT = row_threads<LOGNG>();
    amax = bmax = 0.0;
#pragma unroll
    for (int j = 0; j < band_groups<LOGNG>(); ++j) {
        A[j] = B[j] = 0.0;
        const int p = (int)threadIdx.x + NT * j;
        if (NT * j < b.cnt && p < b.cnt) {
            ga[j] = row_value(h, q0u, wt, W, b.su + p, Ng);            // taken mod Ng
            gb[j] = row_value(h, q0v, wt + 16, W, b.sv + p, Ng);
            A[j] = energy(ga[j]);
            B[j] = energy(gb[j]);
            amax = fmax(amax, A[j]);
            bmax = fmax(bmax, B[j]);
        }
    }
    block_max2<NT>(amax, bmax, red);
}

// (sum |KB|)^2 and sum KB^2 of one axis
__device__ __forceinline__ void weight_sums(const double *wt, int W, double &s1sq, double &s2) {
    double s = 0.0, q = 0.0;
    for (int i = 0; i < W; ++i) {
        s += fabs(wt[i]);
        q = fma(wt[i], wt[i], q);
    }
    s1sq = s * s;
    s2 = q;
}

template <int LOGNG>
constexpr size_t band_count_lds() {
    constexpr size_t lists = 2 * BAND_CAP * 8 + BAND_BINS * 8 + BAND_LIST * 16;
    return spectrum_lds<LOGNG>() > lists ? spectrum_lds<LOGNG>() : lists;
}
template <int LOGNG>
constexpr size_t band_fill_lds() {
    constexpr size_t lists = 2 * BAND_CAP * (16 + 8 + 4 + 2) + 64;
    return spectrum_lds<LOGNG>() > lists ? spectrum_lds<LOGNG>() : lists;
}

// Places, ascending by cell, of this thread's cells among those that can have a kept entry (A_a bmax >= tau, amax B_b
// >= tau): at_a[j], at_b[j], or -1; nca and ncb are their numbers.  s_wc: [PER][NT / 64][4] ints of LDS.
template <int NT, int PER>
__device__ __forceinline__ void candidate_places(const double *A, const double *B, double amax, double bmax, double tau,
                                                 const Band &b, int Ng, int (*s_wc)[NT / 64][4], int *at_a, int *at_b,
                                                 int &nca, int &ncb) {
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    unsigned long long ma[PER], mb[PER];
    const int eu = Ng - b.su, ev = Ng - b.sv;             // positions from here on lie at the axis' start
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int p = tid + NT * j;
        ma[j] = __ballot(p < b.cnt && A[j] * bmax >= tau);
        mb[j] = __ballot(p < b.cnt && amax * B[j] >= tau);
        const unsigned long long ba = __ballot(p < eu) & ma[j], bb = __ballot(p < ev) & mb[j];
        if (lane == 0) {
            s_wc[j][wv][0] = __popcll(ma[j]);
            s_wc[j][wv][1] = __popcll(mb[j]);
            s_wc[j][wv][2] = __popcll(ba);
            s_wc[j][wv][3] = __popcll(bb);
        }
    }
    __syncthreads();
    nca = ncb = 0;
    int na_end = 0, nb_end = 0;                           // candidates before the axis' end
    int pa[PER], pb[PER];                                 // candidates before this wave's cells of group j
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        pa[j] = nca;
        pb[j] = ncb;
        for (int i = 0; i < NW; ++i) {
            const int x = s_wc[j][i][0], y = s_wc[j][i][1];
            if (i < wv) {
                pa[j] += x;
                pb[j] += y;
            }
            nca += x;
            ncb += y;
            na_end += s_wc[j][i][2];
            nb_end += s_wc[j][i][3];
        }
    }
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int p = tid + NT * j;
        at_a[j] = at_b[j] = -1;                           // ascending cells: those past the axis' end come first
        if ((ma[j] >> lane) & 1ull) at_a[j] = pa[j] + __popcll(ma[j] & below) + (p < eu ? nca - na_end : -na_end);
        if ((mb[j] >> lane) & 1ull) at_b[j] = pb[j] + __popcll(mb[j] & below) + (p < ev ? ncb - nb_end : -nb_end);
    }
}

// What the count pass leaves of a row for the fill pass, in the workspace: the candidates of both axes, u then v, each
// ascending by cell, with their values and energies, and what they were made from.  A row keeps some 15 a side; one with
// more than CAND_MAX, or past the first CAND_ROWS rows (which bounds the room), is made again from its spectrum (nca = -1).
// So is a row whose coordinates or threshold are not these: the fill pass makes the rows of the coordinates that it is
// given, and its counts show where they are others than the count pass's.
struct RowCand {
    int nca, ncb;
    double i16_scale;
    double u, v, w, tau;
};
constexpr int CAND_BYTES = 2048, CAND_MAX = (CAND_BYTES - (int)sizeof(RowCand)) / (16 + 8 + 2);
constexpr int64_t CAND_ROWS = 1 << 18;

// append p to list[] (capacity cap, count in *n) for the lanes with keep set, in lane order within a wave
__device__ __forceinline__ void wave_append(bool keep, double p, double *list, int cap, int *n) {
    const unsigned long long m = __ballot(keep);
    if (m == 0) return;
    const int lane = threadIdx.x & 63;
    int at = 0;
    if (lane == 0) at = atomicAdd(n, __popcll(m));
    at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
    if (keep && at < cap) list[at] = p;
}

// walks the nA x nB products with NT threads, without a division per product
struct PairWalk {
    int ia, ib, da, db;
    __device__ PairWalk(int tid, int nt, int nB) {
        ia = tid / nB;
        ib = tid - ia * nB;
        da = nt / nB;
        db = nt - da * nB;
    }
    __device__ void next(int nB) {
        ia += da;
        ib += db;
        if (ib >= nB) {
            ib -= nB;
            ++ia;
        }
    }
};

// Pass 1 for one row per workgroup: tau, kept count, sort key, factor record size; rows it cannot take are listed.
template <int LOGNG>
__global__ __launch_bounds__(row_threads<LOGNG>(), 4) void k_band_count(
    const double *__restrict__ u, const double *__restrict__ v, const double *__restrict__ w, double E, double cell,
    double delta, double L2, int W, double beta, const double2 *__restrict__ tw, double *__restrict__ tau_out,
    int *__restrict__ nnz_out, int *__restrict__ key_out, int *__restrict__ fsz_out, int *__restrict__ err, int64_t r0,
    const RowList list, unsigned char *__restrict__ cand) {
    constexpr int Ng = 1 << LOGNG, NT = row_threads<LOGNG>(), PER = band_groups<LOGNG>();
    extern __shared__ __align__(16) unsigned char smem[];
    double2 *h = (double2 *)smem;
    // after the energies are in registers the spectrum's space holds the lists
    double *eA = (double *)smem, *eB = eA + BAND_CAP;
    unsigned long long *hist = (unsigned long long *)(eB + BAND_CAP);
    double *lp = (double *)(hist + BAND_BINS);
    unsigned long long *lq = (unsigned long long *)(lp + BAND_LIST);
    __shared__ double red[2 * (NT / 64)], s_wt[32], s_tau;
    __shared__ unsigned long long s_above;
    __shared__ int s_n[6];                       // candidates u, v; crossing bin's energies; kept; factors u, v
    __shared__ int s_bin;
    __shared__ int s_wc[PER][NT / 64][4];

    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t k = r0 + blockIdx.x;
    unsigned char *rc = k < CAND_ROWS ? cand + k * CAND_BYTES : nullptr;
    if (rc && tid == 0) ((RowCand *)rc)->nca = -1;
    const double ut = u[k] / cell, vt = v[k] / cell, wk = w[k];
    const bool ok = isfinite(ut) && isfinite(vt) && isfinite(wk) && fabs(ut) < Ng / 2 && fabs(vt) < Ng / 2;
    if (!ok) {
        if (tid == 0) {
            atomicOr(err, 1);
            tau_out[k] = INFINITY;
            nnz_out[k] = 0;
            key_out[k] = 0;
            fsz_out[k] = factor_record_bytes(0, 0);
        }
        return;
    }
    int q0u, q0v;
    row_weights(ut, vt, W, beta, Ng, s_wt, q0u, q0v);
    const Band b = band_of<LOGNG>(wk, L2, W, q0u, q0v);
    if (b.cnt > PER * NT) {                      // uniform over the workgroup
        if (tid == 0) list.push(k);
        return;
    }
    row_spectrum<LOGNG>(h, wk, delta, tw);       // ends with a barrier: the weights are visible
    double s1u, s1v, tu, tv;
    weight_sums(s_wt, W, s1u, tu);
    weight_sums(s_wt + 16, W, s1v, tv);
    const double out = outside_max<LOGNG>(h, b, W, red);
    double2 ga[PER], gb[PER];
    double A[PER], B[PER], amax, bmax;
    band_energies<LOGNG>(h, b, q0u, q0v, s_wt, W, ga, gb, A, B, amax, bmax, red);
    // candidates: 1-D energies of at least alpha times the axis' largest; every entry with another factor has an
    // energy of at most tau_lo = alpha amax bmax.  The band must leave none of them out.
    double alpha = 0x1p-12;
    int shift = 48;                              // 16 bins per octave
    const double norm = 1.0 / ((double)Ng * (double)Ng);
    const bool holds = out * s1u * norm < alpha * amax && out * s1v * norm < alpha * bmax;
    const double T = tu * tv, scale = 0x1p62 / T;
    const unsigned long long target = (unsigned long long)(E * 0x1p62);     // exact: E has 53 bits
    int nA = 0, nB = 0, base = 0;
    double tau_lo = 0.0;
    bool found = false;
    for (int attempt = 0; attempt < 2 && holds; ++attempt) {
        __syncthreads();                         // the spectrum (or the last attempt's lists) is no longer read
        for (int i = tid; i < BAND_BINS; i += NT) hist[i] = 0ull;
        if (tid < 6) s_n[tid] = 0;
        if (tid == 0) s_bin = -1;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (NT * j >= b.cnt) break;
            wave_append(A[j] >= alpha * amax, A[j], eA, BAND_CAP, &s_n[0]);
            wave_append(B[j] >= alpha * bmax, B[j], eB, BAND_CAP, &s_n[1]);
        }
        __syncthreads();
        nA = s_n[0];
        nB = s_n[1];
        if (nA > BAND_CAP || nB > BAND_CAP) break;
        tau_lo = alpha * amax * bmax;
        base = (int)(__double_as_longlong(tau_lo) >> shift);
        PairWalk pw(tid, NT, nB);
        for (int e = tid; e < nA * nB; e += NT, pw.next(nB)) {
            const double p = eA[pw.ia] * eB[pw.ib];
            if (p > tau_lo) {
                const int bin = min((int)(__double_as_longlong(p) >> shift) - base, BAND_BINS - 1);
                atomicAdd(&hist[bin], __double2ull_rn(p * scale));
            }
        }
        __syncthreads();
        if (tid < 64) {
            unsigned long long hb[4], own = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                hb[i] = hist[4 * lane + i];
                own += hb[i];
            }
            unsigned long long incl = own;       // sum over this lane's bins and all higher ones
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long x = __shfl_down(incl, o);
                if (lane + o < 64) incl += x;
            }
            unsigned long long acc = incl - own;
            if (acc < target && incl >= target) {
                int bin = -1;
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    if (bin < 0 && acc + hb[i] >= target) bin = 4 * lane + i;
                    if (bin < 0) acc += hb[i];
                }
                s_bin = bin;
                s_above = acc;
            }
        }
        __syncthreads();
        found = s_bin >= 0;
        if (found || b.cnt < Ng) break;          // a lower alpha needs the whole axis
        alpha = 0x1p-60;
        shift = 50;                              // 4 bins per octave
    }
    if (found) {
        const int bin = s_bin;
        PairWalk pw(tid, NT, nB);
        for (int e = tid; e < nA * nB; e += NT, pw.next(nB)) {
            const double p = eA[pw.ia] * eB[pw.ib];
            if (p > tau_lo && min((int)(__double_as_longlong(p) >> shift) - base, BAND_BINS - 1) == bin) {
                const int at = atomicAdd(&s_n[2], 1);
                if (at < BAND_LIST) {
                    lp[at] = p;
                    lq[at] = __double2ull_rn(p * scale);
                }
            }
        }
        __syncthreads();
        found = s_n[2] <= BAND_LIST;
    }
    if (!found) {                                // uniform over the workgroup
        if (tid == 0) list.push(k);
        return;
    }
    if (tid < 64) {
        const int n = s_n[2];
        const unsigned long long above = s_above;
        double best = 0.0;
        for (int i = lane; i < n; i += 64) {
            const double pi = lp[i];
            unsigned long long s = above;
            for (int j = 0; j < n; ++j) s += lp[j] >= pi ? lq[j] : 0ull;
            if (s >= target) best = fmax(best, pi);
        }
        best = wave_max(best);
        if (lane == 0) s_tau = best;
    }
    __syncthreads();
    const double tau = s_tau;
    int c = 0;
    PairWalk pw(tid, NT, nB);
    for (int e = tid; e < nA * nB; e += NT, pw.next(nB)) c += eA[pw.ia] * eB[pw.ib] >= tau;
    // factors with a kept entry: A_a bmax >= tau, amax B_b >= tau (the fill pass's expressions)
    int na = 0, nb = 0;
    for (int i = tid; i < nA; i += NT) na += eA[i] * bmax >= tau;
    for (int i = tid; i < nB; i += NT) nb += amax * eB[i] >= tau;
    for (int o = 32; o > 0; o >>= 1) {
        c += __shfl_xor(c, o);
        na += __shfl_xor(na, o);
        nb += __shfl_xor(nb, o);
    }
    if constexpr (NT > 64) {
        if (lane == 0) {
            atomicAdd(&s_n[3], c);
            atomicAdd(&s_n[4], na);
            atomicAdd(&s_n[5], nb);
        }
        __syncthreads();
        c = s_n[3];
        na = s_n[4];
        nb = s_n[5];
    }
    if (tid == 0) {
        tau_out[k] = tau;
        nnz_out[k] = c;
        fsz_out[k] = factor_record_bytes(na, nb);
        key_out[k] = row_key(ut, vt, Ng);
    }
    // the fill pass's own condition that the band leaves no kept entry out
    if (!rc || !(out * s1u * norm * bmax < tau && out * s1v * norm * amax < tau)) return;
    int at_a[PER], at_b[PER], nca, ncb;
    candidate_places<NT, PER>(A, B, amax, bmax, tau, b, Ng, s_wc, at_a, at_b, nca, ncb);
    if (nca + ncb > CAND_MAX) return;
    double2 *rg = (double2 *)(rc + sizeof(RowCand));
    double *re = (double *)(rg + nca + ncb);
    uint16_t *rq = (uint16_t *)(re + nca + ncb);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int p = tid + NT * j;
        if (at_a[j] >= 0) {
            rg[at_a[j]] = ga[j];
            re[at_a[j]] = A[j];
            rq[at_a[j]] = (uint16_t)((b.su + p) & (Ng - 1));
        }
        if (at_b[j] >= 0) {
            rg[nca + at_b[j]] = gb[j];
            re[nca + at_b[j]] = B[j];
            rq[nca + at_b[j]] = (uint16_t)((b.sv + p) & (Ng - 1));
        }
    }
    // every tap |g| <= sqrt(amax bmax)
    if (tid == 0) *(RowCand *)rc = RowCand{nca, ncb, sqrt(amax * bmax) / 32767.0, u[k], v[k], wk, tau};
}

// A sorted row from its candidates in LDS (both axes ascending by cell; off and cnt: room for ncb <= BAND_CAP ints each):
// the kept entries in ascending column order, and the factor record.  Called by all NT threads after a barrier.
template <int TK, int NT>
__device__ __forceinline__ void emit_row(int nca, int ncb, const double2 *gA, const double2 *gB, const double *eA,
                                         const double *eB, const uint16_t *ca, const uint16_t *cb, int *off, int *cnt,
                                         double tau, double i16_scale, int Ng, int64_t r, int64_t beg, int len,
                                         int *__restrict__ col, void *__restrict__ val, float *__restrict__ rscale,
                                         const int64_t *__restrict__ frec, unsigned char *__restrict__ fdat,
                                         int *__restrict__ err) {
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    if (TK == WP_TAPS_I16 && tid == 0) rscale[r] = (float)i16_scale;
    for (int ib = tid; ib < ncb; ib += NT) {              // kept entries per candidate row
        const double Bb = eB[ib];
        int c = 0;
        for (int ia = 0; ia < nca; ++ia) c += eA[ia] * Bb >= tau;
        cnt[ib] = c;
    }
    __syncthreads();
    if (tid < 64) {                                       // offsets: lane l takes rows 2l, 2l + 1
        const int c0 = 2 * lane < ncb ? cnt[2 * lane] : 0, c1 = 2 * lane + 1 < ncb ? cnt[2 * lane + 1] : 0;
        int x = c0 + c1;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (2 * lane < ncb) off[2 * lane] = x - c0 - c1;
        if (2 * lane + 1 < ncb) off[2 * lane + 1] = x - c1;
        if (lane == 63 && x != len) atomicOr(err, 2);
    }
    __syncthreads();
    // factor record: candidates ranked by descending energy (ties by ascending cell); a v candidate's kept u
    // candidates are then the first nb of that order, nb = its tap count
    if (fdat) {
        unsigned char *rec = fdat + frec[r];
        const int nu = nca, nv = ncb;
        if ((int64_t)factor_record_bytes(nu, nv) != frec[r + 1] - frec[r]) {
            if (tid == 0) atomicOr(err, 4);
        } else {
            uint16_t *ua = (uint16_t *)rec + 2, *vb = ua + nu, *nbv = vb + nv;
            const int vals = (4 + 2 * nu + 4 * nv + 7) & ~7;
            float2 *gu = (float2 *)(rec + vals), *gv = gu + nu;
            if (tid == 0) {
                *(uint32_t *)rec = (uint32_t)nu | ((uint32_t)nv << 16);
                for (int z = 4 + 2 * nu + 4 * nv; z < vals; ++z) rec[z] = 0;
            }
            for (int ia = tid; ia < nu; ia += NT) {
                const double Aa = eA[ia];
                int rank = 0;
                for (int j = 0; j < nu; ++j) {
                    const double Aj = eA[j];
                    rank += (Aj > Aa) || (Aj == Aa && j < ia);
                }
                ua[rank] = ca[ia];
                gu[rank] = make_float2((float)gA[ia].x, (float)gA[ia].y);
            }
            for (int ib = tid; ib < nv; ib += NT) {
                const double Bb = eB[ib];
                int rank = 0;
                for (int j = 0; j < nv; ++j) {
                    const double Bj = eB[j];
                    rank += (Bj > Bb) || (Bj == Bb && j < ib);
                }
                vb[rank] = cb[ib];
                nbv[rank] = (uint16_t)cnt[ib];
                gv[rank] = make_float2((float)gB[ib].x, (float)gB[ib].y);
            }
        }
    }
    if (!col) return;                                     // factor-record form: no stored taps
    // one wave per candidate row, lanes over the u candidates, ballot-compacted: ascending columns
    for (int ia0 = 0; ia0 < nca; ia0 += 64) {
        const int ia = ia0 + lane;
        const bool in = ia < nca;
        const double Aa = in ? eA[ia] : 0.0;
        const double2 gu = in ? gA[ia] : make_double2(0.0, 0.0);
        const int a = in ? ca[ia] : 0;
        for (int ib = wv; ib < ncb; ib += NW) {
            const bool keep = in && Aa * eB[ib] >= tau;
            const unsigned long long m = __ballot(keep);
            const int o = off[ib];
            if (keep) {
                const int at = o + __popcll(m & below);
                if (at < len) {
                    const double2 g = cmul(gB[ib], gu);
                    const int64_t p = beg + at;
                    col[p] = (int)cb[ib] * Ng + a;
                    if (TK == WP_TAPS_BF16) ((uint32_t *)val)[p] = pack_bf16x2((float)g.x, (float)g.y);
                    else if (TK == WP_TAPS_I16)
                        ((uint32_t *)val)[p] = pack_i16x2((float)(g.x / i16_scale), (float)(g.y / i16_scale));
                    else ((float2 *)val)[p] = make_float2((float)g.x, (float)g.y);
                }
            }
            // each wave owns its rows, so their offsets advance without a barrier
            if (lane == 0 && ia0 + 64 < nca) off[ib] = o + __popcll(m);
        }
        wave_sync();                                      // lane 0's stores before the next round's loads
    }
}

// Pass 2 for the sorted rows marked in `todo`, one per workgroup (the others' workgroups end at once: 65536 of them in 29
// us), from their spectra; rows it cannot take are listed.  Looping over a list of the marked rows instead kept the rows'
// common constants in registers and spilled.
template <int LOGNG, int TK>
__global__ __launch_bounds__(row_threads<LOGNG>(), 4) void k_band_fill(
    const double *__restrict__ u, const double *__restrict__ v, const double *__restrict__ w, double cell, double delta,
    double L2, int W, double beta, const double2 *__restrict__ tw, const double *__restrict__ tau_in,
    const int *__restrict__ perm, const int64_t *__restrict__ rowptr, int *__restrict__ col, void *__restrict__ val,
    float *__restrict__ rscale, const int64_t *__restrict__ frec, unsigned char *__restrict__ fdat,
    int *__restrict__ err, int64_t r0, const int *__restrict__ todo, const RowList list) {
    constexpr int Ng = 1 << LOGNG, NT = row_threads<LOGNG>(), PER = band_groups<LOGNG>();
    extern __shared__ __align__(16) unsigned char smem[];
    double2 *h = (double2 *)smem;
    // after the factors are in registers the spectrum's space holds the candidates, ascending by cell
    double2 *gA = (double2 *)smem, *gB = gA + BAND_CAP;
    double *eA = (double *)(gB + BAND_CAP), *eB = eA + BAND_CAP;
    int *off = (int *)(eB + BAND_CAP);                    // first entry of candidate row ib, then its count
    int *cnt = off + BAND_CAP;
    uint16_t *ca = (uint16_t *)(cnt + BAND_CAP), *cb = ca + BAND_CAP;
    __shared__ double red[2 * (NT / 64)], s_wt[32];
    __shared__ int s_wc[PER][NT / 64][4];

    const int64_t r = r0 + blockIdx.x;
    if (todo[r] == 0) return;
    const int tid = threadIdx.x;
    const int64_t beg = rowptr[r];
    const int len = (int)(rowptr[r + 1] - beg);
    const int k = perm[r];
    const double tau = tau_in[k];
    const double ut = u[k] / cell, vt = v[k] / cell, wk = w[k];
    int q0u, q0v;
    row_weights(ut, vt, W, beta, Ng, s_wt, q0u, q0v);
    const Band b = band_of<LOGNG>(wk, L2, W, q0u, q0v);
    if (b.cnt > PER * NT) {                           // uniform over the workgroup
        if (tid == 0) list.push(r);
        return;
    }
    row_spectrum<LOGNG>(h, wk, delta, tw);           // ends with a barrier: the weights are visible
    double s1u, s1v, tu, tv;
    weight_sums(s_wt, W, s1u, tu);
    weight_sums(s_wt + 16, W, s1v, tv);
    const double out = outside_max<LOGNG>(h, b, W, red);
    double2 ga[PER], gb[PER];
    double A[PER], B[PER], amax, bmax;
    band_energies<LOGNG>(h, b, q0u, q0v, s_wt, W, ga, gb, A, B, amax, bmax, red);
    const double norm = 1.0 / ((double)Ng * (double)Ng);
    const bool holds = out * s1u * norm * bmax < tau && out * s1v * norm * amax < tau;
    const double i16_scale = sqrt(amax * bmax) / 32767.0;     // every tap |g| <= sqrt(amax bmax)
    int at_a[PER], at_b[PER], nca, ncb;
    candidate_places<NT, PER>(A, B, amax, bmax, tau, b, Ng, s_wc, at_a, at_b, nca, ncb);
    if (!holds || nca > BAND_CAP || ncb > BAND_CAP) { // uniform over the workgroup
        if (tid == 0) list.push(r);
        return;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int p = tid + NT * j;
        if (at_a[j] >= 0) {
            ca[at_a[j]] = (uint16_t)((b.su + p) & (Ng - 1));
            eA[at_a[j]] = A[j];
            gA[at_a[j]] = ga[j];
        }
        if (at_b[j] >= 0) {
            cb[at_b[j]] = (uint16_t)((b.sv + p) & (Ng - 1));
            eB[at_b[j]] = B[j];
            gB[at_b[j]] = gb[j];
        }
    }
    __syncthreads();
    emit_row<TK, NT>(nca, ncb, gA, gB, eA, eB, ca, cb, off, cnt, tau, i16_scale, Ng, r, beg, len, col, val, rscale,
                     frec, fdat, err);
}

// Pass 2 for one sorted row per wavefront (and workgroup) from the candidates the count pass left of it, if they are this
// row's; the others are marked in todo.
// Bound by the entries' stores; measured with the count pass in count_rows (builder.hip).
template <int TK>
__global__ __launch_bounds__(64) void k_cand_fill(const double *__restrict__ u, const double *__restrict__ v, const double *__restrict__ w,
                                                  const unsigned char *__restrict__ cand, const double *__restrict__ tau_in,
                                                  int Ng, const int *__restrict__ perm, const int64_t *__restrict__ rowptr,
                                                  int *__restrict__ col, void *__restrict__ val, float *__restrict__ rscale,
                                                  const int64_t *__restrict__ frec, unsigned char *__restrict__ fdat,
                                                  int *__restrict__ err, int64_t r0, int *__restrict__ todo) {
    __shared__ double2 s_g[CAND_MAX];
    __shared__ double s_e[CAND_MAX];
    __shared__ int s_off[CAND_MAX], s_cnt[CAND_MAX];
    __shared__ uint16_t s_q[CAND_MAX];
    const int tid = threadIdx.x;
    const int64_t r = r0 + blockIdx.x;
    const int64_t beg = rowptr[r];
    const int len = (int)(rowptr[r + 1] - beg);
    if (len == 0) {
        if (tid == 0) todo[r] = 0;
        if (fdat && tid == 0) *(uint2 *)(fdat + frec[r]) = make_uint2(0u, 0u);   // nu = nv = 0
        return;
    }
    const int k = perm[r];
    const double tau = tau_in[k], uk = u[k], vk = v[k], wk = w[k];
    RowCand h{-1, 0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const unsigned char *rc = cand + (int64_t)k * CAND_BYTES;
    if (k < CAND_ROWS) h = *(const RowCand *)rc;
    const bool left = h.nca < 0 || h.ncb < 0 || h.nca > CAND_MAX || h.ncb > CAND_MAX - h.nca || h.tau != tau ||
                      h.u != uk || h.v != vk || h.w != wk;                                        // uniform
    if (tid == 0) todo[r] = left;
    if (left) return;
    const int n = h.nca + h.ncb;
    const double2 *rg = (const double2 *)(rc + sizeof(RowCand));
    const double *re = (const double *)(rg + n);
    const uint16_t *rq = (const uint16_t *)(re + n);
    for (int i = tid; i < n; i += 64) {
        s_g[i] = rg[i];
        s_e[i] = re[i];
        s_q[i] = (uint16_t)(rq[i] & (Ng - 1));
    }
    __syncthreads();
    emit_row<TK, 64>(h.nca, h.ncb, s_g, s_g + h.nca, s_e, s_e + h.nca, s_q, s_q + h.nca, s_off, s_cnt, tau, h.i16_scale, Ng, r,
                     beg, len, col, val, rscale, frec, fdat, err);
}

}  // namespace

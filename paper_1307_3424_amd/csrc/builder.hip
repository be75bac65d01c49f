// Builder of the sparse w-projection matrix G (Sections 3.1 and 3.2).
//
// Row k of G, for a visibility at grid coordinates (u~, v~) with component w:
//   1. chirp exp(i pi w l^2) sampled on the padded grid, l = t delta,
//      t in [-Ng/2, Ng/2); phase argument w delta^2 t^2 in FP64 (sincospi);
//   2. its 1-D spectrum h(d) = Ng^-1 sum_t c(t) exp(-2 pi i t d / Ng) (FP64 FFT
//      in LDS).  The linear chirp and the KB window are both separable, so the
//      2-D row is g(q_v, q_u) = g_v(q_v) g_u(q_u) exactly, with
//   3. g_u(q) = sum_i KB(u~ - q'_i) h((q'_i - q) mod Ng) over the W window cells
//      q'_i (u~ - q'_i in [-W/2, W/2)), KB(t) = I0(beta sqrt(1 - (2t/W)^2));
//   4. energies A_a = |g_u(a)|^2, B_b = |g_v(b)|^2; a tap's energy is A_a B_b.
//      Threshold tau = the largest value with K(tau) >= E T, where K(tau) sums
//      the tap energies >= tau and T = K(0) (Section 3.2: keep a fraction E of
//      the row energy), so the kept set {A_a B_b >= tau} (ties kept) is the
//      sort-defined set.  E >= 1 keeps every non-zero tap.
//      Rows are made from a band of cells around the visibility (builder_rows.h).
//      The others (wide chirps, E >= 1) take the whole axes here: tau by bisection
//      on the IEEE-754 bit pattern of non-negative doubles (monotone), 64 steps at
//      most; with B sorted descending and its prefix sums, K(tau) = sum_a A_a
//      PB[#{b: A_a B_b >= tau}] costs O(Ng log Ng).
//   5. CSR: rows are sorted by the Z-order code of their centre cell (stable radix
//      sort; every aligned 32 x 32 tile of cells is then a contiguous range of rows), row lengths are scanned into int64 offsets,
//      and the fill pass writes each row's taps in ascending flattened column
//      q_v Ng + q_u, values g_v g_u rounded to complex float32 (or bf16 pairs).
// Pass 1 (count) computes tau, row lengths, the tile sort, the offsets and the
// adjoint work list sizes; pass 2 (fill) writes the taps, of most rows from the
// candidates that pass 1 left of these coordinates, of the others from row
// factors made again.
#include <cfloat>
#include <climits>
#include <cstdio>

#include "builder_exact.h"
#include "builder_lowrank.h"
#include "builder_rows.h"
#include "builder_sort.h"
#include "builder_util.h"
#include "fft_lds.h"

namespace {

constexpr int ROWS_PER_ITEM = 32;
constexpr int64_t ROW_CHUNK = 1 << 22;     // rows per launch of the per-row kernels

// Whole-axis kernels: threads per row, and the wavefronts per SIMD their registers have to allow.  A row here is long
// serial work and gets more threads than a band row.  Builds on MI355X, band-row threads (64 up to Ng = 512) and the rows'
// loop around the whole body against these: one row of 256 x 256 pixels at E = 1 2230 -> 750 us, 4000 rows of 59000 taps
// 2750 -> 1760, 20000 of 7000 at 512 pixels 7130 -> 4720.
template <int LOGNG>
constexpr int wide_threads() { return LOGNG <= 6 ? 64 : LOGNG <= 11 ? 256 : 512; }
template <int LOGNG>
constexpr int wide_waves() { return LOGNG == 10 ? 5 : 6; }   // Ng = 1024 at E = 1: 2240 us with 5, 2510 with 6

// A function's arguments arrive in vector registers, pointers as generic ones; these are the same in all lanes.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform(int64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)x), hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
    return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double uniform(double x) { return __longlong_as_double(uniform((int64_t)__double_as_longlong(x))); }
template <typename T>
__device__ __forceinline__ T *uniform(T *p) { return as_global((T *)uniform((int64_t)p)); }

// K(tau): energy and, with COUNT, number of taps with A_a B_b >= tau.  Bs sorted descending,
// PB[i] = sum of the first i entries of Bs.
template <int LOGNG, bool COUNT>
__device__ inline void kept_energy(const double *A, const double *Bs, const double *PB, double tau,
                                   double &K, long long &cnt, double *redd, long long *redl) {
    constexpr int Ng = 1 << LOGNG;
    double k = 0.0;
    long long c = 0;
    constexpr int NT = wide_threads<LOGNG>();
    for (int a = threadIdx.x; a < Ng; a += NT) {
        const double Aa = A[a];
        if (!(Aa * Bs[0] >= tau)) continue;
        int lo = 1, hi = Ng;                 // largest n with Aa * Bs[n-1] >= tau
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (Aa * Bs[mid - 1] >= tau) lo = mid; else hi = mid - 1;
        }
        k += Aa * PB[lo];
        c += lo;
    }
    K = block_sum<double, NT>(k, redd);
    if constexpr (COUNT) cnt = block_sum<long long, NT>(c, redl);
}

// ---------------------------------------------------------------------------- pass 1: threshold and count

// Whole-axis form of pass 1 for row k.  The row factors come from the same code as the band's, so either fill pass finds
// the kept set that either count pass counted.  Not inlined: in a loop over rows the compiler keeps the constants of all
// its functions in registers (153 instead of 72 at Ng = 512: three wavefronts per SIMD).
template <int LOGNG>
__device__ __noinline__ void row_count(const double *u, const double *v, const double *w, double E, double cell, double delta,
                                       int W, double beta, const double2 *tw64, double *tau_out, int *nnz_out, int *key_out,
                                       int *fsz_out, int *err, int64_t k) {
    u = uniform(u), v = uniform(v), w = uniform(w), tw64 = uniform(tw64), tau_out = uniform(tau_out);
    nnz_out = uniform(nnz_out), key_out = uniform(key_out), fsz_out = uniform(fsz_out), err = uniform(err);
    E = uniform(E), cell = uniform(cell), delta = uniform(delta), beta = uniform(beta), W = uniform(W), k = uniform(k);
    constexpr int Ng = 1 << LOGNG, BNTH = wide_threads<LOGNG>();
    extern __shared__ __align__(16) unsigned char smem[];
    double2 *h = (double2 *)smem;                 // the spectrum, later PB (Ng+1 doubles)
    double *A = (double *)(smem + spectrum_lds<LOGNG>());       // Ng
    double *B = A + Ng;                           // Ng (sorted descending in place)
    double *PB = (double *)smem;
    __shared__ double redd[BNTH / 64];
    __shared__ long long redl[BNTH / 64];
    __shared__ int redi[BNTH / 64];
    __shared__ double s_wt[32];

    __syncthreads();                                  // the last row's tables are no longer read
    const double ut = u[k] / cell, vt = v[k] / cell, wk = w[k];
    const bool ok = isfinite(ut) && isfinite(vt) && isfinite(wk) && fabs(ut) < Ng / 2 && fabs(vt) < Ng / 2;
    if (!ok) {
        if (threadIdx.x == 0) {
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
    row_spectrum<LOGNG, BNTH>(h, wk, delta, tw64);          // ends with a barrier: the weights are visible
    for (int q = threadIdx.x; q < Ng; q += BNTH) {
        const double2 gu = row_value(h, q0u, s_wt, W, q, Ng);
        const double2 gv = row_value(h, q0v, s_wt + 16, W, q, Ng);
        A[q] = energy(gu);
        B[q] = energy(gv);
    }
    __syncthreads();
    // bitonic sort of B, descending
    for (int kk = 2; kk <= Ng; kk <<= 1) {
        for (int j = kk >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < Ng; i += BNTH) {
                const int ixj = i ^ j;
                if (ixj > i) {
                    const double x0 = B[i], x1 = B[ixj];
                    const bool desc = (i & kk) == 0;
                    if (desc ? (x0 < x1) : (x0 > x1)) { B[i] = x1; B[ixj] = x0; }
                }
            }
            __syncthreads();
        }
    }
    // prefix sums of the sorted B (sequential per wave chunk: Ng values, 256 threads)
    {
        constexpr int PER = (Ng + BNTH - 1) / BNTH;
        double loc[PER];
        double s = 0.0;
        const int b0 = threadIdx.x * PER;
        for (int i = 0; i < PER; ++i) {
            loc[i] = (b0 + i < Ng) ? B[b0 + i] : 0.0;
            s += loc[i];
        }
        // exclusive scan of s across the block (FP64)
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
        double x = s;
        for (int o = 1; o < 64; o <<= 1) {
            double y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        __syncthreads();
        if (lane == 63) redd[wid] = x;
        __syncthreads();
        double off = 0.0;
        for (int i = 0; i < wid; ++i) off += redd[i];
        double run = off + x - s;
        __syncthreads();
        for (int i = 0; i < PER; ++i) {
            if (b0 + i < Ng) PB[b0 + i] = run;
            run += loc[i];
        }
        if (b0 + PER == Ng) PB[Ng] = run;
        __syncthreads();
    }
    double T;
    long long cnt;
    kept_energy<LOGNG, false>(A, B, PB, 0.0, T, cnt, redd, redl);
    double tau;
    if (E >= 1.0) {
        tau = DBL_TRUE_MIN;                        // every non-zero tap
    } else {
        double amax = 0.0;
        for (int a = threadIdx.x; a < Ng; a += BNTH) amax = fmax(amax, A[a]);
        amax = block_max<BNTH>(amax, redd);
        const double target = E * T;
        unsigned long long lo = 0ull;
        unsigned long long hi = (unsigned long long)__double_as_longlong(amax * B[0]) + 1ull;
        while (hi - lo > 1ull) {
            const unsigned long long mid = lo + ((hi - lo) >> 1);
            double Km;
            kept_energy<LOGNG, false>(A, B, PB, __longlong_as_double((long long)mid), Km, cnt, redd, redl);
            if (Km >= target) lo = mid; else hi = mid;
        }
        tau = __longlong_as_double((long long)lo);
    }
    double Kt;
    kept_energy<LOGNG, true>(A, B, PB, tau, Kt, cnt, redd, redl);
    // candidates of the factor record, with the fill pass's expressions: u cells with A_a bmax >= tau,
    // v cells with amax B_b >= tau (B is sorted: B[0] = bmax)
    double amax = 0.0;
    for (int a = threadIdx.x; a < Ng; a += BNTH) amax = fmax(amax, A[a]);
    amax = block_max<BNTH>(amax, redd);
    const double bmax = B[0];
    int na = 0, nb = 0;
    for (int q = threadIdx.x; q < Ng; q += BNTH) {
        na += (A[q] * bmax >= tau);
        nb += (amax * B[q] >= tau);
    }
    na = block_sum<int, BNTH>(na, redi);
    nb = block_sum<int, BNTH>(nb, redi);
    if (threadIdx.x == 0) {
        tau_out[k] = tau;
        nnz_out[k] = (int)cnt;
        fsz_out[k] = factor_record_bytes(na, nb);
        key_out[k] = row_key(ut, vt, Ng);
    }
}

// the listed rows, or with ALL row r0 + blockIdx.x
template <int LOGNG, bool ALL>
__global__ __launch_bounds__(wide_threads<LOGNG>(), wide_waves<LOGNG>()) void k_row_count(
    const double *__restrict__ u, const double *__restrict__ v, const double *__restrict__ w, double E, double cell,
    double delta, int W, double beta, const double2 *__restrict__ tw64, double *__restrict__ tau_out,
    int *__restrict__ nnz_out, int *__restrict__ key_out, int *__restrict__ fsz_out, int *__restrict__ err, int64_t r0,
    const RowList list) {
    const auto row = [&](int64_t k) {
        row_count<LOGNG>(u, v, w, E, cell, delta, W, beta, tw64, tau_out, nnz_out, key_out, fsz_out, err, k);
    };
    if constexpr (ALL) row(r0 + blockIdx.x);
    else list.each(row);
}

// ---------------------------------------------------------------------------- pass 2: fill

// Whole-axis form of pass 2 for sorted row r (not inlined, as row_count).
template <int LOGNG, int TK>
__device__ __noinline__ void row_fill(const double *u, const double *v, const double *w, double cell, double delta, int W,
                                      double beta, const double2 *tw64, const double *tau_in, const int *perm,
                                      const int64_t *rowptr, int *col, void *val, float *rscale, const int64_t *frec,
                                      unsigned char *fdat, int *err, int64_t r) {
    u = uniform(u), v = uniform(v), w = uniform(w), tw64 = uniform(tw64), tau_in = uniform(tau_in), perm = uniform(perm);
    rowptr = uniform(rowptr), col = uniform(col), val = uniform((char *)val), rscale = uniform(rscale), frec = uniform(frec);
    fdat = uniform(fdat), err = uniform(err), cell = uniform(cell), delta = uniform(delta), beta = uniform(beta);
    W = uniform(W), r = uniform(r);
    constexpr int Ng = 1 << LOGNG, BNTH = wide_threads<LOGNG>();
    constexpr int PER = (Ng + BNTH - 1) / BNTH;
    extern __shared__ __align__(16) unsigned char smem[];
    double2 *h = (double2 *)smem;                 // the spectrum
    double *A = (double *)(smem + spectrum_lds<LOGNG>());       // Ng energies along u (those along v are recomputed)
    int *off = (int *)(A + Ng);                   // Ng per-candidate-row output offsets
    uint16_t *ca = (uint16_t *)(off + Ng);        // Ng candidate columns (u)
    uint16_t *cb = ca + Ng;                       // Ng candidate rows (v)
    __shared__ double redd[BNTH / 64];
    __shared__ int redi[BNTH / 64];
    __shared__ int s_nca, s_ncb;
    __shared__ double s_wt[32];

    __syncthreads();                                  // the last row's tables are no longer read
    const int k = perm[r];
    const double tau = tau_in[k];
    const int64_t beg = rowptr[r], len = rowptr[r + 1] - beg;
    if (len == 0) {
        if (fdat && threadIdx.x == 0) *(uint2 *)(fdat + frec[r]) = make_uint2(0u, 0u);   // nu = nv = 0
        return;
    }
    const double ut = u[k] / cell, vt = v[k] / cell, wk = w[k];
    int q0u, q0v;
    row_weights(ut, vt, W, beta, Ng, s_wt, q0u, q0v);
    row_spectrum<LOGNG, BNTH>(h, wk, delta, tw64);          // ends with a barrier: the weights are visible
    double amax = 0.0, bmax = 0.0;
    double bq[PER];                                    // energies along v of this thread's cells q0 + i
    const int q0 = threadIdx.x * PER;
    for (int q = threadIdx.x; q < Ng; q += BNTH) {
        const double Aq = energy(row_value(h, q0u, s_wt, W, q, Ng));
        A[q] = Aq;
        amax = fmax(amax, Aq);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int q = q0 + i;
        bq[i] = q < Ng ? energy(row_value(h, q0v, s_wt + 16, W, q, Ng)) : 0.0;
        bmax = fmax(bmax, bq[i]);
    }
    amax = block_max<BNTH>(amax, redd);                      // its barriers also publish A
    bmax = block_max<BNTH>(bmax, redd);
    // int16 block floating point: every tap |g| <= sqrt(amax bmax), so re / s and im / s fit in +-32767
    const double i16_scale = sqrt(amax * bmax) / 32767.0;
    if (TK == WP_TAPS_I16 && threadIdx.x == 0) rscale[r] = (float)i16_scale;
    // candidate compaction (ascending index); a kept tap needs A_a bmax >= tau and amax B_b >= tau
    {
        int na = 0, nb = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = q0 + i;
            if (q < Ng) {
                na += (A[q] * bmax >= tau);
                nb += (amax * bq[i] >= tau);
            }
        }
        int ta, tb;
        int oa = block_excl_scan<BNTH>(na, redi, ta);
        int ob = block_excl_scan<BNTH>(nb, redi, tb);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = q0 + i;
            if (q < Ng) {
                if (A[q] * bmax >= tau) ca[oa++] = (uint16_t)q;
                if (amax * bq[i] >= tau) cb[ob++] = (uint16_t)q;
            }
        }
        if (threadIdx.x == 0) { s_nca = ta; s_ncb = tb; }
        __syncthreads();
    }
    const int nca = s_nca, ncb = s_ncb;
    // kept taps per candidate row, then offsets
    {
        int cntl[PER];
        int tot = 0;
        for (int i = 0; i < PER; ++i) {
            const int ib = threadIdx.x * PER + i;
            int c = 0;
            if (ib < ncb) {
                const double Bb = energy(row_value(h, q0v, s_wt + 16, W, cb[ib], Ng));
                for (int ia = 0; ia < nca; ++ia) c += (A[ca[ia]] * Bb >= tau);
            }
            cntl[i] = c;
            tot += c;
        }
        int total;
        int o = block_excl_scan<BNTH>(tot, redi, total);
        for (int i = 0; i < PER; ++i) {
            const int ib = threadIdx.x * PER + i;
            if (ib < ncb) off[ib] = o;
            o += cntl[i];
        }
        if (threadIdx.x == 0 && total != len) atomicOr(err, 2);
        __syncthreads();
    }
    // factor record: candidates ranked by descending energy (ties by ascending cell); a v candidate's
    // kept u candidates are then the first nb of that order, nb = its tap count
    if (fdat) {
        unsigned char *rec = fdat + frec[r];
        const int nu = nca, nv = ncb;
        if ((int64_t)factor_record_bytes(nu, nv) != frec[r + 1] - frec[r]) {
            if (threadIdx.x == 0) atomicOr(err, 4);
        } else {
            uint16_t *ua = (uint16_t *)rec + 2, *vb = ua + nu, *nbv = vb + nv;
            const int vals = (4 + 2 * nu + 4 * nv + 7) & ~7;
            float2 *gu = (float2 *)(rec + vals), *gv = gu + nu;
            if (threadIdx.x == 0) {
                *(uint32_t *)rec = (uint32_t)nu | ((uint32_t)nv << 16);
                for (int z = 4 + 2 * nu + 4 * nv; z < vals; ++z) rec[z] = 0;
            }
            for (int ia = threadIdx.x; ia < nu; ia += BNTH) {
                const int a = ca[ia];
                const double Aa = A[a];
                int rank = 0;
                for (int j = 0; j < nu; ++j) {
                    const double Aj = A[ca[j]];
                    rank += (Aj > Aa) || (Aj == Aa && j < ia);
                }
                const double2 g = row_value(h, q0u, s_wt, W, a, Ng);
                ua[rank] = (uint16_t)a;
                gu[rank] = make_float2((float)g.x, (float)g.y);
            }
            for (int ib = threadIdx.x; ib < nv; ib += BNTH) {
                const int b = cb[ib];
                const double2 g = row_value(h, q0v, s_wt + 16, W, b, Ng);
                const double Bb = energy(g);
                int rank = 0;
                for (int j = 0; j < nv; ++j) {
                    const double Bj = energy(row_value(h, q0v, s_wt + 16, W, cb[j], Ng));
                    rank += (Bj > Bb) || (Bj == Bb && j < ib);
                }
                vb[rank] = (uint16_t)b;
                nbv[rank] = (uint16_t)((ib + 1 < nv ? off[ib + 1] : (int)len) - off[ib]);
                gv[rank] = make_float2((float)g.x, (float)g.y);
            }
        }
    }
    if (!col) return;                                // factor-record form: no stored taps
    // emit: one wave per candidate row, ballot-compacted, ascending a
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int ib = wid; ib < ncb; ib += BNTH / 64) {
        const int b = cb[ib];
        const double2 gv = row_value(h, q0v, s_wt + 16, W, b, Ng);
        const double Bb = energy(gv);
        int64_t pos = beg + off[ib];
        for (int ia0 = 0; ia0 < nca; ia0 += 64) {
            const int ia = ia0 + lane;
            int a = 0;
            bool keep = false;
            if (ia < nca) {
                a = ca[ia];
                keep = A[a] * Bb >= tau;
            }
            const unsigned long long m = __ballot(keep);
            if (keep) {
                const int rank = __popcll(m & ((1ull << lane) - 1ull));
                const double2 gu = row_value(h, q0u, s_wt, W, a, Ng);
                const double2 g = cmul(gv, gu);
                const int64_t p = pos + rank;
                if (p < beg + len) {
                    col[p] = b * Ng + a;
                    if (TK == WP_TAPS_BF16) ((uint32_t *)val)[p] = pack_bf16x2((float)g.x, (float)g.y);
                    else if (TK == WP_TAPS_I16)
                        ((uint32_t *)val)[p] = pack_i16x2((float)(g.x / i16_scale), (float)(g.y / i16_scale));
                    else ((float2 *)val)[p] = make_float2((float)g.x, (float)g.y);
                }
            }
            pos += __popcll(m);
        }
    }
}

// the listed sorted rows, or with ALL row r0 + blockIdx.x
template <int LOGNG, int TK, bool ALL>
__global__ __launch_bounds__(wide_threads<LOGNG>(), wide_waves<LOGNG>()) void k_row_fill(
    const double *__restrict__ u, const double *__restrict__ v, const double *__restrict__ w, double cell,
    double delta, int W, double beta, const double2 *__restrict__ tw64, const double *__restrict__ tau_in,
    const int *__restrict__ perm, const int64_t *__restrict__ rowptr, int *__restrict__ col, void *__restrict__ val,
    float *__restrict__ rscale, const int64_t *__restrict__ frec, unsigned char *__restrict__ fdat, int *__restrict__ err,
    int64_t r0, const RowList list) {
    const auto row = [&](int64_t r) {
        row_fill<LOGNG, TK>(u, v, w, cell, delta, W, beta, tw64, tau_in, perm, rowptr, col, val, rscale, frec, fdat, err, r);
    };
    if constexpr (ALL) row(r0 + blockIdx.x);
    else list.each(row);
}


// ---------------------------------------------------------------------------- layout kernels

__global__ void k_gather_nnz(const int *__restrict__ perm, const int *__restrict__ nnz, int64_t *__restrict__ snnz,
                             int64_t M) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < M) snnz[r] = nnz[perm[r]];
}

// row range of every tile: the tile's Z-order code is the row key shifted by the tile's bits
__global__ void k_tile_bounds(const int *__restrict__ skey, int64_t M, int shift, int *__restrict__ tstart,
                              int *__restrict__ tend) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= M) return;
    const int k = skey[r] >> shift;
    if (r == 0 || (skey[r - 1] >> shift) != k) tstart[k] = (int)r;
    if (r == M - 1 || (skey[r + 1] >> shift) != k) tend[k] = (int)r + 1;
}

__global__ void k_tile_chunks(const int *__restrict__ tstart, const int *__restrict__ tend, int T,
                              int *__restrict__ nchunk) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < T) nchunk[t] = (tend[t] - tstart[t] + ROWS_PER_ITEM - 1) / ROWS_PER_ITEM;
}

__global__ void k_write_items(const int *__restrict__ tstart, const int *__restrict__ tend,
                              const int *__restrict__ choff, int T, int ntile, int *__restrict__ work) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    const int s = tstart[t], e = tend[t];
    int it = choff[t];
    int tv, tu;
    demorton2(t, tv, tu);
    (void)ntile;
    for (int r = s; r < e; r += ROWS_PER_ITEM, ++it) {
        work[4 * it + 0] = tv;
        work[4 * it + 1] = tu;
        work[4 * it + 2] = r;
        work[4 * it + 3] = min(r + ROWS_PER_ITEM, e);
    }
}

// ---------------------------------------------------------------------------- transposed copy (gather form of G^H)

__global__ void k_t_count(const int *__restrict__ col, int64_t nnz, int *__restrict__ cnt) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nnz; j += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&cnt[col[j]], 1);
}

template <typename TapT>
__global__ void k_t_fill(const int64_t *__restrict__ rowptr, const int *__restrict__ col, const TapT *__restrict__ val,
                         const int *__restrict__ perm, int64_t M, const int64_t *__restrict__ tcolptr,
                         int *__restrict__ cur, int *__restrict__ trow, TapT *__restrict__ tval) {
    const int lane = threadIdx.x & 63;
    const int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (r >= M) return;
    for (int64_t j = rowptr[r] + lane; j < rowptr[r + 1]; j += 64) {
        const int c = col[j];
        const int64_t pos = tcolptr[c] + atomicAdd(&cur[c], 1);
        trow[pos] = (int)r;
        tval[pos] = val[j];
    }
    (void)perm;
}

// order each cell's entries by sorted row index (a row has at most one entry per cell, so the keys are distinct
// and the order is unique).  A wavefront looks at 64 cells (16 on small grids, to keep the wavefronts many) and
// sorts those of up to TS_WAVE entries, as many whole cells at a time as fit a window.  Longer cells go on lists: up
// to TS_RANK entries a wavefront each; longer ones a workgroup each, up to TS_BIG entries by a bitonic sort of (row,
// position) pairs in LDS, above by one in global memory.  Measured on MI355X against a wavefront and a bitonic LDS sort
// for each cell up to 1024 entries: 13.7M entries over 16.8M cells 7.1 -> 0.16 ms (it launched a wavefront per empty
// cell), 6.8M entries over 262144 cells 0.70 -> 0.19 ms.
constexpr int TS_WAVE = 64, TS_RANK = 256, TS_BIG = 4096;
enum { TSL_MID = 0, TSL_LONG = 1, TSL_N = 2 };     // counts of the two lists (see sort_cells)

// sort one cell's n entries (1 < n <= CAP) in LDS with the NT threads of a group; sync() orders the
// group's LDS accesses
template <typename TapT, int CAP, int NT, typename Sync>
__device__ inline void sort_cell(int64_t b, int n, int lt, int *key, unsigned short *pos, TapT *val,
                                 int *__restrict__ trow, TapT *__restrict__ tval, Sync sync) {
    int P = 2;
    while (P < n) P <<= 1;
    for (int i = lt; i < P; i += NT) {
        key[i] = i < n ? trow[b + i] : INT_MAX;  // padding sorts last
        pos[i] = (unsigned short)i;
        if (i < n) val[i] = tval[b + i];
    }
    sync();
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = lt; i < P; i += NT) {
                const int ixj = i ^ j;
                if (ixj > i) {
                    const int k0 = key[i], k1 = key[ixj];
                    if ((i & k) == 0 ? (k0 > k1) : (k0 < k1)) {
                        key[i] = k1;
                        key[ixj] = k0;
                        const unsigned short p0 = pos[i];
                        pos[i] = pos[ixj];
                        pos[ixj] = p0;
                    }
                }
            }
            sync();
        }
    }
    for (int i = lt; i < n; i += NT) {
        trow[b + i] = key[i];
        tval[b + i] = val[pos[i]];
    }
}

__global__ void k_zero_int(int *p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

// Cells CPW b .. CPW b + CPW - 1 by wavefront b; longer cells go to mid[0 ..] and, above TS_RANK, to long_end[-1 ..]
// downwards.  The wavefront takes as many whole cells at a time as fit TS_WIN entries, a lane four of them: an entry's
// rank is the number of smaller keys of its cell, read from LDS.  Bound by the loads' latency; a cell at a time (one
// entry a lane, ranks by lane broadcast) paid it for every cell: 16.8 M cells of 0.8 entries 983 us.
constexpr int TS_WIN = 256;

template <typename TapT, int CPW>
__global__ __launch_bounds__(256) void k_t_sort_short(const int64_t *__restrict__ tcolptr, int64_t cells,
                                                      int *__restrict__ trow, TapT *__restrict__ tval,
                                                      int *mid, int *long_end, int *__restrict__ count) {
    constexpr int PER = TS_WIN / 64;
    static_assert(TS_WAVE <= TS_WIN, "a short cell fits the window");
    __shared__ int s_key[4][TS_WIN];
    const int lane = threadIdx.x & 63;
    int *sk = s_key[threadIdx.x >> 6];
    const int64_t c = lane < CPW ? ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * CPW + lane : cells;
    int64_t b = INT64_MAX;
    int n = 0;
    if (c < cells) {
        b = tcolptr[c];
        n = (int)(tcolptr[c + 1] - b);
    }
    if (n > TS_RANK) long_end[-1 - atomicAdd(&count[TSL_LONG], 1)] = (int)c;
    else if (n > TS_WAVE) mid[atomicAdd(&count[TSL_MID], 1)] = (int)c;
    const bool mine = n > 1 && n <= TS_WAVE;
    unsigned long long todo = __ballot(mine);
    const int blo = (int)(b & 0xffffffff), bhi = (int)(b >> 32);
    while (todo != 0) {
        const int l0 = __builtin_ctzll(todo);
        const int64_t base = ((int64_t)__builtin_amdgcn_readlane(bhi, l0) << 32) | (unsigned int)__builtin_amdgcn_readlane(blo, l0);
        // this lane's cell relative to the window; lanes without a cell lie past every entry
        const int rel = b - base > TS_WIN ? INT_MAX : (int)(b - base < -1 ? -1 : b - base);
        const unsigned long long in = __ballot(lane >= l0 && rel <= TS_WIN && n <= TS_WIN - rel);
        todo &= ~in;
        const int last = 63 - __builtin_clzll(in);    // l0 is in: a short cell
        const int E = __builtin_amdgcn_readlane(rel, last) + __builtin_amdgcn_readlane(n, last);
        int key[PER], cs[PER], cn[PER], rank[PER];
        TapT v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e = i * 64 + lane;
            cn[i] = rank[i] = 0;
            if (e < E) {
                key[i] = trow[base + e];
                v[i] = tval[base + e];
            }
        }
        // entry e belongs to the last cell that starts at or before it
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (i * 64 >= E) break;
            const int e = i * 64 + lane;
            int l = 0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1)
                if (__shfl(rel, l + o) <= e) l += o;
            cs[i] = __shfl(rel, l);
            const int m = __shfl(n, l);
            cn[i] = e < E && m > 1 && m <= TS_WAVE ? m : 0;
            if (e < E) sk[e] = key[i];
        }
        wave_sync();
#pragma unroll
        for (int i = 0; i < PER; ++i)
            for (int j = 0; j < cn[i]; ++j) rank[i] += sk[cs[i] + j] < key[i];
        __builtin_amdgcn_s_waitcnt(0x0f70);           // vmcnt(0): every value is read before any is overwritten
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (cn[i] > 0) {
                trow[base + cs[i] + rank[i]] = key[i];
                tval[base + cs[i] + rank[i]] = v[i];
            }
        wave_sync();
    }
}

// The listed cells of TS_WAVE + 1 .. TS_RANK entries: one wavefront each (wavefronts loop over the list).  Each 64
// entries are ranked among themselves by lane broadcast and laid out sorted in LDS; an entry's place among the other
// groups is a binary search.  Bound by instruction issue: all ranks by broadcast took 14 instructions an entry pair of
// groups (6.8 M taps at 256 pixels: 137 us, now 96).
template <typename TapT>
__global__ __launch_bounds__(256) void k_t_sort_mid(const int64_t *__restrict__ tcolptr, const int *__restrict__ mid,
                                                    const int *__restrict__ count, int *__restrict__ trow,
                                                    TapT *__restrict__ tval) {
    constexpr int PER = TS_RANK / 64;
    __shared__ int s_key[4][TS_RANK];
    const int lane = threadIdx.x & 63;
    int *sk = s_key[threadIdx.x >> 6];
    const int nm = count[TSL_MID];
    for (int q = blockIdx.x * 4 + (threadIdx.x >> 6); q < nm; q += gridDim.x * 4) {
        const int64_t b = tcolptr[mid[q]];
        const int n = (int)(tcolptr[mid[q] + 1] - b);
        int key[PER], rank[PER];
        TapT v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e = i * 64 + lane;
            key[i] = INT_MAX;
            rank[i] = 0;
            if (e < n) {
                key[i] = trow[b + e];
                v[i] = tval[b + e];
            }
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int m = min(64, n - 64 * i);            // <= 0: no entries in this group
            for (int j = 0; j < m; ++j) rank[i] += __builtin_amdgcn_readlane(key[i], j) < key[i];
            if (i * 64 + lane < n) sk[64 * i + rank[i]] = key[i];
        }
        wave_sync();
#pragma unroll
        for (int g = 0; g < PER; ++g) {
            const int m = min(64, n - 64 * g);
            if (m <= 0) break;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (i == g) continue;
                int lo = 0;                               // keys of group g below this entry's
#pragma unroll
                for (int o = 64; o > 0; o >>= 1)
                    if (lo + o <= m && sk[64 * g + lo + o - 1] < key[i]) lo += o;
                rank[i] += lo;
            }
        }
        wave_sync();                                      // the next cell reuses the slice
        __builtin_amdgcn_s_waitcnt(0x0f70);               // vmcnt(0): every value is read before any is overwritten
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (i * 64 + lane < n) {
                trow[b + rank[i]] = key[i];
                tval[b + rank[i]] = v[i];
            }
    }
}

// A cell of more than TS_BIG entries by a workgroup: a bitonic network in global memory whose comparators all put the
// smaller key first, so that the places past the cell's end, which would hold the largest keys, are never touched.
// N = 256, cells of 2300 entries on average (10000 rows of 59000 taps): build 660 -> 147 ms against a shell sort by one
// thread per cell in a launch of its own.
template <typename TapT>
__device__ __forceinline__ void sort_cell_global(int n, int *kr, TapT *kv) {
    for (int64_t k = 2; k < 2 * (int64_t)n; k <<= 1) {
        for (int64_t j = k >> 1; j > 0; j >>= 1) {
            const int64_t flip = j == k >> 1 ? k - 1 : j;     // a block's first step meets its mirror image
            for (int64_t t = threadIdx.x; t < n; t += 256) {
                const int64_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), p = i ^ flip;
                if (p < n) {
                    const int k0 = kr[i], k1 = kr[p];
                    if (k0 > k1) {
                        kr[i] = k1;
                        kr[p] = k0;
                        const TapT v = kv[i];
                        kv[i] = kv[p];
                        kv[p] = v;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// the listed cells of more than TS_RANK entries: one workgroup per cell (workgroups loop over the list)
template <typename TapT>
__global__ __launch_bounds__(256) void k_t_sort_big(const int64_t *__restrict__ tcolptr, const int *__restrict__ long_end,
                                                    const int *__restrict__ count, int *__restrict__ trow,
                                                    TapT *__restrict__ tval) {
    __shared__ int s_key[TS_BIG];
    __shared__ unsigned short s_pos[TS_BIG];
    __shared__ TapT s_val[TS_BIG];
    const int nl = count[TSL_LONG];
    for (int q = blockIdx.x; q < nl; q += gridDim.x) {
        const int64_t c = long_end[-1 - q];
        const int64_t b = tcolptr[c];
        const int n = (int)(tcolptr[c + 1] - b);
        if (n > TS_BIG) {                        // uniform over the workgroup
            sort_cell_global(n, trow + b, tval + b);
            continue;
        }
        sort_cell<TapT, TS_BIG, 256>(b, n, threadIdx.x, s_key, s_pos, s_val, trow, tval, [] { __syncthreads(); });
        __syncthreads();                         // the next cell reuses the arrays
    }
}

// gather blocks: flag the cells that start a block ...
__global__ void k_gb_flags(const int64_t *__restrict__ tcolptr, int64_t cells, int ent, int *__restrict__ flag) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    const int64_t slot = tcolptr[c] / ent + c / GB_CELLS;
    flag[c] = (c == 0 || slot != tcolptr[c - 1] / ent + (c - 1) / GB_CELLS) ? 1 : 0;
}

// ... and write (first cell, first entry) of block pos[c] for each of them; the pairs from the
// block count up to index n_tblk are (cells, nnz)
__global__ void k_gb_write(const int64_t *__restrict__ tcolptr, const int *__restrict__ flag,
                           const int *__restrict__ pos, int64_t cells, int64_t nnz, int64_t n_tblk,
                           int64_t *__restrict__ tblk) {
    const int64_t n = cells > n_tblk + 1 ? cells : n_tblk + 1;
    const int64_t total = pos[cells];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < cells && flag[i]) {
            const int64_t b = pos[i];
            tblk[2 * b] = i;
            tblk[2 * b + 1] = tcolptr[i];
        }
        if (i >= total && i <= n_tblk) {
            tblk[2 * i] = cells;
            tblk[2 * i + 1] = nnz;
        }
    }
}

inline int64_t align256(int64_t b) { return (b + 255) & ~(int64_t)255; }

struct WsLayout {
    int64_t tau, nnz, key, k0, k1, i0, i1, list, todo, snnz, rowptr, sc32, sc64, tstart, tend, nch, choff, err, count,
        tcnt, sc64t, gpos, fsz, frec, ex, cand, total;
};

// rows2d: the rows are made whole in 2-D (the exact chirp, or a beam per visibility)
WsLayout ws_layout(const wp_plan *p, int64_t M, bool rows2d) {
    const int64_t T = (int64_t)p->ntile * p->ntile;
    WsLayout L;
    int64_t o = 0;
    auto take = [&](int64_t bytes) { int64_t r = o; o += align256(bytes); return r; };
    L.tau = take(8 * M);
    L.nnz = take(4 * M);
    L.key = take(4 * M);
    L.k0 = take(4 * M);
    L.k1 = take(4 * M);
    L.i0 = take(4 * M);
    L.i1 = take(4 * M);
    L.list = take(4 * RowList::rows(M));   // rows for the whole-axis kernels
    L.todo = take(4 * M);                  // marks of the sorted rows the count pass left no candidates of
    L.snnz = take(8 * M);
    L.rowptr = take(8 * (M + 1));
    L.sc32 = take(4 * std::max(rs_scratch_elems(M), scan_scratch_elems(T)));
    L.sc64 = take(8 * scan_scratch_elems(M));
    L.tstart = take(4 * T);
    L.tend = take(4 * T);
    L.nch = take(4 * T);
    L.choff = take(4 * (T + 1));
    L.err = take(16);                      // error flags; bytes of the factor records from byte 8 on
    L.count = take(4 * RowList::COUNTS);   // the list's counters
    const int64_t cells = (int64_t)p->Ng * p->Ng;
    L.tcnt = take(4 * cells);
    L.sc64t = take(8 * scan_scratch_elems(cells));
    L.gpos = take(4 * (cells + 1));
    L.fsz = take(4 * M);
    L.frec = take(8 * (M + 1));
    // the exact chirp's 2-D rows of one chunk (values, or energies in the count pass)
    L.ex = take(rows2d && p->Ng <= EXACT_MAX_NG ? EX_ROW_BYTES_PER_CELL * exact_chunk_rows(p->Ng, M) * p->Ng * p->Ng
                                                : 0);
    L.cand = take(rows2d ? 0 : CAND_BYTES * std::min<int64_t>(M, CAND_ROWS));    // the rows' candidates
    L.total = o;
    return L;
}

// the exact chirp's rows come from the separable expansion above Ng = 512, or when the plan asks for it
// (no beam: a beam's rows stay whole in 2-D)
inline bool exact_lowrank(const wp_plan *p, const double *beam) {
    if (beam || p->chirp != WP_CHIRP_EXACT) return false;
    return p->exact_rows == 1 || (p->exact_rows == 0 && p->Ng > EXACT_MAX_NG);
}

inline RowList row_list(unsigned char *ws, const WsLayout &L, int64_t M) {
    return RowList{(int *)(ws + L.list), (int *)(ws + L.count), RowList::cap(M)};
}

// LDS of the whole-axis kernels: the spectrum and two axes of 8 bytes per cell (energies; offsets and candidates)
template <int LOGNG>
constexpr size_t wide_lds() { return spectrum_lds<LOGNG>() + ((size_t)16 << LOGNG); }
// workgroups of the kernels that loop over a list: what 256 CUs hold by LDS and registers
template <int LOGNG>
constexpr int list_blocks() {
    constexpr int fit = (int)(160 * 1024 / wide_lds<LOGNG>()), waves = 4 * wide_waves<LOGNG>() * 64 / wide_threads<LOGNG>();
    return 256 * (fit < waves ? (fit < 1 ? 1 : fit) : waves);
}

// Pass 1 of the rows.  E < 1: the band kernel, then the whole-axis kernel over the rows it listed; E >= 1 keeps
// every entry, so all rows take the whole axis.  Measured on MI355X, count + fill kernels: 65536 rows at Ng = 4096
// 109 + 12 ms on the whole axes, 2.35 + 2.22 ms in the band, 2.49 + 0.11 ms with the count pass's candidates kept for
// the fill pass (for rows past CAND_ROWS, and of more than CAND_MAX candidates, as before); 32768 rows at Ng = 512
// 3.37 + 0.41, 0.18 + 0.17 and 0.19 + 0.05 ms.
template <int LOGNG>
wp_status count_rows(const wp_plan *p, int64_t M, const double *u, const double *v, const double *w, double E,
                     unsigned char *ws, const WsLayout &L, hipStream_t s) {
    static_assert(wide_lds<LOGNG>() <= 160 * 1024, "LDS budget");
    constexpr int NT = row_threads<LOGNG>();
    int *err = (int *)(ws + L.err);
    const RowList list = row_list(ws, L, M);
    double *tau = (double *)(ws + L.tau);
    int *nnz = (int *)(ws + L.nnz), *key = (int *)(ws + L.key), *fsz = (int *)(ws + L.fsz);
    // one workgroup per row, in launches of at most ROW_CHUNK rows (a grid dimension holds
    // fewer than 2^32 work-items)
    for (int64_t r0 = 0; r0 < M; r0 += ROW_CHUNK) {
        const unsigned n = (unsigned)std::min<int64_t>(ROW_CHUNK, M - r0);
        if (E < 1.0)
            hipLaunchKernelGGL((k_band_count<LOGNG>), dim3(n), dim3(NT), band_count_lds<LOGNG>(), s, u, v, w, E, p->cell,
                               p->delta, p->L * p->L, p->W, p->beta, p->tw64, tau, nnz, key, fsz, err, r0, list,
                               ws + L.cand);
        else
            hipLaunchKernelGGL((k_row_count<LOGNG, true>), dim3(n), dim3(wide_threads<LOGNG>()), wide_lds<LOGNG>(), s, u, v, w, E, p->cell,
                               p->delta, p->W, p->beta, p->tw64, tau, nnz, key, fsz, err, r0, list);
    }
    if (E < 1.0)
        hipLaunchKernelGGL((k_row_count<LOGNG, false>), dim3(list_blocks<LOGNG>()), dim3(wide_threads<LOGNG>()), wide_lds<LOGNG>(), s, u, v, w, E,
                           p->cell, p->delta, p->W, p->beta, p->tw64, tau, nnz, key, fsz, err, (int64_t)0, list);
    return wp_check_launch("build_G_count rows");
}

template <int LOGNG, int TK>
void fill_rows_tk(const wp_plan *p, int64_t M, const double *u, const double *v, const double *w, double E,
                  unsigned char *ws, const WsLayout &L, wp_G *G, hipStream_t s) {
    constexpr int NT = row_threads<LOGNG>(), Ng = 1 << LOGNG;
    int *err = (int *)(ws + L.err), *todo = (int *)(ws + L.todo);
    const RowList list = row_list(ws, L, M);
    const double *tau = (const double *)(ws + L.tau);
    const bool rec = G->frec && G->fdat;
    const int64_t *frec = rec ? (const int64_t *)(ws + L.frec) : nullptr;
    unsigned char *fdat = rec ? (unsigned char *)G->fdat : nullptr;
    for (int64_t r0 = 0; r0 < M; r0 += ROW_CHUNK) {
        const unsigned n = (unsigned)std::min<int64_t>(ROW_CHUNK, M - r0);
        if (E < 1.0)
            hipLaunchKernelGGL((k_cand_fill<TK>), dim3(n), dim3(64), 0, s, u, v, w, ws + L.cand, tau, Ng, G->perm, G->rowptr, G->col,
                               G->val, G->rscale, frec, fdat, err, r0, todo);
        else
            hipLaunchKernelGGL((k_row_fill<LOGNG, TK, true>), dim3(n), dim3(wide_threads<LOGNG>()), wide_lds<LOGNG>(), s, u, v, w, p->cell,
                               p->delta, p->W, p->beta, p->tw64, tau, G->perm, G->rowptr, G->col, G->val, G->rscale,
                               frec, fdat, err, r0, list);
    }
    for (int64_t r0 = 0; E < 1.0 && r0 < M; r0 += ROW_CHUNK)
        hipLaunchKernelGGL((k_band_fill<LOGNG, TK>), dim3((unsigned)std::min<int64_t>(ROW_CHUNK, M - r0)), dim3(NT),
                           band_fill_lds<LOGNG>(), s, u, v, w, p->cell, p->delta, p->L * p->L, p->W, p->beta, p->tw64, tau,
                           G->perm, G->rowptr, G->col, G->val, G->rscale, frec, fdat, err, r0, todo, list);
    if (E < 1.0)
        hipLaunchKernelGGL((k_row_fill<LOGNG, TK, false>), dim3(list_blocks<LOGNG>()), dim3(wide_threads<LOGNG>()), wide_lds<LOGNG>(), s, u, v, w,
                           p->cell, p->delta, p->W, p->beta, p->tw64, tau, G->perm, G->rowptr, G->col, G->val,
                           G->rscale, frec, fdat, err, (int64_t)0, list);
}

template <int LOGNG>
wp_status fill_rows(const wp_plan *p, int64_t M, const double *u, const double *v, const double *w, double E,
                    unsigned char *ws, const WsLayout &L, wp_G *G, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(256), 0, s, (int *)(ws + L.count), RowList::COUNTS);
    if (G->taps == WP_TAPS_BF16) fill_rows_tk<LOGNG, WP_TAPS_BF16>(p, M, u, v, w, E, ws, L, G, s);
    else if (G->taps == WP_TAPS_I16) fill_rows_tk<LOGNG, WP_TAPS_I16>(p, M, u, v, w, E, ws, L, G, s);
    else fill_rows_tk<LOGNG, WP_TAPS_C64>(p, M, u, v, w, E, ws, L, G, s);
    return wp_check_launch("build_G_fill rows");
}

template <typename TapT>
void sort_cells(const wp_G *G, int64_t cells, int *mid, int *count, hipStream_t s) {
    int *long_end = mid + cells;
    TapT *tval = (TapT *)G->tval;
    if (cells > 1 << 20)
        hipLaunchKernelGGL((k_t_sort_short<TapT, 64>), dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, s,
                           G->tcolptr, cells, G->trow, tval, mid, long_end, count);
    else
        hipLaunchKernelGGL((k_t_sort_short<TapT, 16>), dim3((unsigned)((cells + 63) / 64)), dim3(256), 0, s, G->tcolptr,
                           cells, G->trow, tval, mid, long_end, count);
    hipLaunchKernelGGL((k_t_sort_mid<TapT>), dim3(2048), dim3(256), 0, s, G->tcolptr, mid, count, G->trow, tval);
    hipLaunchKernelGGL((k_t_sort_big<TapT>), dim3(1024), dim3(256), 0, s, G->tcolptr, long_end, count, G->trow, tval);
}

template <int LOGNG>
wp_status count_rows_exact(const wp_plan *p, int64_t M, const double *u, const double *v, const double *w,
                           const double *beam, double E, unsigned char *ws, const WsLayout &L, hipStream_t s) {
    const int exact = p->chirp == WP_CHIRP_EXACT;
    constexpr int Ng = 1 << LOGNG;
    const int64_t B = exact_chunk_rows(Ng, M);
    double2 *rows = (double2 *)(ws + L.ex);
    double *en = (double *)(rows + B * Ng * Ng);       // energies beside the values
    for (int64_t k0 = 0; k0 < M; k0 += B) {
        const unsigned nb = (unsigned)std::min<int64_t>(B, M - k0);
        hipLaunchKernelGGL((k_exact_rows<LOGNG>), dim3(Ng / EX_LINES, nb), dim3(BNTH), 0, s, u, v, w, beam, exact,
                           nullptr, k0, p->cell, p->delta, p->W, p->beta, p->tw64, rows);
        hipLaunchKernelGGL((k_exact_cols<LOGNG, true>), dim3(Ng / EX_LINES, nb), dim3(BNTH), 0, s, u, v, w, beam,
                           nullptr, k0, p->cell, p->beta, p->W, p->tw64, rows, en);
        hipLaunchKernelGGL((k_exact_tau<LOGNG>), dim3(nb), dim3(TNT), 0, s, u, v, w, beam, k0, p->cell, E,
                           (const double *)en, (double *)(ws + L.tau), (int *)(ws + L.nnz), (int *)(ws + L.key),
                           (int *)(ws + L.fsz), (int *)(ws + L.err));
    }
    return wp_check_launch("build_G_count exact rows");
}

// the exact chirp's rows from the separable expansion (builder_lowrank.h): one workgroup per row
template <int LOGNG>
wp_status lowrank_rows(const wp_plan *p, int64_t M, const double *u, const double *v, const double *w, double E,
                       unsigned char *ws, const WsLayout &L, const wp_G *G, hipStream_t s) {
    constexpr size_t lds = lowrank_lds<LOGNG>();
    static_assert(lds <= 160 * 1024, "LDS budget");
    const double L2 = p->L * p->L;
    for (int64_t r0 = 0; r0 < M; r0 += ROW_CHUNK) {
        const dim3 g((unsigned)std::min<int64_t>(ROW_CHUNK, M - r0));
        if (!G)
            hipLaunchKernelGGL((k_lowrank_rows<LOGNG, false, WP_TAPS_C64>), g, dim3(BNTH), lds, s, u, v, w, E, p->cell,
                               p->delta, p->W, p->beta, L2, p->tw64, r0, nullptr, (double *)(ws + L.tau),
                               (int *)(ws + L.nnz), (int *)(ws + L.key), (int *)(ws + L.fsz), nullptr, nullptr,
                               nullptr, nullptr, (int *)(ws + L.err));
        else if (G->taps == WP_TAPS_BF16)
            hipLaunchKernelGGL((k_lowrank_rows<LOGNG, true, WP_TAPS_BF16>), g, dim3(BNTH), lds, s, u, v, w, E, p->cell,
                               p->delta, p->W, p->beta, L2, p->tw64, r0, G->perm, (double *)(ws + L.tau), nullptr,
                               nullptr, nullptr, G->rowptr, G->col, G->val, G->rscale, (int *)(ws + L.err));
        else if (G->taps == WP_TAPS_I16)
            hipLaunchKernelGGL((k_lowrank_rows<LOGNG, true, WP_TAPS_I16>), g, dim3(BNTH), lds, s, u, v, w, E, p->cell,
                               p->delta, p->W, p->beta, L2, p->tw64, r0, G->perm, (double *)(ws + L.tau), nullptr,
                               nullptr, nullptr, G->rowptr, G->col, G->val, G->rscale, (int *)(ws + L.err));
        else
            hipLaunchKernelGGL((k_lowrank_rows<LOGNG, true, WP_TAPS_C64>), g, dim3(BNTH), lds, s, u, v, w, E, p->cell,
                               p->delta, p->W, p->beta, L2, p->tw64, r0, G->perm, (double *)(ws + L.tau), nullptr,
                               nullptr, nullptr, G->rowptr, G->col, G->val, G->rscale, (int *)(ws + L.err));
    }
    return wp_check_launch(G ? "build_G_fill exact rows (separable expansion)" : "build_G_count exact rows (separable expansion)");
}

template <int LOGNG>
wp_status fill_rows_exact(const wp_plan *p, int64_t M, const double *u, const double *v, const double *w,
                          const double *beam, const unsigned char *ws, const WsLayout &L, wp_G *G, hipStream_t s) {
    const int exact = p->chirp == WP_CHIRP_EXACT;
    constexpr int Ng = 1 << LOGNG;
    const int64_t B = exact_chunk_rows(Ng, M);
    double2 *rows = (double2 *)(const_cast<unsigned char *>(ws) + L.ex);    // scratch region of the workspace
    const double *tau = (const double *)(ws + L.tau);
    int *err = (int *)(const_cast<unsigned char *>(ws) + L.err);
    for (int64_t r0 = 0; r0 < M; r0 += B) {
        const unsigned nb = (unsigned)std::min<int64_t>(B, M - r0);
        hipLaunchKernelGGL((k_exact_rows<LOGNG>), dim3(Ng / EX_LINES, nb), dim3(BNTH), 0, s, u, v, w, beam, exact,
                           G->perm, r0, p->cell, p->delta, p->W, p->beta, p->tw64, rows);
        hipLaunchKernelGGL((k_exact_cols<LOGNG, false>), dim3(Ng / EX_LINES, nb), dim3(BNTH), 0, s, u, v, w, beam,
                           G->perm, r0, p->cell, p->beta, p->W, p->tw64, rows, nullptr);
        if (G->taps == WP_TAPS_BF16)
            hipLaunchKernelGGL((k_exact_fill<LOGNG, WP_TAPS_BF16>), dim3(nb), dim3(BNTH), 0, s, rows, r0, tau,
                               G->perm, G->rowptr, G->col, G->val, G->rscale, err);
        else if (G->taps == WP_TAPS_I16)
            hipLaunchKernelGGL((k_exact_fill<LOGNG, WP_TAPS_I16>), dim3(nb), dim3(BNTH), 0, s, rows, r0, tau,
                               G->perm, G->rowptr, G->col, G->val, G->rscale, err);
        else
            hipLaunchKernelGGL((k_exact_fill<LOGNG, WP_TAPS_C64>), dim3(nb), dim3(BNTH), 0, s, rows, r0, tau,
                               G->perm, G->rowptr, G->col, G->val, G->rscale, err);
    }
    return wp_check_launch("build_G_fill exact rows");
}

}  // namespace

static int64_t al256(int64_t b) { return (b + 255) & ~(int64_t)255; }

int64_t scan_workspace_bytes(int64_t n) { return al256(4 * scan_scratch_elems(n)); }

wp_status launch_scan_int(const int *in, int *out, int64_t n, void *ws, hipStream_t s) {
    if (n <= 0) return wp_set_error(WP_EINVAL, "scan of %lld elements", (long long)n);
    device_scan<int, int>(in, out, n, (int *)ws, s);
    return wp_check_launch("scan");
}

int64_t sort_workspace_bytes(int64_t n) { return 2 * al256(4 * n) + al256(4 * rs_scratch_elems(n)); }

wp_status launch_sort_pairs(const int *key, int64_t n, int bits, int *keys_out, int *idx_out, void *wsv,
                            hipStream_t s) {
    if (n <= 0) return wp_set_error(WP_EINVAL, "sort of %lld elements", (long long)n);
    if (bits < 1 || bits > 31) return wp_set_error(WP_EINVAL, "sort of %d key bits", bits);
    unsigned char *ws = (unsigned char *)wsv;
    radix_sort(key, n, bits, keys_out, idx_out, (int *)ws, (int *)(ws + al256(4 * n)), (int *)(ws + 2 * al256(4 * n)), s);
    return wp_check_launch("sort");
}

// Every field but the last two sits at the same offset whatever rows2d says: the 2-D rows' chunk or the candidates.  A
// workspace for 2-D rows of a plan whose rows can also be separable holds either.
int64_t builder_workspace_bytes(const wp_plan *p, int64_t M, bool rows2d) {
    const int64_t b = ws_layout(p, M, rows2d).total;
    return rows2d && p->chirp != WP_CHIRP_EXACT ? std::max(b, ws_layout(p, M, false).total) : b;
}

// offsets of the factor records in sorted row order (after the count pass) and their total
wp_status launch_build_factor_bytes(const wp_plan *p, int64_t M, void *wsv, int64_t *bytes, hipStream_t s) {
    unsigned char *ws = (unsigned char *)wsv;
    const WsLayout L = ws_layout(p, M, false);
    const int nthr = 256;
    const dim3 gM((unsigned)((M + nthr - 1) / nthr));
    hipLaunchKernelGGL(k_gather_nnz, gM, dim3(nthr), 0, s, (const int *)(ws + L.i0), (const int *)(ws + L.fsz),
                       (int64_t *)(ws + L.snnz), M);
    device_scan<int64_t, int64_t>((const int64_t *)(ws + L.snnz), (int64_t *)(ws + L.frec), M,
                                  (int64_t *)(ws + L.sc64), s);
    wp_status st = wp_check_launch("build factor offsets");
    if (st != WP_OK) return st;
    // the total also goes next to the error flags (the count pass clears them), where the fill pass
    // checks it against the caller's buffer
    WP_HIP(hipMemcpyAsync(ws + L.err + 8, ws + L.frec + 8 * M, 8, hipMemcpyDeviceToDevice, s));
    WP_HIP(hipMemcpyAsync(bytes, ws + L.frec + 8 * M, 8, hipMemcpyDeviceToHost, s));
    WP_HIP(hipStreamSynchronize(s));
    return WP_OK;
}

wp_status launch_build_count(const wp_plan *p, int64_t M, const double *u, const double *v, const double *w,
                             const double *beam, double E, void *wsv, int64_t *nnz_total, int64_t *nwork,
                             hipStream_t s) {
    unsigned char *ws = (unsigned char *)wsv;
    const bool rows2d = p->chirp == WP_CHIRP_EXACT || beam;
    const WsLayout L = ws_layout(p, M, rows2d);
    const int T = p->ntile * p->ntile;
    WP_HIP(hipMemsetAsync(ws + L.err, 0, L.count + 4 * RowList::COUNTS - L.err, s));     // and the list's counters
    wp_status st;
    if (rows2d && exact_lowrank(p, beam)) {
        switch (p->logNg) {
            case 6: st = lowrank_rows<6>(p, M, u, v, w, E, ws, L, nullptr, s); break;
            case 7: st = lowrank_rows<7>(p, M, u, v, w, E, ws, L, nullptr, s); break;
            case 8: st = lowrank_rows<8>(p, M, u, v, w, E, ws, L, nullptr, s); break;
            case 9: st = lowrank_rows<9>(p, M, u, v, w, E, ws, L, nullptr, s); break;
            case 10: st = lowrank_rows<10>(p, M, u, v, w, E, ws, L, nullptr, s); break;
            case 11: st = lowrank_rows<11>(p, M, u, v, w, E, ws, L, nullptr, s); break;
            case 12: st = lowrank_rows<12>(p, M, u, v, w, E, ws, L, nullptr, s); break;
            default: return wp_set_error(WP_EUNSUPPORTED, "build: Ng = %d", p->Ng);
        }
    } else if (rows2d) {
        switch (p->logNg) {
            case 6: st = count_rows_exact<6>(p, M, u, v, w, beam, E, ws, L, s); break;
            case 7: st = count_rows_exact<7>(p, M, u, v, w, beam, E, ws, L, s); break;
            case 8: st = count_rows_exact<8>(p, M, u, v, w, beam, E, ws, L, s); break;
            case 9: st = count_rows_exact<9>(p, M, u, v, w, beam, E, ws, L, s); break;
            default: return wp_set_error(WP_EUNSUPPORTED, "build: 2-D rows need Ng <= %d (Ng = %d)",
                                         EXACT_MAX_NG, p->Ng);
        }
    } else switch (p->logNg) {
        case 6: st = count_rows<6>(p, M, u, v, w, E, ws, L, s); break;
        case 7: st = count_rows<7>(p, M, u, v, w, E, ws, L, s); break;
        case 8: st = count_rows<8>(p, M, u, v, w, E, ws, L, s); break;
        case 9: st = count_rows<9>(p, M, u, v, w, E, ws, L, s); break;
        case 10: st = count_rows<10>(p, M, u, v, w, E, ws, L, s); break;
        case 11: st = count_rows<11>(p, M, u, v, w, E, ws, L, s); break;
        case 12: st = count_rows<12>(p, M, u, v, w, E, ws, L, s); break;
        default: return wp_set_error(WP_EUNSUPPORTED, "build: Ng = %d", p->Ng);
    }
    if (st != WP_OK) return st;
    // stable sort of the rows by the Z-order code of their centre cell
    const int nthr = 256;
    const dim3 gM((unsigned)((M + nthr - 1) / nthr));
    radix_sort((const int *)(ws + L.key), M, 2 * p->logNg, (int *)(ws + L.k0), (int *)(ws + L.i0), (int *)(ws + L.k1),
               (int *)(ws + L.i1), (int *)(ws + L.sc32), s);
    const int *skey = (const int *)(ws + L.k0), *perm = (const int *)(ws + L.i0);
    hipLaunchKernelGGL(k_gather_nnz, gM, dim3(nthr), 0, s, perm, (const int *)(ws + L.nnz), (int64_t *)(ws + L.snnz), M);
    device_scan<int64_t, int64_t>((const int64_t *)(ws + L.snnz), (int64_t *)(ws + L.rowptr), M,
                                  (int64_t *)(ws + L.sc64), s);
    // adjoint work items: chunks of rows inside each tile
    WP_HIP(hipMemsetAsync(ws + L.tstart, 0, 4 * T, s));
    WP_HIP(hipMemsetAsync(ws + L.tend, 0, 4 * T, s));
    int tbits = 0;
    while ((1 << tbits) < p->tile) ++tbits;
    hipLaunchKernelGGL(k_tile_bounds, gM, dim3(nthr), 0, s, skey, M, 2 * tbits, (int *)(ws + L.tstart),
                       (int *)(ws + L.tend));
    const dim3 gT((unsigned)((T + nthr - 1) / nthr));
    hipLaunchKernelGGL(k_tile_chunks, gT, dim3(nthr), 0, s, (const int *)(ws + L.tstart), (const int *)(ws + L.tend),
                       T, (int *)(ws + L.nch));
    device_scan<int, int>((const int *)(ws + L.nch), (int *)(ws + L.choff), T, (int *)(ws + L.sc32), s);
    if ((st = wp_check_launch("build_G_count layout")) != WP_OK) return st;
    int64_t host_rowptr_end = 0;
    int host_items = 0, host_err = 0;
    WP_HIP(hipMemcpyAsync(&host_rowptr_end, ws + L.rowptr + 8 * M, 8, hipMemcpyDeviceToHost, s));
    WP_HIP(hipMemcpyAsync(&host_items, ws + L.choff + 4 * (int64_t)T, 4, hipMemcpyDeviceToHost, s));
    WP_HIP(hipMemcpyAsync(&host_err, ws + L.err, 4, hipMemcpyDeviceToHost, s));
    WP_HIP(hipStreamSynchronize(s));
    if (host_err & 1)
        return wp_set_error(WP_EINVAL, "build_G_count: a visibility has non-finite (u, v, w), lies outside the band "
                            "|u|,|v| < N/(2L)%s", beam ? " or has a beam that is not finite with sigma > 0" : "");
    if (host_err & 16)
        return wp_set_error(WP_EUNSUPPORTED, "build_G_count: an exact-chirp row spreads over more than %d cells "
                            "(the separable expansion's window); reduce w", LR_WMAX - 2 * LR_MARGIN);
    if (host_err & 8)
        return wp_set_error(WP_EHIP, "build_G_count: an exact-chirp row keeps entries outside its window");
    *nnz_total = host_rowptr_end;
    *nwork = host_items;
    return WP_OK;
}

wp_status launch_build_fill(const wp_plan *p, int64_t M, const double *u, const double *v, const double *w,
                            const double *beam, double E, const void *wsv, wp_G *G, hipStream_t s) {
    unsigned char *ws = (unsigned char *)const_cast<void *>(wsv);
    const bool rows2d = p->chirp == WP_CHIRP_EXACT || beam;
    const WsLayout L = ws_layout(p, M, rows2d);
    const int T = p->ntile * p->ntile;
    WP_HIP(hipMemcpyAsync(G->rowptr, ws + L.rowptr, 8 * (M + 1), hipMemcpyDeviceToDevice, s));
    WP_HIP(hipMemcpyAsync(G->perm, ws + L.i0, 4 * M, hipMemcpyDeviceToDevice, s));
    if (G->frec && G->fdat) {
        int64_t total = 0;
        WP_HIP(hipMemcpyAsync(&total, ws + L.err + 8, 8, hipMemcpyDeviceToHost, s));
        WP_HIP(hipStreamSynchronize(s));
        if (total == 0 || total != G->fbytes)
            return wp_set_error(WP_EINVAL, "factor records: G->fbytes = %lld, the workspace holds %lld (call "
                                "wp_build_factor_bytes after wp_build_G_count)", (long long)G->fbytes, (long long)total);
        WP_HIP(hipMemcpyAsync(G->frec, ws + L.frec, 8 * (M + 1), hipMemcpyDeviceToDevice, s));
    }
    wp_status st;
    if (rows2d && exact_lowrank(p, beam)) {
        switch (p->logNg) {
            case 6: st = lowrank_rows<6>(p, M, u, v, w, E, ws, L, G, s); break;
            case 7: st = lowrank_rows<7>(p, M, u, v, w, E, ws, L, G, s); break;
            case 8: st = lowrank_rows<8>(p, M, u, v, w, E, ws, L, G, s); break;
            case 9: st = lowrank_rows<9>(p, M, u, v, w, E, ws, L, G, s); break;
            case 10: st = lowrank_rows<10>(p, M, u, v, w, E, ws, L, G, s); break;
            case 11: st = lowrank_rows<11>(p, M, u, v, w, E, ws, L, G, s); break;
            case 12: st = lowrank_rows<12>(p, M, u, v, w, E, ws, L, G, s); break;
            default: return wp_set_error(WP_EUNSUPPORTED, "build: Ng = %d", p->Ng);
        }
    } else if (rows2d) {
        switch (p->logNg) {
            case 6: st = fill_rows_exact<6>(p, M, u, v, w, beam, ws, L, G, s); break;
            case 7: st = fill_rows_exact<7>(p, M, u, v, w, beam, ws, L, G, s); break;
            case 8: st = fill_rows_exact<8>(p, M, u, v, w, beam, ws, L, G, s); break;
            case 9: st = fill_rows_exact<9>(p, M, u, v, w, beam, ws, L, G, s); break;
            default: return wp_set_error(WP_EUNSUPPORTED, "build: 2-D rows need Ng <= %d (Ng = %d)",
                                         EXACT_MAX_NG, p->Ng);
        }
    } else switch (p->logNg) {
        case 6: st = fill_rows<6>(p, M, u, v, w, E, ws, L, G, s); break;
        case 7: st = fill_rows<7>(p, M, u, v, w, E, ws, L, G, s); break;
        case 8: st = fill_rows<8>(p, M, u, v, w, E, ws, L, G, s); break;
        case 9: st = fill_rows<9>(p, M, u, v, w, E, ws, L, G, s); break;
        case 10: st = fill_rows<10>(p, M, u, v, w, E, ws, L, G, s); break;
        case 11: st = fill_rows<11>(p, M, u, v, w, E, ws, L, G, s); break;
        case 12: st = fill_rows<12>(p, M, u, v, w, E, ws, L, G, s); break;
        default: return wp_set_error(WP_EUNSUPPORTED, "build: Ng = %d", p->Ng);
    }
    if (st != WP_OK) return st;
    const int nthr = 256;
    const dim3 gT((unsigned)((T + nthr - 1) / nthr));
    hipLaunchKernelGGL(k_write_items, gT, dim3(nthr), 0, s, (const int *)(ws + L.tstart), (const int *)(ws + L.tend),
                       (const int *)(ws + L.choff), T, p->ntile, G->work);
    if ((st = wp_check_launch("build_G_fill layout")) != WP_OK) return st;
    if (G->tcolptr) {
        const int64_t cells = (int64_t)p->Ng * p->Ng;
        int *cnt = (int *)(ws + L.tcnt);          // the workspace is const to callers; this region is scratch
        WP_HIP(hipMemsetAsync(cnt, 0, 4 * cells, s));
        if (G->nnz > 0) {
            int64_t nb = (G->nnz + nthr - 1) / nthr;
            if (nb > 65536) nb = 65536;
            hipLaunchKernelGGL(k_t_count, dim3((unsigned)nb), dim3(nthr), 0, s, G->col, G->nnz, cnt);
        }
        device_scan<int, int64_t>(cnt, G->tcolptr, cells, (int64_t *)(ws + L.sc64t), s);
        WP_HIP(hipMemsetAsync(cnt, 0, 4 * cells, s));
        const dim3 gR((unsigned)((M * 64 + nthr - 1) / nthr));
        if (G->taps != WP_TAPS_C64)
            hipLaunchKernelGGL((k_t_fill<uint32_t>), gR, dim3(nthr), 0, s, G->rowptr, G->col,
                               (const uint32_t *)G->val, G->perm, M, G->tcolptr, cnt, G->trow, (uint32_t *)G->tval);
        else
            hipLaunchKernelGGL((k_t_fill<float2>), gR, dim3(nthr), 0, s, G->rowptr, G->col, (const float2 *)G->val,
                               G->perm, M, G->tcolptr, cnt, G->trow, (float2 *)G->tval);
        const dim3 gC((unsigned)((cells + nthr - 1) / nthr));
        // cnt (free again after the fill) lists the cells longer than a wavefront: each cell is on one list at
        // most, so the two lists grow from its ends; counts in gpos[0 .. TSL_N)
        int *count = (int *)(ws + L.gpos);
        hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(64), 0, s, count, TSL_N);
        if (G->taps != WP_TAPS_C64)
            sort_cells<uint32_t>(G, cells, cnt, count, s);
        else
            sort_cells<float2>(G, cells, cnt, count, s);
        if ((st = wp_check_launch("build_G_fill transpose")) != WP_OK) return st;
        if (G->tblk) {
            // cnt (free again) holds the block-start flags; their scan gives each block's index
            hipLaunchKernelGGL(k_gb_flags, gC, dim3(nthr), 0, s, G->tcolptr, cells, p->gb_ent, cnt);
            int *gpos = (int *)(ws + L.gpos);
            device_scan<int, int>(cnt, gpos, cells, (int *)(ws + L.sc64t), s);
            const int64_t n = cells > G->n_tblk + 1 ? cells : G->n_tblk + 1;
            int64_t nb = (n + nthr - 1) / nthr;
            if (nb > 65536) nb = 65536;
            hipLaunchKernelGGL(k_gb_write, dim3((unsigned)nb), dim3(nthr), 0, s, G->tcolptr, cnt, gpos, cells,
                               G->nnz, G->n_tblk, G->tblk);
            if ((st = wp_check_launch("build_G_fill gather blocks")) != WP_OK) return st;
        }
    }
    // rows of other coordinates than the count pass's are made again: their kept counts must equal its
    int host_err = 0;
    WP_HIP(hipMemcpyAsync(&host_err, ws + L.err, 4, hipMemcpyDeviceToHost, s));
    WP_HIP(hipStreamSynchronize(s));
    if (host_err & 6)
        return wp_set_error(WP_EHIP, "build_G_fill: a row's kept entries or factor record differ from pass 1 (flags %d)",
                            host_err);
    return WP_OK;
}

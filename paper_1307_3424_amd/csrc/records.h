// Both sparse products from the factor records (included by spmv.hip).
//
// A row is y = sum_i g_u(i) sum_{b < nv(i)} g_v(b) X[b, a_i], nv(i) = the v candidates that keep u candidate i (the
// record's staircase read the other way).  Written so, a tap takes four multiply-adds; forming each tap g_v g_u first
// takes eight.  The adjoint folds conj(g_v) y once per v candidate likewise.
//
// Lanes are packed: a row takes ceil(n / P) lanes, n its candidates on the lanes' axis, lane l candidates l,
// l + ceil(n / P), ...; a wavefront takes as many consecutive rows as fit its 64 lanes and its LDS slice.  The
// staircase falls along the candidates' order, so the lanes of one pass have nearly equal trip counts: with P = 2
// 80 % of the lanes' steps are taps, where a power of two of lanes per row had 40 %.  The records of the
// wavefront's rows are one contiguous run, copied to the slice with coalesced loads.
#pragma once

#include "gather_block.h"

namespace {

// ---------------------------------------------------------------------------- packing of rows

// The rows r0 .. r0 + nr - 1 (nr <= 64) of a wavefront, one per lane: record offset (relative to the first row's),
// bytes, header, index in the visibility vector, lanes taken and their running sum.
struct RowGroup {
    int64_t g0;
    int nr, rel, bytes, nl, pl, yi;
    uint32_t hdr;
};

// inclusive prefix sum over the wavefront
__device__ __forceinline__ int wave_prefix(int x, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    return x;
}

// U: lanes over the u candidates, else over the v candidates; P: candidates per lane
template <bool U, int P>
__device__ __forceinline__ RowGroup load_rows(int64_t r0, int nr, const int64_t *__restrict__ frec,
                                              const unsigned char *__restrict__ fdat, const int *__restrict__ perm,
                                              int lane) {
    RowGroup g;
    g.nr = nr;
    g.g0 = nr > 0 ? frec[r0] : 0;
    g.rel = g.bytes = g.nl = g.yi = 0;
    g.hdr = 0;
    if (lane < nr) {
        const int64_t o = frec[r0 + lane];
        g.rel = (int)(o - g.g0);
        g.bytes = (int)(frec[r0 + lane + 1] - o);
        g.yi = perm ? perm[r0 + lane] : (int)(r0 + lane);
        g.hdr = *(const uint32_t *)(fdat + o);
        g.nl = ((U ? (int)(g.hdr & 0xffffu) : (int)(g.hdr >> 16)) + P - 1) / P;
    }
    g.pl = wave_prefix(g.nl, lane);
    return g;
}

// the rows from s on that fit 64 lanes and SLICE bytes (0: row s alone does not)
template <int SLICE>
__device__ __forceinline__ int rows_that_fit(const RowGroup &g, int s, int lane) {
    const int sl = __builtin_amdgcn_readlane(g.pl - g.nl, s), so = __builtin_amdgcn_readlane(g.rel, s);
    const unsigned long long fit =
        __ballot(lane >= s && lane < g.nr && g.pl - sl <= 64 && g.rel + g.bytes - so <= SLICE) >> s;
    return ~fit == 0ull ? 64 : __builtin_ctzll(~fit);
}

// A lane's place in the batch of rows s .. s + cnt - 1, whose records are copied to the slice: row q (a lane of the
// group), lane l of its L, and its record.
struct Place {
    int q, l, L, nu, nv;
    bool on;
    unsigned char *rec;
    uint16_t *ua, *vb, *nb;
    const float2 *gu, *gv;
};

__device__ __forceinline__ Place place_rows(const RowGroup &g, int s, int cnt, const unsigned char *__restrict__ fdat,
                                            unsigned char *slice, int lane) {
    Place p;
    const int sl = __builtin_amdgcn_readlane(g.pl - g.nl, s), so = __builtin_amdgcn_readlane(g.rel, s);
    const int n8 = (__builtin_amdgcn_readlane(g.rel + g.bytes, s + cnt - 1) - so) >> 3;
    const int tot = __builtin_amdgcn_readlane(g.pl, s + cnt - 1) - sl;
    const uint2 *src = (const uint2 *)(fdat + g.g0 + so);
    wave_sync();                                              // the slice's last records are no longer read
    for (int e = lane; e < n8; e += 64) ((uint2 *)slice)[e] = src[e];
    // the last row that starts at or before this lane
    p.q = s;
    for (int j = 1; j < cnt; ++j) p.q += lane >= __builtin_amdgcn_readlane(g.pl - g.nl, s + j) - sl;
    p.on = lane < tot;
    p.L = __shfl(g.nl, p.q);
    p.l = lane - (__shfl(g.pl - g.nl, p.q) - sl);
    const uint32_t h = __shfl((int)g.hdr, p.q);
    p.nu = (int)(h & 0xffffu);
    p.nv = (int)(h >> 16);
    p.rec = slice + (__shfl(g.rel, p.q) - so);
    p.ua = (uint16_t *)p.rec + 2;
    p.vb = p.ua + p.nu;
    p.nb = p.vb + p.nv;
    p.gu = (const float2 *)(p.rec + ((4 + 2 * p.nu + 4 * p.nv + 7) & ~7));
    p.gv = p.gu + p.nu;
    wave_sync();
    return p;
}

// the sum of a row's lanes into its first one
__device__ __forceinline__ void row_sums(const Place &p, float &zr, float &zi, int lane) {
    const int left = p.on ? p.L - p.l : 0;                    // lanes of this row from here on
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float xr = __shfl_down(zr, o), xi = __shfl_down(zi, o);
        if (o < left) {
            zr += xr;
            zi += xi;
        }
    }
}

// ---------------------------------------------------------------------------- degrid

// Lanes over the u candidates, each summing down its column of v candidates: the lanes of a row read neighbouring
// cells of one grid row.  Bound: the texture unit, which returns about one scattered 8-byte value per clock and CU
// (126M taps in 189 us).  Copying each tile's window of the grid to LDS and reading the cells there was slower (285 us,
// 8 items per workgroup): its phases wait on one another and too few wavefronts share a window.
constexpr int DR_NTH = 256, DR_WAVES = DR_NTH / 64, DR_SLICE = 3072, DR_P = 2, DR_U = 4;
constexpr int64_t DR_ROWS_MIN = 24576;     // rows from which packed lanes win (see launch_degrid)

// sum_{b < n} gv[b] X[vb[b], a], DR_U reads in flight; steps past n repeat the last cell with weight zero
__device__ __forceinline__ float2 degrid_column(int n, uint32_t a8, const uint16_t *vb, const float2 *gv,
                                                const float2 *__restrict__ grid, int sh) {
    float ar = 0.f, ai = 0.f;
    for (int b0 = 0; b0 < n; b0 += DR_U) {
        float2 g[DR_U], x[DR_U];
#pragma unroll
        for (int k = 0; k < DR_U; ++k) {
            const int b = min(b0 + k, n - 1);
            g[k] = gv[b];
            x[k] = *(const float2 *)((const unsigned char *)grid + (((uint32_t)vb[b] << sh) + a8));
            if (b0 + k >= n) g[k] = make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int k = 0; k < DR_U; ++k) {
            ar = fmaf(g[k].x, x[k].x, ar);
            ar = fmaf(-g[k].y, x[k].y, ar);
            ai = fmaf(g[k].x, x[k].y, ai);
            ai = fmaf(g[k].y, x[k].x, ai);
        }
    }
    return make_float2(ar, ai);
}

// the v candidates that keep u candidate i: nb falls along them, so the first one with nb <= i ends them
__device__ __forceinline__ int column_length(const uint16_t *nb, int nv, int i) {
    int lo = 0, hi = nv;
    while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if ((int)nb[m] > i) lo = m + 1;
        else hi = m;
    }
    return lo;
}

// a row that does not fit a wavefront's lanes or slice, by the whole wavefront from global memory
__device__ __forceinline__ float2 degrid_row_wide(const unsigned char *__restrict__ rec,
                                                  const float2 *__restrict__ grid, int sh, int lane) {
    const uint32_t hdr = *(const uint32_t *)rec;
    const int nu = (int)(hdr & 0xffffu), nv = (int)(hdr >> 16);
    const uint16_t *ua = (const uint16_t *)rec + 2, *vb = ua + nu, *nb = vb + nv;
    const float2 *gu = (const float2 *)(rec + ((4 + 2 * nu + 4 * nv + 7) & ~7)), *gv = gu + nu;
    float zr = 0.f, zi = 0.f;
    for (int i = lane; i < nu; i += 64) {
        const float2 c = degrid_column(column_length(nb, nv, i), 8u * ua[i], vb, gv, grid, sh), f = gu[i];
        zr = fmaf(f.x, c.x, fmaf(-f.y, c.y, zr));
        zi = fmaf(f.x, c.y, fmaf(f.y, c.x, zi));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        zr += __shfl_xor(zr, o);
        zi += __shfl_xor(zi, o);
    }
    return make_float2(zr, zi);
}

// per: rows per wavefront (at most 64)
__global__ __launch_bounds__(DR_NTH, 4) void k_degrid_records(const int64_t *__restrict__ frec,
                                                           const unsigned char *__restrict__ fdat,
                                                           const float2 *__restrict__ grid,
                                                           const int *__restrict__ perm, float2 *__restrict__ y,
                                                           int64_t M, int per, int logNg) {
    __shared__ __align__(16) unsigned char slices[DR_WAVES][DR_SLICE];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, sh = logNg + 3;
    const int64_t r0 = (xcd_block(blockIdx.x, gridDim.x) * DR_WAVES + wv) * per;
    if (r0 >= M) return;                                      // per wavefront: nothing below syncs the workgroup
    const RowGroup g = load_rows<true, DR_P>(r0, (int)min((int64_t)per, M - r0), frec, fdat, perm, lane);
    if (lane < g.nr && g.nl == 0) y[g.yi] = make_float2(0.f, 0.f);
    for (int s = 0; s < g.nr;) {
        const int cnt = rows_that_fit<DR_SLICE>(g, s, lane);
        if (cnt == 0) {                                       // one long row, by the whole wavefront from memory
            const float2 z = degrid_row_wide(fdat + g.g0 + __builtin_amdgcn_readlane(g.rel, s), grid, sh, lane);
            const int to = __builtin_amdgcn_readlane(g.yi, s);
            if (lane == 0) y[to] = z;
            ++s;
            continue;
        }
        const Place p = place_rows(g, s, cnt, fdat, slices[wv], lane);
        float zr = 0.f, zi = 0.f;
        if (p.on) {
#pragma unroll
            for (int k = 0; k < DR_P; ++k) {
                const int i = p.l + k * p.L;
                if (i < p.nu) {
                    const float2 c = degrid_column(column_length(p.nb, p.nv, i), 8u * p.ua[i], p.vb, p.gv, grid, sh);
                    const float2 f = p.gu[i];
                    zr = fmaf(f.x, c.x, fmaf(-f.y, c.y, zr));
                    zi = fmaf(f.x, c.y, fmaf(f.y, c.x, zi));
                }
            }
        }
        row_sums(p, zr, zi, lane);
        const int to = __shfl(g.yi, p.q);
        if (p.on && p.l == 0) y[to] = make_float2(zr, zi);
        s += cnt;
    }
}

// ---------------------------------------------------------------------------- adjoint

// Tile by tile of the uv grid: the adjoint's work items are rows of one 32 x 32-cell tile each (rows sorted by
// Z-order), and their records reach a window of the tile and a halo.  A workgroup accumulates the window of a run
// of items of one tile in LDS and adds it to the grid once.  Lanes over the v candidates, each adding along its
// row of u candidates: lanes of a row add to different window rows (stride of 65 values: different banks).
// Bound: vector issue, about 25 instructions per tap and lane, most of them the conversion to fixed point: 61 % of the
// SIMDs' cycles at 600000 rows and 2048 pixels (446 us), with 39 of 64 lanes active; LDS busy 32 %, texture data unit 57 %.
constexpr int RT_NTH = 512, RT_WAVES = RT_NTH / 64, RT_ITEMS = 8, RT_SLICE = 1536, RT_P = 1;
constexpr int RT_WS = 64, RT_LD = RT_WS + 1, RT_PLANE = RT_WS * RT_LD;
constexpr int RT_ROWS = RT_WAVES * 64;                // rows of a window: a wavefront's share is one group

struct TileView {
    int v0, u0, mask, logNg;
};

// x (a float of at most 2^62 in modulus) as a 64-bit integer, rounded to nearest: both halves are exact in float
__device__ __forceinline__ unsigned long long to_fixed(float x) {
    const float hi = rintf(x * 0x1p-32f);
    const int lo = __float2int_rn(fmaf(hi, -0x1p32f, x));
    const int h = (int)hi + (lo >> 31);
    return ((unsigned long long)(unsigned int)h << 32) | (unsigned int)lo;
}

// turns a lane's share of its row's columns into window byte offsets 8 du, and gives its v candidates: window row,
// kept u candidates, factor.  Returns whether any of them lies outside the window.
__device__ __forceinline__ bool place_taps(const Place &p, const TileView &t, int *dv, int *n, float2 *f) {
    bool out = false;
    if (p.on)
        for (int k = p.l; k < p.nu; k += p.L) {
            const int du = ((int)p.ua[k] - t.u0) & t.mask;
            out |= du >= RT_WS;
            p.ua[k] = (uint16_t)(8 * du);
        }
#pragma unroll
    for (int k = 0; k < RT_P; ++k) {
        const int b = p.l + k * p.L;
        dv[k] = n[k] = 0;
        f[k] = make_float2(0.f, 0.f);
        if (p.on && b < p.nv) {
            dv[k] = ((int)p.vb[b] - t.v0) & t.mask;
            n[k] = p.nb[b];
            f[k] = p.gv[b];
            out |= dv[k] >= RT_WS;
        }
    }
    return out;
}

// adds conj(g_u(i)) h, i < n, along window row dv; ua holds window byte offsets 8 du.  SAFE: all inside the window.
template <bool SAFE>
__device__ __forceinline__ void scatter_add(int dv, int n, float2 h, const uint16_t *ua, const float2 *gu,
                                            unsigned long long *win, float *__restrict__ grid, const TileView &t,
                                            int exp, bool fixed) {
    unsigned char *row = (unsigned char *)(win + dv * RT_LD);
    for (int i = 0; i < n; ++i) {
        const int o = ua[i];
        const float2 g = gu[i];
        const float cr = fmaf(g.x, h.x, g.y * h.y), ci = fmaf(g.x, h.y, -g.y * h.x);       // conj(g) h
        if (SAFE || (fixed && dv < RT_WS && o < 8 * RT_WS)) {
            atomicAdd((unsigned long long *)(row + o), to_fixed(cr));
            atomicAdd((unsigned long long *)(row + 8 * RT_PLANE + o), to_fixed(ci));
        } else {
            const int64_t e = ((int64_t)((dv + t.v0) & t.mask) << t.logNg) | (((o >> 3) + t.u0) & t.mask);
            unsafeAtomicAdd(&grid[2 * e], ldexpf(cr, -exp));
            unsafeAtomicAdd(&grid[2 * e + 1], ldexpf(ci, -exp));
        }
    }
}

// a row that does not fit a wavefront's lanes or slice, by the whole wavefront from global memory: lane l takes
// u candidates l, l + 64, ...
__device__ __forceinline__ void scatter_row_wide(const unsigned char *__restrict__ rec, float2 yk,
                                                 unsigned long long *win, float *__restrict__ grid, const TileView &t,
                                                 int exp, bool fixed, int lane) {
    const uint32_t hdr = *(const uint32_t *)rec;
    const int nu = (int)(hdr & 0xffffu), nv = (int)(hdr >> 16);
    const uint16_t *ua = (const uint16_t *)rec + 2, *vb = ua + nu, *nbv = vb + nv;
    const float2 *gu = (const float2 *)(rec + ((4 + 2 * nu + 4 * nv + 7) & ~7)), *gv = gu + nu;
    for (int i = lane; i < nu; i += 64) {
        const int du = ((int)ua[i] - t.u0) & t.mask;
        const float2 g = gu[i];
        const float hr = fmaf(g.x, yk.x, g.y * yk.y), hi = fmaf(g.x, yk.y, -g.y * yk.x);   // conj(g_u) y
        for (int b = 0; b < nv && i < (int)nbv[b]; ++b) {
            const float2 f = gv[b];
            const float cr = fmaf(f.x, hr, f.y * hi), ci = fmaf(f.x, hi, -f.y * hr);
            const int dv = ((int)vb[b] - t.v0) & t.mask;
            if (fixed && dv < RT_WS && du < RT_WS) {
                unsigned long long *p = win + dv * RT_LD + du;
                atomicAdd(p, to_fixed(cr));
                atomicAdd(p + RT_PLANE, to_fixed(ci));
            } else {
                const int64_t e = ((int64_t)vb[b] << t.logNg) | ua[i];
                unsafeAtomicAdd(&grid[2 * e], ldexpf(cr, -exp));
                unsafeAtomicAdd(&grid[2 * e + 1], ldexpf(ci, -exp));
            }
        }
    }
}

// rows [rb, re) of the next run of items of one tile, from item i on
__device__ __forceinline__ void next_run(const int *__restrict__ work, int &i, int end, int &tv, int &tu, int &rb,
                                         int &re) {
    tv = work[4 * (int64_t)i];
    tu = work[4 * (int64_t)i + 1];
    rb = work[4 * (int64_t)i + 2];
    re = work[4 * (int64_t)i + 3];
    for (++i; i < end; ++i) {
        const int *w = work + 4 * (int64_t)i;
        if (w[0] != tv || w[1] != tu || w[2] != re || w[3] - rb > RT_ROWS) break;
        re = w[3];
    }
}

// workgroup b: items [b per, b per + per), per <= RT_ITEMS; with parts > 1 (per = 1), one of that many parts of an
// item's rows
__global__ __launch_bounds__(RT_NTH, 4) void k_scatter_records(const int *__restrict__ work, int n_work, int per, int parts,
                                                            const int64_t *__restrict__ frec,
                                                            const unsigned char *__restrict__ fdat,
                                                            const int *__restrict__ perm,
                                                            const float2 *__restrict__ y, float *__restrict__ grid,
                                                            int logNg, int tile, int halo) {
    __shared__ unsigned long long win[2 * RT_PLANE];          // real plane, imaginary plane
    __shared__ __align__(16) unsigned char slices[RT_WAVES][RT_SLICE];
    __shared__ double s_red[RT_WAVES];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t blk = blockIdx.x / parts;           // round-robin over XCDs: the uv centre's items are heavier
    const int part = blockIdx.x % parts;
    const int end = (int)min((int64_t)n_work, (blk + 1) * per);
    TileView t;
    t.logNg = logNg;
    t.mask = (1 << logNg) - 1;
    int tv = 0, tu = 0, rb = 0, run_end = 0;
    for (int i = (int)(blk * per); i < end || rb < run_end;) {
        if (rb >= run_end) {
            next_run(work, i, end, tv, tu, rb, run_end);
            if (parts > 1) {
                const int64_t n = run_end - rb;
                run_end = rb + (int)(n * (part + 1) / parts);
                rb += (int)(n * part / parts);
            }
            if (rb >= run_end) continue;
        }
        const int re = min(run_end, rb + RT_ROWS);    // the builder's items hold 32 rows; longer ones go in pieces
        t.v0 = (tv * tile - halo) & t.mask;
        t.u0 = (tu * tile - halo) & t.mask;
        const int share = (re - rb + RT_WAVES - 1) / RT_WAVES;
        const int r0 = rb + wv * share;
        const RowGroup g = load_rows<false, RT_P>(r0, max(0, min(share, re - r0)), frec, fdat, perm, lane);
        float2 yk = make_float2(0.f, 0.f), fu = yk, fv = yk;      // and the row's first factors: its largest tap
        if (lane < g.nr) {
            const int nu = (int)(g.hdr & 0xffffu), nv = (int)(g.hdr >> 16);
            const float2 *f = (const float2 *)(fdat + g.g0 + g.rel + ((4 + 2 * nu + 4 * nv + 7) & ~7));
            yk = y[g.yi];
            if (nu > 0 && nv > 0) {
                fu = f[0];
                fv = f[nu];
            }
        }
        __syncthreads();                              // the last run's window has been flushed
        for (int e = threadIdx.x; e < 2 * RT_PLANE; e += RT_NTH) win[e] = 0ull;
        // Fixed point: every partial sum of a cell is at most S = sum over the run's rows of |y_k| max |G_k.|, max |G_k.| the
        // product of the row's two first factors, so with a unit of 2^-exp, 2^61 <= 2^exp S < 2^62, it stays within int64.
        // The unit is 2^-61 S or less.  The scatter of stored taps has 2^-61 of (W I0)^2 |y_k| over an item's 32 rows; a run
        // is eight items, but (W I0)^2 is W (any chirp) to W^2 (short ones) times a row's largest tap.
        // S not finite: every tap goes straight to the grid, which then holds what the sum gives.
        double bsum = sqrt(((double)yk.x * yk.x + (double)yk.y * yk.y) * ((double)fu.x * fu.x + (double)fu.y * fu.y) *
                           ((double)fv.x * fv.x + (double)fv.y * fv.y));
        for (int o = 32; o > 0; o >>= 1) bsum += __shfl_xor(bsum, o);
        if (lane == 0) s_red[wv] = bsum;
        __syncthreads();
        double S = 0.0;
        for (int k = 0; k < RT_WAVES; ++k) S += s_red[k];
        const bool fixed = S < 1e300;
        int exp = 0;
        if (fixed && S > 0.0) {
            (void)frexp(S, &exp);                     // S < 2^exp
            exp = min(62 - exp, 120);
        }
        yk.x = ldexpf(yk.x, exp);
        yk.y = ldexpf(yk.y, exp);
        for (int s = 0; s < g.nr;) {
            const int cnt = rows_that_fit<RT_SLICE>(g, s, lane);
            if (cnt == 0) {
                const float2 yw = make_float2(__shfl(yk.x, s), __shfl(yk.y, s));
                scatter_row_wide(fdat + g.g0 + __builtin_amdgcn_readlane(g.rel, s), yw, win, grid, t, exp, fixed, lane);
                ++s;
                continue;
            }
            const Place p = place_rows(g, s, cnt, fdat, slices[wv], lane);
            int dv[RT_P], n[RT_P];
            float2 f[RT_P];
            const bool safe = !__any(place_taps(p, t, dv, n, f)) && fixed;
            wave_sync();
            const float yr = __shfl(yk.x, p.q), yc = __shfl(yk.y, p.q);
#pragma unroll
            for (int k = 0; k < RT_P; ++k) {
                const float2 h = make_float2(fmaf(f[k].x, yr, f[k].y * yc), fmaf(f[k].x, yc, -f[k].y * yr));   // conj(g_v) y
                if (safe) scatter_add<true>(dv[k], n[k], h, p.ua, p.gu, win, grid, t, exp, fixed);
                else scatter_add<false>(dv[k], n[k], h, p.ua, p.gu, win, grid, t, exp, fixed);
            }
            s += cnt;
        }
        __syncthreads();
        // consecutive lanes add consecutive floats
        for (int e = threadIdx.x; e < 2 * RT_WS * RT_WS; e += RT_NTH) {
            const int dv = e / (2 * RT_WS), du = (e >> 1) % RT_WS, im = e & 1;
            const long long a = (long long)win[im * RT_PLANE + dv * RT_LD + du];
            if (a != 0) {
                const int64_t c = ((int64_t)((t.v0 + dv) & t.mask) << logNg) | ((t.u0 + du) & t.mask);
                unsafeAtomicAdd(&grid[2 * c + im], (float)ldexp((double)a, -exp));
            }
        }
        rb = re;
    }
}

}  // namespace

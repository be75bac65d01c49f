// Learned surrogate of the sparsified rows: the network's forward and backward
// passes, Adam, the training loop, the exact training targets taken from rows the
// builder made, and the per-row energy error of the surrogate against exact rows.
//
// The surrogate maps (w, du, dv) -- w and the offset of (u~, v~) from its nearest
// grid cell c = floor(u~ + 1/2) -- to the taps of the row (Section 3.1 kernel,
// Section 3.2 energy rule) on the 32 x 32 cells (c_v - 16 .. c_v + 15) x
// (c_u - 16 .. c_u + 15), modulo Ng.  Output 2 p (+1) is the real (imaginary) part
// of box cell p = 32 oy + ox, times the output scale s_out.
//
// Mixed precision: products W_l a_{l-1} (l = 2..4) and the backward products take
// bfloat16 operands with FP32 accumulation; the first layer (3 inputs), biases,
// GELU, the loss, bias and W1 gradients and Adam run in FP32.
#include <cmath>
#include <cstring>

#include "mlp_pass.h"

using namespace mlpc;

namespace {

constexpr int NTH = 256;

// ---------------------------------------------------------------------------- elementwise kernels

__global__ void k_adam(float *__restrict__ p, float *__restrict__ m1, float *__restrict__ m2,
                       const float *__restrict__ g, int64_t n, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
    for (int64_t e = (int64_t)blockIdx.x * NTH + threadIdx.x; e < n; e += (int64_t)gridDim.x * NTH) {
        const float ge = g[e];
        const float a = b1 * m1[e] + (1.0f - b1) * ge;
        const float b = b2 * m2[e] + (1.0f - b2) * ge * ge;
        m1[e] = a;
        m2[e] = b;
        p[e] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
    }
}

// features (2 w / w_top - 1, 2 du, 2 dv) with du = u~ - floor(u~ + 1/2)
__global__ void k_features(const double *__restrict__ u, const double *__restrict__ v, const double *__restrict__ w,
                           int64_t n, double cell, double half, double w_top, float *__restrict__ feat,
                           int *__restrict__ err) {
    const int64_t k = (int64_t)blockIdx.x * NTH + threadIdx.x;
    if (k >= n) return;
    const double ut = u[k] / cell, vt = v[k] / cell, wk = w[k];
    if (!(isfinite(ut) && isfinite(vt) && isfinite(wk) && fabs(ut) < half && fabs(vt) < half)) atomicOr(err, 1);
    const double du = ut - floor(ut + 0.5), dv = vt - floor(vt + 0.5);
    feat[3 * k] = (float)(2.0 * wk / w_top - 1.0);
    feat[3 * k + 1] = (float)(2.0 * du);
    feat[3 * k + 2] = (float)(2.0 * dv);
}

__device__ inline int box_cell(double gt, int Ng) {
    const long long c = (long long)floor(gt + 0.5) + Ng / 2;
    return (int)(((c % Ng) + Ng) % Ng);
}

__device__ inline double wave_sum(double x) {
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off);
    return __shfl(x, 0);
}

// exact training targets: row of visibility k (sorted row r, k = perm[r]) scattered
// into its box, divided by s_out; lost[k] = row energy outside the box / row energy
__global__ void k_box_targets(const int64_t *__restrict__ rowptr, const int *__restrict__ col,
                              const float2 *__restrict__ val, const int *__restrict__ perm, int64_t M,
                              const double *__restrict__ u, const double *__restrict__ v, double cell, int logNg,
                              float inv_s, float *__restrict__ target, float *__restrict__ lost) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * (NTH / 64) + (threadIdx.x >> 6);
    if (r >= M) return;
    const int Ng = 1 << logNg;
    const int k = perm[r];
    const int cu = box_cell(u[k] / cell, Ng), cv = box_cell(v[k] / cell, Ng);
    double tot = 0.0, out = 0.0;
    for (int64_t e = rowptr[r] + lane; e < rowptr[r + 1]; e += 64) {
        const int c = col[e];
        const int oy = ((c >> logNg) - cv + BOX / 2) & (Ng - 1);
        const int ox = ((c & (Ng - 1)) - cu + BOX / 2) & (Ng - 1);
        const float2 g = val[e];
        const double e2 = (double)g.x * g.x + (double)g.y * g.y;
        tot += e2;
        if (oy < BOX && ox < BOX) {
            float *t = target + (int64_t)k * NOUT + 2 * (oy * BOX + ox);
            t[0] = g.x * inv_s;
            t[1] = g.y * inv_s;
        } else {
            out += e2;
        }
    }
    tot = wave_sum(tot);
    out = wave_sum(out);
    if (lane == 0) lost[k] = tot > 0.0 ? (float)(out / tot) : 0.0f;
}

// features of sorted rows r0 .. r0 + n - 1
__global__ void k_gather_feat(const float *__restrict__ feat, const int *__restrict__ perm, int64_t r0, int n,
                              float *__restrict__ out) {
    const int i = blockIdx.x * NTH + threadIdx.x;
    if (i >= 3 * n) return;
    out[i] = feat[3 * (int64_t)perm[r0 + i / 3] + i % 3];
}

// eps[k] = ||t - g||^2 / ||g||^2 for sorted rows r0 .. r0 + n - 1 (network outputs o in that order)
__global__ __launch_bounds__(NTH) void k_row_errors(const float *__restrict__ o, int64_t r0, int n,
                                                    const int64_t *__restrict__ rowptr, const int *__restrict__ col,
                                                    const float2 *__restrict__ val, const int *__restrict__ perm,
                                                    const double *__restrict__ u, const double *__restrict__ v,
                                                    double cell, int logNg, float s_out, float *__restrict__ eps,
                                                    float *__restrict__ energy) {
    __shared__ float2 box[NTH / 64][BOX * BOX];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i = blockIdx.x * (NTH / 64) + wv;
    const bool live = i < n;
    const int Ng = 1 << logNg;
    const int64_t r = r0 + (live ? i : 0);
    const int k = perm[r];
    float2 *bx = box[wv];
    for (int p = lane; p < BOX * BOX; p += 64) {
        const float2 t = live ? ((const float2 *)(o + (int64_t)i * NOUT))[p] : make_float2(0.f, 0.f);
        bx[p] = make_float2(t.x * s_out, t.y * s_out);
    }
    __syncthreads();
    double tot = 0.0, out = 0.0;
    if (live) {
        const int cu = box_cell(u[k] / cell, Ng), cv = box_cell(v[k] / cell, Ng);
        for (int64_t e = rowptr[r] + lane; e < rowptr[r + 1]; e += 64) {
            const int c = col[e];
            const int oy = ((c >> logNg) - cv + BOX / 2) & (Ng - 1);
            const int ox = ((c & (Ng - 1)) - cu + BOX / 2) & (Ng - 1);
            const float2 g = val[e];
            tot += (double)g.x * g.x + (double)g.y * g.y;
            if (oy < BOX && ox < BOX) {
                float2 &b = bx[oy * BOX + ox];
                b.x -= g.x;
                b.y -= g.y;
            } else {
                out += (double)g.x * g.x + (double)g.y * g.y;
            }
        }
    }
    __syncthreads();
    double d = 0.0;
    for (int p = lane; p < BOX * BOX; p += 64) d += (double)bx[p].x * bx[p].x + (double)bx[p].y * bx[p].y;
    d = wave_sum(d);
    tot = wave_sum(tot);
    out = wave_sum(out);
    if (live && lane == 0) {
        eps[k] = tot > 0.0 ? (float)((d + out) / tot) : 0.0f;
        if (energy) energy[k] = (float)tot;
    }
}

// Check lattice: node i = (iw nd + iv) nd + iu at w = w_top iw / (nw - 1) and offsets du = -1/2 + iu / (nd - 1)
// (dv likewise) from the centre cell; the last offset node sits just below +1/2, so that it keeps the
// centre cell (at +1/2 the nearest cell would change).
__global__ void k_lattice_coords(int nw, int nd, double w_top, double cell, double *__restrict__ u,
                                 double *__restrict__ v, double *__restrict__ w) {
    const int64_t i = (int64_t)blockIdx.x * NTH + threadIdx.x;
    const int64_t n = (int64_t)nw * nd * nd;
    if (i >= n) return;
    const int iu = (int)(i % nd), iv = (int)((i / nd) % nd), iw = (int)(i / ((int64_t)nd * nd));
    auto off = [nd](int j) { return j == nd - 1 ? 0.5 - 0x1p-20 : -0.5 + (double)j / (double)(nd - 1); };
    u[i] = off(iu) * cell;
    v[i] = off(iv) * cell;
    w[i] = w_top * (double)iw / (double)(nw - 1);
}

// Run-time per-row check of network rows k0 .. k0 + n - 1 (caller order; outputs o of those rows), from
// the check lattice alone (no exact row):
//   est = max( largest node error of the lattice cell holding (w, du, dv),
//              (| ||t|| - sqrt(K) | / sqrt(K))^2 )
// with K the kept energy interpolated trilinearly between the cell's nodes.  The second term is a lower
// bound of the row's error ||t - g||^2 / ||g||^2 by the reverse triangle inequality when K = ||g||^2.
// A row outside the lattice (w beyond the trained range) or with a non-finite value gets +infinity.
__global__ __launch_bounds__(NTH) void k_row_check(const float *__restrict__ o, int64_t k0, int n,
                                                   const float *__restrict__ feat, const float *__restrict__ table,
                                                   int nw, int nd, float s_out, float *__restrict__ est) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * (NTH / 64) + (threadIdx.x >> 6);
    if (i >= n) return;
    const float *oi = o + (int64_t)i * NOUT;
    double e = 0.0;
    for (int p = lane; p < NOUT; p += 64) e += (double)oi[p] * oi[p];
    e = wave_sum(e);
    if (lane != 0) return;
    const int64_t k = k0 + i;
    const float *f = feat + 3 * k;
    const double wf = (0.5 * ((double)f[0] + 1.0)) * (nw - 1);
    const double uf = (0.5 * (double)f[1] + 0.5) * (nd - 1), vf = (0.5 * (double)f[2] + 0.5) * (nd - 1);
    float r = INFINITY;
    if (wf >= 0.0 && wf <= (double)(nw - 1) && uf >= 0.0 && uf <= (double)(nd - 1) && vf >= 0.0 &&
        vf <= (double)(nd - 1) && isfinite(e)) {
        const int iw = min((int)wf, nw - 2), iu = min((int)uf, nd - 2), iv = min((int)vf, nd - 2);
        const double tw = wf - iw, tu = uf - iu, tv = vf - iv;
        const int64_t nodes = (int64_t)nw * nd * nd;
        float emax = 0.0f;
        double K = 0.0;
        for (int c = 0; c < 8; ++c) {
            const int a = c & 1, b = (c >> 1) & 1, d = c >> 2;
            const int64_t node = ((int64_t)(iw + d) * nd + (iv + b)) * nd + (iu + a);
            const float en = table[node];
            emax = (en > emax || en != en) ? en : emax;            // a NaN node error propagates
            K += (a ? tu : 1.0 - tu) * (b ? tv : 1.0 - tv) * (d ? tw : 1.0 - tw) * (double)table[nodes + node];
        }
        const double tn = (double)s_out * sqrt(e);
        const double lb = K > 0.0 ? (tn - sqrt(K)) * (tn - sqrt(K)) / K : INFINITY;
        r = fmaxf(emax, (float)lb);
        if (emax != emax) r = emax;
    }
    est[k] = r;
}

int blocks_for(int64_t n, int per = NTH) { return (int)std::min<int64_t>((n + per - 1) / per, 65536); }

// the weights' bfloat16 fragments from the parameters
wp_status refresh_fragments(wp_mlp *m, hipStream_t s) {
    constexpr int n = (4 * H * H + 2 * NOUT * H) / 8;
    k_mlp_fragments<<<(n + NTH - 1) / NTH, NTH, 0, s>>>(m->params, m->WF2, m->WT2, m->WF3, m->WT3, m->WF4, m->WT4);
    return wp_check_launch("k_mlp_fragments");
}

PassArgs pass_args(const wp_mlp *m, int n, const float *feat) {
    PassArgs a{};
    a.feat = feat;
    a.map = RowMap{1, 0, INT64_MAX};
    a.rows = n;
    a.params = m->params;
    a.WF2 = m->WF2; a.WF3 = m->WF3; a.WF4 = m->WF4;
    a.WT2 = m->WT2; a.WT3 = m->WT3; a.WT4 = m->WT4;
    return a;
}

wp_status check_mlp(const wp_mlp *m) {
    if (!m) return wp_set_error(WP_EINVAL, "mlp is NULL");
    return WP_OK;
}

// Forward and backward of n rows (a multiple of 64), row i being sample map(i) of X and T: gradients into m->grad,
// the sum of squared errors into m->loss (add: added to it).  Two launches: the pass (a workgroup per 32 rows) and
// the weight gradients (160 tiles, from 2048 rows on the batch in two halves: 320 workgroups).
// Measured on MI355X at 8192 rows: 54 + 25 us, against 445 us for layer-by-layer products (64 x 64 and 128 x 128 tiles,
// operands staged through LDS, FP32 pre-activations, outputs and output gradients written and read again).
wp_status mlp_backward(wp_mlp *m, int n, const float *X, const float *T, const RowMap &map, bool add, hipStream_t s) {
    PassArgs a = pass_args(m, n, X);
    a.targ = T;
    a.map = map;
    a.scale = 2.0f / (float)((int64_t)n * NOUT);
    a.a1F = m->a1F; a.a2F = m->a2F; a.a3F = m->a3F;
    a.dOF = m->dOF; a.dz3F = m->dz3F; a.dz2F = m->dz2F;
    a.part = m->part;
    a.lpart = m->lpart;
    a.grad = m->grad;
    const int nrb = n / PR;
    k_mlp_train<<<nrb, PNT, TRAIN_GRAD_LDS, s>>>(a);
    wp_status st = wp_check_launch("k_mlp_train");
    if (st != WP_OK) return st;
    const int chunk = nrb >= 64 ? (nrb + 1) / 2 : nrb, splits = (nrb + chunk - 1) / chunk;
    k_mlp_wgrad<<<GTILES * splits + GRB, GNT, 0, s>>>(a, nrb, splits, chunk, m->loss, add ? 1 : 0);
    return wp_check_launch("k_mlp_wgrad");
}

wp_status mlp_adam(wp_mlp *m, float lr, float b1, float b2, float eps, hipStream_t s) {
    m->step += 1;
    const float c1 = (float)(1.0 - std::pow((double)b1, (double)m->step));
    const float c2 = (float)(1.0 - std::pow((double)b2, (double)m->step));
    k_adam<<<blocks_for(NPARAM, NTH * 4), NTH, 0, s>>>(m->params, m->m1, m->m2, m->grad, NPARAM, lr, b1, b2, eps, c1,
                                                       c2);
    wp_status st = wp_check_launch("k_adam");
    return st != WP_OK ? st : refresh_fragments(m, s);
}

int64_t gcd64(int64_t a, int64_t b) {
    while (b) {
        const int64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}

}  // namespace

// Shares of the outputs: twice as many workgroups until there are two per CU.  Measured on MI355X: 10007 rows 44 us (82
// layer by layer), 1000 rows 17 us, one row 11 us.
wp_status mlp_forward(wp_mlp *m, int n, const float *X, float *out, uint16_t *a3, hipStream_t s) {
    if (n <= 0 || (!out && !a3)) return WP_OK;
    PassArgs a = pass_args(m, n, X);
    a.out = out;
    a.a3 = a3;
    const int nb = (n + PR - 1) / PR;
    int shares = 1;
    while (out && shares < NOUT / H && nb * shares < 512) shares *= 2;
    k_mlp_infer<<<dim3(nb, shares), PNT, 0, s>>>(a);
    return wp_check_launch("k_mlp_infer");
}

// ---------------------------------------------------------------------------- C ABI

extern "C" {

int64_t wp_mlp_param_count(void) { return NPARAM; }

wp_status wp_mlp_create(wp_mlp **out, int max_batch) {
    if (!out) return wp_set_error(WP_EINVAL, "out is NULL");
    *out = nullptr;
    if (max_batch < 64 || max_batch > (1 << 20) || max_batch % 64)
        return wp_set_error(WP_EINVAL, "max_batch = %d: need a multiple of 64 in [64, 2^20]", max_batch);
    wp_mlp *m = (wp_mlp *)calloc(1, sizeof(wp_mlp));
    if (!m) return wp_set_error(WP_ENOMEM, "mlp allocation");
    m->max_batch = max_batch;
    m->w_top = 1.0;
    m->s_out = 1.0;
    if (hipGetDevice(&m->device) != hipSuccess) {
        free(m);
        return wp_set_error(WP_EHIP, "hipGetDevice failed");
    }
    const int64_t B = max_batch;
    struct { void **p; int64_t bytes; } a[] = {
        {(void **)&m->params, NPARAM * 4}, {(void **)&m->m1, NPARAM * 4}, {(void **)&m->m2, NPARAM * 4},
        {(void **)&m->grad, NPARAM * 4},
        {(void **)&m->WF2, (int64_t)H * H * 2}, {(void **)&m->WT2, (int64_t)H * H * 2},
        {(void **)&m->WF3, (int64_t)H * H * 2}, {(void **)&m->WT3, (int64_t)H * H * 2},
        {(void **)&m->WF4, (int64_t)NOUT * H * 2}, {(void **)&m->WT4, (int64_t)NOUT * H * 2},
        {(void **)&m->a1F, B * H * 2}, {(void **)&m->a2F, B * H * 2},
        {(void **)&m->a3F, B * H * 2}, {(void **)&m->dOF, B * NOUT * 2}, {(void **)&m->dz3F, B * H * 2},
        {(void **)&m->dz2F, B * H * 2}, {(void **)&m->part, B / PR * PN * 4}, {(void **)&m->lpart, B / PR * 8},
        {(void **)&m->o, B * NOUT * 4}, {(void **)&m->xb, B * 3 * 4},
        {(void **)&m->loss, 8},
    };
    for (auto &e : a) {
        if (hipMalloc(e.p, e.bytes) != hipSuccess) {
            wp_mlp_destroy(m);
            return wp_set_error(WP_ENOMEM, "mlp buffers (%lld bytes)", (long long)e.bytes);
        }
    }
    WP_HIP(hipMemset(m->params, 0, NPARAM * 4));
    WP_HIP(hipMemset(m->m1, 0, NPARAM * 4));
    WP_HIP(hipMemset(m->m2, 0, NPARAM * 4));
    *out = m;
    return WP_OK;
}

wp_status wp_mlp_destroy(wp_mlp *m) {
    if (!m) return WP_OK;
    void *bufs[] = {m->params, m->m1, m->m2, m->grad, m->WF2, m->WT2, m->WF3, m->WT3, m->WF4, m->WT4, m->a1F,
                    m->a2F, m->a3F, m->dOF, m->dz3F, m->dz2F, m->part, m->lpart, m->o, m->xb, m->loss};
    for (void *b : bufs)
        if (b) (void)hipFree(b);
    free(m);
    return WP_OK;
}

wp_status wp_mlp_set_params(wp_mlp *m, const float *params, double w_top, double s_out) {
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (!params) return wp_set_error(WP_EINVAL, "params is NULL");
    if (!(w_top > 0.0) || !std::isfinite(w_top)) return wp_set_error(WP_EINVAL, "w_top = %g: need > 0", w_top);
    if (!(s_out > 0.0) || !std::isfinite(s_out)) return wp_set_error(WP_EINVAL, "s_out = %g: need > 0", s_out);
    for (int64_t i = 0; i < NPARAM; ++i)
        if (!std::isfinite(params[i])) return wp_set_error(WP_EINVAL, "params[%lld] is not finite", (long long)i);
    WP_HIP(hipMemcpy(m->params, params, NPARAM * 4, hipMemcpyHostToDevice));
    WP_HIP(hipMemset(m->m1, 0, NPARAM * 4));
    WP_HIP(hipMemset(m->m2, 0, NPARAM * 4));
    m->step = 0;
    m->w_top = w_top;
    m->s_out = s_out;
    if ((st = refresh_fragments(m, 0)) != WP_OK) return st;
    WP_HIP(hipDeviceSynchronize());
    return WP_OK;
}

wp_status wp_mlp_get_params(const wp_mlp *m, float *params, double *w_top, double *s_out) {
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (!params) return wp_set_error(WP_EINVAL, "params is NULL");
    WP_HIP(hipDeviceSynchronize());
    WP_HIP(hipMemcpy(params, m->params, NPARAM * 4, hipMemcpyDeviceToHost));
    if (w_top) *w_top = m->w_top;
    if (s_out) *s_out = m->s_out;
    return WP_OK;
}

wp_status wp_mlp_features(const wp_plan *p, const wp_mlp *m, int64_t n, const double *u, const double *v,
                          const double *w, float *feat, int *err, void *stream) {
    if (!p) return wp_set_error(WP_EINVAL, "plan is NULL");
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (n < 0) return wp_set_error(WP_EINVAL, "n < 0");
    if (n == 0) return WP_OK;
    if (!u || !v || !w || !feat || !err) return wp_set_error(WP_EINVAL, "NULL array");
    k_features<<<blocks_for(n), NTH, 0, (hipStream_t)stream>>>(u, v, w, n, p->cell, p->Ng / 2.0, m->w_top, feat, err);
    return wp_check_launch("k_features");
}

wp_status wp_mlp_forward(wp_mlp *m, int n, const float *feat, float *out, void *stream) {
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (n < 0 || n > m->max_batch) return wp_set_error(WP_EINVAL, "n = %d: need 0 <= n <= max_batch = %d", n, m->max_batch);
    if (n > 0 && (!feat || !out)) return wp_set_error(WP_EINVAL, "NULL array");
    return mlp_forward(m, n, feat, out, nullptr, (hipStream_t)stream);
}

wp_status wp_mlp_gradients(wp_mlp *m, int n, const float *feat, const float *target, float *grads, double *loss,
                           void *stream) {
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (n < 64 || n > m->max_batch || n % 64)
        return wp_set_error(WP_EINVAL, "n = %d: need a multiple of 64 in [64, max_batch = %d]", n, m->max_batch);
    if (!feat || !target) return wp_set_error(WP_EINVAL, "NULL array");
    hipStream_t s = (hipStream_t)stream;
    if ((st = mlp_backward(m, n, feat, target, RowMap{1, 0, INT64_MAX}, false, s)) != WP_OK) return st;
    if (grads) WP_HIP(hipMemcpyAsync(grads, m->grad, NPARAM * 4, hipMemcpyDeviceToDevice, s));
    if (loss) {
        double acc = 0.0;
        WP_HIP(hipMemcpyAsync(&acc, m->loss, 8, hipMemcpyDeviceToHost, s));
        WP_HIP(hipStreamSynchronize(s));
        *loss = acc / ((double)n * NOUT);
    }
    return WP_OK;
}

wp_status wp_mlp_adam_step(wp_mlp *m, float lr, float beta1, float beta2, float eps, void *stream) {
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (!(lr >= 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps >= 0.0f))
        return wp_set_error(WP_EINVAL, "Adam hyper-parameters out of range");
    return mlp_adam(m, lr, beta1, beta2, eps, (hipStream_t)stream);
}

wp_status wp_mlp_train(wp_mlp *m, int64_t n, const float *feat, const float *target, int batch, int epochs,
                       float lr_max, double *loss_hist, void *stream) {
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (batch < 64 || batch > m->max_batch || batch % 64)
        return wp_set_error(WP_EINVAL, "batch = %d: need a multiple of 64 in [64, max_batch = %d]", batch, m->max_batch);
    if (n < batch) return wp_set_error(WP_EINVAL, "n = %lld < batch", (long long)n);
    if (epochs < 1) return wp_set_error(WP_EINVAL, "epochs < 1");
    if (!feat || !target) return wp_set_error(WP_EINVAL, "NULL array");
    if (!(lr_max > 0.0f)) return wp_set_error(WP_EINVAL, "lr_max must be > 0");
    hipStream_t s = (hipStream_t)stream;
    const int64_t nb = n / batch;
    const int64_t T = nb * epochs, warm = std::max<int64_t>(1, T / 32);
    int64_t t = 0;
    for (int e = 0; e < epochs; ++e) {
        // per-epoch order: sample (a i + c) mod n, a coprime to n
        int64_t a = (int64_t)((0x9E3779B97F4A7C15ull * (uint64_t)(e + 1)) % (uint64_t)n) | 1;
        while (gcd64(a, n) != 1) a += 2;
        const int64_t c = (int64_t)((0xD1B54A32D192ED03ull * (uint64_t)(e + 7)) % (uint64_t)n);
        for (int64_t b = 0; b < nb; ++b, ++t) {
            const RowMap map{a, (c + a * b * batch) % n, n};
            if ((st = mlp_backward(m, batch, feat, target, map, b > 0, s)) != WP_OK) return st;
            const double ramp = std::min(1.0, (double)(t + 1) / (double)warm);
            const float lr = (float)(lr_max * ramp * 0.5 * (1.0 + std::cos(M_PI * (double)t / (double)T)));
            if ((st = mlp_adam(m, lr, 0.9f, 0.999f, 1e-8f, s)) != WP_OK) return st;
        }
        if (loss_hist) {
            double acc = 0.0;
            WP_HIP(hipMemcpyAsync(&acc, m->loss, 8, hipMemcpyDeviceToHost, s));
            WP_HIP(hipStreamSynchronize(s));
            loss_hist[e] = acc / ((double)nb * batch * NOUT);
        }
    }
    return WP_OK;
}

wp_status wp_mlp_output_scale(const wp_plan *p, double *s_out) {
    if (!p) return wp_set_error(WP_EINVAL, "plan is NULL");
    if (!s_out) return wp_set_error(WP_EINVAL, "s_out is NULL");
    // A row's energy is (sum over the u window of KB^2) (sum over the v window of KB^2): shifts of
    // the chirp spectrum are orthonormal because the chirp has unit modulus on the padded grid.
    // T0: that energy for a visibility on a cell centre; s_out = sqrt(T0 / BOX^2).
    double e = 0.0;
    const int base = -p->W / 2 + 1;
    for (int i = 0; i < p->W; ++i) {
        const double t = -(double)(base + i);
        const double r = 1.0 - (2.0 * t / p->W) * (2.0 * t / p->W);
        if (r < 0.0) continue;
        const double x = p->beta * std::sqrt(r);
        double term = 1.0, sum = 1.0;          // I0(x) = sum (x/2)^2k / (k!)^2
        for (int k = 1; k < 200 && term > 1e-17 * sum; ++k) {
            term *= (x * x / 4.0) / ((double)k * (double)k);
            sum += term;
        }
        e += sum * sum;
    }
    *s_out = std::sqrt(e * e / (double)(BOX * BOX));
    return WP_OK;
}

wp_status wp_mlp_box_targets(const wp_plan *p, const wp_G *G, const double *u, const double *v, double s_out,
                             float *target, float *lost, void *stream) {
    if (!p) return wp_set_error(WP_EINVAL, "plan is NULL");
    if (!G) return wp_set_error(WP_EINVAL, "G is NULL");
    if (G->taps != WP_TAPS_C64 || (G->nnz > 0 && (!G->col || !G->val)))
        return wp_set_error(WP_EINVAL, "box targets need stored complex64 taps");
    if (!(s_out > 0.0)) return wp_set_error(WP_EINVAL, "s_out must be > 0");
    if (p->Ng < 2 * BOX) return wp_set_error(WP_EINVAL, "Ng = %d < %d", p->Ng, 2 * BOX);
    if (G->M == 0) return WP_OK;
    if (!u || !v || !target || !lost || !G->rowptr || !G->perm) return wp_set_error(WP_EINVAL, "NULL array");
    hipStream_t s = (hipStream_t)stream;
    wp_status st = launch_fill_zero(target, G->M * NOUT, s);
    if (st != WP_OK) return st;
    k_box_targets<<<(int)((G->M + 3) / 4), NTH, 0, s>>>(G->rowptr, G->col, (const float2 *)G->val, G->perm, G->M, u, v,
                                                        p->cell, p->logNg, (float)(1.0 / s_out), target, lost);
    return wp_check_launch("k_box_targets");
}

}  // extern "C"

namespace {
wp_status row_errors(const wp_plan *p, wp_mlp *m, const wp_G *G, const double *u, const double *v, const float *feat,
                     float *eps, float *energy, void *stream) {
    if (!p) return wp_set_error(WP_EINVAL, "plan is NULL");
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (!G) return wp_set_error(WP_EINVAL, "G is NULL");
    if (G->taps != WP_TAPS_C64 || (G->nnz > 0 && (!G->col || !G->val)))
        return wp_set_error(WP_EINVAL, "the energy check needs stored complex64 taps");
    if (p->Ng < 2 * BOX) return wp_set_error(WP_EINVAL, "Ng = %d < %d", p->Ng, 2 * BOX);
    if (G->M == 0) return WP_OK;
    if (!u || !v || !feat || !eps || !G->rowptr || !G->perm) return wp_set_error(WP_EINVAL, "NULL array");
    hipStream_t s = (hipStream_t)stream;
    const int chunk = m->max_batch;
    for (int64_t r0 = 0; r0 < G->M; r0 += chunk) {
        const int nr = (int)std::min<int64_t>(chunk, G->M - r0);
        k_gather_feat<<<(3 * nr + NTH - 1) / NTH, NTH, 0, s>>>(feat, G->perm, r0, nr, m->xb);
        if ((st = wp_check_launch("k_gather_feat")) != WP_OK) return st;
        if ((st = mlp_forward(m, nr, m->xb, m->o, nullptr, s)) != WP_OK) return st;
        k_row_errors<<<(nr + 3) / 4, NTH, 0, s>>>(m->o, r0, nr, G->rowptr, G->col, (const float2 *)G->val, G->perm, u,
                                                  v, p->cell, p->logNg, (float)m->s_out, eps, energy);
        if ((st = wp_check_launch("k_row_errors")) != WP_OK) return st;
    }
    return WP_OK;
}

}  // namespace

extern "C" {

wp_status wp_mlp_row_errors(const wp_plan *p, wp_mlp *m, const wp_G *G, const double *u, const double *v,
                            const float *feat, float *eps, void *stream) {
    return row_errors(p, m, G, u, v, feat, eps, nullptr, stream);
}

wp_status wp_mlp_lattice_coords(const wp_plan *p, const wp_mlp *m, int nw, int nd, double *u, double *v, double *w,
                                void *stream) {
    if (!p) return wp_set_error(WP_EINVAL, "plan is NULL");
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (nw < 2 || nd < 2 || (int64_t)nw * nd * nd > (1 << 26))
        return wp_set_error(WP_EINVAL, "lattice %d x %d x %d: need nw, nd >= 2 and at most 2^26 nodes", nw, nd, nd);
    if (!u || !v || !w) return wp_set_error(WP_EINVAL, "NULL array");
    if (!(m->w_top > 0.0)) return wp_set_error(WP_EINVAL, "the network's w_top is not set");
    const int64_t n = (int64_t)nw * nd * nd;
    k_lattice_coords<<<(int)((n + NTH - 1) / NTH), NTH, 0, (hipStream_t)stream>>>(nw, nd, m->w_top, p->cell, u, v, w);
    return wp_check_launch("k_lattice_coords");
}

wp_status wp_mlp_check_table(const wp_plan *p, wp_mlp *m, const wp_G *G, int nw, int nd, const double *u,
                             const double *v, const float *feat, float *table, void *stream) {
    if (!G) return wp_set_error(WP_EINVAL, "G is NULL");
    if (nw < 2 || nd < 2 || G->M != (int64_t)nw * nd * nd)
        return wp_set_error(WP_EINVAL, "G->M = %lld is not the lattice's %d x %d x %d nodes", (long long)G->M, nw, nd,
                            nd);
    if (!table) return wp_set_error(WP_EINVAL, "table is NULL");
    return row_errors(p, m, G, u, v, feat, table, table + G->M, stream);
}

wp_status wp_mlp_row_check(const wp_plan *p, wp_mlp *m, int nw, int nd, const float *table, int64_t n,
                           const float *feat, float *est, void *stream) {
    if (!p) return wp_set_error(WP_EINVAL, "plan is NULL");
    wp_status st = check_mlp(m);
    if (st != WP_OK) return st;
    if (nw < 2 || nd < 2 || (int64_t)nw * nd * nd > (1 << 26))
        return wp_set_error(WP_EINVAL, "lattice %d x %d x %d: need nw, nd >= 2 and at most 2^26 nodes", nw, nd, nd);
    if (n < 0) return wp_set_error(WP_EINVAL, "n = %lld", (long long)n);
    if (n == 0) return WP_OK;
    if (!table || !feat || !est) return wp_set_error(WP_EINVAL, "NULL array");
    hipStream_t s = (hipStream_t)stream;
    for (int64_t k0 = 0; k0 < n; k0 += m->max_batch) {
        const int nr = (int)std::min<int64_t>(m->max_batch, n - k0);
        if ((st = mlp_forward(m, nr, feat + 3 * k0, m->o, nullptr, s)) != WP_OK) return st;
        k_row_check<<<(nr + 3) / 4, NTH, 0, s>>>(m->o, k0, nr, feat, table, nw, nd, (float)m->s_out, est);
        if ((st = wp_check_launch("k_row_check")) != WP_OK) return st;
    }
    return WP_OK;
}

}  // extern "C"

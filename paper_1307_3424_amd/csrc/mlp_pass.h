// The surrogate network's forward and backward passes (included by mlp.hip).
//
// k_mlp_infer and k_mlp_train take 32 rows through all layers in one workgroup: the activations stay in LDS and
// registers, the weights stream from L2 as ready-made MFMA fragments, and in training the loss, its gradient and the
// chain back to the first layer follow in the same kernel, so no pre-activation, output or output gradient is stored
// in FP32.  k_mlp_wgrad then forms the weight gradients dW_l = dz_l^T a_(l-1) from the fragments k_mlp_train left, reading
// every operand straight from memory in fragment order (no LDS, no transposition).
//
// Fragment order.  v_mfma_f32_32x32x16_bf16 takes from lane l eight consecutive k (8 (l / 32) ..) of row l % 32 of
// each operand, and leaves column l % 32 of the product in lane l, rows 8 (r / 4) + 4 (l / 32) + r % 4 in its
// registers r.  Weights are kept as [tile of 32 rows][step of 16 k][lane][8].  An activation or a gradient used as an
// operand of a weight gradient (reduced over the batch) is kept as the product left it: registers 0..7 and 8..15
// of lane l are its two fragments of a 32-row block; the k order they imply is the same for both operands, which
// is all a sum over the batch needs.
//
// Bound of k_mlp_train: the weights' stream, 2.6 MB per workgroup through the CU's 64-byte-per-clock L1 (20 us for 256
// workgroups); the products themselves 10 us and the other arithmetic 14 us, which overlap only in part.  Two groups of
// eight wavefronts taking the output slabs in turn were slower (61 against 54 us at 8192 rows: 38 spilled registers, and
// both groups in the same phase).  Measured: see mlp_forward and mlp_backward.
#pragma once

#include "mlp_core.h"

namespace mlpc {

constexpr int PR = 32;                    // rows per workgroup
constexpr int PNT = 512, PW = PNT / 64;   // threads, wavefronts: wavefront w makes 32 columns of each 256
constexpr int PLD = H + 8;                // LDS row stride (bfloat16)
constexpr int KS = H / 16;                // MFMA steps over a depth of 256
constexpr int FRAG = 512;                 // elements of one fragment: 64 lanes x 8
static_assert(PW * 32 == H, "a wavefront per 32 hidden units");

// partial sums of one workgroup: b4, b3, b2, b1, W1
constexpr int PB4 = 0, PB3 = NOUT, PB2 = PB3 + H, PB1 = PB2 + H, PW1 = PB1 + H, PN = PW1 + 3 * H;

// row i of the batch is sample (a i + c) mod n of feat / targ
struct RowMap {
    int64_t a, c, n;
};

struct PassArgs {
    const float *feat, *targ;             // targ: training
    RowMap map;
    int rows;
    const float *params;
    const uint16_t *WF2, *WF3, *WF4;      // fragments of W_l (rows: outputs), [tile][step][lane][8]
    const uint16_t *WT2, *WT3, *WT4;      // of W_l^T (rows: inputs)
    float *out;                           // outputs [rows][NOUT], or NULL
    uint16_t *a3;                         // last hidden layer [rows][H], or NULL
    float scale;                          // training: 2 / (rows NOUT)
    uint16_t *a1F, *a2F, *a3F, *dOF, *dz3F, *dz2F;
    float *part;                          // [workgroups][PN]
    double *lpart;                        // [workgroups]
    float *grad;                          // weight gradients, cleared here for k_mlp_wgrad
};

__device__ __forceinline__ bf16x8 load_frag(const uint16_t *p, int lane) {
    return __builtin_bit_cast(bf16x8, *(const u32x4 *)(p + lane * 8));
}

// gelu(x) = x Phi(x) (error-function form) and its derivative Phi(x) + x phi(x).  A branch-free pair from one
// exponential and a degree-9 erfcx polynomial was as exact against FP64 and 2 us faster at 8192 training rows, but its
// last bits turn one bfloat16 activation in 10^4 the other way, which shows in the outputs; not kept.
__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_both(float x, float &grad) {
    const float e = 1.0f + erff(x * 0.70710678118654752f);
    grad = 0.5f * e + x * expf(-0.5f * x * x) * 0.39894228040143268f;
    return 0.5f * x * e;
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// a 32 x 32 block's 16 registers as bfloat16 pairs (round to nearest even, one instruction a pair)
struct Packed {
    uint32_t u[8];
    __device__ __forceinline__ explicit Packed(const float *v) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const f32x2 f = {v[2 * e], v[2 * e + 1]};
            u[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
        }
    }
    // the block's two fragments
    __device__ __forceinline__ void to_frags(uint16_t *p, int lane) const {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const u32x4 f = {u[4 * k], u[4 * k + 1], u[4 * k + 2], u[4 * k + 3]};
            *(u32x4 *)(p + k * FRAG + lane * 8) = f;
        }
    }
    // its column l % 32 into an LDS tile, columns col0 ..
    __device__ __forceinline__ void to_tile(uint16_t *t, int col0, int lane) const {
        uint16_t *q = t + 4 * (lane >> 5) * PLD + col0 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) q[(8 * (r >> 2) + (r & 3)) * PLD] = (uint16_t)(u[r >> 1] >> (16 * (r & 1)));
    }
};

__device__ __forceinline__ bf16x8 tile_frag(const uint16_t *t, int s, int lane) {
    return __builtin_bit_cast(bf16x8, *(const u32x4 *)(t + (lane & 31) * PLD + 16 * s + 8 * (lane >> 5)));
}

__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

// the KS fragments of one 256-deep product, asked for ahead of their use
struct Frags {
    bf16x8 f[KS];
    __device__ __forceinline__ void load(const uint16_t *p, int lane) {
#pragma unroll
        for (int s = 0; s < KS; ++s) f[s] = load_frag(p + s * FRAG, lane);
    }
};

// acc += A tile (32 x 256) times b
__device__ __forceinline__ f32x16 tile_product(const uint16_t *t, const Frags &b, f32x16 acc, int lane) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tile_frag(t, s, lane), b.f[s], acc, 0, 0, 0);
        if (s % 4 == 3) __builtin_amdgcn_sched_barrier(0);    // four of the tile's fragments in registers at a time
    }
    return acc;
}

// the first layer's pre-activations of this lane's column, 16 rows, to f
template <class F>
__device__ __forceinline__ void hidden1(const PassArgs &p, const float (*xs)[4], int col, int lane, F f) {
    const float *W1 = p.params + OW1 + 3 * col;
    const float w0 = W1[0], w1 = W1[1], w2 = W1[2], b = p.params[OB1 + col];
    float z[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float *x = xs[acc_row(r, lane)];
        z[r] = x[0] * w0 + x[1] * w1 + x[2] * w2 + b;
    }
    f(z);
}

// sum over the 32 rows of a block's column, in lanes 0 .. 31
__device__ __forceinline__ float column_sum(const float *v) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) s += v[r];
    return s + __shfl_xor(s, 32);
}

// A wavefront's registers hold the weight fragments of its next products; they are asked for as soon as the last
// product has used its own, ahead of its epilogue and the barrier.  The workgroups of one XCD (every eighth) start at
// different output slabs, so that its CUs do not all want the same lines of L2 at once.
// Inference: blockIdx.y takes the outputs in gridDim.y equal shares (each share makes the hidden layers again: a
// seventh of the work), so that few rows still fill the GPU and many put two workgroups on a CU.
constexpr size_t TRAIN_GRAD_LDS = (size_t)3 * 16 * PNT * 4;   // gelu' of the three layers

__global__ __launch_bounds__(PNT, 4) void k_mlp_infer(const PassArgs p) {
    __shared__ __align__(16) uint16_t tile[2][PR * PLD];
    __shared__ float xs[PR][4];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = (int)blockIdx.x * PR, col = 32 * w + (lane & 31);
    const int per = NOUT / H / gridDim.y, s0 = blockIdx.y * per, rot = (int)(blockIdx.x >> 3) % per;
    Frags f;
    f.load(p.WF2 + w * KS * FRAG, lane);
    if (tid < PR) {
        const int64_t i = min(i0 + tid, p.rows - 1);          // rows past the end repeat the last one
#pragma unroll
        for (int c = 0; c < 3; ++c) xs[tid][c] = p.feat[3 * i + c];
    }
    __syncthreads();
    hidden1(p, xs, col, lane, [&](const float *z) {
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = gelu(z[r]);
        Packed(v).to_tile(tile[0], 32 * w, lane);
    });
#pragma unroll
    for (int l = 2; l <= 3; ++l) {
        __syncthreads();
        const f32x16 z = tile_product(tile[l & 1], f, zero16(), lane);
        f.load(l == 2 ? p.WF3 + w * KS * FRAG : p.WF4 + (int64_t)((s0 + rot) * PW + w) * KS * FRAG, lane);
        const float b = p.params[(l == 2 ? OB2 : OB3) + col];
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = gelu(z[r] + b);
        Packed(v).to_tile(tile[(l + 1) & 1], 32 * w, lane);   // read last before this layer's barrier
    }
    __syncthreads();
    const uint16_t *t3 = tile[0];                             // a3
    if (p.a3 && blockIdx.y == 0) {
        for (int e = tid; e < PR * H / 8; e += PNT) {
            const int r = e / (H / 8), c = (e % (H / 8)) * 8;
            if (i0 + r < p.rows) *(u32x4 *)(p.a3 + (int64_t)(i0 + r) * H + c) = *(const u32x4 *)(t3 + r * PLD + c);
        }
    }
    if (!p.out) return;                                       // uniform over the grid
#pragma unroll 1
    for (int it = 0; it < per; ++it) {
        const int oc = (s0 + (it + rot) % per) * H + col;
        const float b4 = p.params[OB4 + oc];
        const f32x16 o = tile_product(t3, f, zero16(), lane);
        f.load(p.WF4 + (int64_t)((s0 + (it + 1 + rot) % per) * PW + w) * KS * FRAG, lane);   // the last one not used
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = i0 + acc_row(r, lane);
            if (i < p.rows) p.out[(int64_t)i * NOUT + oc] = o[r] + b4;
        }
    }
}

__global__ __launch_bounds__(PNT, 2) void k_mlp_train(const PassArgs p) {
    __shared__ __align__(16) uint16_t tile[3][PR * PLD];
    __shared__ float xs[PR][4];
    __shared__ uint32_t src[PR];                              // samples (fewer than 2^31)
    __shared__ double s_loss[PW];
    extern __shared__ float s_grad[];                         // [3][16][PNT]
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t blk = blockIdx.x;
    const int i0 = (int)blk * PR, col = 32 * w + (lane & 31);
    Frags f, ft;                                              // of the next products
    f.load(p.WF2 + w * KS * FRAG, lane);
    if (tid < PR) {
        const int64_t q = (p.map.a * (i0 + tid) + p.map.c) % p.map.n;
        src[tid] = (uint32_t)q;
#pragma unroll
        for (int c = 0; c < 3; ++c) xs[tid][c] = p.feat[3 * q + c];
    }
    {                                                         // clear this workgroup's share of the weight gradients
        const int64_t per = (NPARAM + gridDim.x - 1) / gridDim.x;
        for (int64_t e = blk * per + tid; e < min((blk + 1) * per, NPARAM); e += PNT) p.grad[e] = 0.f;
    }
    __syncthreads();
    uint16_t *t3 = tile[2];                                   // a3
    {
        hidden1(p, xs, col, lane, [&](const float *z) {
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float g;
                v[r] = gelu_both(z[r], g);
                s_grad[r * PNT + tid] = g;
            }
            const Packed pk(v);
            pk.to_tile(tile[0], 32 * w, lane);
            pk.to_frags(p.a1F + (blk * PW + w) * 2 * FRAG, lane);
        });
    }
    __syncthreads();
    {
        const f32x16 z = tile_product(tile[0], f, zero16(), lane);
        f.load(p.WF3 + w * KS * FRAG, lane);
        const float b = p.params[OB2 + col];
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float g;
            v[r] = gelu_both(z[r] + b, g);
            s_grad[(16 + r) * PNT + tid] = g;
        }
        const Packed pk(v);
        pk.to_tile(tile[1], 32 * w, lane);
        pk.to_frags(p.a2F + (blk * PW + w) * 2 * FRAG, lane);
    }
    __syncthreads();
    {
        const f32x16 z = tile_product(tile[1], f, zero16(), lane);
        const float b = p.params[OB3 + col];
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float g;
            v[r] = gelu_both(z[r] + b, g);
            s_grad[(32 + r) * PNT + tid] = g;
        }
        const Packed pk(v);
        pk.to_tile(t3, 32 * w, lane);
        pk.to_frags(p.a3F + (blk * PW + w) * 2 * FRAG, lane);
    }
    const int rot = (int)(blk >> 3) % (NOUT / H);
    f.load(p.WF4 + (int64_t)(rot * PW + w) * KS * FRAG, lane);
    __syncthreads();
    // layer 4, 256 outputs at a time: each wavefront's output gradients go to an LDS tile (two in turn), and
    // the product with W4 gathers the gradient of the last hidden layer
    f32x16 da = zero16();
    double loss = 0.0;
#pragma unroll 1
    for (int it = 0; it < NOUT / H; ++it) {
        const int sl = (it + rot) % (NOUT / H), oc = sl * H + col;       // this lane's output
        const float b4 = p.params[OB4 + oc];
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = p.targ[(uint64_t)src[acc_row(r, lane)] * NOUT + oc];
        ft.load(p.WT4 + ((int64_t)w * (NOUT / 16) + sl * KS) * FRAG, lane);
        const f32x16 o = tile_product(t3, f, zero16(), lane);
        f.load(it + 1 < NOUT / H ? p.WF4 + (int64_t)((sl + 1) % (NOUT / H) * PW + w) * KS * FRAG : p.WT3 + w * KS * FRAG, lane);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float d = (o[r] + b4) - v[r];
            loss += (double)d * d;
            v[r] = d * p.scale;
        }
        const float cs = column_sum(v);
        if (lane < 32) p.part[blk * PN + PB4 + oc] = cs;
        const Packed pk(v);
        pk.to_frags(p.dOF + ((blk * (NOUT / 32)) + sl * PW + w) * 2 * FRAG, lane);
        uint16_t *dt = tile[it & 1];
        pk.to_tile(dt, 32 * w, lane);
        __syncthreads();                                      // the other tile's readers are done by the next one
        // wavefront w: hidden units 32 w .. + 31, outputs sl H .. + 255 as depth
        da = tile_product(dt, ft, da, lane);
    }
    ft.load(p.WT2 + w * KS * FRAG, lane);
    for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off);
    if (lane == 0) s_loss[w] = loss;
    __syncthreads();                                          // a3 and the gradients' tiles are no longer read
    if (tid == 0) {
        double s = 0.0;
        for (int k = 0; k < PW; ++k) s += s_loss[k];
        p.lpart[blk] = s;
    }
    // the chain back through layers 3, 2 and 1: dz_l = da_l gelu'(z_l)
    float v[16];
    {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = da[r] * s_grad[(32 + r) * PNT + tid];
        const float cs = column_sum(v);
        if (lane < 32) p.part[blk * PN + PB3 + col] = cs;
        const Packed pk(v);
        pk.to_frags(p.dz3F + (blk * PW + w) * 2 * FRAG, lane);
        pk.to_tile(tile[2], 32 * w, lane);
    }
    __syncthreads();
    {
        da = tile_product(tile[2], f, zero16(), lane);
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = da[r] * s_grad[(16 + r) * PNT + tid];
        const float cs = column_sum(v);
        if (lane < 32) p.part[blk * PN + PB2 + col] = cs;
        const Packed pk(v);
        pk.to_frags(p.dz2F + (blk * PW + w) * 2 * FRAG, lane);
        pk.to_tile(tile[0], 32 * w, lane);
    }
    __syncthreads();
    {
        da = tile_product(tile[0], ft, zero16(), lane);
        float s0 = 0.f, s1 = 0.f, s2 = 0.f, sb = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float d = da[r] * s_grad[r * PNT + tid];
            const float *x = xs[acc_row(r, lane)];
            s0 += d * x[0];
            s1 += d * x[1];
            s2 += d * x[2];
            sb += d;
        }
        s0 += __shfl_xor(s0, 32);
        s1 += __shfl_xor(s1, 32);
        s2 += __shfl_xor(s2, 32);
        sb += __shfl_xor(sb, 32);
        if (lane < 32) {
            float *q = p.part + blk * PN;
            q[PW1 + 3 * col] = s0;
            q[PW1 + 3 * col + 1] = s1;
            q[PW1 + 3 * col + 2] = s2;
            q[PB1 + col] = sb;
        }
    }
}

// Weight gradients: C[m][n] += sum over the batch of A[.][m] B[.][n], A and B as fragments of 32-row blocks.  A
// workgroup makes a 64 x 64 tile; its wavefronts take every eighth block of its share of the batch, the next one's
// eight fragments on their way while the last one's multiply, and their sums meet in LDS.  Roles by block index: tiles
// of layers 4, 3 and 2, times `splits` shares of the batch, then the column sums.  Bound: the fragments through L1 (335
// MB at 8192 rows: 10 us).  Splitting the batch over workgroups instead of wavefronts cost 1.7 us per share in float
// atomics (16 shares: 46 us).
constexpr int GNT = 512, GW = GNT / 64;
constexpr int GN = H / 64, GT4 = NOUT / 64 * GN, GT3 = H / 64 * GN, GTILES = GT4 + 2 * GT3;
constexpr int GRC = 64, GRB = PN / GRC;   // column sums: 64 columns a workgroup, rows over its wavefronts
static_assert(PN % GRC == 0, "column sums");

__global__ __launch_bounds__(GNT, 4) void k_mlp_wgrad(const PassArgs p, int nrb, int splits, int chunk,
                                                      double *__restrict__ loss, int add_loss) {
    __shared__ float red[GW / 2][64 * 64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((int)blockIdx.x >= GTILES * splits) {                 // column sums of the partials
        const int q = (int)blockIdx.x - GTILES * splits, c = q * GRC + lane;
        float s = 0.f;
#pragma unroll 8
        for (int i = w; i < nrb; i += GW) s += p.part[(int64_t)i * PN + c];
        red[0][w * GRC + lane] = s;
        __syncthreads();
        if (w == 0) {
            s = 0.f;
            for (int k = 0; k < GW; ++k) s += red[0][k * GRC + lane];
            const int64_t at = c < PB3 ? OB4 + c : c < PB2 ? OB3 + (c - PB3) : c < PB1 ? OB2 + (c - PB2)
                             : c < PW1 ? OB1 + (c - PB1) : OW1 + (c - PW1);
            p.grad[at] = s;
        }
        if (q == 0 && w == 1) {                               // the loss: one wavefront over the workgroups' sums
            double d = 0.0;
            for (int i = lane; i < nrb; i += 64) d += p.lpart[i];
            for (int off = 32; off > 0; off >>= 1) d += __shfl_xor(d, off);
            if (lane == 0) *loss = add_loss ? *loss + d : d;
        }
        return;
    }
    // the four tiles of one A column run on one XCD, so its L2 serves A to three of them
    const int lb = (int)xcd_block(blockIdx.x, GTILES * splits);
    int mt = lb % GTILES;
    const int sp = lb / GTILES;
    const uint16_t *A, *B;
    float *C;
    int ntile;                                                // fragments per block of A
    if (mt < GT4) {
        A = p.dOF; B = p.a3F; C = p.grad + OW4; ntile = NOUT / 32;
    } else if ((mt -= GT4) < GT3) {
        A = p.dz3F; B = p.a2F; C = p.grad + OW3; ntile = H / 32;
    } else {
        mt -= GT3;
        A = p.dz2F; B = p.a1F; C = p.grad + OW2; ntile = H / 32;
    }
    const int m0 = 2 * (mt / GN), n0 = 2 * (mt % GN);
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = zero16();
    struct Step {                                             // one 16-row step of a block: two fragments a side
        bf16x8 a[2], b[2];
    };
    auto load = [&](Step &f, int rb, int k) {
        const uint16_t *a = A + ((int64_t)rb * ntile + m0) * 2 * FRAG, *b = B + ((int64_t)rb * (H / 32) + n0) * 2 * FRAG;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            f.a[i] = load_frag(a + (2 * i + k) * FRAG, lane);
            f.b[i] = load_frag(b + (2 * i + k) * FRAG, lane);
        }
    };
    auto multiply = [&](const Step &f) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
    };
    const int rb1 = min(nrb, (sp + 1) * chunk);
    Step f0, f1;                                              // each step's registers reload as soon as it is multiplied
    int rb = sp * chunk + w;
    if (rb < rb1) {
        load(f0, rb, 0);
        load(f1, rb, 1);
#pragma unroll 1
        for (; rb < rb1; rb += GW) {
            const int next = rb + GW < rb1 ? rb + GW : rb;    // the last one loads its own again
            multiply(f0);
            load(f0, next, 0);
            multiply(f1);
            load(f1, next, 1);
        }
    }
    // sums over the wavefronts: the upper half's, the lower half added, then each wavefront an eighth of the tile
    auto slot = [&](int k, int i, int j, int r) -> float & { return red[k][((i * 2 + j) * 16 + r) * 64 + lane]; };
    if (w >= GW / 2)
#pragma unroll
        for (int e = 0; e < 64; ++e) slot(w - GW / 2, e >> 5, (e >> 4) & 1, e & 15) = acc[e >> 5][(e >> 4) & 1][e & 15];
    __syncthreads();
    if (w < GW / 2)
#pragma unroll
        for (int e = 0; e < 64; ++e) slot(w, e >> 5, (e >> 4) & 1, e & 15) += acc[e >> 5][(e >> 4) & 1][e & 15];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 64 / GW; ++q) {
        const int e = w * (64 / GW) + q, i = e >> 5, j = (e >> 4) & 1, r = e & 15;
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < GW / 2; ++k) s += red[k][e * 64 + lane];
        float *c = C + (int64_t)(32 * (m0 + i) + acc_row(r, lane)) * H + 32 * (n0 + j) + acc_col(lane);
        if (splits > 1) unsafeAtomicAdd(c, s);
        else *c = s;
    }
}

// the weights' fragments: thread (matrix, fragment, lane) packs eight values
__global__ void k_mlp_fragments(const float *__restrict__ params, uint16_t *__restrict__ WF2, uint16_t *__restrict__ WT2,
                                uint16_t *__restrict__ WF3, uint16_t *__restrict__ WT3, uint16_t *__restrict__ WF4,
                                uint16_t *__restrict__ WT4) {
    constexpr int E2 = H * H / 8, E4 = NOUT * H / 8;
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 4 * E2 + 2 * E4) return;
    const float *W;
    uint16_t *dst;
    bool tr;                                                  // fragments of the transpose
    int depth;                                                // k extent
    if (e < 4 * E2) {
        const int q = e / E2;
        e -= q * E2;
        W = params + (q < 2 ? OW2 : OW3);
        dst = q == 0 ? WF2 : q == 1 ? WT2 : q == 2 ? WF3 : WT3;
        tr = q & 1;
        depth = H;
    } else {
        e -= 4 * E2;
        tr = e >= E4;
        if (tr) e -= E4;
        W = params + OW4;
        dst = tr ? WT4 : WF4;
        depth = tr ? NOUT : H;
    }
    const int lane = e & 63, f = e >> 6, steps = depth / 16, s = f % steps, tl = f / steps;
    const int row = 32 * tl + (lane & 31), k = 16 * s + 8 * (lane >> 5);
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = tr ? W[(int64_t)(k + i) * H + row] : W[(int64_t)row * H + k + i];
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = pack_bf16x2(x[2 * i], x[2 * i + 1]);
    *(u32x4 *)(dst + (int64_t)e * 8) = o;
}

}  // namespace mlpc

// Internal: sizes of the surrogate network and the bfloat16 MFMA tile machinery
// shared by its training kernels (mlp.hip) and the surrogate operator (surrogate.hip).
//
// Network: 3 -> H -> H -> H -> NOUT with GELU after the hidden layers; NOUT =
// 2 BOX^2 outputs are the real and imaginary parts of the taps of a BOX x BOX
// box of grid cells.  Parameters are packed in FP32 in the order
// W1 [H,3], b1 [H], W2 [H,H], b2, W3 [H,H], b3, W4 [NOUT,H], b4 [NOUT]
// (row-major, W_l maps layer l-1 to layer l).
//
// Matrix products: C[M,N] = A[M,K] B[N,K]^T with bfloat16 operands and FP32
// accumulation on v_mfma_f32_32x32x16_bf16; the surrogate's register-staged
// operands sit in LDS K-contiguous, BK = 32 deep, rows padded to LDK elements.
#pragma once

#include "common.h"

namespace mlpc {

constexpr int H = 256;
constexpr int BOX = 32;
constexpr int NOUT = 2 * BOX * BOX;
constexpr int64_t OW1 = 0;
constexpr int64_t OB1 = OW1 + (int64_t)H * 3;
constexpr int64_t OW2 = OB1 + H;
constexpr int64_t OB2 = OW2 + (int64_t)H * H;
constexpr int64_t OW3 = OB2 + H;
constexpr int64_t OB3 = OW3 + (int64_t)H * H;
constexpr int64_t OW4 = OB3 + H;
constexpr int64_t OB4 = OW4 + (int64_t)NOUT * H;
constexpr int64_t NPARAM = OB4 + NOUT;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 32;
constexpr int LDK = BK + 8;   // 80-byte LDS rows: consecutive rows start 20 banks apart

__device__ inline uint16_t to_bf16(float f) { return (uint16_t)bf16_bits_rne(f); }
__device__ inline float from_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// acc[fm][fn] += A rows [arow0 + 32 fm, +32) times B rows [brow0 + 32 fn, +32), one BK-deep step;
// LDS row strides SA and SB (elements).  Lane l feeds A[row l % 32][k 8 (l / 32) .. +7] and
// B[row l % 32][same k].
template <int FM, int FN, int SA = LDK, int SB = LDK>
__device__ __forceinline__ void mma_bk(f32x16 (&acc)[FM][FN], const uint16_t *As, const uint16_t *Bs, int arow0,
                                       int brow0, int lane) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
        bf16x8 a[FM], b[FN];
        const int ko = kk + 8 * (lane >> 5), ro = lane & 31;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
            a[fm] = __builtin_bit_cast(bf16x8, *(const u32x4 *)(As + (arow0 + 32 * fm + ro) * SA + ko));
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
            b[fn] = __builtin_bit_cast(bf16x8, *(const u32x4 *)(Bs + (brow0 + 32 * fn + ro) * SB + ko));
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
                acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[fm], b[fn], acc[fm][fn], 0, 0, 0);
    }
}

// position of accumulator register r of lane l inside its 32 x 32 block
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
__device__ __forceinline__ int acc_col(int lane) { return lane & 31; }

}  // namespace mlpc

// surrogate network object (mlp.hip)
struct wp_mlp {
    int device;
    int max_batch;
    double w_top, s_out;
    int64_t step;                          // Adam steps taken
    float *params, *m1, *m2, *grad;        // [NPARAM] FP32: parameters, Adam moments, gradients
    uint16_t *WF2, *WF3, *WF4;             // bfloat16 fragments of W2, W3, W4 (mlp_pass.h) ...
    uint16_t *WT2, *WT3, *WT4;             // ... and of their transposes
    uint16_t *a1F, *a2F, *a3F;             // [max_batch H] activations, fragments
    uint16_t *dOF, *dz3F, *dz2F;           // [max_batch NOUT], [max_batch H] gradients, fragments
    float *part;                           // [max_batch / 32][PN] bias and W1 gradients per workgroup
    double *lpart;                         // [max_batch / 32] squared errors per workgroup
    float *o;                              // [max_batch NOUT] outputs
    float *xb;                             // [max_batch 3] gathered features
    double *loss;                          // [1] running sum of squared errors
};

// forward pass of n <= max_batch feature rows: the outputs with `out`, the last hidden layer
// (bfloat16, row-major) with `a3`
wp_status mlp_forward(wp_mlp *m, int n, const float *feat, float *out, uint16_t *a3, hipStream_t s);

// Device-wide exclusive scan and the stable radix sort of (key, index) pairs, shared by the row builder and the
// surrogate's set-up.
#pragma once

#include "common.h"

namespace {

// ---------------------------------------------------------------------------- device-wide scan

constexpr int SCAN_NTH = 256, SCAN_IPT = 8, SCAN_TILE = SCAN_NTH * SCAN_IPT;

template <typename T>
__device__ inline T block_excl_scan_T(T v, T *red, T &total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    T x = v;
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    __syncthreads();
    if (lane == 63) red[wid] = x;
    __syncthreads();
    T off = 0, tot = 0;
    for (int i = 0; i < SCAN_NTH / 64; ++i) {
        if (i < wid) off += red[i];
        tot += red[i];
    }
    total = tot;
    return off + x - v;
}

// out[i] = sum_{j<i} in[j] within each tile of SCAN_TILE; bsum[tile] = tile total; in may be out
template <typename Tin, typename T>
__global__ __launch_bounds__(SCAN_NTH) void k_scan_tiles(const Tin *in, T *out, int64_t n, T *bsum) {
    __shared__ T red[SCAN_NTH / 64];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_IPT;
    T loc[SCAN_IPT];
    T s = 0;
    for (int i = 0; i < SCAN_IPT; ++i) {
        loc[i] = (base + i < n) ? (T)in[base + i] : (T)0;
        s += loc[i];
    }
    T total;
    T run = block_excl_scan_T(s, red, total);
    for (int i = 0; i < SCAN_IPT; ++i) {
        if (base + i < n) out[base + i] = run;
        run += loc[i];
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// exclusive scan of n values into out[0..n] (out[n] = total) by one workgroup, tile after tile; in may be out
template <typename Tin, typename T>
__global__ __launch_bounds__(SCAN_NTH) void k_scan_one(const Tin *in, T *out, int64_t n) {
    __shared__ T red[SCAN_NTH / 64];
    T carry = 0;
    for (int64_t t0 = 0; t0 < n; t0 += SCAN_TILE) {
        const int64_t base = t0 + threadIdx.x * SCAN_IPT;
        T loc[SCAN_IPT];
        T s = 0;
        for (int i = 0; i < SCAN_IPT; ++i) {
            loc[i] = (base + i < n) ? (T)in[base + i] : (T)0;
            s += loc[i];
        }
        T total;
        T run = carry + block_excl_scan_T(s, red, total);
        for (int i = 0; i < SCAN_IPT; ++i) {
            if (base + i < n) out[base + i] = run;
            run += loc[i];
        }
        carry += total;
    }
    if (threadIdx.x == 0) out[n] = carry;
}

// out[0..n) += boff[tile]; out[n] = the total
template <typename T>
__global__ __launch_bounds__(SCAN_NTH) void k_scan_add(T *__restrict__ out, int64_t n, const T *__restrict__ boff) {
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    const T o = boff[blockIdx.x];
    for (int i = threadIdx.x; i < SCAN_TILE; i += SCAN_NTH)
        if (base + i < n) out[base + i] += o;
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = boff[gridDim.x];
}

// scratch of device_scan: the tiles' totals, scanned in place, and their sum
inline int64_t scan_scratch_elems(int64_t n) { return (n + SCAN_TILE - 1) / SCAN_TILE + 1; }

// Exclusive scan of n >= 1 inputs into out[0..n], out[n] = total: one launch for up to SCAN_ONE values (a
// workgroup takes a tile per 2 us or so, less than two more launches), else tiles, their totals, and the sums.
constexpr int64_t SCAN_ONE = 2 * SCAN_TILE;
template <typename Tin, typename T>
void device_scan(const Tin *in, T *out, int64_t n, T *scratch, hipStream_t s) {
    if (n <= SCAN_ONE) {
        hipLaunchKernelGGL((k_scan_one<Tin, T>), dim3(1), dim3(SCAN_NTH), 0, s, in, out, n);
        return;
    }
    const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    hipLaunchKernelGGL((k_scan_tiles<Tin, T>), dim3(nb), dim3(SCAN_NTH), 0, s, in, out, n, scratch);
    hipLaunchKernelGGL((k_scan_one<T, T>), dim3(1), dim3(SCAN_NTH), 0, s, scratch, scratch, nb);
    hipLaunchKernelGGL((k_scan_add<T>), dim3(nb), dim3(SCAN_NTH), 0, s, out, n, scratch);
}

// ---------------------------------------------------------------------------- stable radix sort

// Least significant digit first, up to 8 bits per pass: a histogram of every tile of RS_TILE pairs, one scan of
// them (digit by digit, tiles in order), and the move.  Within a tile a wavefront takes a run of consecutive
// pairs 64 at a time and ranks equal digits by ballots, so the order is stable without atomics' luck.
// Three passes of three to five launches replace one partition per bit (24 of four to six launches at Ng = 4096):
// 0.9 -> 0.12 ms at 65536 pairs of 24 bits, 0.5 -> 0.1 ms at 32768 of 18 on MI355X.
constexpr int RS_NTH = 256, RS_WAVES = RS_NTH / 64, RS_IPL = 16, RS_RUN = 64 * RS_IPL, RS_TILE = RS_WAVES * RS_RUN;
constexpr int RS_DIGITS = 256;

__global__ __launch_bounds__(RS_NTH) void k_rs_hist(const int *__restrict__ keys, int64_t n, int shift, int mask,
                                                    int ntile, int *__restrict__ hist) {
    __shared__ int cnt[RS_DIGITS];
    for (int d = threadIdx.x; d <= mask; d += RS_NTH) cnt[d] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * RS_TILE;
    for (int i = threadIdx.x; i < RS_TILE; i += RS_NTH)
        if (t0 + i < n) atomicAdd(&cnt[(keys[t0 + i] >> shift) & mask], 1);
    __syncthreads();
    for (int d = threadIdx.x; d <= mask; d += RS_NTH) hist[(int64_t)d * ntile + blockIdx.x] = cnt[d];
}

// iin NULL: the indices are the positions
__global__ __launch_bounds__(RS_NTH) void k_rs_move(const int *__restrict__ kin, const int *__restrict__ iin,
                                                    int64_t n, int shift, int mask, int bits, int ntile,
                                                    const int *__restrict__ off, int *__restrict__ kout,
                                                    int *__restrict__ iout) {
    __shared__ int pos[RS_WAVES][RS_DIGITS];          // first the waves' counts, then their next positions
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int d = threadIdx.x; d < RS_WAVES * RS_DIGITS; d += RS_NTH) (&pos[0][0])[d] = 0;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * RS_TILE + wv * RS_RUN;
    int key[RS_IPL], rank[RS_IPL];
    volatile int *wp = pos[wv];
#pragma unroll
    for (int i = 0; i < RS_IPL; ++i) {
        const int64_t e = r0 + i * 64 + lane;
        const bool in = e < n;
        key[i] = in ? kin[e] : 0;
        const int d = (key[i] >> shift) & mask;
        unsigned long long same = __ballot(in);       // lanes with this lane's digit
        for (int b = 0; b < bits; ++b) {
            const unsigned long long one = __ballot((d >> b) & 1);
            same &= ((d >> b) & 1) ? one : ~one;
        }
        const int before = in ? wp[d] : 0;
        rank[i] = before + __popcll(same & ((1ull << lane) - 1ull));
        __builtin_amdgcn_wave_barrier();
        if (in && (same >> lane) == 1ull) wp[d] = before + __popcll(same);      // the digit's last lane
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int d = threadIdx.x; d <= mask; d += RS_NTH) {
        int at = off[(int64_t)d * ntile + blockIdx.x];
        for (int w = 0; w < RS_WAVES; ++w) {
            const int c = pos[w][d];
            pos[w][d] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RS_IPL; ++i) {
        const int64_t e = r0 + i * 64 + lane;
        if (e < n) {
            const int to = pos[wv][(key[i] >> shift) & mask] + rank[i];
            kout[to] = key[i];
            iout[to] = iin ? iin[e] : (int)e;
        }
    }
}

inline int rs_tiles(int64_t n) { return (int)((n + RS_TILE - 1) / RS_TILE); }
// scratch ints of radix_sort: the histograms (scanned in place, with their total) and the scan's own
inline int64_t rs_scratch_elems(int64_t n) {
    const int64_t h = (int64_t)RS_DIGITS * rs_tiles(n) + 1;
    return h + scan_scratch_elems(h);
}

// Sorts key[0..n) by its low `bits` bits (1..31), stably: keys_out / idx_out hold the sorted keys and the input
// position of each; k1 / i1 are temporaries of n ints.  key is not written unless it is keys_out or k1.
inline void radix_sort(const int *key, int64_t n, int bits, int *keys_out, int *idx_out, int *k1, int *i1, int *scratch,
                       hipStream_t s) {
    const int passes = (bits + 7) / 8, nt = rs_tiles(n);
    int *hist = scratch, *sc = scratch + (int64_t)RS_DIGITS * nt + 1;
    const int *kin = key, *iin = nullptr;
    int shift = 0;
    for (int q = 0; q < passes; ++q) {
        const int b = (bits - shift + passes - q - 1) / (passes - q), mask = (1 << b) - 1;
        int *ko = (passes - q) & 1 ? keys_out : k1, *io = (passes - q) & 1 ? idx_out : i1;   // the last pass lands in out
        hipLaunchKernelGGL(k_rs_hist, dim3(nt), dim3(RS_NTH), 0, s, kin, n, shift, mask, nt, hist);
        const int64_t nh = (int64_t)(mask + 1) * nt;
        device_scan<int, int>(hist, hist, nh, sc, s);
        hipLaunchKernelGGL(k_rs_move, dim3(nt), dim3(RS_NTH), 0, s, kin, iin, n, shift, mask, b, nt, hist, ko, io);
        kin = ko;
        iin = io;
        shift += b;
    }
}

}  // namespace

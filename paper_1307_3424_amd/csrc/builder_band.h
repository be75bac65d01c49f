// The band of cells around a visibility from which builder_rows.h makes a row of the linear chirp, and what it must
// show of the cells outside.  Host code too: a test walks every cell of every axis.
#pragma once

#include <hip/hip_runtime.h>

constexpr int BAND_MARGIN = 64;           // cells beyond the chirp's reach: the tail's bound is below 2^-13 of the
                                          // row's largest 1-D energy there up to supports of 64 cells

// Cells (su + p) mod Ng and (sv + p) mod Ng, p < cnt, of the two axes: the band, or the whole axis where the band
// reads all of h (su = sv = 0).  Every h(d) a cell of the band reads has |d| <= D.
struct Band {
    int su, sv, cnt, D;
};

// Window cells q0 .. q0 + W - 1 of the two axes; cell q reads h(q0 + i - q), i < W, so the cell next to the band reads
// W - 1 values from inside |d| <= D.  D is W - 1 cells wider than the margin for them, as far as `room` cells hold the
// band: a band that would fit without them is not given up for them.  cnt > room: too wide.
__host__ __device__ __forceinline__ Band row_band(int Ng, int room, double reach, int W, int q0u, int q0v) {
    Band b;
    const int least = (int)fmin(reach, (double)Ng) + 1 + BAND_MARGIN, most = (room + W - 2) / 2;
    b.D = least + W - 1;
    if (b.D > most) b.D = least > most ? least : most;
    b.cnt = 2 * b.D - W + 2;
    b.su = (q0u + W - 1 - b.D) & (Ng - 1);
    b.sv = (q0v + W - 1 - b.D) & (Ng - 1);
    if (b.cnt >= Ng || b.D >= Ng / 2) {       // the whole axis, also where the band leaves out only the few cells opposite
        b.su = b.sv = 0;
        b.cnt = Ng;
    }
    return b;
}

// the smallest |d| of an h(d) that a cell outside the band reads
__host__ __device__ __forceinline__ int outside_from(const Band &b, int W) { return b.D + 2 - W; }

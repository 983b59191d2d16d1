// What the LDS kernels share, and the body of the whole-grid pass that keeps a batched grid in LDS
// (batched.hip).
//
// Each of 256 threads computes a 4-column x RS-row block from a register ring of input rows (three 16-byte
// LDS reads per row); every tap is a register operand of one FMA.  Per cell the FP32 order is the centre
// product, then one FMA per footprint tap in row-major (dy, dx) order.
#pragma once

#include "internal.h"
#include "storage.h"

namespace st {

constexpr int NT = 256;  // threads per workgroup

__device__ __forceinline__ bool tap_in(int shape, int dy, int dx) {
    return shape == SHAPE_BOX || dy == 0 || dx == 0;
}


// Map the launch's block index to a tile so that each of the 8 XCDs (which receive blocks
// round-robin) works on a contiguous band of tiles; vertically adjacent tiles then share
// their halo rows through the same L2.
__device__ __forceinline__ int64_t xcd_tile(int64_t bid, int64_t ntiles) {
    const int64_t q = ntiles / 8, rem = ntiles % 8;
    const int64_t k = bid % 8, i = bid / 8;
    return k * q + (k < rem ? k : rem) + i;
}

// Whole-grid body: one workgroup keeps a small grid (plus an r-deep halo of b) resident in LDS
// for all `steps` steps, so the grid never round-trips through HBM between steps.  Buffer column
// bc holds grid column bc - 8, buffer row br holds grid row br - R.  `lds` must hold
// resident_lds_bytes(R, rows, cols) bytes.
__host__ __device__ inline int resident_bw(int64_t cols) { return int(((8 + cols + 8 + 7) / 8) * 8); }

__host__ __device__ inline size_t resident_lds_bytes(int R, int64_t rows, int64_t cols) {
    return (size_t(2) * size_t(rows + 2 * R) * size_t(resident_bw(cols)) + MAXK) * sizeof(float);
}

template <int R, int SHAPE, int RS>
__device__ __forceinline__ void resident_body(const float* src, float* dst, int rows, int cols, float b, int steps,
                                              const float* w, float* lds) {
    constexpr int K = 2 * R + 1;
    constexpr int OFF = 8;
    const int BW = resident_bw(cols), BH = rows + 2 * R;
    // buffers by offset arithmetic on the LDS base (keeps the compiler on LDS instructions)
    float* wsh = lds + 2 * BH * BW;
    if (threadIdx.x < K * K) wsh[threadIdx.x] = w[threadIdx.x];
    for (int k = threadIdx.x; k < 2 * BH * BW; k += NT) lds[k] = b;
    __syncthreads();
    for (int k = threadIdx.x; k < rows * cols; k += NT) {
        const int i = k / cols, j = k - i * cols;
        lds[(i + R) * BW + OFF + j] = src[k];
    }
    __syncthreads();
    float wreg[K * K];
#pragma unroll
    for (int q = 0; q < K * K; ++q) wreg[q] = wsh[q];
    const int ngx = (cols + 3) >> 2;
    const int nseg = (rows + RS - 1) / RS;
    for (int s = 0; s < steps; ++s) {
        const float* sb = lds + (s & 1) * (BH * BW);
        float* db = lds + ((s + 1) & 1) * (BH * BW);
        for (int it = threadIdx.x; it < ngx * nseg; it += NT) {
            const int seg = it / ngx;
            const int gx0 = 4 * (it - seg * ngx);
            const int bc = OFF + gx0;
            const int r0 = R + seg * RS;
            float v[RS + 2 * R][12];
#pragma unroll
            for (int j = 0; j < RS + 2 * R; ++j) {
                const int br = min(r0 - R + j, BH - 1);
                const float4* p = reinterpret_cast<const float4*>(sb + br * BW + bc - 4);
                const float4 q0 = p[0], q1 = p[1], q2 = p[2];
                v[j][0] = q0.x; v[j][1] = q0.y; v[j][2] = q0.z; v[j][3] = q0.w;
                v[j][4] = q1.x; v[j][5] = q1.y; v[j][6] = q1.z; v[j][7] = q1.w;
                v[j][8] = q2.x; v[j][9] = q2.y; v[j][10] = q2.z; v[j][11] = q2.w;
                if (j < 2 * R) continue;
                const int kr = j - 2 * R;
                float o[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) o[c] = wreg[R * K + R] * v[kr + R][4 + c];
#pragma unroll
                for (int dy = -R; dy <= R; ++dy)
#pragma unroll
                    for (int dx = -R; dx <= R; ++dx) {
                        if ((dy == 0 && dx == 0) || !tap_in(SHAPE, dy, dx)) continue;
                        const float wt = wreg[(dy + R) * K + dx + R];
#pragma unroll
                        for (int c = 0; c < 4; ++c) o[c] = __builtin_fmaf(wt, v[kr + R + dy][4 + c + dx], o[c]);
                    }
                const int gy = seg * RS + kr;
                if (gy >= rows) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (gx0 + c < cols) db[(gy + R) * BW + bc + c] = o[c];  // halo cells keep b
            }
        }
        __syncthreads();
    }
    const float* fin = lds + (steps & 1) * (BH * BW);
    for (int k = threadIdx.x; k < rows * cols; k += NT) {
        const int i = k / cols, j = k - i * cols;
        dst[k] = fin[(i + R) * BW + OFF + j];
    }
}

}  // namespace st

// Constant-weight Jacobi pass on register tiles (block_body.h): the kernels of ST_VARIANT_TILED and of
// plans that were never tuned.  Per cell the FP32 order of Sec. IV-E (centre product, then one FMA per
// footprint tap in row-major order), cells outside the grid hold b at every level (Sec. IV-A), and
// 16-bit fields are rounded after every level, so results are those of every other variant.
#pragma once

#include "block_body.h"

namespace st {

struct BlockArgs {
    const void* src;
    void* dst;
    int64_t rows, cols;
    int64_t tiles_x, first;  // tiles across; the first tile of this launch
    const int* stop;  // nullable: when it holds a nonzero value the pass does nothing
    float b;
    int tb;           // levels of this pass
    float w[MAXK];
    double* sums;     // sweep_block_sums: per tile, over its cells x, sum((x - x before the last level)^2), sum(x^2)
};
using BlockFn = void (*)(BlockArgs);

// The sweep_block_sums kernel of a tile (block::kDefs), solve_pass.hip.
BlockFn sums_lookup(int storage, int shape, int r, int def);

namespace block {

// One level: `w` the dense weights, `wx` those of a star's side taps.
template <int S, int R, int SHAPE, int V, int RW, int NW>
__device__ __forceinline__ void level(const float* w, const float* wx, const float* buf, int wave, int lane, float (&o)[RW][V]) {
    constexpr int K = 2 * R + 1, N = RW + 2 * R;
    constexpr bool BOX = SHAPE == SHAPE_BOX;
    constexpr int E = BOX ? V + 2 * R : V, C0 = BOX ? R : 0;
    float x[N][E];  // rows -R .. RW + R - 1 of this wavefront's frame; a box needs the sides of all of them
#pragma unroll
    for (int k = 0; k < N; ++k) {
        float q[V];
        if (k < R || k >= R + RW) {
            halo_row<R, V, RW, NW>(buf, wave, lane, k - R, q);
        } else {
#pragma unroll
            for (int c = 0; c < V; ++c) q[c] = o[k - R][c];
        }
        if constexpr (BOX) {
            with_sides<R, V>(q, x[k]);
        } else {
#pragma unroll
            for (int c = 0; c < V; ++c) x[k][c] = q[c];
        }
    }
    if constexpr (BOX) {
        // the rows that need no halo row first: they hide the LDS reads
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int k = RW <= 2 * R ? i : i < RW - 2 * R ? i + R : i < RW - R ? i - (RW - 2 * R) : i;
#pragma unroll
            for (int c = 0; c < V; ++c) o[k][c] = w[R * K + R] * x[k + R][C0 + c];
#pragma unroll
            for (int dy = -R; dy <= R; ++dy)
#pragma unroll
                for (int dx = -R; dx <= R; ++dx) {
                    if (dy == 0 && dx == 0) continue;
#pragma unroll
                    for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(w[(dy + R) * K + dx + R], x[k + R + dy][C0 + c + dx], o[k][c]);
                }
        }
    } else {
#pragma unroll
        for (int k = 0; k < RW; ++k) {
#pragma unroll
            for (int c = 0; c < V; ++c) o[k][c] = w[R * K + R] * x[k + R][c];
#pragma unroll
            for (int dy = -R; dy < 0; ++dy)
#pragma unroll
                for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(w[(dy + R) * K + R], x[k + R + dy][c], o[k][c]);
        }
        side_taps<R, V, RW>(o, x + R, wx);
#pragma unroll
        for (int k = 0; k < RW; ++k)
#pragma unroll
            for (int dy = 1; dy <= R; ++dy)
#pragma unroll
                for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(w[(dy + R) * K + R], x[k + R + dy][c], o[k][c]);
    }
    round_rows<S, V, RW>(o);
}

// Every level of a pass over the tile at `at`; EDGE tiles check rows and columns.  With SUMS also this
// lane's part of the tile's two sums.
template <int S, int R, int SHAPE, int V, int RW, int NW, bool EDGE, bool SUMS>
__device__ __forceinline__ void tile_levels(const BlockArgs& a, const TileAt& at, float* lds, double (&sum)[2]) {
    const int lane = int(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int64_t y0 = at.ty + wave * RW, x0 = at.tx + lane * V;
    bool col_ok[V];
#pragma unroll
    for (int c = 0; c < V; ++c) col_ok[c] = !EDGE || (x0 + c >= 0 && x0 + c < a.cols);
    const bool all_cols = !EDGE || (x0 >= 0 && x0 + V <= a.cols);
    float o[RW][V];
#pragma unroll
    for (int k = 0; k < RW; ++k) {
        const int64_t y = y0 + k;
        if constexpr (!EDGE) {
            load_cells<S, V>(a.src, y * a.cols + x0, o[k]);
        } else {
#pragma unroll
            for (int c = 0; c < V; ++c) o[k][c] = a.b;
            if (y >= 0 && y < a.rows) {
                if (all_cols) {
                    load_cells<S, V>(a.src, y * a.cols + x0, o[k]);
                } else {
#pragma unroll
                    for (int c = 0; c < V; ++c)
                        if (col_ok[c]) {
                            float one[1];
                            load_cells<S, 1>(a.src, y * a.cols + x0 + c, one);
                            o[k][c] = one[0];
                        }
                }
            }
        }
    }
    float wx[2 * R];  // a star's side taps, in registers for the DPP instructions
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) wx[i] = a.w[R * (2 * R + 1) + (i < R ? i : i + 1)];
    constexpr size_t HALF = lds_floats(R, V, RW, NW) / 2;
    auto step = [&](int l) __attribute__((always_inline)) {
        float* buf = lds + (l & 1) * HALF;
        if (has_rows<RW, NW>(wave, R * l)) publish<R, V, RW>(buf, wave, lane, o);
        __syncthreads();
        if (!has_rows<RW, NW>(wave, R * (l + 1))) return;
        level<S, R, SHAPE, V, RW, NW>(a.w, wx, buf, wave, lane, o);
        if constexpr (EDGE) {
#pragma unroll
            for (int k = 0; k < RW; ++k) {
                const bool row_ok = y0 + k >= 0 && y0 + k < a.rows;
#pragma unroll
                for (int c = 0; c < V; ++c) o[k][c] = row_ok && col_ok[c] ? o[k][c] : a.b;
            }
        }
    };
    [[maybe_unused]] float before[RW][V];
    if constexpr (SUMS) {
        for (int l = 0; l < a.tb - 1; ++l) step(l);
#pragma unroll
        for (int k = 0; k < RW; ++k)
#pragma unroll
            for (int c = 0; c < V; ++c) before[k][c] = o[k][c];
        step(a.tb - 1);
    } else {
        for (int l = 0; l < a.tb; ++l) step(l);
    }
    const int H = R * a.tb, HL = margin_cols(R, a.tb, V) / V;
    if (lane < HL || lane >= 64 - HL) return;
#pragma unroll
    for (int k = 0; k < RW; ++k) {
        const int row = wave * RW + k;
        const int64_t y = y0 + k;
        if (row < H || row >= NW * RW - H || (EDGE && y >= a.rows)) continue;
        if constexpr (SUMS) {
#pragma unroll
            for (int c = 0; c < V; ++c) {
                const double x = col_ok[c] ? double(o[k][c]) : 0.0, d = col_ok[c] ? x - double(before[k][c]) : 0.0;
                sum[0] = __builtin_fma(d, d, sum[0]);
                sum[1] = __builtin_fma(x, x, sum[1]);
            }
        }
        if (all_cols) {
            store_cells<S, V>(a.dst, y * a.cols + x0, o[k]);
        } else {
#pragma unroll
            for (int c = 0; c < V; ++c)
                if (col_ok[c]) {
                    const float one[1] = {o[k][c]};
                    store_cells<S, 1>(a.dst, y * a.cols + x0 + c, one);
                }
        }
    }
}

}  // namespace block

template <int S, int R, int SHAPE, int V, int RW, int NW>
__global__ __launch_bounds__(64 * NW) void sweep_block(BlockArgs a) {
    extern __shared__ float4 lds4[];
    if (a.stop && __hip_atomic_load(a.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const block::TileAt at =
        block::tile_at<R, V, RW, NW>(a.first + block::xcd_order(blockIdx.x, gridDim.x), a.tiles_x, a.rows, a.cols, a.tb);
    float* lds = reinterpret_cast<float*>(lds4);
    double sum[2];
    if (at.edge) block::tile_levels<S, R, SHAPE, V, RW, NW, true, false>(a, at, lds, sum);
    else block::tile_levels<S, R, SHAPE, V, RW, NW, false, false>(a, at, lds, sum);
}

// The same pass, which also sums how far its last level moved the cells: a lane has the cell before and
// after it in registers, so a convergence check reads no field at all.  Against a last step and two norms
// kernels of its own (three launches, two fields read), per check of 20 steps of star r = 1: 79 -> 58 us at
// 2048^2, 617 -> 424 us at 8192^2, 42 -> 25 us at 256^2; an interval of one step at 2048^2 33 -> 27 us.
template <int S, int R, int SHAPE, int V, int RW, int NW>
__global__ __launch_bounds__(64 * NW) void sweep_block_sums(BlockArgs a) {
    extern __shared__ float4 lds4[];
    if (a.stop && __hip_atomic_load(a.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int64_t t = a.first + block::xcd_order(blockIdx.x, gridDim.x);
    const block::TileAt at = block::tile_at<R, V, RW, NW>(t, a.tiles_x, a.rows, a.cols, a.tb);
    float* lds = reinterpret_cast<float*>(lds4);
    double sum[2] = {0.0, 0.0};
    if (at.edge) block::tile_levels<S, R, SHAPE, V, RW, NW, true, true>(a, at, lds, sum);
    else block::tile_levels<S, R, SHAPE, V, RW, NW, false, true>(a, at, lds, sum);
    __shared__ double part[NW][2];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        sum[0] += __shfl_down(sum[0], d);
        sum[1] += __shfl_down(sum[1], d);
    }
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6][0] = sum[0];
        part[threadIdx.x >> 6][1] = sum[1];
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double q = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) q += part[w][threadIdx.x];
        a.sums[2 * t + threadIdx.x] = q;
    }
}

}  // namespace st

// Batched grids on register tiles (block_body.h): a pass of every grid of a stencil class in one launch,
// each workgroup one tile of one grid, and small grids whose every step runs in one workgroup.
//
// A pass computes what the single-grid kernel does (sweep_block.h), so results are bitwise the same.  What
// bounds it is FP32 issue, plus the margins: the tile of a class is chosen on the host (batched.hip).
// Whole grids: with the grid and its halo in one 128 x 128 tile no margin is lost and nothing but the first
// load and the last store touches memory; a level costs what its cells do, one barrier and a row exchange.
//
// Tuned batches of mixed classes, before (tiles and whole grids in LDS, one kernel for all classes) and
// after, us: 100 grids of sides up to 256, 50 steps 850 and 300; 64 of up to 1024, 30 steps 609 and 275; 256
// of up to 2048, 40 steps, most of which march, 2190 and 1935-1963 (four tunings).
#include "batched.h"
#include "sweep_block.h"

namespace st {

namespace {

__device__ __forceinline__ void fill_args(const BatchDesc& d, BlockArgs& a) {
    a.rows = d.rows;
    a.cols = d.cols;
    a.stop = nullptr;
    a.b = d.b;
    a.sums = nullptr;
}
// A footprint's weights, loaded before the first store (scalar registers).
template <int R>
__device__ __forceinline__ void load_w(const BatchDesc& d, BlockArgs& a) {
#pragma unroll
    for (int t = 0; t < (2 * R + 1) * (2 * R + 1); ++t) a.w[t] = d.w[t];
}

template <int R, int SH, int V, int RW, int NW>
__global__ __launch_bounds__(64 * NW) void batched_block(BlockPassArgs q) {
    extern __shared__ float4 lds4[];
    const int64_t o = q.first + block::xcd_order(blockIdx.x, gridDim.x);
    const int k = upper_index(q.tile_prefix, q.n + 1, o);
    const BatchDesc& d = q.desc[q.order[k]];
    const int P = d.passes, p = q.p;
    BlockArgs a;
    fill_args(d, a);
    load_w<R>(d, a);
    a.src = p == 0 ? d.in : (((P - p) % 2 == 0) ? d.out : d.ws);  // written by pass p - 1
    a.dst = ((P - 1 - p) % 2 == 0) ? d.out : d.ws;
    a.tb = d.steps / P + (p < d.steps % P);  // equally deep passes, give or take a level
    const block::TileAt at = block::tile_at<R, V, RW, NW>(o - q.tile_prefix[k], d.tiles_x, d.rows, d.cols, a.tb);
    // (a shallower pass has wider tiles: the last ones may lie beyond the grid)
    if (at.ty + R * a.tb >= d.rows || at.tx + block::margin_cols(R, a.tb, V) >= d.cols) return;
    float* lds = reinterpret_cast<float*>(lds4);
    double sum[2];
    if (at.edge) block::tile_levels<ST_F32, R, SH, V, RW, NW, true, false>(a, at, lds, sum);
    else block::tile_levels<ST_F32, R, SH, V, RW, NW, false, false>(a, at, lds, sum);
}

constexpr int WV = 2, WRW = 8, WNW = 16;  // the 128 x 128 tile of whole grids
template <int R, int SH>
__global__ __launch_bounds__(64 * WNW) void batched_whole(BlockPassArgs q) {
    extern __shared__ float4 lds4[];
    float* lds = reinterpret_cast<float*>(lds4);
    const BatchDesc& d = q.desc[q.order[blockIdx.x]];
    BlockArgs a;
    fill_args(d, a);
    load_w<R>(d, a);
    const int lane = int(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    // the grid sits R rows and a lane's columns or more inside the tile; the cells around it hold b
    const int rows = int(a.rows), cols = int(a.cols);
    const int y0 = wave * WRW - R, x0 = lane * WV - block::margin_cols(R, 1, WV);
    float o[WRW][WV];
    bool ok[WRW][WV];
#pragma unroll
    for (int k = 0; k < WRW; ++k)
#pragma unroll
        for (int c = 0; c < WV; ++c) {
            ok[k][c] = unsigned(y0 + k) < unsigned(rows) && unsigned(x0 + c) < unsigned(cols);
            o[k][c] = ok[k][c] ? d.in[int64_t(y0 + k) * cols + x0 + c] : a.b;
        }
    float wx[2 * R];
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) wx[i] = a.w[R * (2 * R + 1) + (i < R ? i : i + 1)];
    constexpr size_t HALF = block::lds_floats(R, WV, WRW, WNW) / 2;
    const bool used = y0 + WRW > 0 && y0 < rows;  // some row of the grid is this wavefront's
    for (int l = 0; l < d.steps; ++l) {
        float* buf = lds + (l & 1) * HALF;
        block::publish<R, WV, WRW>(buf, wave, lane, o);
        __syncthreads();
        if (!used) continue;
        block::level<ST_F32, R, SH, WV, WRW, WNW>(a.w, wx, buf, wave, lane, o);
#pragma unroll
        for (int k = 0; k < WRW; ++k)
#pragma unroll
            for (int c = 0; c < WV; ++c) o[k][c] = ok[k][c] ? o[k][c] : a.b;
    }
#pragma unroll
    for (int k = 0; k < WRW; ++k)
#pragma unroll
        for (int c = 0; c < WV; ++c)
            if (ok[k][c]) d.out[int64_t(y0 + k) * cols + x0 + c] = o[k][c];
}

template <int R, int SH>
BlockPassFn block_pass_fn(int def) {
    switch (def) {
        case 0: return batched_block<R, SH, 1, 8, 8>;
        case 1: return batched_block<R, SH, 2, 4, 8>;
        case 2: return batched_block<R, SH, 2, 8, 8>;
        case 3: return batched_block<R, SH, 4, 4, 8>;
        case 4: return batched_block<R, SH, 2, 8, 16>;
    }
    return nullptr;
}

}  // namespace

BlockPassFn batched_block_lookup(int shape, int r, int def) {
    switch (r) {
        case 1: return shape == SHAPE_BOX ? block_pass_fn<1, SHAPE_BOX>(def) : block_pass_fn<1, SHAPE_STAR>(def);
        case 2: return shape == SHAPE_BOX ? block_pass_fn<2, SHAPE_BOX>(def) : block_pass_fn<2, SHAPE_STAR>(def);
        case 3: return shape == SHAPE_BOX ? block_pass_fn<3, SHAPE_BOX>(def) : block_pass_fn<3, SHAPE_STAR>(def);
    }
    return nullptr;
}

BlockPassFn batched_whole_lookup(int shape, int r) {
    switch (r) {
        case 1: return shape == SHAPE_BOX ? batched_whole<1, SHAPE_BOX> : batched_whole<1, SHAPE_STAR>;
        case 2: return shape == SHAPE_BOX ? batched_whole<2, SHAPE_BOX> : batched_whole<2, SHAPE_STAR>;
        case 3: return shape == SHAPE_BOX ? batched_whole<3, SHAPE_BOX> : batched_whole<3, SHAPE_STAR>;
    }
    return nullptr;
}

}  // namespace st

// Variable-coefficient (conservative) heat step: a 5-point Jacobi update (paper Sec. II-C)
// whose weights come from a diffusivity field kappa:
//   u'(c) = u(c) + sum_{nb in N, W, E, S} kf (u(nb) - u(c)),  kf = (kappa(c) + kappa(nb)) / 2,
// with u(nb) := b and kappa(nb) := kappa(c) across the grid edge.  FP32 order: acc = u(c), then
// acc = fma(0.5f * (kappa(c) + kappa(nb)), u(nb) - u(c), acc) for nb = N, W, E, S.
//
// varcoef_naive: one step per launch, one thread per cell.
// varcoef_block: tb steps per launch on register tiles (block_body.h).
#include <algorithm>

#include "block_body.h"
#include "internal.h"

namespace st {

namespace {

constexpr int NT = 256;

__device__ __forceinline__ float vc_update(float uc, float kc, float un, float kn, float uw, float kw, float ue,
                                           float ke, float us, float ks) {
    float acc = uc;
    acc = __builtin_fmaf(0.5f * (kc + kn), un - uc, acc);
    acc = __builtin_fmaf(0.5f * (kc + kw), uw - uc, acc);
    acc = __builtin_fmaf(0.5f * (kc + ke), ue - uc, acc);
    acc = __builtin_fmaf(0.5f * (kc + ks), us - uc, acc);
    return acc;
}

__global__ __launch_bounds__(NT) void varcoef_naive(SweepArgs a) {
    const int64_t n = a.rows * a.cols;
    const float* u = static_cast<const float*>(a.src);
    const float* k = a.kappa;
    // grid-stride: the grid is capped on the host, so any cell count fits one launch
    for (int64_t idx = int64_t(blockIdx.x) * NT + threadIdx.x; idx < n; idx += int64_t(gridDim.x) * NT) {
        const int64_t i = idx / a.cols, j = idx - i * a.cols;
        const float uc = u[idx], kc = k[idx];
        const bool hn = i > 0, hw = j > 0, he = j + 1 < a.cols, hs = i + 1 < a.rows;
        const float un = hn ? u[idx - a.cols] : a.b, kn = hn ? k[idx - a.cols] : kc;
        const float uw = hw ? u[idx - 1] : a.b, kw = hw ? k[idx - 1] : kc;
        const float ue = he ? u[idx + 1] : a.b, ke = he ? k[idx + 1] : kc;
        const float us = hs ? u[idx + a.cols] : a.b, ks = hs ? k[idx + a.cols] : kc;
        static_cast<float*>(a.dst)[idx] = vc_update(uc, kc, un, kn, uw, kw, ue, ke, us, ks);
    }
}

// The depths that a plan accepts per tile: the LDS that two buffers of the field and one of kappa would take,
// the halo around the tile included.  No kernel keeps them; the limit decides which calls are refused, and
// stays what it was.
size_t vlds_bytes(int tb, int TX, int TY) {
    const int off = ((tb + 4 + 3) / 4) * 4;
    const int bw = ((off + TX + tb + 8 + 3) / 4) * 4, bh = TY + 2 * tb;
    return size_t(3) * size_t(bw) * size_t(bh) * sizeof(float);
}

struct VArgs {
    const float* src;
    const float* kappa;
    float* dst;
    int64_t rows, cols;
    int64_t tiles_x, tiles;  // of one field
    int64_t first, blocks;   // the tiles of this launch, of all fields: `blocks` from `first` on
    int fields;              // fields one after another in src, kappa and dst
    float b;
    int tb;
    // windows of larger fields: rows x cols cells of each at window_origin(); kappa always, src if src_whole,
    // is then the larger field, w.rows x w.cols, and dst holds the windows one after another
    VcWindows w;
    int src_whole;
};

// A pass on register tiles (block_body.h).  The diffusivity enters once per pass as face values,
// 0.5f (kappa(c) + kappa(nb)), which two cells share: V north faces per row (one row more than the
// wavefront's) and V + 1 west faces, so that a level is four subtractions and four FMAs per cell.
// Rows and columns of kappa clamp at the grid's edge, which is the rule kappa(nb) := kappa(c).
// Bound by the vector ALU: at 1024^2 x 16 steps the LDS-tile kernel this replaced took 80 us.
template <int V, int RW, int NW, bool EDGE>
__device__ __forceinline__ void vc_levels(const VArgs& a, const block::TileAt& at, int64_t f, float* lds) {
    using namespace block;
    const int lane = int(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int64_t y0 = at.ty + wave * RW, x0 = at.tx + lane * V;
    const int64_t field = f * a.rows * a.cols;
    const float* src = a.src + field;
    const float* kap = a.kappa + field;
    int64_t pitch = a.cols, src_pitch = a.cols;
    if (a.w.yx) {
        pitch = a.w.cols;
        const int64_t at0 = f * a.w.rows * pitch + window_origin(a.w.yx[2 * f], a.w.reach, a.w.rows, a.rows) * pitch +
                            window_origin(a.w.yx[2 * f + 1], a.w.reach, pitch, a.cols);
        kap = a.kappa + at0;
        if (a.src_whole) {
            src = a.src + at0;
            src_pitch = pitch;
        }
    }
    float* dst = a.dst + field;
    bool col_ok[V];
#pragma unroll
    for (int c = 0; c < V; ++c) col_ok[c] = !EDGE || (x0 + c >= 0 && x0 + c < a.cols);
    const bool all_cols = !EDGE || (x0 >= 0 && x0 + V <= a.cols);
    auto load_row = [&](const float* base, int64_t pitch, int64_t y, float (&q)[V]) {  // y inside the grid; columns clamped
        if (all_cols) {
            load_cells<ST_F32, V>(base, y * pitch + x0, q);
        } else {
#pragma unroll
            for (int c = 0; c < V; ++c) {
                const int64_t x = x0 + c < 0 ? 0 : x0 + c >= a.cols ? a.cols - 1 : x0 + c;
                float one[1];
                load_cells<ST_F32, 1>(base, y * pitch + x, one);
                q[c] = one[0];
            }
        }
    };
    auto clamp_row = [&](int64_t y) { return y < 0 ? int64_t(0) : y >= a.rows ? a.rows - 1 : y; };
    float o[RW][V], fn[RW + 1][V], fw[RW][V + 1];
    {
        float k[RW + 2][V];
#pragma unroll
        for (int r = 0; r < RW + 2; ++r) load_row(kap, pitch, clamp_row(y0 - 1 + r), k[r]);
#pragma unroll
        for (int r = 0; r < RW; ++r) load_row(src, src_pitch, clamp_row(y0 + r), o[r]);
#pragma unroll
        for (int r = 0; r <= RW; ++r)
#pragma unroll
            for (int c = 0; c < V; ++c) fn[r][c] = 0.5f * (k[r + 1][c] + k[r][c]);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const float kw = prev_lane(k[r + 1][V - 1]), ke = next_lane(k[r + 1][0]);
#pragma unroll
            for (int c = 0; c <= V; ++c)
                fw[r][c] = 0.5f * ((c < V ? k[r + 1][c < V ? c : 0] : ke) + (c > 0 ? k[r + 1][c > 0 ? c - 1 : 0] : kw));
        }
    }
    auto outside = [&]() {  // cells outside the grid hold b
        if constexpr (EDGE) {
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const bool row_ok = y0 + r >= 0 && y0 + r < a.rows;
#pragma unroll
                for (int c = 0; c < V; ++c) o[r][c] = row_ok && col_ok[c] ? o[r][c] : a.b;
            }
        }
    };
    outside();
    constexpr size_t HALF = lds_floats(1, V, RW, NW) / 2;
    for (int l = 0; l < a.tb; ++l) {
        float* buf = lds + (l & 1) * HALF;
        if (has_rows<RW, NW>(wave, l)) publish<1, V, RW>(buf, wave, lane, o);
        __syncthreads();
        if (!has_rows<RW, NW>(wave, l + 1)) continue;
        float x[RW + 2][V];
        halo_row<1, V, RW, NW>(buf, wave, lane, -1, x[0]);
        halo_row<1, V, RW, NW>(buf, wave, lane, RW, x[RW + 1]);
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < V; ++c) x[r + 1][c] = o[r][c];
        // the rows that need no halo row first: they hide the LDS reads
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int r = i < RW - 2 ? i + 1 : i == RW - 2 ? 0 : RW - 1;
            const float(&u)[V] = x[r + 1];
            const float w = prev_lane(u[V - 1]), e = next_lane(u[0]);
#pragma unroll
            for (int c = 0; c < V; ++c) {
                float acc = u[c];
                acc = __builtin_fmaf(fn[r][c], x[r][c] - u[c], acc);
                acc = __builtin_fmaf(fw[r][c], (c > 0 ? u[c > 0 ? c - 1 : 0] : w) - u[c], acc);
                acc = __builtin_fmaf(fw[r][c + 1], (c + 1 < V ? u[c + 1 < V ? c + 1 : 0] : e) - u[c], acc);
                acc = __builtin_fmaf(fn[r + 1][c], x[r + 2][c] - u[c], acc);
                o[r][c] = acc;
            }
        }
        outside();
    }
    const int HL = margin_cols(1, a.tb, V) / V;
    if (lane < HL || lane >= 64 - HL) return;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int row = wave * RW + r;
        const int64_t y = y0 + r;
        if (row < a.tb || row >= NW * RW - a.tb || (EDGE && y >= a.rows)) continue;
        if (all_cols) {
            store_cells<ST_F32, V>(dst, y * a.cols + x0, o[r]);
        } else {
#pragma unroll
            for (int c = 0; c < V; ++c)
                if (col_ok[c]) {
                    const float one[1] = {o[r][c]};
                    store_cells<ST_F32, 1>(dst, y * a.cols + x0 + c, one);
                }
        }
    }
}

template <int V, int RW, int NW>
__global__ __launch_bounds__(64 * NW) void varcoef_block(VArgs a) {
    extern __shared__ float4 lds4[];
    float* lds = reinterpret_cast<float*>(lds4);
    const int64_t t = a.first + block::xcd_order(blockIdx.x, a.blocks), f = t / a.tiles;
    const block::TileAt at = block::tile_at<1, V, RW, NW>(t - f * a.tiles, a.tiles_x, a.rows, a.cols, a.tb);
    if (at.edge) vc_levels<V, RW, NW, true>(a, at, f, lds);
    else vc_levels<V, RW, NW, false>(a, at, f, lds);
}

using VcFn = void (*)(VArgs);

VcFn varcoef_lookup(int def) {
    switch (def) {
        case 0: return varcoef_block<1, 8, 8>;
        case 1: return varcoef_block<2, 4, 8>;
        case 2: return varcoef_block<2, 8, 8>;
        case 3: return varcoef_block<4, 4, 8>;
        case 4: return varcoef_block<2, 8, 16>;
    }
    return nullptr;
}

}  // namespace

size_t varcoef_lds_bytes(int tb, int tx, int ty) { return vlds_bytes(tb, tx, ty); }

// A pass of `levels` levels on register tiles over `fields` fields (or windows) of rows x cols cells.
static int launch_vc_block(int tile, VArgs a, hipStream_t s) {
    const block::Cover c = block::pick(tile, VARCOEF_OPS, 1, a.tb, a.rows, a.cols);
    if (c.def < 0) return fail(ST_EUNSUPPORTED, "temporal block too deep for the tile");
    if (c.tiles * a.fields >= int64_t(1) << 31) return fail(ST_EUNSUPPORTED, "too many tiles for one launch");
    const block::Def& d = block::kDefs[c.def];
    VcFn fn = varcoef_lookup(c.def);
    const size_t lds = block::lds_floats(1, d.v, d.rw, d.nw) * sizeof(float);
    if (int rc = prepare_lds(reinterpret_cast<const void*>(fn), lds)) return rc;
    a.tiles_x = c.tiles_x;
    a.tiles = c.tiles;
    clear_stale_error();
    launch_runs(c.tiles * a.fields, 64 * d.nw, [&](int64_t first, int64_t n) {
        a.first = first;
        a.blocks = n;
        hipLaunchKernelGGL(fn, dim3(unsigned(n)), dim3(64 * d.nw), lds, s, a);
    });
    ST_LAUNCH_CHECK("varcoef_block");
    return ST_OK;
}

int varcoef_launch(const st_plan* p, const float* src, float* dst, const float* kappa, int levels, hipStream_t s) {
    if (levels <= 0) {  // naive reference path
        SweepArgs a;
        a.src = src;
        a.dst = dst;
        a.kappa = kappa;
        a.rows = p->rows;
        a.cols = p->cols;
        a.b = p->bq;
        a.tb = 1;
        const int64_t n = p->rows * p->cols;
        clear_stale_error();
        hipLaunchKernelGGL(varcoef_naive, dim3(unsigned(std::min<int64_t>((n + NT - 1) / NT, kNaiveMaxBlocks))),
                           dim3(NT), 0, s, a);
        ST_LAUNCH_CHECK("varcoef_naive");
        return ST_OK;
    }
    return launch_vc_block(tile_index(p->tile_x, p->tile_y),
                           VArgs{src, kappa, dst, p->rows, p->cols, 0, 0, 0, 0, 1, p->bq, levels, VcWindows{}, 0}, s);
}

int varcoef_windows(const float* u0, const float* kappa, const VcWindows& w, int64_t rows, int64_t cols, int fields,
                    int64_t steps, float* out, float* scratch, hipStream_t s) {
    constexpr int kDepth = 8;  // 64 x 64 tiles that store 48 x 48: the fastest for windows of a few hundred cells
    const int64_t passes = (steps + kDepth - 1) / kDepth;
    const float* src = u0;
    for (int64_t k = 0; k < passes; ++k) {
        float* dst = (passes - 1 - k) % 2 == 0 ? out : scratch;
        const int levels = int(steps / passes + (k < steps % passes));
        if (int rc = launch_vc_block(0, VArgs{src, kappa, dst, rows, cols, 0, 0, 0, 0, fields, 0.0f, levels, w, k == 0}, s)) return rc;
        src = dst;
    }
    return ST_OK;
}

}  // namespace st

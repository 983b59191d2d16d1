// Jacobi sweep kernels for constant-weight star and box stencils (paper Sec. II-C update,
// Sec. IV-A fixed halo, Sec. IV-E centre-first accumulation).
//
// Kernels:
//   sweep_naive   one step per launch, one thread per cell, neighbours read straight from
//                 global memory with a bounds test.  The plain GPU reference path.
//   sweep_block   tb steps per launch (temporal blocking) on register tiles, see block_body.h and
//                 sweep_block.h.
//   sweep_step    one step per launch on LDS tiles, for footprints and sizes where no step is to be saved.
//   sweep_stream  tb steps per launch on LDS tiles, persistent workgroups, the next tile copied into
//                 LDS by DMA while the current one computes.
// All use the same per-cell FP32 order (centre product, then one FMA per footprint tap in
// row-major order), so their results are bitwise identical for every tb and tile.
#include <algorithm>
#include <map>
#include <mutex>

#include "internal.h"
#include "march_layout.h"
#include "storage.h"
#include "sweep_block.h"
#include "sweep_body.h"

namespace st {

namespace {


// ---------------------------------------------------------------------------
// naive kernel
// ---------------------------------------------------------------------------
template <int S, int R, int SHAPE>
__global__ __launch_bounds__(256) void sweep_naive(SweepArgs a) {
    using F = Fmt<S>;
    using T = typename F::T;
    const int64_t n = a.rows * a.cols;
    const T* src = static_cast<const T*>(a.src);
    auto at = [&](int64_t y, int64_t x) -> float {
        return (y < 0 || y >= a.rows || x < 0 || x >= a.cols) ? a.b : F::ld(src[y * a.cols + x]);
    };
    constexpr int K = 2 * R + 1;
    // grid-stride: the grid is capped on the host, so any cell count fits one launch
    for (int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x; idx < n; idx += int64_t(gridDim.x) * 256) {
        const int64_t i = idx / a.cols, j = idx - i * a.cols;
        float acc = a.w[R * K + R] * at(i, j);
#pragma unroll
        for (int dy = -R; dy <= R; ++dy)
#pragma unroll
            for (int dx = -R; dx <= R; ++dx) {
                if ((dy == 0 && dx == 0) || !tap_in(SHAPE, dy, dx)) continue;
                acc = __builtin_fmaf(a.w[(dy + R) * K + dx + R], at(i + dy, j + dx), acc);
            }
        static_cast<T*>(a.dst)[idx] = F::st(acc);
    }
}

// ---------------------------------------------------------------------------
// one step on LDS tiles
// ---------------------------------------------------------------------------
// A workgroup stages its 128 x 64 tile and an R-deep halo into LDS, 16-byte chunks (whole ones: tiled_step),
// all in flight before the first is written, and each thread computes 4 columns x 8 rows from a register
// ring of input rows, three 16-byte LDS reads per row.  Stars are bound by HBM (16384 x 8192 FP32, r = 1:
// 195 us, 5.5 TB/s), the largest boxes by FP32 issue (r = 4 at 16384 x 8192: 328 us, 66 TFLOP/s).
constexpr int STX = 128, STY = 64, SRS = 8;
template <int S, int R>
struct StepGeo {
    static constexpr int VEC = Fmt<S>::VEC;
    static constexpr int OFF = 8;  // buffer column of the tile's first
    static constexpr int LO = (OFF - R) / VEC * VEC, HI = (OFF + STX + R + VEC - 1) / VEC * VEC;  // staged columns
    static constexpr int BW = (OFF + STX + 8 + 7) / 8 * 8, BH = STY + 2 * R, NCH = (HI - LO) / VEC, TOTAL = BH * NCH;
    static constexpr int PER = (TOTAL + NT - 1) / NT;  // chunks per thread
};
template <int S, int R, int SHAPE>
__global__ __launch_bounds__(NT) void sweep_step(SweepArgs a) {
    using F = Fmt<S>;
    using T = typename F::T;
    using G = StepGeo<S, R>;
    constexpr int K = 2 * R + 1;
    __shared__ float4 buf4[G::BH * G::BW / 4];
    __shared__ float wsh[K * K];
    float* buf = reinterpret_cast<float*>(buf4);
    if (a.stop && __hip_atomic_load(a.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int64_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t y0 = t / a.tiles_x * STY, x0 = t % a.tiles_x * STX;
    const T* src = static_cast<const T*>(a.src);
    T* dst = static_cast<T*>(a.dst);
    // (weights reach vector registers through LDS: 81 of them do not fit the scalar registers)
    if (threadIdx.x < K * K) wsh[threadIdx.x] = a.w[threadIdx.x];
    uint4 raw[G::PER];
    bool in[G::PER];
#pragma unroll
    for (int u = 0; u < G::PER; ++u) {
        const int k = int(threadIdx.x) + u * NT;
        const int64_t gy = y0 - R + k / G::NCH, gx = x0 - G::OFF + G::LO + k % G::NCH * G::VEC;
        in[u] = k < G::TOTAL && gy >= 0 && gy < a.rows && gx >= 0 && gx < a.cols;
        if (in[u]) raw[u] = *reinterpret_cast<const uint4*>(src + gy * a.cols + gx);
    }
#pragma unroll
    for (int u = 0; u < G::PER; ++u) {
        const int k = int(threadIdx.x) + u * NT;
        if (k >= G::TOTAL) break;
        float v[G::VEC];
        if (in[u]) {
            widen_chunk<S>(raw[u], v);
        } else {
#pragma unroll
            for (int e = 0; e < G::VEC; ++e) v[e] = a.b;
        }
        float4* p = reinterpret_cast<float4*>(buf + k / G::NCH * G::BW + G::LO + k % G::NCH * G::VEC);
#pragma unroll
        for (int e = 0; e < G::VEC; e += 4) p[e / 4] = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
    }
    __syncthreads();
    float wreg[K * K];
#pragma unroll
    for (int q = 0; q < K * K; ++q) wreg[q] = wsh[q];
    static_assert(STX / 4 * (STY / SRS) == NT, "a block of cells per thread");
    const int seg = int(threadIdx.x) / (STX / 4), c4 = 4 * (int(threadIdx.x) % (STX / 4));
    const float* rows = buf + seg * SRS * G::BW + G::OFF + c4 - 4;
    const int64_t gx = x0 + c4;
    float v[SRS + 2 * R][12];
#pragma unroll
    for (int j = 0; j < SRS + 2 * R; ++j) {
        const float4* p = reinterpret_cast<const float4*>(rows + j * G::BW);
        const float4 q0 = p[0], q1 = p[1], q2 = p[2];
        v[j][0] = q0.x; v[j][1] = q0.y; v[j][2] = q0.z; v[j][3] = q0.w;
        v[j][4] = q1.x; v[j][5] = q1.y; v[j][6] = q1.z; v[j][7] = q1.w;
        v[j][8] = q2.x; v[j][9] = q2.y; v[j][10] = q2.z; v[j][11] = q2.w;
        if (j < 2 * R) continue;
        const int k = j - 2 * R;  // the output row that this input row completes
        float o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = wreg[R * K + R] * v[k + R][4 + c];
#pragma unroll
        for (int dy = -R; dy <= R; ++dy)
#pragma unroll
            for (int dx = -R; dx <= R; ++dx) {
                if ((dy == 0 && dx == 0) || !tap_in(SHAPE, dy, dx)) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c) o[c] = __builtin_fmaf(wreg[(dy + R) * K + dx + R], v[k + R + dy][4 + c + dx], o[c]);
            }
        const int64_t gy = y0 + seg * SRS + k;
        if (gy < a.rows && gx < a.cols) store4<S>(dst + gy * a.cols + gx, o);
    }
}

// ---------------------------------------------------------------------------
// persistent streaming kernel (FP32, cols % 4 == 0): LDS-DMA double buffering
// ---------------------------------------------------------------------------
// Each workgroup loops over tiles (stride = grid size).  While it computes tile i from one LDS
// staging buffer, the hardware copies tile i+1 into the other with global_load_lds_dwordx4 (no
// registers involved), so the load of the next tile hides behind the arithmetic of this one.
// Staging layout is dense: buffer column 0 holds global column x0 - A, every staged row is
// exactly BW = 4 * NCH floats, so 64 consecutive 16-byte chunks of one DMA instruction land
// contiguously, lane by lane.  Chunks that fall outside the grid are fetched from a clamped
// in-bounds address and then overwritten with b by the lane that fetched them.
struct SGeo {
    int H, A, bw, bh, nch, total;
};

__host__ __device__ inline SGeo sgeometry(int R, int tb, int TX, int TY) {
    SGeo g;
    g.H = R * tb;
    g.A = ((g.H + 3) & ~3) + 8;
    g.bw = (g.A + TX + g.H + 8 + 3) & ~3;
    g.bh = TY + 2 * g.H;
    g.nch = g.bw / 4;
    g.total = g.bh * g.nch;
    return g;
}

__host__ __device__ inline size_t stream_lds_bytes(int R, int tb, int TX, int TY) {
    SGeo g = sgeometry(R, tb, TX, TY);
    return (size_t(tb > 1 ? 3 : 2) * size_t(g.bw) * size_t(g.bh) + MAXK) * sizeof(float);
}

// Issue (or, with FIX, repair) this lane's share of the DMA of one tile into `buf`.
template <bool FIX>
__device__ __forceinline__ void stream_stage(const float* src, int64_t rows, int64_t cols, float b, const SGeo& g,
                                             int64_t y0, int64_t x0, float* buf) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int k = 64 * wave + lane;
    int row = k / g.nch, cc = k - row * g.nch;
    const int dq = NT / g.nch, dr = NT % g.nch;
    for (int j = 0; j * NT < g.total; ++j, k += NT) {
        if (k < g.total) {
            const int64_t gy = y0 - g.H + row, gx = x0 - g.A + 4 * cc;
            const bool in = gy >= 0 && gy < rows && gx >= 0 && gx + 4 <= cols;
            if (FIX) {
                if (!in) reinterpret_cast<float4*>(buf)[k] = make_float4(b, b, b, b);
            } else {
                const float* gp = in ? src + gy * cols + gx : src;
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void*)(gp),
                    (__attribute__((address_space(3))) void*)(buf + 4 * (j * NT + 64 * wave)), 16, 0,
                    0);
            }
        }
        row += dq;
        cc += dr;
        if (cc >= g.nch) {
            cc -= g.nch;
            ++row;
        }
    }
}

template <int R, int SHAPE, int TX, int TY, int RS>
__global__ __launch_bounds__(NT) void sweep_stream(SweepArgs a) {
    constexpr int K = 2 * R + 1;
    extern __shared__ float4 lds4[];
    float* lds = reinterpret_cast<float*>(lds4);
    const int tb = a.tb;
    const SGeo g = sgeometry(R, tb, TX, TY);
    const int H = g.H, A = g.A, BW = g.bw, BH = g.bh;
    // Buffers are picked by offset arithmetic on the LDS base (an array of pointers would make the
    // compiler lose the LDS address space and fall back to flat loads).
    float* mid = lds + 2 * BH * BW;
    float* wsh = mid + (tb > 1 ? BH * BW : 0);
    const int64_t rows = a.rows, cols = a.cols;
    const float b = a.b;
    const float* src = static_cast<const float*>(a.src);
    float* dst = static_cast<float*>(a.dst);
    const int64_t ntiles = a.tiles_x * a.tiles_y;
    if (threadIdx.x < K * K) wsh[threadIdx.x] = a.w[threadIdx.x];

    int64_t t = blockIdx.x;
    if (t < ntiles) {
        const int64_t m = xcd_tile(t, ntiles);
        stream_stage<false>(src, rows, cols, b, g, (m / a.tiles_x) * TY, (m % a.tiles_x) * TX, lds);
    }
    float wreg[K * K];
    for (int it = 0; t < ntiles; ++it, t += gridDim.x) {
        const int64_t m = xcd_tile(t, ntiles);
        const int64_t y0 = (m / a.tiles_x) * TY, x0 = (m % a.tiles_x) * TX;
        float* cur = lds + (it & 1) * (BH * BW);
        // Every wave waits for its own DMA of the current tile; the barrier then orders all of
        // them before the out-of-grid repair (same chunks) and the repair before any read.
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        stream_stage<true>(src, rows, cols, b, g, y0, x0, cur);
        __syncthreads();
        if (it == 0) {
#pragma unroll
            for (int q = 0; q < K * K; ++q) wreg[q] = wsh[q];
        }
        const int64_t tn = t + gridDim.x;
        if (tn < ntiles) {
            const int64_t mn = xcd_tile(tn, ntiles);
            stream_stage<false>(src, rows, cols, b, g, (mn / a.tiles_x) * TY, (mn % a.tiles_x) * TX,
                                lds + ((it + 1) & 1) * (BH * BW));
        }
        const float* sb = cur;
        for (int l = 1; l <= tb; ++l) {
            const int E = R * (tb - l);
            const bool last = (l == tb);
            float* db = (l & 1) ? mid : cur;
            const int g0 = (A - E) & ~3;
            const int g1 = (A + TX + E + 3) & ~3;
            const int ngx = (g1 - g0) >> 2;
            const int HL = TY + 2 * E;
            const int nseg = (HL + RS - 1) / RS;
            const int nitems = ngx * nseg;
            for (int item = threadIdx.x; item < nitems; item += NT) {
                const int seg = item / ngx;
                const int bc = g0 + 4 * (item - seg * ngx);
                const int r0 = H - E + seg * RS;
                const int nr = min(RS, HL - seg * RS);
                const int64_t gx0 = x0 - A + bc;
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
                    if (kr >= nr) continue;
                    const int brow = r0 + kr;
                    const int64_t gy = y0 - H + brow;
                    if (last) {
                        if (gy >= rows) continue;
                        if (gx0 + 4 <= cols) {
                            *reinterpret_cast<float4*>(dst + gy * cols + gx0) = make_float4(o[0], o[1], o[2], o[3]);
                        } else {
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                if (gx0 + c < cols) dst[gy * cols + gx0 + c] = o[c];
                        }
                    } else {
                        const bool row_in = gy >= 0 && gy < rows;
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const int64_t gx = gx0 + c;
                            o[c] = (row_in && gx >= 0 && gx < cols) ? o[c] : b;
                        }
                        *reinterpret_cast<float4*>(db + brow * BW + bc) = make_float4(o[0], o[1], o[2], o[3]);
                    }
                }
            }
            __syncthreads();
            sb = db;
        }
    }
}

// ---------------------------------------------------------------------------
// dispatch tables
// ---------------------------------------------------------------------------
struct TileDef {
    int tx, ty;
};
constexpr TileDef kTiles[] = {{64, 64}, {128, 32}, {128, 64}, {256, 32}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

using KernelFn = void (*)(SweepArgs);

template <int S, int R, int SH>
BlockFn block_fn(int def) {
    switch (def) {
        case 0: return sweep_block<S, R, SH, 1, 8, 8>;
        case 1: return sweep_block<S, R, SH, 2, 4, 8>;
        case 2: return sweep_block<S, R, SH, 2, 8, 8>;
        case 3: return sweep_block<S, R, SH, 4, 4, 8>;
        case 4: return sweep_block<S, R, SH, 2, 8, 16>;
    }
    return nullptr;
}

template <int S, int SH>
BlockFn block_fn_r(int r, int def) {
    switch (r) {
        case 1: return block_fn<S, 1, SH>(def);
        case 2: return block_fn<S, 2, SH>(def);
        case 3: return block_fn<S, 3, SH>(def);
        case 4: return block_fn<S, 4, SH>(def);
    }
    return nullptr;
}

BlockFn block_lookup(int storage, int shape, int r, int def) {
    if (storage == ST_F32)
        return shape == SHAPE_BOX ? block_fn_r<ST_F32, SHAPE_BOX>(r, def) : block_fn_r<ST_F32, SHAPE_STAR>(r, def);
    if (storage == ST_BF16)
        return shape == SHAPE_BOX ? block_fn_r<ST_BF16, SHAPE_BOX>(r, def) : block_fn_r<ST_BF16, SHAPE_STAR>(r, def);
    if (storage == ST_F16)
        return shape == SHAPE_BOX ? block_fn_r<ST_F16, SHAPE_BOX>(r, def) : block_fn_r<ST_F16, SHAPE_STAR>(r, def);
    return nullptr;
}

// Operations of a cell and level.
double cell_ops(const st_plan* p) {
    const int k = 2 * p->radius + 1;
    return p->kind == KIND_VARCOEF ? VARCOEF_OPS : p->shape == SHAPE_BOX ? k * k + 1 : 2 * k;
}

// The register tiles of a pass.  One that sums keeps to the plan's tile as far as that goes: with the cells
// before the last level in registers too the tallest tile, which others pick, spills (star r = 1 at 2048^2, 20
// steps a check as 16 + 4 levels on 256 x 32 tiles 56 us, as 10 + 10 on picked ones 60).
block::Cover plan_cover(const st_plan* p, int levels, bool sums) {
    if (sums) return block::cover(tile_index(p->tile_x, p->tile_y), p->radius, levels, p->rows, p->cols);
    return block::pick(tile_index(p->tile_x, p->tile_y), cell_ops(p), p->radius, levels, p->rows, p->cols);
}

// A pass on register tiles; with `sums` its last level's sums per tile (sweep_block_sums), `tiles` of them.
int launch_block(const st_plan* p, const void* src, void* dst, int levels, double* sums, int64_t* tiles, hipStream_t s) {
    const block::Cover c = plan_cover(p, levels, sums);
    if (c.def < 0) return fail(ST_EUNSUPPORTED, "temporal block too deep for the tile");
    if (c.tiles >= int64_t(1) << 31) return fail(ST_EUNSUPPORTED, "too many tiles for one launch");
    const block::Def& d = block::kDefs[c.def];
    BlockFn fn = sums ? sums_lookup(p->storage, p->shape, p->radius, c.def) : block_lookup(p->storage, p->shape, p->radius, c.def);
    if (!fn) return fail(ST_EUNSUPPORTED, "no tiled kernel for this storage/shape/radius/tile");
    const size_t lds = block::lds_floats(p->radius, d.v, d.rw, d.nw) * sizeof(float);
    if (int rc = prepare_lds(reinterpret_cast<const void*>(fn), lds)) return rc;
    BlockArgs a;
    a.src = src;
    a.dst = dst;
    a.rows = p->rows;
    a.cols = p->cols;
    a.tiles_x = c.tiles_x;
    a.stop = p->stop;
    a.b = p->bq;
    a.tb = levels;
    a.sums = sums;
    std::memcpy(a.w, p->w, sizeof(a.w));
    clear_stale_error();
    launch_runs(c.tiles, 64 * d.nw, [&](int64_t first, int64_t n) {
        a.first = first;
        hipLaunchKernelGGL(fn, dim3(unsigned(n)), dim3(64 * d.nw), lds, s, a);
    });
    ST_LAUNCH_CHECK("sweep_block");
    if (tiles) *tiles = c.tiles;
    return ST_OK;
}

template <int S, int SH>
KernelFn step_fn_r(int r) {
    switch (r) {
        case 1: return sweep_step<S, 1, SH>;
        case 2: return sweep_step<S, 2, SH>;
        case 3: return sweep_step<S, 3, SH>;
        case 4: return sweep_step<S, 4, SH>;
    }
    return nullptr;
}

KernelFn step_lookup(int storage, int shape, int r) {
    if (storage == ST_F32) return shape == SHAPE_BOX ? step_fn_r<ST_F32, SHAPE_BOX>(r) : step_fn_r<ST_F32, SHAPE_STAR>(r);
    if (storage == ST_BF16) return shape == SHAPE_BOX ? step_fn_r<ST_BF16, SHAPE_BOX>(r) : step_fn_r<ST_BF16, SHAPE_STAR>(r);
    if (storage == ST_F16) return shape == SHAPE_BOX ? step_fn_r<ST_F16, SHAPE_BOX>(r) : step_fn_r<ST_F16, SHAPE_STAR>(r);
    return nullptr;
}

template <int S, int SH>
KernelFn naive_fn_r(int r) {
    switch (r) {
        case 1: return sweep_naive<S, 1, SH>;
        case 2: return sweep_naive<S, 2, SH>;
        case 3: return sweep_naive<S, 3, SH>;
        case 4: return sweep_naive<S, 4, SH>;
    }
    return nullptr;
}

template <int SH>
KernelFn stream_fn_r(int r, int tile) {
#define ST_STREAM_TILES(R)                                  \
    switch (tile) {                                         \
        case 0: return sweep_stream<R, SH, 64, 64, 4>;      \
        case 1: return sweep_stream<R, SH, 128, 32, 4>;     \
        case 2: return sweep_stream<R, SH, 128, 64, 8>;     \
        case 3: return sweep_stream<R, SH, 256, 32, 8>;     \
    }                                                       \
    return nullptr;
    switch (r) {
        case 1: ST_STREAM_TILES(1)
        case 2: ST_STREAM_TILES(2)
        case 3: ST_STREAM_TILES(3)
        case 4: ST_STREAM_TILES(4)
    }
#undef ST_STREAM_TILES
    return nullptr;
}

KernelFn stream_lookup(int shape, int r, int tile) {
    return shape == SHAPE_BOX ? stream_fn_r<SHAPE_BOX>(r, tile) : stream_fn_r<SHAPE_STAR>(r, tile);
}

KernelFn naive_lookup(int storage, int shape, int r) {
    if (storage == ST_F32) return shape == SHAPE_BOX ? naive_fn_r<ST_F32, SHAPE_BOX>(r) : naive_fn_r<ST_F32, SHAPE_STAR>(r);
    if (storage == ST_BF16) return shape == SHAPE_BOX ? naive_fn_r<ST_BF16, SHAPE_BOX>(r) : naive_fn_r<ST_BF16, SHAPE_STAR>(r);
    if (storage == ST_F16) return shape == SHAPE_BOX ? naive_fn_r<ST_F16, SHAPE_BOX>(r) : naive_fn_r<ST_F16, SHAPE_STAR>(r);
    return nullptr;
}

void fill_args(const st_plan* p, const void* src, void* dst, const float* kappa, SweepArgs& a) {
    a.src = src;
    a.dst = dst;
    a.kappa = kappa;
    a.rows = p->rows;
    a.cols = p->cols;
    a.b = p->bq;
    a.stop = p->stop;
    std::memcpy(a.w, p->w, sizeof(a.w));
}

int launch_step(const st_plan* p, const void* src, void* dst, hipStream_t s) {
    SweepArgs a;
    fill_args(p, src, dst, nullptr, a);
    a.tiles_x = (p->cols + STX - 1) / STX;
    a.tiles_y = (p->rows + STY - 1) / STY;
    clear_stale_error();
    hipLaunchKernelGGL(step_lookup(p->storage, p->shape, p->radius), dim3(unsigned(a.tiles_x * a.tiles_y)), dim3(NT), 0, s, a);
    ST_LAUNCH_CHECK("sweep_step");
    return ST_OK;
}

}  // namespace

int tile_index(int tx, int ty) {
    for (int i = 0; i < kNumTiles; ++i)
        if (kTiles[i].tx == tx && kTiles[i].ty == ty) return i;
    return -1;
}

bool tile_supported(int shape, int radius, int tx, int ty) {
    (void)shape;
    (void)radius;
    return tile_index(tx, ty) >= 0;
}

int supported_tiles(int* xy, int cap) {
    for (int i = 0; i < kNumTiles && i < cap; ++i) {
        xy[2 * i] = kTiles[i].tx;
        xy[2 * i + 1] = kTiles[i].ty;
    }
    return kNumTiles;
}

bool tile_replaced(const st_plan* p, int levels) {
    const int def = tile_index(p->tile_x, p->tile_y);
    return block::cover(def, p->radius, levels, p->rows, p->cols).def == def &&
           block::pick(def, cell_ops(p), p->radius, levels, p->rows, p->cols).def != def;
}

// The depths that a tiled plan accepts per tile: as many levels as two LDS buffers of the tile and the halo
// around it (16-byte chunks) would hold.  No kernel keeps them: register tiles hold any r tb up to 39 on one
// tile or another, but the limit decides which calls are refused, and stays what it was.
static size_t accepted_lds_bytes(int r, int tb, int tx, int ty) {
    const int h = r * tb, off = (h + 4 + 7) / 8 * 8, bw = (off + tx + h + 7 + 7) / 8 * 8;
    return (size_t(tb > 1 ? 2 : 1) * size_t(bw) * size_t(ty + 2 * h) + MAXK) * sizeof(float);
}

int max_tb(const st_plan* p, int tx, int ty) {
    int tb = 1;
    if (is_march(p->variant)) return march_max_tb(p->shape, p->radius, march_vmax(p->variant));
    if (p->variant == VARIANT_RESIDENT) return std::max(1, std::min(64, resident_max_tb(p)));
    if (p->variant == VARIANT_MFMA) return 1;
    if (p->variant == VARIANT_STREAM) {
        while (tb < 16 && stream_lds_bytes(p->radius, tb + 1, tx, ty) <= lds_limit()) ++tb;
    } else {
        while (tb < 16 && accepted_lds_bytes(p->radius, tb + 1, tx, ty) <= lds_limit()) ++tb;
    }
    return tb;
}

bool stream_usable(const st_plan* p) { return p->storage == ST_F32 && p->cols % 4 == 0; }

int launch_naive(const st_plan* p, const void* src, void* dst, const float* kappa, hipStream_t s) {
    KernelFn fn = naive_lookup(p->storage, p->shape, p->radius);
    if (!fn) return fail(ST_EUNSUPPORTED, "no naive kernel for this storage/shape/radius");
    SweepArgs a;
    fill_args(p, src, dst, kappa, a);
    a.tb = 1;
    a.tiles_x = a.tiles_y = 0;
    const int64_t n = p->rows * p->cols;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, kNaiveMaxBlocks);
    clear_stale_error();
    hipLaunchKernelGGL(fn, dim3(unsigned(blocks)), dim3(256), 0, s, a);
    ST_LAUNCH_CHECK("sweep_naive");
    return ST_OK;
}

// Passes of the tiled variant that the row-marching kernels run faster (columns per lane; 0: register
// tiles).  Marching recomputes a few rows per segment instead of a margin around every tile, but needs a
// grid that gives each wavefront the device holds a segment much longer than its warm-up.  Measured side
// after side (GStencil/s, register tiles / marching): star r = 2 at tb 6, 2048^2 1000 / 1071, 3000^2
// 1450 / 1573, 4096^2 1588 / 2201; box r = 1 at tb 6, 2000 x 3000 1550 / 1310, 4096^2 1802 / 2155.  Boxes
// of r >= 3 hold few rows in flight either way, and one-column marching wins from 1.5 10^6 cells on (box
// r = 3 at tb 2, 1000^2 168 / 153, 1448^2 218 / 251, 4096^2 424 / 491; at 16384^2 eight columns reach 720).
// Eight columns (four at widths that are no multiple of eight) pay where their bands hold grid in at least
// 0.62 of their lanes (4 10^7 cells of box r = 3, 12 steps at tb 2, ms, eight columns / one column: 1200 wide
// 0.95 / 1.20, 1000 wide 1.17 / 1.18, 520 wide 1.40 / 1.13, 64 wide 5.3 / 1.8), and on grids narrower than a tile register tiles beat a band of
// 256 columns where they hold most of their rows (10^7 cells, 100 wide: star r = 2 118 / 85, box r = 1 124 / 88,
// but star r = 1 70 / 59 to 219 / 222 and star r = 3 177 / 170, at 40 wide 327 / 401; star r = 2 at two levels
// 39 / 48).
int tiled_march_columns(const st_plan* p, int levels) {
    if (p->kind != KIND_CONST || p->bc != ST_BC_CONST) return 0;
    const int64_t cells = p->rows * p->cols;
    const bool big_box = p->shape == SHAPE_BOX && p->radius >= 3;
    if (cells < (big_box ? 1500000 : 8000000)) return 0;
    if (levels >= 4 && p->cols < 128 && ((p->shape == SHAPE_STAR && p->radius == 2) || (p->shape == SHAPE_BOX && p->radius == 1))) return 0;
    int vmax = 4;
    if (big_box) {
        const int V = p->cols % 8 ? 4 : 8;  // (launch_march: rows of whole vectors of eight)
        const int64_t bands = march::band_count(p->cols, V, march::halo_lanes(p->radius, levels, V), false);
        vmax = cells >= int64_t(1) << 25 && double(p->cols) >= 0.62 * double(bands * 64 * V) ? 8 : 1;
    }
    return vmax && levels <= march_max_tb(p->shape, p->radius, vmax) ? vmax : 0;
}

// Passes of one level of the tiled variant that run on LDS tiles: no step is saved, so a register tile's
// margins and a marching wavefront's warm-up only cost.  Rows and buffers must be whole 16-byte chunks.  us a
// step, LDS tiles / what runs otherwise: star r = 1 FP32 512^2 4.7 / 4.9, 16384 x 8192 195 / 240; star r = 4
// BF16 2000 x 3000 8.2 / 13.5; box r = 2 BF16 2000 x 3000 9.5 / 15.6; box r = 4 FP32 1024^2 9.1 / 11.7, 4096^2
// 42 / 55, BF16 40 / 59.  The marching kernels keep what they run faster: 16-bit stars and boxes of r = 1 of some
// sizes (star r = 1 3000 x 4000 11.7 / 9.9, r = 3 8192^2 55 / 50, r = 4 8192^2 55 / 51, box r = 1 4096^2
// 15.8 / 14.5), box r = 3 in FP32 (4096^2 34 / 32), and large boxes narrower than a tile (250000 x 40, r = 4
// 74 / 47).
bool tiled_step(const st_plan* p, const void* src, const void* dst) {
    if (p->kind != KIND_CONST || p->bc != ST_BC_CONST || p->variant != VARIANT_TILED) return false;
    const bool f32 = p->storage == ST_F32, box = p->shape == SHAPE_BOX;
    if (p->cols % (f32 ? 4 : 8) || reinterpret_cast<uintptr_t>(src) % 16 || reinterpret_cast<uintptr_t>(dst) % 16) return false;
    const int64_t cells = p->rows * p->cols;
    const int64_t tiles = (p->cols + STX - 1) / STX * ((p->rows + STY - 1) / STY);
    if (tiles >= int64_t(1) << 24) return false;  // threads of a launch
    const bool big = box && p->radius == 4;
    if (tiles < 256 && (p->tile_x != STX || p->tile_y != STY))  // a small grid: the plan's tile spreads it
        return big && p->tile_x * p->tile_y == STX * STY;
    if (big) return p->cols >= STX || cells < 1500000;
    const int V = tiled_march_columns(p, 1);
    if (!V) return true;  // (register tiles were never faster)
    // lanes that hold grid: 60000 x 200 (0.78 of either) box r = 3 FP32 32 / 28, 100000 x 256 (1.0 of the tiles,
    // 0.5 of the bands) box r = 1 BF16 21 / 28
    const double fill = double(cells) / double(tiles * STX * STY);
    const double bands = double(march::band_count(p->cols, V, march::halo_lanes(p->radius, 1, V), false));
    const double march_fill = double(p->cols) / (bands * 64 * V);
    if (fill < 0.8) return fill > 1.2 * march_fill && !(box && p->radius == 3);
    if (p->cols < 512) return true;
    if (box && p->radius == 3 && f32) return cells < 6000000 || cells >= int64_t(1) << 25;
    if (f32 || box) return f32 || p->radius != 1 || cells >= 100000000;
    const int64_t from[] = {8000000, 0, 8000000, 60000000}, to[] = {20000000, 0, 100000000, 100000000};
    return cells < from[p->radius - 1] || cells >= to[p->radius - 1];
}

// Boxes whose arithmetic hides the HBM trip of every step, where the tiles of a step are whole and share out
// evenly among the compute units.  us a step, single / two at a time: r = 4 1000 x 2000 FP32 (256 tiles) 9.8 /
// 13, 4096^2 42 / 60, but 5000 x 400 (316 tiles) 16 / 13; r = 3 in 16 bits 4096^2 29 / 38, but 666 x 3000 (264
// tiles) 10.4 / 9.2; FP32 r = 3 only on grids that marching bands fit worse: 15625 x 128 8.7 / 10.6, 6000 x 8192
// 93 / 78.  Grids of few tiles wait for launches: 300^2, r = 4, two at a time 53 / 49 for six steps.
bool single_steps(const st_plan* p) {
    if (p->shape != SHAPE_BOX || p->radius < 3) return false;
    const int64_t cells = p->rows * p->cols, tiles = (p->cols + STX - 1) / STX * ((p->rows + STY - 1) / STY);
    if (cells < 1500000) return false;
    const double fill = double(cells) / double((tiles + 255) / 256 * 256 * STX * STY);
    if (p->radius == 4 || p->storage != ST_F32) return fill >= 0.75;
    const double bands = double(march::band_count(p->cols, 1, march::halo_lanes(3, 2, 1), false));
    return cells < 6000000 && fill >= 1.2 * double(p->cols) / (bands * 64);
}

int launch_pass(const st_plan* p, const void* src, void* dst, const float* kappa, int levels, hipStream_t s) {
    if (p->flags & ST_FLAG_NAIVE) {
        // the reference path: one launch per step through the workspace is handled by the caller
        return fail(ST_EUNSUPPORTED, "launch_pass called on a naive plan");
    }
    const int ti = tile_index(p->tile_x, p->tile_y);
    if (p->variant == VARIANT_MFMA && levels == 1 && mfma_usable(p)) return launch_mfma(p, src, dst, s);
    if (is_march(p->variant) && march_usable(p) &&
        levels <= march_max_tb(p->shape, p->radius, march_vmax(p->variant)))
        return launch_march(p, src, dst, levels, march_vmax(p->variant), s);
    const bool aligned = (reinterpret_cast<uintptr_t>(src) % 16) == 0 && (reinterpret_cast<uintptr_t>(dst) % 16) == 0;
    if (p->variant == VARIANT_STREAM && stream_usable(p) && aligned) {
        KernelFn fn = stream_lookup(p->shape, p->radius, ti);
        if (!fn) return fail(ST_EUNSUPPORTED, "no streaming kernel for this shape/radius/tile");
        const size_t lds = stream_lds_bytes(p->radius, levels, p->tile_x, p->tile_y);
        if (int rc = prepare_lds(reinterpret_cast<const void*>(fn), lds)) return rc;
        SweepArgs a;
        fill_args(p, src, dst, kappa, a);
        a.tb = levels;
        a.tiles_x = (p->cols + p->tile_x - 1) / p->tile_x;
        a.tiles_y = (p->rows + p->tile_y - 1) / p->tile_y;
        const int64_t ntiles = a.tiles_x * a.tiles_y;
        int blocks = 0;
        if (int rc = resident_blocks(reinterpret_cast<const void*>(fn), lds, &blocks)) return rc;
        clear_stale_error();
        hipLaunchKernelGGL(fn, dim3(unsigned(std::min<int64_t>(ntiles, blocks))), dim3(NT), lds, s, a);
        ST_LAUNCH_CHECK("sweep_stream");
        return ST_OK;
    }
    if (levels == 1 && tiled_step(p, src, dst)) return launch_step(p, src, dst, s);
    if (p->variant == VARIANT_TILED)
        if (const int vmax = tiled_march_columns(p, levels)) return launch_march(p, src, dst, levels, vmax, s);
    return launch_block(p, src, dst, levels, nullptr, nullptr, s);
}

int64_t sums_tiles(const st_plan* p, int levels) {
    if (p->kind != KIND_CONST || p->bc != ST_BC_CONST) return 0;
    const block::Cover c = plan_cover(p, levels, true);
    return c.def < 0 || c.tiles >= int64_t(1) << 31 ? 0 : c.tiles;
}

double block_work(const st_plan* p, int levels) {
    const block::Cover c = plan_cover(p, levels, true);
    if (c.def < 0) return HUGE_VAL;
    const block::Def& d = block::kDefs[c.def];
    return double(c.tiles) * (64 * d.v * d.rw * d.nw) * levels;
}

int launch_sums(const st_plan* p, const void* src, void* dst, int levels, double* sums, int64_t* tiles, hipStream_t s) {
    return launch_block(p, src, dst, levels, sums, tiles, s);
}

}  // namespace st

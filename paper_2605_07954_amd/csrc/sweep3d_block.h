// 3D star passes with temporal blocking: register tiles (block_body.h) that march along z.
//
// A workgroup owns NW RW rows x 64 V columns of the (y, x) plane and walks up the planes of a z segment
// with T levels in flight: iteration t takes input plane t and advances level l (1 .. T) by one plane,
// t - R l.  Each level keeps the 2R + 1 planes it reads in registers; the ring slots become fixed
// registers because the plane loop is unrolled over the ring length (a level's newest plane t - R l
// sits in slot (u - R l) mod (2R + 1), u = t mod (2R + 1)).  A star reads its (y, x) neighbours on the
// centre plane only, and that plane was complete an iteration ago, so all levels publish the outer rows
// of their centre planes into LDS first and one barrier serves the whole iteration.  The next input
// plane is loaded, raw, while this one computes.  The pass stores the tile without its outer R T rows
// and columns; a segment recomputes R T planes at either end.
//
// One level per pass is bound by HBM (8 bytes per update; LDS tiles of whole cache lines reach 4.4 TB/s,
// 560 GStencil/s for the 7-point star at 512^3, and run single levels of large FP32 stars); T levels divide
// the bytes by T.  Measured there at T = 1 .. 7: 424, 900, 1216, 1468, 1590, 1646, 1331 GStencil/s -- at
// T = 1 4.4 TB/s (64 columns that start inside a cache line read three lines for two and write parts of lines:
// 1.45 GB for 1.05), at T = 5 4.1 TB/s and vector issue on 0.61 of the cycles; the work grows with the tile's
// margin (64 x 64 cells for (64 - 2T)^2), and T = 7 spills registers.  Sixteen wavefronts of four rows beat eight of eight (1193 at T = 3) and 128-column tiles
// (997), which leave fewer wavefronts to a SIMD.
#pragma once

#include "block_body.h"

namespace st {

struct Args3B {
    const void* src;
    void* dst;
    int64_t planes, rows, cols;
    int64_t tiles_x, tiles, zseg;  // tiles of a plane; planes per segment
    int64_t first;                 // the first (segment, tile) of this launch
    float b;
    float wc;                                     // the centre weight
    float wz[2 * ST_MAX_RADIUS_3D], wy[2 * ST_MAX_RADIUS_3D], wx[2 * ST_MAX_RADIUS_3D];  // offsets -R .. -1, 1 .. R
};

struct Args3X {
    const void* src;
    void* dst;
    int64_t planes, rows, cols;
    int64_t tiles_x, tiles, zseg, first;
    float b;
    float w[MAXK3];  // dense, row-major in (dz, dy, dx)
};

namespace block {

__host__ __device__ constexpr int mod(int a, int k) { return ((a % k) + k) % k; }

// A raw plane of a wavefront's rows as loaded (rows and columns clamped into the grid).
template <int S, int V, int RW>
struct RawPlane {
    typename VecOf<typename Fmt<S>::T, V>::type r[RW];
};

// What a wavefront needs of its place in the tile, and its accesses to the fields.
template <int S, int V, int RW, bool EDGE>
struct Place3 {
    using Tp = typename Fmt<S>::T;
    const void* src;
    void* dst;
    int64_t planes, rows, cols, plane, y0, x0;
    bool col_ok[V], all_cols;
    float b;

    __device__ __forceinline__ void fetch(int64_t z, RawPlane<S, V, RW>& p) const {
        const int64_t zz = z < 0 ? 0 : z >= planes ? planes - 1 : z;
#pragma unroll
        for (int k = 0; k < RW; ++k) {
            int64_t y = y0 + k;
            if (EDGE) y = y < 0 ? 0 : y >= rows ? rows - 1 : y;
            const Tp* row = static_cast<const Tp*>(src) + zz * plane + y * cols;
            if (all_cols) {
                p.r[k] = *(const __attribute__((address_space(1))) typename VecOf<Tp, V>::type*)(row + x0);
            } else {
#pragma unroll
                for (int c = 0; c < V; ++c) {
                    const int64_t x = x0 + c < 0 ? 0 : x0 + c >= cols ? cols - 1 : x0 + c;
                    const Tp q = *(const __attribute__((address_space(1))) Tp*)(row + x);
                    if constexpr (V == 1) p.r[k] = q;
                    else p.r[k][c] = q;
                }
            }
        }
    }
    __device__ __forceinline__ void widen(const RawPlane<S, V, RW>& p, float (*in)[V]) const {
#pragma unroll
        for (int k = 0; k < RW; ++k)
#pragma unroll
            for (int c = 0; c < V; ++c) {
                if constexpr (V == 1) in[k][c] = Fmt<S>::ld(p.r[k]);
                else in[k][c] = Fmt<S>::ld(p.r[k][c]);
            }
    }
    // Cells outside the grid hold b.  Selects, no branches: the levels of an iteration stay one block of
    // code whose LDS reads the compiler can move ahead.
    __device__ __forceinline__ void settle(float (*p)[V], int64_t z) const {
        if constexpr (EDGE) {
            const bool z_ok = z >= 0 && z < planes;
#pragma unroll
            for (int k = 0; k < RW; ++k) {
                const bool row_ok = z_ok && y0 + k >= 0 && y0 + k < rows;
#pragma unroll
                for (int c = 0; c < V; ++c) p[k][c] = row_ok && col_ok[c] ? p[k][c] : b;
            }
        }
    }
    // Rows [lo, hi) of the tile (this wavefront's first is `row0`) of plane z.
    __device__ __forceinline__ void store(const float (*o)[V], int64_t z, int row0, int lo, int hi) const {
#pragma unroll
        for (int k = 0; k < RW; ++k) {
            const int64_t y = y0 + k;
            if (row0 + k < lo || row0 + k >= hi || (EDGE && y >= rows)) continue;
            const int64_t off = z * plane + y * cols + x0;
            if (all_cols) {
                float q[V];
#pragma unroll
                for (int c = 0; c < V; ++c) q[c] = o[k][c];
                store_cells<S, V>(dst, off, q);
            } else {
#pragma unroll
                for (int c = 0; c < V; ++c)
                    if (col_ok[c]) {
                        const float one[1] = {o[k][c]};
                        store_cells<S, 1>(dst, off + c, one);
                    }
            }
        }
    }
};

template <int S, int V, int RW, bool EDGE, typename Args>
__device__ __forceinline__ Place3<S, V, RW, EDGE> place3(const Args& a, const TileAt& at, int wave, int lane) {
    Place3<S, V, RW, EDGE> p;
    p.src = a.src;
    p.dst = a.dst;
    p.planes = a.planes;
    p.rows = a.rows;
    p.cols = a.cols;
    p.plane = a.rows * a.cols;
    p.y0 = at.ty + wave * RW;
    p.x0 = at.tx + lane * V;
#pragma unroll
    for (int c = 0; c < V; ++c) p.col_ok[c] = !EDGE || (p.x0 + c >= 0 && p.x0 + c < a.cols);
    p.all_cols = !EDGE || (p.x0 >= 0 && p.x0 + V <= a.cols);
    p.b = a.b;
    return p;
}

template <int S, int R, int T, int V, int RW, int NW, bool EDGE>
__device__ __forceinline__ void march3d(const Args3B& a, const TileAt& at, int64_t z0, int64_t z1, float* lds) {
    constexpr int K = 2 * R + 1;
    const int lane = int(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const auto pl = place3<S, V, RW, EDGE>(a, at, wave, lane);
    float wx[2 * R];
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) wx[i] = a.wx[i];
    // ring[l]: the planes that level l + 1 reads
    float ring[T][K][RW][V];
#pragma unroll
    for (int l = 0; l < T; ++l)
#pragma unroll
        for (int s = 0; s < K; ++s)
#pragma unroll
            for (int k = 0; k < RW; ++k)
#pragma unroll
                for (int c = 0; c < V; ++c) ring[l][s][k][c] = 0.0f;
    constexpr size_t LVL = lds_floats(R, V, RW, NW) / 2;  // floats of one level's published rows
    const int HL = margin_cols(R, T, V) / V;
    const int64_t tend = z1 - 1 + R * T;
    RawPlane<S, V, RW> next;
    int64_t t = z0 - R * T;
    pl.fetch(t, next);
    int par = 0;
    for (;;) {
#pragma unroll
        for (int u = 0; u < K; ++u) {
            if (t > tend) return;
            // input plane t into its slot; the next one on its way (past the last: clamped, unused)
            pl.widen(next, ring[0][u]);
            pl.settle(ring[0][u], t);
            pl.fetch(t + 1, next);
            float* buf = lds + par * (T * LVL);
            par ^= 1;
#pragma unroll
            for (int l = 0; l < T; ++l) publish<R, V, RW>(buf + l * LVL, wave, lane, ring[l][mod(u - R * l - R, K)]);
            __syncthreads();
            float halo[T][2 * R][V];  // the centre planes' rows beyond the wavefront's own
#pragma unroll
            for (int l = 0; l < T; ++l)
#pragma unroll
                for (int k = 0; k < 2 * R; ++k) halo_row<R, V, RW, NW>(buf + l * LVL, wave, lane, k < R ? k - R : k - R + RW, halo[l][k]);
#pragma unroll
            for (int l = 0; l < T; ++l) {
                const int64_t z = t - R * (l + 1);  // the plane that level l + 1 completes
                const int ctr = mod(u - R * l - R, K);
                float x[RW + 2 * R][V];  // rows -R .. RW + R - 1 of the centre plane
#pragma unroll
                for (int k = 0; k < RW + 2 * R; ++k) {
#pragma unroll
                    for (int c = 0; c < V; ++c)
                        x[k][c] = k < R ? halo[l][k < R ? k : 0][c] : k >= R + RW ? halo[l][k >= R + RW ? k - RW : 0][c]
                                                                              : ring[l][ctr][k < R || k >= R + RW ? 0 : k - R][c];
                }
                float o[RW][V];
#pragma unroll
                for (int k = 0; k < RW; ++k) {
#pragma unroll
                    for (int c = 0; c < V; ++c) o[k][c] = a.wc * x[k + R][c];
#pragma unroll
                    for (int d = -R; d < 0; ++d)
#pragma unroll
                        for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(a.wz[d + R], ring[l][mod(ctr + d, K)][k][c], o[k][c]);
#pragma unroll
                    for (int d = -R; d < 0; ++d)
#pragma unroll
                        for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(a.wy[d + R], x[k + R + d][c], o[k][c]);
                }
                side_taps<R, V, RW>(o, x + R, wx);
#pragma unroll
                for (int k = 0; k < RW; ++k) {
#pragma unroll
                    for (int d = 1; d <= R; ++d)
#pragma unroll
                        for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(a.wy[d + R - 1], x[k + R + d][c], o[k][c]);
#pragma unroll
                    for (int d = 1; d <= R; ++d)
#pragma unroll
                        for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(a.wz[d + R - 1], ring[l][mod(ctr + d, K)][k][c], o[k][c]);
                }
                round_rows<S, V, RW>(o);
                if (l + 1 < T) {
                    pl.settle(o, z);
                    const int s = mod(u - R * (l + 1), K);
#pragma unroll
                    for (int k = 0; k < RW; ++k)
#pragma unroll
                        for (int c = 0; c < V; ++c) ring[l + 1 < T ? l + 1 : 0][s][k][c] = o[k][c];
                } else if (z >= z0 && lane >= HL && lane < 64 - HL) {
                    pl.store(o, z, wave * RW, R * T, NW * RW - R * T);
                }
            }
            ++t;
        }
    }
}

// Boxes read the (y, x) neighbours of every plane, so each level holds its 2R + 1 planes with the R rows
// beyond the wavefront's own at either side: the newest plane's outer rows cross LDS once, at the start
// of an iteration.  A level therefore trails the one below by R + 1 planes (its newest plane is
// t - (R + 1) l), and the levels run from the last down, each reading a ring that the one below then
// extends.  Side columns come by lane shifts, once per row and plane.
template <int S, int R, int T, int V, int RW, int NW, bool EDGE>
__device__ __forceinline__ void march3d_box(const Args3X& a, const TileAt& at, int64_t z0, int64_t z1, float* lds) {
    constexpr int K = 2 * R + 1, N = RW + 2 * R, LAG = R + 1;
    const int lane = int(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const auto pl = place3<S, V, RW, EDGE>(a, at, wave, lane);
    float ring[T][K][N][V];  // ring[l]: the planes that level l + 1 reads, rows -R .. RW + R - 1
#pragma unroll
    for (int l = 0; l < T; ++l)
#pragma unroll
        for (int s = 0; s < K; ++s)
#pragma unroll
            for (int k = 0; k < N; ++k)
#pragma unroll
                for (int c = 0; c < V; ++c) ring[l][s][k][c] = 0.0f;
    constexpr size_t LVL = lds_floats(R, V, RW, NW) / 2;
    const int HL = margin_cols(R, T, V) / V;
    const int64_t tend = z1 - 1 + LAG * (T - 1) + R;
    RawPlane<S, V, RW> next;
    int64_t t = z0 - R * T;
    pl.fetch(t, next);
    int par = 0;
    for (;;) {
#pragma unroll
        for (int u = 0; u < K; ++u) {
            if (t > tend) return;
            pl.widen(next, &ring[0][u][R]);
            pl.settle(&ring[0][u][R], t);
            pl.fetch(t + 1, next);
            float* buf = lds + par * (T * LVL);
            par ^= 1;
#pragma unroll
            for (int l = 0; l < T; ++l) {
                float own[RW][V];
#pragma unroll
                for (int k = 0; k < RW; ++k)
#pragma unroll
                    for (int c = 0; c < V; ++c) own[k][c] = ring[l][mod(u - LAG * l, K)][R + k][c];
                publish<R, V, RW>(buf + l * LVL, wave, lane, own);
            }
            __syncthreads();
#pragma unroll
            for (int l = 0; l < T; ++l)
#pragma unroll
                for (int k = 0; k < 2 * R; ++k) {
                    const int row = k < R ? k - R : k - R + RW;
                    halo_row<R, V, RW, NW>(buf + l * LVL, wave, lane, row, ring[l][mod(u - LAG * l, K)][row + R]);
                }
#pragma unroll
            for (int l = T - 1; l >= 0; --l) {
                const int ctr = mod(u - LAG * l - R, K);
                const int64_t z = t - LAG * l - R;  // the plane that level l + 1 completes
                float o[RW][V];
#pragma unroll
                for (int k = 0; k < RW; ++k)
#pragma unroll
                    for (int c = 0; c < V; ++c) o[k][c] = a.w[((R * K) + R) * K + R] * ring[l][ctr][k + R][c];
#pragma unroll
                for (int dz = -R; dz <= R; ++dz) {
                    float e[N][V + 2 * R];
#pragma unroll
                    for (int k = 0; k < N; ++k) with_sides<R, V>(ring[l][mod(ctr + dz, K)][k], e[k]);
#pragma unroll
                    for (int dy = -R; dy <= R; ++dy)
#pragma unroll
                        for (int dx = -R; dx <= R; ++dx) {
                            if (dz == 0 && dy == 0 && dx == 0) continue;
                            const float w = a.w[((dz + R) * K + dy + R) * K + dx + R];
#pragma unroll
                            for (int k = 0; k < RW; ++k)
#pragma unroll
                                for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(w, e[k + R + dy][R + c + dx], o[k][c]);
                        }
                }
                round_rows<S, V, RW>(o);
                if (l + 1 < T) {
                    pl.settle(o, z);
                    const int s = mod(u + 1 - LAG * (l + 1), K);
#pragma unroll
                    for (int k = 0; k < RW; ++k)
#pragma unroll
                        for (int c = 0; c < V; ++c) ring[l + 1 < T ? l + 1 : 0][s][R + k][c] = o[k][c];
                } else if (z >= z0 && lane >= HL && lane < 64 - HL) {
                    pl.store(o, z, wave * RW, R * T, NW * RW - R * T);
                }
            }
            ++t;
        }
    }
}

}  // namespace block

template <int S, int R, int T, int V, int RW, int NW>
__global__ __launch_bounds__(64 * NW) void sweep3d_block(Args3B a) {
    extern __shared__ float4 lds4[];
    const int64_t at0 = a.first + blockIdx.x, seg = at0 / a.tiles, tile = at0 - seg * a.tiles;
    const block::TileAt at = block::tile_at<R, V, RW, NW>(tile, a.tiles_x, a.rows, a.cols, T);
    const int64_t z0 = seg * a.zseg, z1 = z0 + a.zseg < a.planes ? z0 + a.zseg : a.planes;
    float* lds = reinterpret_cast<float*>(lds4);
    if (at.edge || z0 < R * T || z1 + R * T > a.planes) block::march3d<S, R, T, V, RW, NW, true>(a, at, z0, z1, lds);
    else block::march3d<S, R, T, V, RW, NW, false>(a, at, z0, z1, lds);
}

template <int S, int R, int T, int V, int RW, int NW>
__global__ __launch_bounds__(64 * NW) void sweep3d_block_box(Args3X a) {
    extern __shared__ float4 lds4[];
    const int64_t at0 = a.first + blockIdx.x, seg = at0 / a.tiles, tile = at0 - seg * a.tiles;
    const block::TileAt at = block::tile_at<R, V, RW, NW>(tile, a.tiles_x, a.rows, a.cols, T);
    const int64_t z0 = seg * a.zseg, z1 = z0 + a.zseg < a.planes ? z0 + a.zseg : a.planes;
    float* lds = reinterpret_cast<float*>(lds4);
    if (at.edge || z0 < R * T || z1 + R * T > a.planes) block::march3d_box<S, R, T, V, RW, NW, true>(a, at, z0, z1, lds);
    else block::march3d_box<S, R, T, V, RW, NW, false>(a, at, z0, z1, lds);
}

}  // namespace st

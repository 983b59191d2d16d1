// Register-tile temporal blocking: the body shared by the constant-weight kernels (sweep_block.h)
// and the variable-coefficient one (varcoef.hip).
//
// A workgroup of NW wavefronts keeps a tile of NW RW rows x 64 V columns in registers for all levels
// of a pass: wavefront w holds rows [w RW, (w + 1) RW), each lane V consecutive columns of them.  A
// level reads its east and west neighbours from the next lanes (DPP wave shifts) and its north and
// south neighbours beyond the wavefront's own rows from LDS, where every wavefront publishes its
// outer R rows before the level's one barrier (two buffers alternate).  A cell therefore costs its
// taps plus a few instructions per row, against twelve LDS floats read per row of four cells when the
// whole tile lives in LDS, and nothing but the R outer rows crosses LDS.  The tile's outer R rows and
// columns of cells become invalid with every level, so a pass of T levels stores the tile without its
// outer R T cells; wavefronts whose rows are all past use skip the arithmetic.
#pragma once

#include "internal.h"
#include "star_rows.h"
#include "storage.h"

namespace st {
namespace block {

// lane l receives lane l - 1's (l + 1's) value, lane 0 (63) zero
__device__ __forceinline__ float prev_lane(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float next_lane(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}

// rows a wavefront publishes: its outer R on either side, or all of them
__host__ __device__ constexpr int pub_rows(int R, int RW) { return 2 * R < RW ? 2 * R : RW; }
__host__ __device__ constexpr int pub_slot(int R, int RW, int k) {
    return 2 * R >= RW ? k : k < R ? k : k - RW + 2 * R;
}
__host__ __device__ constexpr bool published(int R, int RW, int k) { return 2 * R >= RW || k < R || k >= RW - R; }

// floats of the two exchange buffers
__host__ __device__ constexpr size_t lds_floats(int R, int V, int RW, int NW) {
    return size_t(2) * NW * pub_rows(R, RW) * 64 * V;
}

// Columns of the margin a pass of `levels` levels leaves unstored at either side: whole lanes.
__host__ __device__ constexpr int margin_cols(int R, int levels, int V) { return (R * levels + V - 1) / V * V; }

template <int V>
struct alignas(V == 2 ? 8 : V == 4 ? 16 : 4) Pack {
    float v[V];
};

// Publish this wavefront's outer rows into `buf` (its base), or read halo row d (1 .. R) above / below.
template <int R, int V, int RW>
__device__ __forceinline__ void publish(float* buf, int wave, int lane, const float (&o)[RW][V]) {
    constexpr int PR = pub_rows(R, RW);
#pragma unroll
    for (int k = 0; k < RW; ++k)
        if (published(R, RW, k)) {
            Pack<V> p;
#pragma unroll
            for (int c = 0; c < V; ++c) p.v[c] = o[k][c];
            *reinterpret_cast<Pack<V>*>(buf + ((wave * PR + pub_slot(R, RW, k)) * 64 + lane) * V) = p;
        }
}

// Row `k` of this wavefront's frame (k < 0: above its rows, k >= RW: below) as its owner published it.  A
// row beyond the tile reads some published row instead: it feeds cells that are past use only.
template <int R, int V, int RW, int NW>
__device__ __forceinline__ void halo_row(const float* buf, int wave, int lane, int k, float (&x)[V]) {
    constexpr int PR = pub_rows(R, RW);
    const int up = k < 0 ? (-k + RW - 1) / RW : -(k / RW);  // wavefronts above this one
    const int w = min(max(wave - up, 0), NW - 1);
    const Pack<V> p = *reinterpret_cast<const Pack<V>*>(buf + ((w * PR + pub_slot(R, RW, k + up * RW)) * 64 + lane) * V);
#pragma unroll
    for (int c = 0; c < V; ++c) x[c] = p.v[c];
}

// One row of a lane's cells with R columns from the neighbouring lanes at either side.
template <int R, int V>
__device__ __forceinline__ void with_sides(const float (&x)[V], float (&e)[V + 2 * R]) {
#pragma unroll
    for (int c = 0; c < V; ++c) e[R + c] = x[c];
#pragma unroll
    for (int c = -1; c >= -R; --c) e[R + c] = prev_lane(e[R + c + V]);
#pragma unroll
    for (int c = V; c < V + R; ++c) e[R + c] = next_lane(e[R + c - V]);
}

// A level's cells rounded to the storage type (16-bit types two at a time).
template <int S, int V, int RW>
__device__ __forceinline__ void round_rows(float (&o)[RW][V]) {
    if constexpr (S != ST_F32) {
        static_assert(RW * V % 2 == 0, "pairs");
#pragma unroll
        for (int i = 0; i < RW * V; i += 2) Fmt<S>::rnd2(o[i / V][i % V], o[(i + 1) / V][(i + 1) % V]);
    }
}

// The side taps of a star on RW rows: o[k][c] += w[dx] x[k][c + dx], dx = -R .. -1, then 1 .. R.
template <int R, int V, int RW>
__device__ __forceinline__ void side_taps(float (&o)[RW][V], const float (*x)[V], const float* w) {
    constexpr int N = V == 1 && RW >= 8 ? 8 : V == 4 ? 2 : 4;  // rows per block of StarRows
    if constexpr (StarRows<R, V, N>::exists && RW % N == 0) {
#pragma unroll
        for (int k = 0; k < RW; k += N) StarRows<R, V, N>::apply(o + k, x + k, w);
    } else {
#pragma unroll
        for (int k = 0; k < RW; ++k) {
            float q[V], e[V + 2 * R];
#pragma unroll
            for (int c = 0; c < V; ++c) q[c] = x[k][c];
            with_sides<R, V>(q, e);
#pragma unroll
            for (int d = -R; d <= R; ++d) {
                if (d == 0) continue;
#pragma unroll
                for (int c = 0; c < V; ++c) o[k][c] = __builtin_fmaf(w[d < 0 ? d + R : d + R - 1], e[R + c + d], o[k][c]);
            }
        }
    }
}

// Whether wavefront `wave` holds a row of [lo, NW RW - lo).
template <int RW, int NW>
__device__ __forceinline__ bool has_rows(int wave, int lo) {
    return (wave + 1) * RW > lo && wave * RW < NW * RW - lo;
}

// V consecutive elements at any element alignment (global memory takes vector accesses that are only
// element-aligned).
template <typename T, int V>
struct VecOf {
    typedef T type __attribute__((ext_vector_type(V), aligned(sizeof(T))));
};
template <typename T>
struct VecOf<T, 1> {
    typedef T type;
};
template <int S, int V>
__device__ __forceinline__ void load_cells(const void* base, int64_t off, float (&x)[V]) {
    using T = typename Fmt<S>::T;
    using G = const __attribute__((address_space(1))) typename VecOf<T, V>::type;
    const auto q = *(G*)(static_cast<const T*>(base) + off);
    if constexpr (V == 1) {
        x[0] = Fmt<S>::ld(q);
    } else {
#pragma unroll
        for (int c = 0; c < V; ++c) x[c] = Fmt<S>::ld(q[c]);
    }
}
template <int S, int V>
__device__ __forceinline__ void store_cells(void* base, int64_t off, const float (&x)[V]) {
    using T = typename Fmt<S>::T;
    using VT = typename VecOf<T, V>::type;
    VT q;
    if constexpr (V == 1) {
        q = Fmt<S>::st(x[0]);
    } else {
#pragma unroll
        for (int c = 0; c < V; ++c) q[c] = Fmt<S>::st(x[c]);
    }
    *(__attribute__((address_space(1))) VT*)(static_cast<T*>(base) + off) = q;
}

// The tile of one workgroup: rows [ty, ty + NW RW) and columns [tx, tx + 64 V) of the grid (its
// margins included, so possibly beyond the grid).
struct TileAt {
    int64_t ty, tx;
    bool edge;  // some cell of it lies outside the grid
};

// Blocks go to the 8 XCDs in turn; give each a contiguous run of tiles, so that neighbours share an L2.
__device__ __forceinline__ int64_t xcd_order(int64_t bid, int64_t n) {
    const int64_t q = n / 8, rem = n % 8, k = bid % 8, i = bid / 8;
    return k * q + (k < rem ? k : rem) + i;
}

template <int R, int V, int RW, int NW>
__device__ __forceinline__ TileAt tile_at(int64_t t, int64_t tiles_x, int64_t rows, int64_t cols, int levels) {
    const int H = R * levels, HC = margin_cols(R, levels, V);
    TileAt a;
    a.ty = (t / tiles_x) * (NW * RW - 2 * H) - H;
    a.tx = (t % tiles_x) * (64 * V - 2 * HC) - HC;
    a.edge = a.ty < 0 || a.tx < 0 || a.ty + NW * RW > rows || a.tx + 64 * V > cols;
    return a;
}

// Register tiles: V columns per lane, RW rows per wavefront, NW wavefronts.  A plan's tile picks the one
// of its size (pick).  A pass whose margins would leave less than a quarter of a tile in either direction
// takes the last, whose 128 x 128 cells hold every depth a plan accepts (r tb <= 39).  Eight wavefronts of
// eight rows beat sixteen of four on the same tile (star r = 1, 8192^2, tb 8: 3109 against 2756
// GStencil/s): half the rows cross LDS, and two or three workgroups share a compute unit.
struct Def {
    int v, rw, nw;
};
constexpr Def kDefs[] = {{1, 8, 8}, {2, 4, 8}, {2, 8, 8}, {4, 4, 8}, {2, 8, 16}};
constexpr int kTall = 4;

// Tiles of one pass of `levels` levels of radius r with definition `def` (-1: the tile of no plan).
struct Cover {
    int def;
    int64_t tiles_x, tiles;
};
inline Cover cover(int def, int r, int levels, int64_t rows, int64_t cols) {
    auto out_rows = [&](int d) { return kDefs[d].nw * kDefs[d].rw - 2 * r * levels; };
    auto out_cols = [&](int d) { return 64 * kDefs[d].v - 2 * margin_cols(r, levels, kDefs[d].v); };
    if (def < 0 || 4 * out_rows(def) < kDefs[def].nw * kDefs[def].rw || out_cols(def) < 16 * kDefs[def].v) def = kTall;
    if (out_rows(def) < 1 || out_cols(def) < 1) return Cover{-1, 0, 0};
    const int64_t tx = (cols + out_cols(def) - 1) / out_cols(def);
    return Cover{def, tx, tx * ((rows + out_rows(def) - 1) / out_rows(def))};
}

// The tile that a plan's pass runs on: the plan's own (`def`), unless its margins would leave less than
// two fifths of its cells and another is estimated to take less than 0.85 of its time: the instructions that
// a compute unit issues per level (`ops` a cell, a few per row, and the exchange) for the most tiles that one of
// the 256 gets, each after the first at 0.7 of it (their waits overlap).  The constants are fitted to 4 passes of
// every tile at 12 grids up to 2000^2, six footprints, 3 to 16 levels: of 1024 choices 495 are more than 3 % faster
// than the own tile, and 4 slower (the most 5 %).
// Three passes at 2000^2, us, own tile / picked: star r = 4, 64 x 64, 6 levels (6 % kept) 592 / 157 (LDS tiles,
// whose halo lies around the tile, took 295); box r = 2, 64 x 64, 12 levels 1429 / 351; star r = 4, 128 x 64, 4
// levels (38 %) 95 / 89.  From two fifths up the own tile was never slower than LDS tiles.  Small grids are
// often best on small tiles all the same: star r = 1 at 512^2, 64 x 64, 16 levels (25 %) 8.0 us a pass, on the
// next tile 9.7.
inline Cover pick(int def, double ops, int r, int levels, int64_t rows, int64_t cols) {
    const Cover own = cover(def, r, levels, rows, cols);
    if (own.def == def) {
        const Def& d = kDefs[def];
        const double keep = double(d.nw * d.rw - 2 * r * levels) * (64 * d.v - 2 * margin_cols(r, levels, d.v));
        if (keep >= 0.4 * d.nw * d.rw * 64 * d.v) return own;
    }
    auto time = [&](const Cover& c) {
        const Def& d = kDefs[c.def];
        const double share = 0.3 + 0.7 * double((c.tiles + 255) / 256);  // (tiles on one compute unit overlap)
        return share * d.nw * (d.rw * d.v * ops + 4.0 * d.rw + 15.0);
    };
    Cover best = own;
    if (own.def < 0) return own;
    double best_t = time(own) * (own.def == def ? 0.85 : 1.0);
    for (int i = 0; i <= kTall; ++i) {
        const Cover c = cover(i, r, levels, rows, cols);
        if (c.def == i && time(c) < best_t) {
            best_t = time(c);
            best = c;
        }
    }
    return best;
}

}  // namespace block

// Which of the tiles of stencil_tiles() this is (-1: none), in the order of block::kDefs.
int tile_index(int tx, int ty);

}  // namespace st

// 3D Jacobi stencil (the update of Sec. II-C on a planes x rows x cols grid, the constant halo of
// Sec. IV-A, the centre-first FP32 order of Sec. IV-E extended to (dz, dy, dx)):
//   u'(k, i, j) = sum_{dz, dy, dx in [-r, r]} W[dz+r][dy+r][dx+r] ~u(k+dz, i+dy, j+dx),
// per cell acc = W_c u_c, then one FMA per footprint tap in row-major (dz, dy, dx) order (star:
// the taps on the three axes; box: all of them).
//
// Stars, and boxes of radius 1, run several levels per pass on register tiles (sweep3d_block.h).
//
// Boxes of radius 2 (125 taps: their weights alone fill the scalar registers), and single levels of large
// FP32 stars (ring_pass), run on LDS tiles, one level per pass.  One workgroup owns a TY x TX column of the grid and marches along z over a segment of planes:
// the 2r + 1 input planes of the current output plane sit in an LDS ring, each with its r-deep
// (y, x) halo; every iteration stores a plane fetched earlier into the slot the oldest plane leaves,
// starts fetching the plane after next into registers (two register sets, so two planes are in
// flight), and computes its cells of the output plane from the ring meanwhile.  A wavefront covers one row of the
// tile (64 consecutive columns), so loads and stores are coalesced and LDS reads of one tap hit 64
// consecutive words.  Boxes are bound by LDS (one read per tap and cell), stars by HBM.
#include <algorithm>

#include "internal.h"
#include "storage.h"
#include "sweep3d_block.h"

namespace st {

namespace {

constexpr int TX = 64, TY = 32, NT3 = 256;
constexpr int ROWS_PER_THREAD = TY / (NT3 / TX);  // 8

struct Args3 {
    const void* src;
    void* dst;
    int64_t planes, rows, cols;
    int64_t tiles_x, tiles_y, zseg;  // tile grid and planes per segment
    float b;
    float w[MAXK3];
};

// One plane of the tile with its r-deep (y, x) halo, in the storage type's FP32 values: fetched into
// registers (PER values per thread) while the previous plane computes, stored into LDS afterwards.
template <int R>
struct PlaneRegs {
    static constexpr int PW = TX + 2 * R, PH = TY + 2 * R, PS = PW * PH;
    static constexpr int PER = (PS + NT3 - 1) / NT3;
    float v[PER];
};

template <int S, int R>
__device__ __forceinline__ void fetch_plane(const Args3& a, PlaneRegs<R>& p, int64_t z, int64_t y0, int64_t x0) {
    using T = typename Fmt<S>::T;
    using P = PlaneRegs<R>;
    const T* src = static_cast<const T*>(a.src);
    const bool zin = z >= 0 && z < a.planes;
#pragma unroll
    for (int j = 0; j < P::PER; ++j) {
        const int k = int(threadIdx.x) + NT3 * j;
        const int py = k / P::PW, px = k % P::PW;
        const int64_t y = y0 - R + py, x = x0 - R + px;
        float v = a.b;
        if (k < P::PS && zin && y >= 0 && y < a.rows && x >= 0 && x < a.cols) v = Fmt<S>::ld(src[(z * a.rows + y) * a.cols + x]);
        p.v[j] = v;
    }
}

template <int R>
__device__ __forceinline__ void store_plane(float* slot, const PlaneRegs<R>& p) {
    using P = PlaneRegs<R>;
#pragma unroll
    for (int j = 0; j < P::PER; ++j) {
        const int k = int(threadIdx.x) + NT3 * j;
        if (k < P::PS) slot[k] = p.v[j];
    }
}

template <int S, int R, int SHAPE>
__global__ __launch_bounds__(NT3) void sweep3d(Args3 a) {
    constexpr int K = 2 * R + 1;
    using P = PlaneRegs<R>;
    constexpr int PW = P::PW, PS = P::PS;
    __shared__ float ring[K][PS];
    const int64_t t = blockIdx.x;
    const int64_t tile = t % (a.tiles_x * a.tiles_y), seg = t / (a.tiles_x * a.tiles_y);
    const int64_t y0 = (tile / a.tiles_x) * TY, x0 = (tile % a.tiles_x) * TX;
    const int64_t z0 = seg * a.zseg, z1 = z0 + a.zseg < a.planes ? z0 + a.zseg : a.planes;
    const int tx = threadIdx.x % TX, ty0 = threadIdx.x / TX;
    using T = typename Fmt<S>::T;
    T* dst = static_cast<T*>(a.dst);
    // planes z0 - R .. z0 + R - 1 into slots; plane z lives in slot (z - z0 + R) mod K
    P pre;
    for (int q = 0; q < 2 * R; ++q) {
        fetch_plane<S, R>(a, pre, z0 - R + q, y0, x0);
        store_plane<R>(ring[q], pre);
    }
    // planes fetched two ahead (two register sets, the loop unrolled by two): twice the bytes in
    // flight per workgroup while a plane computes
    P pre2;
    fetch_plane<S, R>(a, pre, z0 + R, y0, x0);
    if (z0 + 1 < z1) fetch_plane<S, R>(a, pre2, z0 + 1 + R, y0, x0);
    auto compute = [&](int64_t z) {
        const int c_slot = int((z - z0 + R) % K);
#pragma unroll
        for (int rr = 0; rr < ROWS_PER_THREAD; ++rr) {
            const int ty = ty0 + rr * (NT3 / TX);
            const int o = (ty + R) * PW + tx + R;  // the cell's offset within a plane tile
            float acc = a.w[(R * K + R) * K + R] * ring[c_slot][o];
#pragma unroll
            for (int dz = -R; dz <= R; ++dz) {
                const float* pl = ring[(c_slot + dz + K) % K];
#pragma unroll
                for (int dy = -R; dy <= R; ++dy)
#pragma unroll
                    for (int dx = -R; dx <= R; ++dx) {
                        const int nz = (dz != 0) + (dy != 0) + (dx != 0);
                        if (nz == 0 || (SHAPE == SHAPE_STAR && nz > 1)) continue;
                        acc = __builtin_fmaf(a.w[((dz + R) * K + dy + R) * K + dx + R], pl[o + dy * PW + dx], acc);
                    }
            }
            const int64_t y = y0 + ty, x = x0 + tx;
            if (y < a.rows && x < a.cols) dst[(z * a.rows + y) * a.cols + x] = Fmt<S>::st(acc);
        }
    };
    for (int64_t z = z0; z < z1; z += 2) {
        store_plane<R>(ring[int((z - z0 + 2 * R) % K)], pre);  // plane z + R
        __syncthreads();
        if (z + 2 < z1) fetch_plane<S, R>(a, pre, z + 2 + R, y0, x0);
        compute(z);
        __syncthreads();  // every thread is done with the slot the next store overwrites
        if (z + 1 >= z1) break;
        store_plane<R>(ring[int((z + 1 - z0 + 2 * R) % K)], pre2);  // plane z + 1 + R
        __syncthreads();
        if (z + 3 < z1) fetch_plane<S, R>(a, pre2, z + 3 + R, y0, x0);
        compute(z + 1);
        __syncthreads();
    }
}

// The kernels on LDS tiles: boxes of radius 2, FP32 stars.
using Fn3 = void (*)(Args3);
Fn3 ring_lookup(int shape, int r, int storage) {
    if (shape == SHAPE_STAR) return storage != ST_F32 ? nullptr : r == 1 ? sweep3d<ST_F32, 1, SHAPE_STAR> : sweep3d<ST_F32, 2, SHAPE_STAR>;
    if (r != 2) return nullptr;
    if (storage == ST_F32) return sweep3d<ST_F32, 2, SHAPE_BOX>;
    if (storage == ST_BF16) return sweep3d<ST_BF16, 2, SHAPE_BOX>;
    if (storage == ST_F16) return sweep3d<ST_F16, 2, SHAPE_BOX>;
    return nullptr;
}

// Single levels of an FP32 star that run on LDS tiles: their 64 columns start on cache lines where the rows
// do, while a register tile's start inside them (1.45 GB moved for 1.05 at 512^3, r = 1).  The widths
// (a multiple of 16) and sizes where that is faster; us a step, LDS tiles / register tiles.  r = 1: 256^3
// 35 / 36, 400^3 145 / 154, 512^3 241 / 331, 4 x 8192^2 502 / 611; at other widths 300^3 56 / 52, 450^3
// 236 / 210.  r = 2, larger halos to load, from fields beyond the 256 MB cache on: 400^3 197 / 163; 512^3
// 266 / 348, 640^3 680 / 645, 64 x 2048^2 516 / 658.  16-bit fields: 512^3 391 / 208.
bool ring_pass(const st_plan* p) {
    return p->shape == SHAPE_STAR && p->storage == ST_F32 && p->cols % 16 == 0 &&
           field_cells(p) >= (p->radius == 1 ? int64_t(1) << 24 : int64_t(1) << 26);
}

// Stars and boxes of radius 1 on register tiles (sweep3d_block.h): one column per lane, four rows per
// wavefront; sixteen wavefronts (64 x 64 tiles) for stars, eight (64 x 32) for boxes, whose levels hold six
// rows of three planes (two levels at 512^3: 650 GStencil/s, sixteen wavefronts 587, eight rows 575).
constexpr int BV = 1, BRW = 4, BNW_STAR = 16, BNW_BOX = 8;
constexpr int MAX_LEVELS_STAR1 = 6, MAX_LEVELS_STAR2 = 2, MAX_LEVELS_BOX1 = 2;

template <int S>
const void* block3(int shape, int r, int levels) {
#define ST_STAR3(R, T) \
    if (shape == SHAPE_STAR && r == R && levels == T) return reinterpret_cast<const void*>(sweep3d_block<S, R, T, BV, BRW, BNW_STAR>);
#define ST_BOX3(T) \
    if (shape == SHAPE_BOX && r == 1 && levels == T) return reinterpret_cast<const void*>(sweep3d_block_box<S, 1, T, BV, BRW, BNW_BOX>);
    ST_STAR3(1, 1) ST_STAR3(1, 2) ST_STAR3(1, 3) ST_STAR3(1, 4) ST_STAR3(1, 5) ST_STAR3(1, 6)
    ST_STAR3(2, 1) ST_STAR3(2, 2)
    ST_BOX3(1) ST_BOX3(2)
#undef ST_STAR3
#undef ST_BOX3
    return nullptr;
}

const void* block3(const st_plan* p, int levels) {
    if (p->storage == ST_F32) return block3<ST_F32>(p->shape, p->radius, levels);
    if (p->storage == ST_BF16) return block3<ST_BF16>(p->shape, p->radius, levels);
    if (p->storage == ST_F16) return block3<ST_F16>(p->shape, p->radius, levels);
    return nullptr;
}

bool on_tiles(const st_plan* p) { return p->shape == SHAPE_STAR || p->radius == 1; }

// How a pass of `levels` levels covers the grid, and its cost in units of one level's arithmetic on one
// plane of a tile (0.235 us): a workgroup takes zseg + 2 r levels iterations of 3 + levels units (loads,
// exchange and barrier, then the levels), and the launch as many rounds of workgroups as the device needs
// for all of them; its bytes at 4.4 TB/s (a third of what the field takes when it fits the 256 MB cache)
// and a launch of about 15 units are the other bounds.  The model ranks depths as measured: 512^3 1, 2, 3, 4, 5, 6
// levels 424, 900, 1216, 1468, 1590, 1646 GStencil/s; 100^3 x 20 steps 193, 124, 112, 106, 144 us for
// 1 .. 5; 40 x 500 x 500 439, 249, 210, 191, 228 us.
struct Cover3 {
    int64_t tiles_x, tiles, zseg;
    double cost;
};
int cover3(const st_plan* p, int levels, Cover3* c) {
    const int r = p->radius, nw = p->shape == SHAPE_STAR ? BNW_STAR : BNW_BOX;
    const void* fn = block3(p, levels);
    if (!fn) return fail(ST_EUNSUPPORTED, "no 3D kernel for this storage/shape/radius");
    const size_t lds = block::lds_floats(r, BV, BRW, nw) * levels * sizeof(float);
    if (int rc = prepare_lds(fn, lds)) return rc;
    int slots = 0;
    if (int rc = resident_blocks_of(fn, lds, 64 * nw, &slots)) return rc;
    const int out_rows = nw * BRW - 2 * r * levels, out_cols = 64 * BV - 2 * block::margin_cols(r, levels, BV);
    c->tiles_x = (p->cols + out_cols - 1) / out_cols;
    c->tiles = c->tiles_x * ((p->rows + out_rows - 1) / out_rows);
    double best = 0.0;
    for (int64_t segs = 1; segs <= std::min<int64_t>(p->planes, 64); ++segs) {
        const int64_t zs = (p->planes + segs - 1) / segs, n = (p->planes + zs - 1) / zs;
        const double cost = double((c->tiles * n + slots - 1) / slots) * double(zs + 2 * r * levels) * (3 + levels);
        if (best == 0.0 || cost < best) {
            best = cost;
            c->zseg = zs;
        }
    }
    const double bytes = 2.0 * double(field_cells(p)) * double(elem_size(p->storage));
    const double rate = levels == 1 && ring_pass(p) ? 4.4e6 : 3.5e6;  // bytes per us
    c->cost = std::max(best, bytes / rate / 0.235 * (bytes > 2e8 ? 1.0 : 1.0 / 3.0)) + 15.0;
    return ST_OK;
}

int launch_tiles(const st_plan* p, const void* src, void* dst, int levels, hipStream_t s) {
    Cover3 c;
    if (int rc = cover3(p, levels, &c)) return rc;
    const int64_t grid = c.tiles * ((p->planes + c.zseg - 1) / c.zseg);
    if (grid > (int64_t(1) << 31) - 1) return fail(ST_EUNSUPPORTED, "3D grid too large for one launch");
    const int r = p->radius, k = 2 * r + 1, nw = p->shape == SHAPE_STAR ? BNW_STAR : BNW_BOX;
    const size_t lds = block::lds_floats(r, BV, BRW, nw) * levels * sizeof(float);
    auto fill = [&](auto& a) {
        a.src = src;
        a.dst = dst;
        a.planes = p->planes;
        a.rows = p->rows;
        a.cols = p->cols;
        a.tiles_x = c.tiles_x;
        a.tiles = c.tiles;
        a.zseg = c.zseg;
        a.b = p->bq;
    };
    clear_stale_error();
    if (p->shape == SHAPE_STAR) {
        Args3B a;
        fill(a);
        const float* w = p->w3 + (r * k + r) * k + r;  // the centre weight
        a.wc = w[0];
        for (int i = 0; i < 2 * r; ++i) {
            const int d = i < r ? i - r : i - r + 1;
            a.wz[i] = w[d * k * k];
            a.wy[i] = w[d * k];
            a.wx[i] = w[d];
        }
        launch_runs(grid, 64 * nw, [&](int64_t first, int64_t n) {
            a.first = first;
            hipLaunchKernelGGL(reinterpret_cast<void (*)(Args3B)>(const_cast<void*>(block3(p, levels))), dim3(unsigned(n)),
                               dim3(64 * nw), lds, s, a);
        });
    } else {
        Args3X a;
        fill(a);
        std::memcpy(a.w, p->w3, sizeof(a.w));
        launch_runs(grid, 64 * nw, [&](int64_t first, int64_t n) {
            a.first = first;
            hipLaunchKernelGGL(reinterpret_cast<void (*)(Args3X)>(const_cast<void*>(block3(p, levels))), dim3(unsigned(n)),
                               dim3(64 * nw), lds, s, a);
        });
    }
    ST_LAUNCH_CHECK("sweep3d_block");
    return ST_OK;
}

}  // namespace

// Levels per pass: the depth of the least cost per step.
int max_levels_3d(st_plan* p) {
    if (!on_tiles(p)) return 1;
    if (p->levels3 == 0) {
        const int most = p->shape == SHAPE_BOX ? MAX_LEVELS_BOX1 : p->radius == 1 ? MAX_LEVELS_STAR1 : MAX_LEVELS_STAR2;
        double best = 0.0;
        for (int t = 1; t <= most; ++t) {
            Cover3 c;
            if (cover3(p, t, &c) != ST_OK) break;
            if (best == 0.0 || c.cost / t < best) {
                best = c.cost / t;
                p->levels3 = t;
            }
        }
        if (p->levels3 == 0) return 1;
    }
    return p->levels3;
}

int launch_3d(const st_plan* p, const void* src, void* dst, int levels, hipStream_t s) {
    if (on_tiles(p) && !(levels == 1 && ring_pass(p))) return launch_tiles(p, src, dst, levels, s);
    Fn3 fn = ring_lookup(p->shape, p->radius, p->storage);
    if (!fn) return fail(ST_EUNSUPPORTED, "no 3D kernel for this storage/shape/radius");
    Args3 a;
    a.src = src;
    a.dst = dst;
    a.planes = p->planes;
    a.rows = p->rows;
    a.cols = p->cols;
    a.b = p->bq;
    std::memcpy(a.w, p->w3, sizeof(a.w));
    a.tiles_x = (p->cols + TX - 1) / TX;
    a.tiles_y = (p->rows + TY - 1) / TY;
    int blocks = 0;
    if (int rc = resident_blocks(reinterpret_cast<const void*>(fn), 0, &blocks)) return rc;
    // z segments so that the launch about fills the device once; each segment reloads 2r planes
    const int64_t tiles = a.tiles_x * a.tiles_y;
    const int64_t segs = std::max<int64_t>(1, std::min<int64_t>(p->planes, (blocks + tiles - 1) / tiles));
    a.zseg = (p->planes + segs - 1) / segs;
    const int64_t nseg = (p->planes + a.zseg - 1) / a.zseg;
    const int64_t grid = tiles * nseg;
    if (grid > (int64_t(1) << 31) - 1) return fail(ST_EUNSUPPORTED, "3D grid too large for one launch");
    clear_stale_error();
    hipLaunchKernelGGL(fn, dim3(unsigned(grid)), dim3(NT3), 0, s, a);
    ST_LAUNCH_CHECK("sweep3d");
    return ST_OK;
}

}  // namespace st

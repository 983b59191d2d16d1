// Row-marching Jacobi pass (paper Sec. II-C update with the fixed halo of Sec. IV-A; per cell the
// FP32 order of Sec. IV-E: the centre product, then one FMA per footprint tap in row-major order, the
// same order as the tiled kernels, so results agree bit for bit).  Fields may be stored as FP32,
// BF16 or FP16; arithmetic is FP32 and every level is rounded to the storage type.
//
// One wavefront owns a band of columns, V per lane (V = 8 or 4 with one or two 16-byte loads, or one
// 8-byte load, per lane and row; for narrow grids of an odd width V = 4 with one element access
// per column; or V = 1, many short tasks for small grids), and walks down a segment of rows.  Each
// input row is read from HBM once per band; the r columns a lane needs on either side
// come from neighbouring lanes through DPP wave shifts (the value at column c < 0 is the previous
// lane's value at column c + V, so the side columns are produced nearest first, one shift each),
// and the pass uses neither LDS nor barriers.  The rows a lane needs sit in a register ring whose
// slots become fixed registers because the row loop is unrolled over the ring length.  With several
// levels per pass further rings hold the intermediate levels.  Level l is exact on columns at
// least r*l away from the band's loaded edge, so a band writes V (64 - 2 H) columns with
// H = ceil(r tb / V) halo lanes per side (with a halo of +0 the bands at the grid's sides write
// theirs too, see march_layout.h).  A wavefront lowers its priority as its task progresses, so the
// tasks sharing a SIMD finish together (march_body.h).
//
// Segments are sized on the host so that the number of (band, segment) tasks is close to the number
// of wavefronts the device holds at once: every wavefront runs one task of about equal duration (the
// tasks that take the grid's edge checks get proportionally shorter segments, see march_layout.h).  A
// plan may ask for longer segments (stencil_set_march_segment), which the autotuner does for small
// grids.

#include <algorithm>
#include <cmath>

#include "march_kern.h"

namespace st {

using march_k::MarchArgs;
using march_k::MarchFn;
using march_k::MWAVES;

namespace {

MarchFn march_lookup(int storage, int mode, int shape, int r, int levels, bool xbc, bool periodic) {
    const bool box = shape == SHAPE_BOX;
    if (xbc) {
        if (storage == ST_F32)
            return box ? march_lookup_xbc_f32_box(mode, r, levels, periodic) : march_lookup_xbc_f32_star(mode, r, levels, periodic);
        if (storage == ST_BF16)
            return box ? march_lookup_xbc_bf16_box(mode, r, levels, periodic) : march_lookup_xbc_bf16_star(mode, r, levels, periodic);
        if (storage == ST_F16)
            return box ? march_lookup_xbc_f16_box(mode, r, levels, periodic) : march_lookup_xbc_f16_star(mode, r, levels, periodic);
        return nullptr;
    }
    if (storage == ST_F32) return box ? march_lookup_f32_box(mode, r, levels) : march_lookup_f32_star(mode, r, levels);
    if (storage == ST_BF16) return box ? march_lookup_bf16_box(mode, r, levels) : march_lookup_bf16_star(mode, r, levels);
    if (storage == ST_F16) return box ? march_lookup_f16_box(mode, r, levels) : march_lookup_f16_star(mode, r, levels);
    return nullptr;
}

}  // namespace

int march_max_tb(int shape, int radius, int vmax) {
    if (vmax == 8) {  // never deeper than the four-column kernels it falls back to
        if (shape == SHAPE_STAR) return radius == 1 ? 8 : radius == 2 ? 4 : radius == 3 ? 3 : 2;
        return radius == 1 ? 3 : radius == 2 ? 2 : radius == 3 ? 2 : 1;
    }
    if (shape == SHAPE_STAR) return radius == 1 ? 8 : radius == 2 ? 6 : radius == 3 ? 4 : 3;
    return radius == 1 ? 6 : radius == 2 ? 3 : 2;
}

bool march_usable(const st_plan* p) { return p->kind == KIND_CONST && p->radius <= 4; }

// Passes at widths that are no multiple of four where four elements per lane are faster than one vector all the
// same: at such widths the vector form can need a band more, and its rows start on no vector boundary, so that
// what its single access saves depends on what else the kernel does.  Measured at 2000 x 2003, 3000 x 3002 and 4099 x 5003 (one pass, us, vector / elements):
//   boxes of r = 4, two levels: periodic BF16 328 / 206, 709 / 445, 1057 / 645, FP32 384 / 307, 825 / 615, 1284 /
//   925 (at 700 x 257 123 / 127); framed FP32 375 / 314, 803 / 620, 1116 / 884 (framed BF16: no difference);
//   stars of r = 1 (halo value 0; 0.5), four levels: FP32 43 / 38, 62 / 55, 106 / 100; 44 / 38, 65 / 55, 110 / 100
//   (at 1000 x 701 19 / 24), F16 38 / 36, 51 / 48, 76 / 72; 40 / 35, 56 / 47, 72 / 70, BF16 34 / 36, 46 / 46, 74 /
//   69; 36 / 35, 50 / 45, 73 / 67; five, F16: 40 / 47, 60 / 62, 95 / 87; 45 / 47, 67 / 61, 93 / 85 (BF16 54 / 59
//   and FP32 56 / 64 at 3000 x 3002); six, FP32: 45 / 56, 66 / 62, 106 / 105; 48 / 55, 72 / 63, 110 / 104, BF16 43 /
//   53, 62 / 62, 92 / 92; 49 / 53, 71 / 61, 97 / 90;
//   boxes of r = 1, six levels: FP32 65 / 65, 94 / 88, 147 / 144; 72 / 65, 93 / 88, 147 / 141, BF16 64 / 67, 95 /
//   90, 153 / 146; 73 / 67, 95 / 90, 153 / 146 (at 1000 x 701 34 / 42; 39 / 41);
//   stars of r = 4, three levels, BF16: 71 / 83, 93 / 109, 176 / 155.
static bool element_accesses(const st_plan* p, int levels) {
    if (p->cols % 4 == 0) return false;
    const bool f32 = p->storage == ST_F32;
    const int64_t cells = p->rows * p->cols;
    if (p->bc != ST_BC_CONST)
        return p->shape == SHAPE_BOX && p->radius == 4 && levels == 2 && (p->bc == ST_BC_PERIODIC || f32);
    if (p->radius == 1 && p->shape == SHAPE_BOX) return levels == 6 && cells >= 2500000;
    if (p->radius == 1) {
        if (levels == 4) return cells >= (f32 ? 2500000 : 6000000);
        return (levels == 6 || (levels == 5 && p->storage == ST_F16)) && cells >= 6000000;
    }
    return p->radius == 4 && levels == 3 && !f32 && cells >= 15000000;
}

int launch_march(const st_plan* p, const void* src, void* dst, int levels, int vmax, hipStream_t s) {
    // Four columns per lane with one vector access per lane and row, at any width and alignment, when no
    // lane's vector straddles the grid's side (march_layout.h; 4099 x 5003, halo 1.5, us a pass with four
    // element accesses / one vector: star r = 3 at tb 1 42 / 34, tb 3 48 / 46, box r = 3 at tb 2 99 / 78);
    // else, on narrow grids, element accesses (mode 0).  Eight columns per lane where rows are whole and
    // aligned vectors of eight (at other widths four are faster: star r = 2 at tb 4 41.5 / 46.8, box r = 3
    // at tb 2 76 / 98).  vmax 1: one column per lane, any width.  48 steps of the tuned plan: 704 -> 607 us.
    // (periodic and framed grids have no eight-column kernels: they take four columns per lane)
    const bool xbc = p->bc != ST_BC_CONST;
    if (xbc && vmax == 8) vmax = 4;
    const bool aligned = (reinterpret_cast<uintptr_t>(src) % 16) == 0 && (reinterpret_cast<uintptr_t>(dst) % 16) == 0;
    const int mode = vmax == 1 ? 1 : vmax == 8 && aligned && p->cols % 8 == 0 ? 8 : march::whole_lanes(p->cols, 4) && !element_accesses(p, levels) ? 4 : 0;
    const int V = mode == 8 ? 8 : mode == 1 ? 1 : 4;
    MarchFn fn = march_lookup(p->storage, mode, p->shape, p->radius, levels, xbc, p->bc == ST_BC_PERIODIC);
    if (!fn) return fail(ST_EUNSUPPORTED, "no row-marching kernel for this shape/radius/depth");
    MarchArgs a;
    a.src = src;
    a.dst = dst;
    a.b = p->bq;
    a.bc = p->bc;
    a.frame = p->frame;
    a.stop = p->stop;
    std::memcpy(a.w, p->w, sizeof(a.w));
    // A constant halo of +0 with whole-lane accesses (vector, or one column per lane): the first
    // band starts at column 0 and the last ends at the last column (march_layout.h).
    const float zero = 0.0f;
    const bool zero_sides =
        !xbc && mode != 0 && std::memcmp(&p->bq, &zero, sizeof(float)) == 0 && p->cols >= 2 * 64 * V;
    int blocks = 0;
    if (int rc = resident_blocks(reinterpret_cast<const void*>(fn), 0, &blocks)) return rc;
    const int taps = p->shape == SHAPE_STAR ? 4 * p->radius + 1 : (2 * p->radius + 1) * (2 * p->radius + 1);
    if (!march::plan_march_tasks(a.map, p->rows, p->cols, V, p->radius, levels, taps, int64_t(blocks) * MWAVES,
                                 p->seg_min, zero_sides))
        return fail(ST_EUNSUPPORTED, "too many marching tasks for one pass");
    const int64_t grid = (a.map.tasks + MWAVES - 1) / MWAVES;
    clear_stale_error();
    hipLaunchKernelGGL(fn, dim3(unsigned(grid)), dim3(64 * MWAVES), 0, s, a);
    ST_LAUNCH_CHECK("sweep_march");
    return ST_OK;
}

}  // namespace st

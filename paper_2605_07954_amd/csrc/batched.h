// What the batched kernels share with the host side of a batch (batched.hip): the descriptor table's
// entries and the register-tile kernels of batched_block.hip.
#pragma once

#include "internal.h"

namespace st {

struct BatchDesc {
    const float* in;
    float* out;
    float* ws;
    int64_t rows, cols;
    int64_t tiles_x, tiles_y;  // register tiles: columns and rows of tiles; marching engine: bands and segments
    int64_t seg;               // marching engine: output rows per task
    int r, shape, tb, steps, passes, resident;
    int zero_sides;  // marching engine: bands start and end at the grid's sides (march_layout.h)
    float b;
    float w[MAXK];
};

// One pass of the grids order[0 .. n) of a stencil class on register tiles, or with p < 0 all steps of
// grids that fit one tile each.
struct BlockPassArgs {
    const BatchDesc* desc;
    const int* order;
    const int64_t* tile_prefix;  // prefix sums of tiles over `order` (n + 1 of them; p >= 0)
    int n;
    int p;
    int64_t first;  // the first tile of this launch
};
using BlockPassFn = void (*)(BlockPassArgs);
// The kernel of a class with tile `def` (block::kDefs), or of whole grids in one tile.
BlockPassFn batched_block_lookup(int shape, int r, int def);
BlockPassFn batched_whole_lookup(int shape, int r);

// largest index i in [0, n) with a[i] <= x (a ascending, a[0] <= x)
__device__ __forceinline__ int upper_index(const int64_t* a, int n, int64_t x) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a[mid] <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

}  // namespace st

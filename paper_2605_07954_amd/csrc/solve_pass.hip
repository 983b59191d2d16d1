// The last pass of a convergence interval on register tiles: it also sums, per tile, how far its last
// level moved the cells (sweep_block_sums).
#include "sweep_block.h"

namespace st {

namespace {

template <int S, int R, int SH>
BlockFn sums_fn(int def) {
    switch (def) {
        case 0: return sweep_block_sums<S, R, SH, 1, 8, 8>;
        case 1: return sweep_block_sums<S, R, SH, 2, 4, 8>;
        case 2: return sweep_block_sums<S, R, SH, 2, 8, 8>;
        case 3: return sweep_block_sums<S, R, SH, 4, 4, 8>;
        case 4: return sweep_block_sums<S, R, SH, 2, 8, 16>;
    }
    return nullptr;
}

template <int S, int SH>
BlockFn sums_fn_r(int r, int def) {
    switch (r) {
        case 1: return sums_fn<S, 1, SH>(def);
        case 2: return sums_fn<S, 2, SH>(def);
        case 3: return sums_fn<S, 3, SH>(def);
        case 4: return sums_fn<S, 4, SH>(def);
    }
    return nullptr;
}

template <int S>
BlockFn sums_fn_shape(int shape, int r, int def) {
    return shape == SHAPE_BOX ? sums_fn_r<S, SHAPE_BOX>(r, def) : sums_fn_r<S, SHAPE_STAR>(r, def);
}

}  // namespace

BlockFn sums_lookup(int storage, int shape, int r, int def) {
    switch (storage) {
        case ST_F32: return sums_fn_shape<ST_F32>(shape, r, def);
        case ST_BF16: return sums_fn_shape<ST_BF16>(shape, r, def);
        case ST_F16: return sums_fn_shape<ST_F16>(shape, r, def);
    }
    return nullptr;
}

}  // namespace st

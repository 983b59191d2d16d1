// Batched sweep: many independent grids of uneven size and mixed stencil shape, run by one call.
//
// Small grids are resident: one workgroup keeps the grid for all of its steps, in registers where it
// fits a 128 x 128 tile with its halo (batched_block.hip), else in LDS, so it never round-trips through
// HBM.  The other grids run in passes: pass p of every grid of a stencil class is one multi-grid kernel
// whose workgroups each take one (grid, tile) of that pass on register tiles, or whose wavefronts each
// take one (grid, band, segment), so a pass of a class costs one launch instead of one per grid.  Passes
// follow each other on a stream, so the dependency of a tile on its neighbours' previous pass (the
// halo exchange of the paper's tiles, Sec. IV-B/C) is carried by the kernel boundary; with ST_FLAG_GRAPH
// the classes and the resident grids run on parallel branches, forked from and joined into the caller's
// stream.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <new>
#include <vector>

#include "batched.h"
#include "block_body.h"
#include "internal.h"
#include "march_body.h"
#include "sweep_body.h"

namespace st {

namespace {

constexpr int SIMDS = 1024;  // 256 compute units of four
constexpr int kRS = 8;  // rows per thread of the LDS-resident kernel

__device__ __forceinline__ void dispatch_resident(const BatchDesc& d, float* lds) {
    const int rows = int(d.rows), cols = int(d.cols);
    if (d.shape == SHAPE_BOX) {
        switch (d.r) {
            case 1: resident_body<1, SHAPE_BOX, kRS>(d.in, d.out, rows, cols, d.b, d.steps, d.w, lds); break;
            case 2: resident_body<2, SHAPE_BOX, kRS>(d.in, d.out, rows, cols, d.b, d.steps, d.w, lds); break;
            default: resident_body<3, SHAPE_BOX, kRS>(d.in, d.out, rows, cols, d.b, d.steps, d.w, lds); break;
        }
    } else {
        switch (d.r) {
            case 1: resident_body<1, SHAPE_STAR, kRS>(d.in, d.out, rows, cols, d.b, d.steps, d.w, lds); break;
            case 2: resident_body<2, SHAPE_STAR, kRS>(d.in, d.out, rows, cols, d.b, d.steps, d.w, lds); break;
            default: resident_body<3, SHAPE_STAR, kRS>(d.in, d.out, rows, cols, d.b, d.steps, d.w, lds); break;
        }
    }
}

// The LDS-resident grids: one workgroup per grid for all of its steps.
__global__ __launch_bounds__(NT) void batched_resident(const BatchDesc* desc, const int* res) {
    extern __shared__ float4 lds4[];
    dispatch_resident(desc[res[blockIdx.x]], reinterpret_cast<float*>(lds4));
}

// Marching engine: one launch runs `levels` (the template TB) levels of pass p for the grids
// order[s0 .. s0+n) of one stencil class; wavefront task -> (grid, band, segment) through the class's
// task prefix sums.  Four columns per lane, one vector access per lane and row at any alignment; grids
// narrower than a band run on register tiles.
struct MarchPassArgs {
    const BatchDesc* desc;
    const int* order;            // the class's grids, ordered by passes then last-pass depth, descending
    const int64_t* task_prefix;  // prefix sums of tasks over `order`
    int s0, n;                   // the slice of `order` this launch covers
    int p;                       // pass index
};

constexpr int MW = 4;  // wavefronts per workgroup of the marching engine
constexpr int MV = 4;  // columns per lane of the marching engine

// LDS of a batched marching workgroup: the input rows that the two wavefronts of a pair share (2 r tb
// rows of 64 lanes x 16 bytes per pair).
constexpr size_t march_share_bytes(int r, int tb) { return size_t(MW / 2) * 2 * r * tb * 64 * sizeof(float4); }

// (Star r = 3 at four levels takes 175 registers, two wavefronts per SIMD.  Held to 168 for three it keeps 13
// values in scratch, and 256 mixed grids with that class at this depth took 2.9-3.1 ms instead of 2.0.)
template <int R, int SH, int TB>
__global__ __launch_bounds__(64 * MW) void batched_march(MarchPassArgs a) {
    extern __shared__ float4 shared_rows[];
    const int lane = int(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int64_t* pre = a.task_prefix + a.s0;
    const int64_t task_in = pre[0] + int64_t(blockIdx.x) * MW + wave;
    const bool active = task_in < pre[a.n];
    // a wavefront past the launch's last task computes as that task (its setup is then a plain load
    // chain from the descriptor table, like the others') but stages nothing and stops at the barrier
    const int64_t task = active ? task_in : pre[a.n] - 1;
    // a grid's tasks go down each band in turn, so a workgroup's wavefronts take neighbouring
    // segments.  Wavefronts 0 and 2 march upwards and 1 and 3 downwards, so the pairs 0-1 and 2-3
    // meet at their start: each stages its own half of the 2 r tb input rows around the boundary in
    // LDS, and both read the whole overlap from there instead of reading it from HBM twice.
    const bool up = !(wave & 1);
    constexpr int H = march::halo_lanes(R, TB, MV);
    constexpr int64_t RT = int64_t(R) * TB;
    const int k = upper_index(pre, a.n + 1, task);
    const BatchDesc& d = a.desc[a.order[a.s0 + k]];
    const int64_t t = task - pre[k];
    const int64_t segi = t % d.tiles_y, band = t / d.tiles_y;
    const int64_t y0 = segi * d.seg;
    const int64_t y1 = y0 + d.seg < d.rows ? y0 + d.seg : d.rows;
    // the partner: the next task for an upward wavefront, the previous one for a downward one
    const int64_t pt = up ? task + 1 : task - 1;
    bool paired = false;
    if (active && pt >= pre[k] && pt < pre[k + 1] && pt < pre[a.n]) {
        const int64_t tp = pt - pre[k];
        paired = tp / d.tiles_y == band && (up ? tp % d.tiles_y == segi + 1 : tp % d.tiles_y + 1 == segi);
    }
    const int64_t yb = up ? y1 : y0;  // the pair's boundary
    const int P = d.passes, p = a.p;
    const float* src = p == 0 ? d.in : (((P - p) % 2 == 0) ? d.out : d.ws);  // written by pass p-1
    float* dst = ((P - 1 - p) % 2 == 0) ? d.out : d.ws;
    const march::MarchView v{src, dst, d.rows, d.cols, d.b, march::BC_CONST, nullptr};
    const march::BandCols bc = march::band_cols(d.cols, d.tiles_x, d.zero_sides, band, MV, H);
    const int64_t X0 = bc.x0;
    float4* mine = shared_rows + (wave >> 1) * (2 * RT * 64);
    if (paired) {  // each stages the rows on its own side of the boundary
        march::stage_rows<ST_F32, R, MV, TB>(v, lane, y0, y1, X0, up ? yb - RT : yb, yb - RT, mine);
    }
    __syncthreads();  // every wavefront of the workgroup reaches it once
    if (!active) return;
    const march::SharedRows sh{paired ? mine : nullptr, yb - RT, yb + RT};
    // input rows in flight: one ring length, except box r >= 3 with several levels (registers)
    constexpr int D = SH == SHAPE_STAR || R <= 2 || TB == 1 ? 2 * R + 1 : 0;
    march::march_task_dir<ST_F32, R, MV, SH, TB, D>(v, d.w, lane, y0, y1, X0, up, sh, bc.lo, bc.hi);
}

using MarchPassFn = void (*)(MarchPassArgs);

template <int SH>
MarchPassFn batched_march_fn(int r, int levels) {
#define ST_BMARCH(R, TB) \
    if (r == R && levels == TB) return batched_march<R, SH, TB>;
    if constexpr (SH == SHAPE_STAR) {
        ST_BMARCH(1, 1) ST_BMARCH(1, 2) ST_BMARCH(1, 3) ST_BMARCH(1, 4) ST_BMARCH(1, 5) ST_BMARCH(1, 6)
        ST_BMARCH(1, 7) ST_BMARCH(1, 8)
        ST_BMARCH(2, 1) ST_BMARCH(2, 2) ST_BMARCH(2, 3) ST_BMARCH(2, 4) ST_BMARCH(2, 5) ST_BMARCH(2, 6)
        ST_BMARCH(3, 1) ST_BMARCH(3, 2) ST_BMARCH(3, 3) ST_BMARCH(3, 4)
    } else {
        ST_BMARCH(1, 1) ST_BMARCH(1, 2) ST_BMARCH(1, 3) ST_BMARCH(1, 4) ST_BMARCH(1, 5) ST_BMARCH(1, 6)
        ST_BMARCH(2, 1) ST_BMARCH(2, 2) ST_BMARCH(2, 3)
        ST_BMARCH(3, 1) ST_BMARCH(3, 2)
    }
#undef ST_BMARCH
    return nullptr;
}

MarchPassFn batched_march_lookup(int shape, int r, int levels) {
    return shape == SHAPE_BOX ? batched_march_fn<SHAPE_BOX>(r, levels) : batched_march_fn<SHAPE_STAR>(r, levels);
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// The branches of a batch: the LDS-resident grids, each class's one-workgroup grids, and each class's
// passes on either engine.
constexpr int BRANCHES = 19;

// Each branch's stream and the event that joins it, made when the branch is first used and kept as long as
// the batch.  (A hipGraph per batch, captured from such streams and made again whenever a class changed,
// ended the process in a host segmentation fault now and then, three times on record, each in a run that
// captured, instantiated and destroyed many of them; the cause was not found, so nothing is captured.)
struct Branches {
    hipStream_t side[BRANCHES] = {};
    hipEvent_t fork = nullptr, join[BRANCHES] = {};
    bool make(int i) {
        return (fork || hipEventCreateWithFlags(&fork, hipEventDisableTiming) == hipSuccess) &&
               (side[i] || hipStreamCreateWithFlags(&side[i], hipStreamNonBlocking) == hipSuccess) &&
               (join[i] || hipEventCreateWithFlags(&join[i], hipEventDisableTiming) == hipSuccess);
    }
    ~Branches() {
        for (int i = 0; i < BRANCHES; ++i)
            if (side[i]) (void)hipStreamSynchronize(side[i]);
        for (int i = 0; i < BRANCHES; ++i) {
            if (join[i]) (void)hipEventDestroy(join[i]);
            if (side[i]) (void)hipStreamDestroy(side[i]);
        }
        if (fork) (void)hipEventDestroy(fork);
    }
};

}  // namespace

}  // namespace st

using namespace st;

struct st_batch {
    int n;
    uint32_t flags;
    std::vector<BatchDesc> desc;
    std::vector<int> res;              // one-workgroup grids: LDS-resident, then each class's on register tiles
    int n_lds;                         // the LDS-resident ones
    int whole_first[6], whole_n[6];    // per class: its grids on register tiles in `res`
    std::vector<int> zero_steps;       // grids with steps == 0 (copied, not computed)
    std::vector<int> tiled;            // grids that are neither resident nor zero-step, in input order
    std::vector<int> tb_max, plan_tb;  // per grid: deepest pass on register tiles, and its plan's
    // per stencil class (slot = shape * 3 + r - 1): engine (0 = register tiles, 1 = marching) and depth
    int engine[6], depth[6];
    int64_t seg_min[6];  // marching: least output rows per task (0: the tasks about fill the device once)
    struct MLaunch {
        int s0, n, p, levels;
        int64_t tasks;
    };
    struct Passes {
        int64_t seg = 0;               // marching: output rows per task (the longest a grid's segment may be)
        int def = 0;                   // register tiles: which of block::kDefs
        std::vector<int> order;        // the class's grids by passes, then last-pass depth
        std::vector<int64_t> prefix;   // task (tile) prefix sums over `order`
        std::vector<MLaunch> launches; // in pass order
    } march[6], tile[6];               // per class, its grids on either engine
    size_t off_desc, off_res, off_order[12], off_prefix[12], off_fields, ws_bytes;  // tables: march, then tile
    std::vector<size_t> field_off;     // per grid: workspace offset of its ping-pong field (0 = none)
    size_t lds_res;
    Branches branches;  // ST_FLAG_GRAPH only
    // staging
    void* pinned;
    size_t pinned_bytes;
    hipEvent_t staged;
    bool staged_valid;
    std::vector<const void*> last_in;
    std::vector<void*> last_out;
    void* last_ws;
};

namespace {

// LDS budget per workgroup of the batched kernels: two workgroups per CU when the device allows
// 80 KiB per workgroup.
size_t batch_lds_budget() { return std::min<size_t>(80 * 1024, lds_limit()); }

}  // namespace

// Whether grids of this width march when their class does: narrower than a band, they would leave lanes idle.
static bool marches_at(int64_t cols) { return cols >= 64 * MV; }

static int class_slot(const BatchDesc& d) { return d.shape * 3 + d.r - 1; }

// Whether a grid and the halo around it fit the tile of batched_whole.
static bool fits_tile(const BatchDesc& d) {
    const block::Def& t = block::kDefs[block::kTall];
    return d.rows + 2 * d.r <= t.nw * t.rw && d.cols + block::margin_cols(d.r, 1, t.v) + d.r <= 64 * t.v;
}

// Marching engine: output rows per task for a class, so that its tasks about fill the device once
// (`waves`: the wavefronts of the class's kernel the device holds at once).
static int64_t march_segment(int64_t band_rows, int64_t waves) {
    const int64_t seg = (band_rows + waves - 1) / waves;
    return std::min<int64_t>(2048, std::max<int64_t>(8, seg));
}

// Wavefronts of the marching kernel for (shape, radius, depth) resident at once (4096 if unknown).
static int64_t march_waves(int shape, int r, int tb) {
    MarchPassFn fn = batched_march_lookup(shape, r, tb);
    int blocks = 0;
    if (!fn || resident_blocks(reinterpret_cast<const void*>(fn), march_share_bytes(r, tb), &blocks) != ST_OK ||
        blocks < 1) {
        (void)hipGetLastError();
        return 4096;
    }
    return int64_t(blocks) * MW;
}

// Depth of a grid's deepest pass on register tiles: its steps spread evenly over the passes.
static int even_depth(const BatchDesc& d) { return (d.steps + d.passes - 1) / d.passes; }

// Register tile of a class: the least estimated time, from the instructions that a wavefront issues per level
// (its cells' taps, a few per row, and the exchange), over the SIMDs the device has, plus one workgroup's own
// time, which is what small batches wait for.  A tile must keep a quarter of its sides as block::cover asks.
static int class_tile(const st_batch* B, const std::vector<int>& grids) {
    int best = block::kTall;
    double best_t = HUGE_VAL;
    for (int def = 0; def <= block::kTall; ++def) {
        const block::Def& t = block::kDefs[def];
        double work = 0.0;
        int steps = 0;
        bool fits = true;
        double level = 0.0;
        for (int g : grids) {
            const BatchDesc& d = B->desc[g];
            const block::Cover c = block::cover(def, d.r, even_depth(d), d.rows, d.cols);
            fits = fits && c.def == def;
            const int taps = d.shape == SHAPE_BOX ? (2 * d.r + 1) * (2 * d.r + 1) : 4 * d.r + 1;
            level = t.rw * t.v * (taps + 1.0) + 6.0 * t.rw + 40.0;
            work += double(c.tiles) * t.nw * level * d.steps;
            steps = std::max(steps, d.steps);
        }
        const double time = work / SIMDS + level * steps * t.nw / 4.0;
        if (fits && time < best_t) {
            best_t = time;
            best = def;
        }
    }
    return best;
}

// Pass structure from each class's engine and depth: the order by (passes, depth of the last pass)
// descending, the task or tile prefix sums, and the launches.  Register tiles: at pass p the grids with
// more than p passes are a prefix of the order, one launch.  Marching: bands and segments per grid; at pass
// p the full-depth grids are a prefix of the order and the grids finishing with a shallower pass follow in
// groups of equal depth.
static void build_passes(st_batch* B) {
    for (int c = 0; c < 6; ++c) B->march[c] = B->tile[c] = st_batch::Passes();
    for (int g : B->tiled) {
        BatchDesc& d = B->desc[g];
        const int c = class_slot(d);
        const bool marches = B->engine[c] == 1 && marches_at(d.cols);
        // (beside a marching class its narrow grids take about twelve rows of margin: 80 grids 110 to 255 wide, 40
        // steps, us at 2 levels / 12 / r / more: star r = 1 641 / 361 / 357, r = 2 862 / 702 / 674, r = 3 1418 / 1140
        // / 1562, box r = 1 834 / 633 / 644, r = 2 1438 / 1369 / 1459, r = 3 2447 / 2476 / 3850)
        d.tb = marches ? B->depth[c]
                       : std::min(B->engine[c] == 1 ? 12 / d.r : B->depth[c] > 0 ? B->depth[c] : B->plan_tb[g], B->tb_max[g]);
        d.passes = (d.steps + d.tb - 1) / d.tb;
        if (marches) {
            const float zero = 0.0f;
            d.zero_sides = std::memcmp(&d.b, &zero, sizeof zero) == 0 && d.cols >= 2 * 64 * MV;
            d.tiles_x = march::band_count(d.cols, MV, march::halo_lanes(d.r, d.tb, MV), d.zero_sides);
        }
        (marches ? B->march : B->tile)[c].order.push_back(g);
    }
    for (int c = 0; c < 6; ++c) {
        st_batch::Passes& M = B->tile[c];
        if (M.order.empty()) continue;
        std::stable_sort(M.order.begin(), M.order.end(), [&](int a, int b) { return B->desc[a].passes > B->desc[b].passes; });
        M.def = class_tile(B, M.order);
        M.prefix.assign(1, 0);
        for (int g : M.order) {
            BatchDesc& d = B->desc[g];
            const block::Cover t = block::cover(M.def, d.r, even_depth(d), d.rows, d.cols);
            d.tiles_x = t.tiles_x;
            d.tiles_y = t.tiles / t.tiles_x;
            M.prefix.push_back(M.prefix.back() + t.tiles);
        }
        int n = int(M.order.size());
        for (int p = 0; p < B->desc[M.order[0]].passes; ++p) {
            while (B->desc[M.order[n - 1]].passes <= p) --n;
            M.launches.push_back({0, n, p, 0, M.prefix[n]});
        }
    }
    for (int c = 0; c < 6; ++c) {
        st_batch::Passes& M = B->march[c];
        if (M.order.empty()) continue;
        const int tb = B->depth[c];
        auto last_depth = [&](int g) { return B->desc[g].steps - (B->desc[g].passes - 1) * tb; };
        std::stable_sort(M.order.begin(), M.order.end(), [&](int a, int b) {
            const BatchDesc &da = B->desc[a], &db = B->desc[b];
            return da.passes != db.passes ? da.passes > db.passes : last_depth(a) > last_depth(b);
        });
        int64_t band_rows = 0;
        for (int g : M.order) band_rows += B->desc[g].tiles_x * B->desc[g].rows;
        const int64_t seg =
            std::max(march_segment(band_rows, march_waves(c / 3, c % 3 + 1, tb)), B->seg_min[c]);
        M.seg = seg;
        M.prefix.assign(1, 0);
        for (int g : M.order) {
            BatchDesc& d = B->desc[g];
            d.seg = std::min<int64_t>(seg, d.rows);
            d.tiles_y = (d.rows + d.seg - 1) / d.seg;  // segments
            M.prefix.push_back(M.prefix.back() + d.tiles_x * d.tiles_y);
        }
        const int P = B->desc[M.order[0]].passes;
        const int n = int(M.order.size());
        for (int p = 0; p < P; ++p) {
            // grids at pass p: passes > p (a prefix); those with passes == p + 1 run their last depth
            int a = 0;
            while (a < n && B->desc[M.order[a]].passes > p) ++a;
            int full = 0;
            while (full < a && (B->desc[M.order[full]].passes > p + 1 || last_depth(M.order[full]) == tb)) ++full;
            auto push = [&](int s0, int e, int levels) {
                if (e > s0) M.launches.push_back({s0, e - s0, p, levels, M.prefix[e] - M.prefix[s0]});
            };
            push(0, full, tb);
            for (int s0 = full; s0 < a;) {
                const int lv = last_depth(M.order[s0]);
                int e = s0;
                while (e < a && last_depth(M.order[e]) == lv) ++e;
                push(s0, e, lv);
                s0 = e;
            }
        }
    }
}

extern "C" int stencil_batch_create(st_batch** out, int n, st_plan* const* plans, const int64_t* steps,
                                    uint32_t flags) {
    if (!out) return fail(ST_EINVAL, "out is NULL");
    *out = nullptr;
    if (n < 1 || !plans || !steps) return fail(ST_EINVAL, "need n >= 1 plans and steps");
    if (flags & ~ST_FLAG_GRAPH) return fail(ST_EINVAL, "unknown batch flag bits");
    st_batch* B = new (std::nothrow) st_batch();
    if (!B) return fail(ST_ENOMEM, "batch allocation failed");
    B->n = n;
    B->flags = flags;
    B->desc.resize(n);
    B->field_off.assign(n, 0);
    B->tb_max.assign(n, 0);
    B->plan_tb.assign(n, 0);
    std::vector<int> tiled, whole[6];
    size_t lds_res = 0;
    for (int g = 0; g < n; ++g) {
        const st_plan* p = plans[g];
        if (!p || steps[g] < 0 || steps[g] > (int64_t(1) << 30)) {
            delete B;
            return fail(ST_EINVAL, "NULL plan, or steps outside [0, 2^30]");
        }
        if (p->kind != KIND_CONST || p->storage != ST_F32 || p->radius > 3 || p->bc != ST_BC_CONST) {
            delete B;
            return fail(ST_EUNSUPPORTED, "batched grids must be FP32 constant-weight plans with a constant halo, r <= 3");
        }
        BatchDesc& d = B->desc[g];
        std::memset(&d, 0, sizeof(d));
        d.rows = p->rows;
        d.cols = p->cols;
        d.r = p->radius;
        d.shape = p->shape;
        d.b = p->bq;
        d.steps = int(steps[g]);
        std::memcpy(d.w, p->w, sizeof(d.w));
        if (steps[g] == 0) {  // plain copy in -> out, enqueued by stencil_run_batched
            B->zero_steps.push_back(g);
            continue;
        }
        const size_t rl = resident_lds_bytes(p->radius, p->rows, p->cols);
        if (rl <= batch_lds_budget()) {
            d.resident = 1;
            d.passes = 1;
            d.tb = d.steps;
            if (fits_tile(d)) {
                whole[class_slot(d)].push_back(g);
            } else {
                lds_res = std::max(lds_res, rl);
                B->res.push_back(g);
            }
            continue;
        }
        // deepest pass that leaves a third of the tallest tile; the plan's depth, capped by it, is the
        // starting point
        B->tb_max[g] = std::min(16, 39 / p->radius);
        B->plan_tb[g] = std::max(1, p->tb);
        tiled.push_back(g);
    }
    B->tiled = tiled;
    B->n_lds = int(B->res.size());
    for (int c = 0; c < 6; ++c) {
        B->whole_first[c] = int(B->res.size());
        B->whole_n[c] = int(whole[c].size());
        B->res.insert(B->res.end(), whole[c].begin(), whole[c].end());
    }
    for (int c = 0; c < 6; ++c) {
        B->engine[c] = 0;
        B->depth[c] = 0;  // 0: each grid keeps its plan's depth (capped)
        B->seg_min[c] = 0;
    }
    build_passes(B);
    // workspace: descriptor table, queue tables, one ping-pong field per tiled grid with two or more
    // steps (any depth the autotuner may pick below the step count needs it)
    size_t off = 0;
    B->off_desc = off;
    off = align256(off + size_t(n) * sizeof(BatchDesc));
    B->off_res = off;
    off = align256(off + std::max<size_t>(B->res.size(), 1) * sizeof(int));
    for (int t = 0; t < 12; ++t) {  // room for every grid of the class on either engine
        const size_t m = size_t(std::count_if(tiled.begin(), tiled.end(), [&](int g) { return class_slot(B->desc[g]) == t % 6; }));
        B->off_order[t] = off;
        off = align256(off + std::max<size_t>(m, 1) * sizeof(int));
        B->off_prefix[t] = off;
        off = align256(off + (m + 1) * sizeof(int64_t));
    }
    B->off_fields = off;
    for (int g : tiled) {
        if (B->desc[g].steps >= 2) {
            B->field_off[g] = off;
            off = align256(off + size_t(B->desc[g].rows * B->desc[g].cols) * sizeof(float));
        }
    }
    B->ws_bytes = std::max<size_t>(off, 256);
    B->lds_res = lds_res;
    B->pinned = nullptr;
    B->pinned_bytes = B->off_fields - B->off_desc;
    B->staged = nullptr;
    B->staged_valid = false;
    B->last_ws = nullptr;
    *out = B;
    return ST_OK;
}

extern "C" int stencil_batch_workspace_bytes(const st_batch* batch, size_t* bytes) {
    if (!batch || !bytes) return fail(ST_EINVAL, "NULL argument");
    *bytes = batch->ws_bytes;
    return ST_OK;
}

extern "C" int stencil_batch_destroy(st_batch* batch) {
    if (!batch) return ST_OK;
    if (batch->staged) {
        (void)hipEventSynchronize(batch->staged);
        (void)hipEventDestroy(batch->staged);
    }
    if (batch->pinned) (void)hipHostFree(batch->pinned);
    delete batch;
    return ST_OK;
}

// The launches of table t (march[0 .. 5], then tile[0 .. 5]), in pass order, on stream `s`.
static const st_batch::Passes& passes_of(const st_batch* B, int t) { return t < 6 ? B->march[t] : B->tile[t - 6]; }
static int enqueue_passes(st_batch* B, int t, char* ws, hipStream_t s) {
    const st_batch::Passes& M = passes_of(B, t);
    const BatchDesc& d0 = B->desc[M.order[0]];
    const BatchDesc* desc = reinterpret_cast<const BatchDesc*>(ws + B->off_desc);
    const int* order = reinterpret_cast<const int*>(ws + B->off_order[t]);
    const int64_t* prefix = reinterpret_cast<const int64_t*>(ws + B->off_prefix[t]);
    for (const st_batch::MLaunch& L : M.launches) {
        clear_stale_error();
        if (t >= 6) {
            if (L.tasks >= int64_t(1) << 31) return fail(ST_EUNSUPPORTED, "too many tiles for one launch");
            const block::Def& tile = block::kDefs[M.def];
            BlockPassFn fn = batched_block_lookup(d0.shape, d0.r, M.def);
            const size_t lds = block::lds_floats(d0.r, tile.v, tile.rw, tile.nw) * sizeof(float);
            if (int rc = prepare_lds(reinterpret_cast<const void*>(fn), lds)) return rc;
            launch_runs(L.tasks, 64 * tile.nw, [&](int64_t first, int64_t n) {
                hipLaunchKernelGGL(fn, dim3(unsigned(n)), dim3(64 * tile.nw), lds, s, BlockPassArgs{desc, order, prefix, L.n, L.p, first});
            });
            ST_LAUNCH_CHECK("batched_block");
            continue;
        }
        MarchPassFn fn = batched_march_lookup(d0.shape, d0.r, L.levels);
        if (!fn) return fail(ST_EUNSUPPORTED, "no batched marching kernel for this class/depth");
        MarchPassArgs a;
        a.desc = desc;
        a.order = order;
        a.task_prefix = prefix;
        a.s0 = L.s0;
        a.n = L.n;
        a.p = L.p;
        const int64_t blocks = (L.tasks + MW - 1) / MW;
        hipLaunchKernelGGL(fn, dim3(unsigned(blocks)), dim3(64 * MW), march_share_bytes(d0.r, L.levels), s, a);
        ST_LAUNCH_CHECK("batched_march");
    }
    return ST_OK;
}

// Class c's grids that one workgroup each keeps in registers.
static int enqueue_whole(st_batch* B, int c, char* ws, hipStream_t s) {
    const BatchDesc& d0 = B->desc[B->res[size_t(B->whole_first[c])]];
    const block::Def& t = block::kDefs[block::kTall];
    BlockPassFn fn = batched_whole_lookup(d0.shape, d0.r);
    const size_t lds = block::lds_floats(d0.r, t.v, t.rw, t.nw) * sizeof(float);
    if (int rc = prepare_lds(reinterpret_cast<const void*>(fn), lds)) return rc;
    clear_stale_error();
    hipLaunchKernelGGL(fn, dim3(unsigned(B->whole_n[c])), dim3(64 * t.nw), lds, s,
                       BlockPassArgs{reinterpret_cast<const BatchDesc*>(ws + B->off_desc),
                                     reinterpret_cast<const int*>(ws + B->off_res) + B->whole_first[c], nullptr, B->whole_n[c], -1, 0});
    ST_LAUNCH_CHECK("batched_whole");
    return ST_OK;
}

static bool branch_used(const st_batch* B, int i) {
    if (i == 0) return B->n_lds > 0;
    return i <= 6 ? B->whole_n[i - 1] > 0 : !passes_of(B, i - 7).order.empty();
}
static int enqueue_branch(st_batch* B, int i, char* ws, hipStream_t s) {
    if (i > 6) return enqueue_passes(B, i - 7, ws, s);
    if (i > 0) return enqueue_whole(B, i - 1, ws, s);
    if (int rc = prepare_lds(reinterpret_cast<const void*>(batched_resident), B->lds_res)) return rc;
    clear_stale_error();
    hipLaunchKernelGGL(batched_resident, dim3(unsigned(B->n_lds)), dim3(NT), B->lds_res, s,
                       reinterpret_cast<const BatchDesc*>(ws + B->off_desc), reinterpret_cast<const int*>(ws + B->off_res));
    ST_LAUNCH_CHECK("batched_resident");
    return ST_OK;
}

// Enqueue the batch's kernels: with ST_FLAG_GRAPH, where there is more than one branch, each on its own
// stream forked from and joined into `s`.  A caller that captures `s` gets them one after another.
static int enqueue_batch(st_batch* B, char* ws, hipStream_t s) {
    int used = 0;
    for (int i = 0; i < BRANCHES; ++i) used += branch_used(B, i);
    bool fork = (B->flags & ST_FLAG_GRAPH) && used > 1;
    if (fork) {
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &st) != hipSuccess) clear_stale_error();
        fork = st == hipStreamCaptureStatusNone;
    }
    Branches& br = B->branches;
    if (fork) {
        for (int i = 0; i < BRANCHES; ++i)
            if (branch_used(B, i) && !br.make(i)) return fail(ST_EHIP, "stream/event creation failed");
        ST_HIP_CHECK(hipEventRecord(br.fork, s));
    }
    // A failed branch ends the loop, but what was enqueued before it is joined all the same: the caller's
    // stream is the only one that the caller can wait for.
    int rc = ST_OK;
    hipError_t e = hipSuccess;
    for (int i = 0; i < BRANCHES && !rc && e == hipSuccess; ++i) {
        if (!branch_used(B, i)) continue;
        if (fork && (e = hipStreamWaitEvent(br.side[i], br.fork, 0)) != hipSuccess) break;
        rc = enqueue_branch(B, i, ws, fork ? br.side[i] : s);
        if (!fork) continue;
        e = hipEventRecord(br.join[i], br.side[i]);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, br.join[i], 0);
        if (e != hipSuccess) (void)hipStreamSynchronize(br.side[i]);
    }
    if (!rc && e != hipSuccess) {
        clear_stale_error();
        rc = fail(ST_EHIP, std::string("fork/join of the batch's streams: ") + hipGetErrorString(e));
    }
    return rc;
}

extern "C" int stencil_run_batched(st_batch* B, const void* const* ins, void* const* outs, void* workspace,
                                   size_t ws_bytes, void* stream) {
    if (!B || !ins || !outs) return fail(ST_EINVAL, "NULL argument");
    if (!workspace || ws_bytes < B->ws_bytes) return fail(ST_ENOWS, "workspace too small");
    for (int g = 0; g < B->n; ++g) {
        if (!ins[g] || !outs[g]) return fail(ST_EINVAL, "NULL grid pointer");
        const size_t bytes = size_t(B->desc[g].rows * B->desc[g].cols) * sizeof(float);
        const char* x = static_cast<const char*>(ins[g]);
        const char* y = static_cast<const char*>(outs[g]);
        if (x < y + bytes && y < x + bytes) return fail(ST_EALIAS, "in and out overlap");
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    // stage the descriptor tables when any pointer changed since the last run
    bool changed = !B->staged_valid || B->last_ws != workspace;
    for (int g = 0; g < B->n && !changed; ++g) changed = B->last_in[g] != ins[g] || B->last_out[g] != outs[g];
    if (changed) {
        if (!B->pinned) {
            ST_HIP_CHECK(hipHostMalloc(&B->pinned, B->pinned_bytes, hipHostMallocDefault));
            ST_HIP_CHECK(hipEventCreateWithFlags(&B->staged, hipEventDisableTiming));
        } else {
            ST_HIP_CHECK(hipEventSynchronize(B->staged));  // the previous copy out of the staging buffer is done
        }
        char* h = static_cast<char*>(B->pinned);
        for (int g = 0; g < B->n; ++g) {
            BatchDesc d = B->desc[g];
            d.in = static_cast<const float*>(ins[g]);
            d.out = static_cast<float*>(outs[g]);
            d.ws = B->field_off[g] ? reinterpret_cast<float*>(ws + B->field_off[g]) : nullptr;
            std::memcpy(h + g * sizeof(BatchDesc), &d, sizeof(d));
        }
        if (!B->res.empty()) std::memcpy(h + (B->off_res - B->off_desc), B->res.data(), B->res.size() * sizeof(int));
        for (int t = 0; t < 12; ++t) {
            const st_batch::Passes& M = passes_of(B, t);
            if (M.order.empty()) continue;
            std::memcpy(h + (B->off_order[t] - B->off_desc), M.order.data(), M.order.size() * sizeof(int));
            std::memcpy(h + (B->off_prefix[t] - B->off_desc), M.prefix.data(), M.prefix.size() * sizeof(int64_t));
        }
        ST_HIP_CHECK(hipMemcpyAsync(ws + B->off_desc, h, B->pinned_bytes, hipMemcpyHostToDevice, s));
        ST_HIP_CHECK(hipEventRecord(B->staged, s));
        B->staged_valid = true;
        B->last_in.assign(ins, ins + B->n);
        B->last_out.assign(outs, outs + B->n);
        B->last_ws = workspace;
    }
    for (int g : B->zero_steps)
        ST_HIP_CHECK(hipMemcpyAsync(outs[g], ins[g], size_t(B->desc[g].rows * B->desc[g].cols) * sizeof(float),
                                    hipMemcpyDeviceToDevice, s));
    return enqueue_batch(B, ws, s);
}

extern "C" int stencil_batch_set_class(st_batch* B, int shape, int radius, int engine, int depth) {
    if (!B) return fail(ST_EINVAL, "batch is NULL");
    if ((shape != SHAPE_STAR && shape != SHAPE_BOX) || radius < 1 || radius > 3 || (engine != 0 && engine != 1))
        return fail(ST_EINVAL, "bad class or engine");
    if (depth < 1 || depth > 16 || (engine == 1 && depth > march_max_tb(shape, radius, 1)))
        return fail(ST_EUNSUPPORTED, "depth out of range for this engine");
    const int c = shape * 3 + radius - 1;
    B->engine[c] = engine;
    B->depth[c] = depth;
    build_passes(B);
    B->staged_valid = false;
    return ST_OK;
}

extern "C" int stencil_batch_set_segment(st_batch* B, int shape, int radius, int64_t min_rows) {
    if (!B) return fail(ST_EINVAL, "batch is NULL");
    if ((shape != SHAPE_STAR && shape != SHAPE_BOX) || radius < 1 || radius > 3 || min_rows < 0)
        return fail(ST_EINVAL, "bad class or segment length");
    const int c = shape * 3 + radius - 1;
    B->seg_min[c] = min_rows;
    build_passes(B);
    B->staged_valid = false;
    return ST_OK;
}

extern "C" int stencil_batch_get_segment(const st_batch* B, int shape, int radius, int64_t* rows) {
    if (!B || !rows) return fail(ST_EINVAL, "NULL argument");
    if ((shape != SHAPE_STAR && shape != SHAPE_BOX) || radius < 1 || radius > 3)
        return fail(ST_EINVAL, "bad class");
    const int c = shape * 3 + radius - 1;
    *rows = B->march[c].order.empty() ? 0 : B->march[c].seg;
    return ST_OK;
}

// Coordinate descent over the stencil classes (shape, radius) of the non-resident grids: for each
// class in turn, time the whole batch (branches that run beside each other share the device, so what is
// fastest alone need not be) with every candidate engine and depth -- register
// tiles with the class's depth capped at 1, 2, 3, 4, 6, 8, 12 or 16, or marching with 1 .. the
// deepest its radius allows, each marching depth with the default segments and with those that make
// at most one, two, three or four tasks per SIMD (a pass waits for its busiest SIMD) --
// keep the fastest, then move to the next class; then each class's best six once more.
extern "C" int stencil_batch_autotune(st_batch* B, const void* const* ins, void* const* outs, void* workspace,
                                      size_t ws_bytes, int* tb_out, int* engine_out, void* stream) {
    if (!B || !ins || !outs) return fail(ST_EINVAL, "NULL argument");
    if (!workspace || ws_bytes < B->ws_bytes) return fail(ST_ENOWS, "workspace too small");
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (tb_out) std::fill(tb_out, tb_out + 6, 0);
    if (engine_out) std::fill(engine_out, engine_out + 6, 0);
    bool present[6] = {}, wide[6] = {};  // (wide: some grid of the class marches)
    int deepest[6] = {};
    for (int g : B->tiled) {
        const int c = class_slot(B->desc[g]);
        present[c] = true;
        wide[c] = wide[c] || marches_at(B->desc[g].cols);
        deepest[c] = std::max(deepest[c], B->tb_max[g]);
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = ST_OK;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) rc = fail(ST_EHIP, "hipEventCreate");
    // fill: marching segments such that the class's tasks are at most that many wavefronts a SIMD
    auto apply = [&](int c, int engine, int depth, int fill) {
        B->engine[c] = engine;
        B->depth[c] = depth;
        B->seg_min[c] = 0;
        build_passes(B);
        if (engine == 1 && fill && !B->march[c].order.empty()) {
            auto tasks = [&](int64_t seg) {
                int64_t n = 0;
                for (int g : B->march[c].order) n += B->desc[g].tiles_x * ((B->desc[g].rows + seg - 1) / seg);
                return n;
            };
            int64_t lo = 1, hi = int64_t(1) << 31;  // the shortest segment that fits
            while (lo < hi) {
                const int64_t mid = lo + (hi - lo) / 2;
                if (tasks(mid) <= int64_t(SIMDS) * fill) hi = mid; else lo = mid + 1;
            }
            if (lo < int64_t(1) << 31) {
                B->seg_min[c] = lo;
                build_passes(B);
            }
        }
        B->staged_valid = false;  // descriptor tables changed
    };
    // the fastest of `runs` runs after one that warms up and stages the tables
    auto timed = [&](int runs, float* ms) -> int {
        if (int r = stencil_run_batched(B, ins, outs, workspace, ws_bytes, stream)) return r;
        *ms = 1e30f;
        for (int i = 0; i < runs; ++i) {
            if (hipEventRecord(e0, s) != hipSuccess) return fail(ST_EHIP, "hipEventRecord");
            if (int r = stencil_run_batched(B, ins, outs, workspace, ws_bytes, stream)) return r;
            float t = 0.0f;
            if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                hipEventElapsedTime(&t, e0, e1) != hipSuccess)
                return fail(ST_EHIP, "hipEventRecord/Synchronize/ElapsedTime");
            *ms = std::min(*ms, t);
        }
        return ST_OK;
    };
    static const int kCaps[] = {1, 2, 3, 4, 6, 8, 12, 16};
    struct Cand {
        int engine, depth, fill;
        float ms;
    };
    std::vector<Cand> cands[6];
    // every candidate once, the other classes as they are; then each class's best few again, the others tuned
    for (int sweep = 0; sweep < 2; ++sweep)
        for (int c = 0; c < 6 && rc == ST_OK; ++c) {
            if (!present[c]) continue;
            std::vector<Cand>& cs = cands[c];
            if (sweep == 0) {
                for (int cap : kCaps)
                    if (cap <= deepest[c]) cs.push_back({0, cap, 0, 0.0f});
                for (int t = 1; wide[c] && t <= march_max_tb(c / 3, c % 3 + 1, 1); ++t)
                    for (int m : {0, 1, 2, 3, 4}) cs.push_back({1, t, m, 0.0f});
            }
            for (Cand& cd : cs) {
                apply(c, cd.engine, cd.depth, cd.fill);
                if ((rc = timed(1 + 2 * sweep, &cd.ms))) break;
            }
            if (rc) break;
            std::stable_sort(cs.begin(), cs.end(), [](const Cand& x, const Cand& y) { return x.ms < y.ms; });
            cs.resize(std::min<size_t>(cs.size(), 6));
            apply(c, cs[0].engine, cs[0].depth, cs[0].fill);
            if (tb_out) tb_out[c] = cs[0].depth;
            if (engine_out) engine_out[c] = cs[0].engine;
        }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    return rc;
}

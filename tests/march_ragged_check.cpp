// Host check of the row-marching layout at widths that are no multiple of a lane's columns: every lane of
// every band holds V columns of the grid or none, and the stored lanes cover the grid and lie deep enough
// inside their band's loaded columns (or the grid's side) to be exact.
#include <algorithm>
#include <cstdio>
#include <utility>
#include <vector>

#include "../paper_2605_07954_amd/csrc/march_layout.h"

using namespace st::march;

int main() {
    long layouts = 0;
    for (int V : {4, 8})
        for (int r = 1; r <= 4; ++r)
            for (int levels = 1; levels <= 8; ++levels) {
                const int H = halo_lanes(r, levels, V), reach = r * levels;
                if (64 - 2 * H < 2) continue;
                for (int64_t cols = 64 * V; cols < 64 * V * 6; ++cols) {
                    if (!whole_lanes(cols, V)) return std::printf("FAIL whole_lanes %lld %d\n", (long long)cols, V), 1;
                    for (int zs = 0; zs <= (cols >= 128 * V); ++zs) {
                        TaskMap m{};
                        if (!plan_march_tasks(m, 300, cols, V, r, levels, 4 * r + 1, 2048, 0, zs != 0))
                            return std::printf("FAIL no layout\n"), 1;
                        std::vector<std::pair<int64_t, int64_t>> spans;
                        for (int b = 0; b < m.bands; ++b) {
                            const BandCols c = band_cols(m, b, V, H);
                            const int lo = c.lo < 0 ? H : c.lo, hi = c.hi < 0 ? 64 - H : c.hi;
                            for (int lane = 0; lane < 64; ++lane) {
                                const int64_t g = c.x0 + int64_t(V) * lane;
                                const int64_t in = std::min(cols, g + V) - std::max<int64_t>(0, g);
                                if (in > 0 && in < V)
                                    return std::printf("FAIL cols %lld V %d r %d levels %d zs %d: band %d lane %d straddles\n",
                                                       (long long)cols, V, r, levels, zs, b, lane), 1;
                            }
                            const int64_t s0 = std::max<int64_t>(0, c.x0 + int64_t(V) * lo), s1 = std::min(cols, c.x0 + int64_t(V) * hi);
                            const bool left = s0 - c.x0 >= reach || (s0 == 0 && c.x0 == 0 && zs), right = c.x0 + 64 * V - s1 >= reach || (s1 == cols && zs);
                            if (!left || !right)
                                return std::printf("FAIL cols %lld V %d r %d levels %d zs %d: band %d stores too far out\n",
                                                   (long long)cols, V, r, levels, zs, b), 1;
                            spans.push_back({s0, s1});
                        }
                        std::sort(spans.begin(), spans.end());
                        int64_t covered = 0;
                        for (auto& q : spans) {
                            if (q.first > covered) return std::printf("FAIL cols %lld V %d: gap\n", (long long)cols, V), 1;
                            covered = std::max(covered, q.second);
                        }
                        if (covered < cols) return std::printf("FAIL cols %lld V %d: end\n", (long long)cols, V), 1;
                        ++layouts;
                    }
                }
            }
    std::printf("ok: %ld layouts\n", layouts);
    return 0;
}

// Which kernel a head of the given shape takes on a device with `cus` compute units, and how its launch is
// planned (csrc/plan.hpp, no HIP): compiled and run by helpers.plan_route.
// usage: plan_route M V_act d k cus                          ->   one line "key=value ..."
//        plan_route batched V_core V_arc d k cus rows...     the batched head with so many draft rows per sequence (up to 64 chunks)
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "plan.hpp"

using namespace evospec;

static void print_tiles(const TileRoute& r, int M, int V_act, int cus) {
    const int tiles = ((V_act + kGemmSlab - 1) / kGemmSlab) * ((M + kTileRows - 1) / kTileRows);
    if (!r.small) std::printf("kernel=gemm");
    else std::printf("kernel=tile stages=%d", tiles > cus ? 2 : 4);
    if (r.parts) std::printf(" parts=1");
}

static void print_slab(const Plan& p) {
    std::printf("kernel=slab tiles=%d blocks=%d shared=%d segments=%d lists=%d rows=%d", p.nw, p.mb, p.ks, p.segs, p.n_slabs, p.rt);
}

static int batched(int n, char** a) {
    const int V_core = std::atoi(a[0]), V_arc = std::atoi(a[1]), d = std::atoi(a[2]), k = std::atoi(a[3]), cus = std::atoi(a[4]);
    int M = 0, chunks = 0, max_rows = 0;
    for (int i = 5; i < n; ++i) M += std::atoi(a[i]);
    const bool one_set = V_core == 0 || V_arc == 0;
    const TileRoute r = V_core > 0 ? tile_route(M, V_core, d, k, cus, one_set, core_workspace_bytes(M, d, V_core, k)) : TileRoute{};
    for (int i = 5, m0 = 0, end = 0; i < n; ++i)
        for (end += std::atoi(a[i]); m0 < end; ++chunks) {
            const int limit = r.tiles ? m0 + kMTile : (m0 / kMTile + 1) * kMTile, to = end < limit ? end : limit;
            if (to - m0 > max_rows) max_rows = to - m0;
            m0 = to;
        }
    if (chunks < 1 || chunks > kMaxChunks) return 1;
    if (r.tiles) print_tiles(r, M, V_core, cus);
    else if (V_core > 0) print_slab(make_plan(kMTile, V_core, d, k, cus, 1, one_set));
    if (V_arc > 0) {
        const bool split = !one_set && split_rows(max_rows, V_arc, d, k, cus, chunks);
        const Plan p = make_plan(split ? kSplitRows : max_rows, V_arc, d, k, cus, split ? 2 * chunks : chunks, one_set);
        RowBound b;
        if (r.tiles) choose_bound(&b, p.n_slabs, k);
        std::printf(" chunks=%d split=%d arc_tiles=%d arc_blocks=%d bound=%d", chunks, split ? 1 : 0, p.nw, p.mb, b.q);
    }
    if (r.tiles && r.small && !one_set)
        std::printf(" joint=%d", joint_tiles(M, V_core, d, cus, true, make_tile_batch_plan(max_rows, V_arc, k).n_slabs, chunks) ? 1 : 0);
    if (!r.tiles && !one_set) {                                // both sets in one launch
        const JointPlan j = make_joint_plan(M, V_core, V_arc, chunks, d, k, cus);
        std::printf(" joint_tiles=%d joint_blocks=%d joint_slabs=%d", j.core.nw, j.core.mb, j.core.n_slabs);
    }
    std::printf("\n");
    return 0;
}

int main(int argc, char** argv) {
    if (argc > 7 && !std::strcmp(argv[1], "batched")) return batched(argc - 2, argv + 2);
    if (argc != 6) return 1;
    const int M = std::atoi(argv[1]), V_act = std::atoi(argv[2]), d = std::atoi(argv[3]), k = std::atoi(argv[4]), cus = std::atoi(argv[5]);
    const TileRoute r = tile_route(M, V_act, d, k, cus, true, workspace_upper_bound(V_act, k));
    const int rows = M < kMTile ? M : kMTile;                  // (the first pass)
    if (r.tiles) print_tiles(r, M, V_act, cus);
    else if (use_narrow(rows, d, V_act, cus)) std::printf("kernel=narrow lists=%d", make_narrow_plan(rows, V_act, k, cus).n_slabs);
    else print_slab(make_plan(rows, V_act, d, k, cus));
    std::printf("\n");
    return 0;
}

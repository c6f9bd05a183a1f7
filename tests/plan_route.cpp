// Which kernel a head of the given shape takes on a device with `cus` compute units, and how its launch is
// planned (csrc/plan.hpp, no HIP): compiled and run by helpers.plan_route.
// usage: plan_route M V_act d k cus                          ->   one line "key=value ..."
//        plan_route batched LAYOUT V_core V_arc d k cus rows...     the batched head with so many draft rows per sequence (up to 64 chunks)
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "plan.hpp"

using namespace evospec;

static void print_tiles(const TileRoute& r, int M, int V_act, int cus, int beside = 0) {
    const int tiles = beside + ((V_act + kGemmSlab - 1) / kGemmSlab) * ((M + kTileRows - 1) / kTileRows);
    if (!r.small) std::printf("kernel=gemm");
    else std::printf("kernel=tile stages=%d", tiles > cus ? 2 : 4);
    if (r.parts) std::printf(" parts=1");
}

static void print_slab(const Plan& p) {
    std::printf("kernel=slab tiles=%d blocks=%d shared=%d segments=%d lists=%d rows=%d", p.nw, p.mb, p.ks, p.segs, p.n_slabs, p.rt);
}

// (the decisions of evospec_active_lmhead_topk_segmented, in its order)
static int batched(int n, char** a) {
    const bool packed = !std::strcmp(a[0], "packed");
    const int V_core = std::atoi(a[1]), V_arc = std::atoi(a[2]), d = std::atoi(a[3]), k = std::atoi(a[4]), cus = std::atoi(a[5]);
    std::vector<int32_t> row_off(1, 0);
    for (int i = 6; i < n; ++i) row_off.push_back(row_off.back() + std::atoi(a[i]));
    const int S = (int)row_off.size() - 1, M = row_off[S];
    const bool one_set = V_core == 0 || V_arc == 0;
    const TileRoute r = batch_route(row_off.data(), S, V_core, V_arc, d, k, cus, packed, core_workspace_bytes(M, d, V_core, k));
    const ChunkCount c = count_chunks(row_off.data(), S, r.tiles);
    if (c.n < 1 || c.n > kMaxChunks) return 1;
    const int pt_slabs = make_tile_batch_plan(c.max_rows, V_arc, k).n_slabs;
    const bool joint = !one_set && (r.tiles ? r.small && joint_tiles(M, V_core, d, cus, packed, pt_slabs, c.n) : joint_slabs(M, V_core, V_arc, c.n));
    const JointPlan j = joint && !r.tiles ? make_joint_plan(M, V_core, V_arc, c.n, d, k, cus) : JointPlan{};
    if (r.tiles) print_tiles(r, M, V_core, cus, joint ? pt_slabs * c.n : 0);
    else if (V_core > 0) print_slab(joint ? j.core : make_plan(kMTile, V_core, d, k, cus, 1, one_set));
    std::printf(" chunks=%d joint=%d", c.n, joint ? 1 : 0);
    if (V_arc > 0) {                                           // a joint launch neither shares out rows nor has a bound
        const bool split = !joint && !one_set && split_rows(c.max_rows, V_arc, d, k, cus, c.n);
        const Plan p = joint ? (r.tiles ? make_tile_batch_plan(c.max_rows, V_arc, k) : j.arc)
                             : make_plan(split ? kSplitRows : c.max_rows, V_arc, d, k, cus, split ? 2 * c.n : c.n, one_set);
        RowBound b;
        const long tiles = ((V_core + 127l) / 128) * ((M + 127l) / 128);
        const bool takes = !r.small || !packed || (tiles > cus && !w_in_registers(M, V_core, d, cus));      // a kernel for it
        if (r.tiles && !joint && takes) choose_bound(&b, p.n_slabs, k);
        std::printf(" split=%d arc_tiles=%d arc_blocks=%d arc_slabs=%d bound=%d", split ? 1 : 0, p.nw, p.mb, p.n_slabs, b.q);
    }
    std::printf("\n");
    return 0;
}

int main(int argc, char** argv) {
    if (argc > 8 && !std::strcmp(argv[1], "batched")) return batched(argc - 2, argv + 2);
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

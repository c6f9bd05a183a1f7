// Which kernel a head of the given shape takes on a device with `cus` compute units, and how its launch is
// planned (csrc/plan.hpp, no HIP): compiled and run by helpers.plan_route.
// usage: plan_route M V_act d k cus   ->   one line "key=value ..."
#include <cstdio>
#include <cstdlib>

#include "plan.hpp"

using namespace evospec;

int main(int argc, char** argv) {
    if (argc != 6) return 1;
    const int M = std::atoi(argv[1]), V_act = std::atoi(argv[2]), d = std::atoi(argv[3]), k = std::atoi(argv[4]), cus = std::atoi(argv[5]);
    if (use_gemm(M, d)) {
        const int tiles = ((V_act + kGemmSlab - 1) / kGemmSlab) * ((M + kTileRows - 1) / kTileRows);
        if (use_small_tiles(M, V_act, d, k, cus)) std::printf("kernel=tile stages=%d\n", tiles > cus ? 2 : 4);
        else std::printf("kernel=gemm\n");
        return 0;
    }
    const int rows = M < kMTile ? M : kMTile;                  // (the first pass)
    if (use_narrow(rows, d, V_act, cus)) {
        const NarrowPlan p = make_narrow_plan(rows, V_act, k, cus);
        std::printf("kernel=narrow lists=%d\n", p.n_slabs);
        return 0;
    }
    const Plan p = make_plan(rows, V_act, d, k, cus);
    std::printf("kernel=slab tiles=%d blocks=%d shared=%d lists=%d rows=%d\n", p.nw, p.mb, p.ks, p.n_slabs, p.rt);
    return 0;
}

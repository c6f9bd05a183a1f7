// Host-only check of the launch planning in csrc/plan.hpp (no HIP): compiled and run by
// tests/test_plan_host.py.  Prints "ok" or the first violated invariant.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <vector>

#include "plan.hpp"

using namespace evospec;

#define REQUIRE(cond, ...) do { if (!(cond)) { std::printf("FAILED %s: ", #cond); std::printf(__VA_ARGS__); std::printf("\n"); return 1; } } while (0)

int main() {
    const int cus[] = {256, 304, 64};
    const int ds[] = {8, 64, 2048, 4096, 4104, 8192};
    const int ks[] = {1, 10, 16, 17, 64};
    const int rows_list[] = {1, 16, 17, 32, 33, 60, 64};
    for (int cu : cus)
        for (int d : ds)
            for (int k : ks)
                for (int rows : rows_list)
                    for (int V_act = 1; V_act <= 200000; V_act = V_act < 300 ? V_act + 1 : V_act + V_act / 7 + 13) {
                        if (k > V_act) continue;
                        for (int replicas : {1, 16}) {
                            const Plan p = make_plan(rows, V_act, d, k, cu, replicas);
                            REQUIRE(p.nw >= 4 && p.nw <= 12 && (p.ks == 1 || p.ks == 2 || p.ks == 4) && p.nw * p.ks <= 16 && p.mb % p.ks == 0, "shape nw=%d ks=%d", p.nw, p.ks);
                            REQUIRE(p.rt == 16 * p.nw, "rt=%d", p.rt);
                            REQUIRE(p.mb == mb_for_rows(rows) && 16 * p.mb >= rows, "mb=%d rows=%d", p.mb, rows);
                            REQUIRE((long)p.n_slabs * p.rt >= V_act && (long)(p.n_slabs - 1) * p.rt < V_act, "slabs=%d rt=%d V_act=%d", p.n_slabs, p.rt, V_act);
                            REQUIRE(p.lds_bytes <= (size_t)kLdsLimit, "lds=%zu", p.lds_bytes);
                            REQUIRE(p.gl >= 0 && p.gl <= 2, "gl=%d", p.gl);
                            REQUIRE(p.segs == 1 || (p.segs == 2 && d % 2048 == 0 && p.ks <= 2), "segments=%d d=%d ks=%d", p.segs, d, p.ks);
                            // (partial sums of a shared tile, and of the other segment, behind one another)
                            REQUIRE(p.lds_bytes >= 2ull * 16 * p.mb * kHStride * 2 + slab_level_bytes(p.nw * p.ks, p.mb, p.segs), "lds=%zu segments=%d", p.lds_bytes, p.segs);
                            // without sharing, as where two sets meet: a logit's sum runs front to back
                            const Plan q = make_plan(rows, V_act, d, k, cu, replicas, false);
                            REQUIRE(q.ks == 1 && q.segs == 1 && q.rt == p.rt, "two sets ks=%d segments=%d", q.ks, q.segs);
                            for (int chunks : {1, 4, 16})
                                if (split_rows(rows, V_act, d, k, cu, chunks)) {
                                    const Plan s = make_plan(kSplitRows, V_act, d, k, cu, 2 * chunks, false);
                                    REQUIRE(rows > kSplitRows && s.mb == mb_for_rows(kSplitRows) && s.ks == 1 && (long)s.n_slabs * 2 * chunks <= cu, "shared out rows=%d V_act=%d chunks=%d", rows, V_act, chunks);
                                }
                            // the workspace the ABI asks callers for covers the plan's own layout
                            REQUIRE(p.stats_off >= (size_t)p.n_slabs * kMTile * k * 8, "stats_off");
                            REQUIRE(p.total_bytes <= workspace_upper_bound(V_act, k), "total=%zu bound=%zu V_act=%d k=%d nw=%d", p.total_bytes,
                                    workspace_upper_bound(V_act, k), V_act, k, p.nw);
                        }
                    }
    // the shapes the benchmark configurations run with on 256 CUs (measured best of a sweep over nw)
    REQUIRE(make_plan(60, 36864, 4096, 10, 256).nw == 9, "36,864 rows");
    REQUIRE(make_plan(60, 32256, 4096, 10, 256).nw == 9, "32,256 rows: not the 1 MiB slabs of 8 wavefronts");
    REQUIRE(make_plan(8, 18432, 4096, 10, 256).nw == 5, "18,432 rows");
    REQUIRE(make_plan(60, 8448, 4096, 10, 256).nw == 4, "8,448 rows");
    REQUIRE(make_plan(60, 151936, 4096, 10, 256).nw == 10, "151,936 rows");
    // wavefronts that share a tile: not with one block of draft rows, not on several rounds with two, not on request
    REQUIRE(make_plan(60, 8448, 4096, 10, 256).ks == 4 && make_plan(60, 18432, 4096, 10, 256).ks == 2 && make_plan(60, 36864, 4096, 10, 256).ks == 1, "shared tiles");
    REQUIRE(make_plan(24, 8448, 4096, 10, 256).ks == 2 && make_plan(24, 51446, 512, 10, 256).ks == 1 && make_plan(60, 51446, 512, 10, 256).ks == 2, "rounds");
    REQUIRE(make_plan(16, 8448, 4096, 10, 256).ks == 1 && make_plan(60, 8448, 4096, 10, 256, 1, false).ks == 1, "no shared tiles");
    // the bound's groups: pairs of a lane's logits from k = lanes of a draft row on; then they are no coarser than a lane
    for (int nw = 4; nw <= 12; ++nw)
        for (int k = 1; k <= 64; ++k) {
            REQUIRE(fine_groups(k, nw) == (k >= 4 * nw), "fine_groups");
            REQUIRE(!fine_groups(k, nw) || group_level_for(k, nw) == 0, "level of pairs");
        }
    // few draft rows: when, and everything the kernel assumes of its plan
    REQUIRE(use_narrow(1, 4096, 151936, 256) && use_narrow(16, 4096, 151936, 256) && use_narrow(8, 4096, 18432, 256) && use_narrow(16, 8, 4096, 256), "few rows");
    REQUIRE(!use_narrow(17, 256, 100, 256) && !use_narrow(1, 4104, 100, 256) && !use_narrow(9, 4096, 18432, 256) && !use_narrow(8, 256, 36864, 256) && use_narrow(8, 256, 24576, 256), "the other kernel");
    for (int cu : cus)
        for (int M = 1; M <= kNarrowRows; ++M)
            for (int k : {1, 10, 17, 64})
                for (int V_act = k; V_act <= 2000000; V_act = V_act < 300 ? V_act + 1 : V_act + V_act / 7 + 13) {
                    const NarrowPlan p = make_narrow_plan(M, V_act, k, cu);
                    const int tiles = (V_act + 15) / 16, most = p.base_tiles + (p.rem_tiles > 0);
                    REQUIRE(p.n_slabs >= 1 && p.base_tiles >= 1 && p.rem_tiles >= 0 && p.rem_tiles < p.n_slabs, "V_act=%d", V_act);
                    REQUIRE((long)p.n_slabs * p.base_tiles + p.rem_tiles == tiles, "tiles V_act=%d", V_act);
                    REQUIRE(most <= kNarrowMaxTiles && p.z_stride >= most * 16 + 4 && p.z_stride % 4 == 0, "most=%d", most);
                    REQUIRE(p.lds_bytes <= (size_t)kLdsLimit, "lds=%zu", p.lds_bytes);
                    REQUIRE(p.stats_off >= (size_t)p.n_slabs * M * k * 8 && p.total_bytes >= p.stats_off + (size_t)p.n_slabs * M * 8, "layout");
                    REQUIRE(p.total_bytes <= workspace_upper_bound(V_act, k), "total=%zu V_act=%d M=%d k=%d", p.total_bytes, V_act, M, k);
                }
    // packed layout sizes
    REQUIRE(packed_d(4096) == 4096 && packed_d(8) == 256 && packed_d(264) == 512, "packed_d");
    REQUIRE(packed_rows(36864) == 36864 && packed_rows(1) == 16 && packed_rows(17) == 32, "packed_rows");
    REQUIRE(matrix_elems(33, 72, true) == 48u * 256u && matrix_elems(33, 72, false) == 33u * 72u, "matrix_elems");
    // updates past the caches: sets of 128 MiB and more, packed ones up to 512 rows
    REQUIRE(update_past_caches(512, 16384, 4096, true) && !update_past_caches(513, 16384, 4096, true), "packed updates");
    REQUIRE(update_past_caches(9000, 16384, 4096, false) && !update_past_caches(8, 16383, 4096, false), "row-major updates");
    REQUIRE(!update_past_caches(8, 16368, 4096, true) && !update_past_caches(8, 40000, 2056, false), "small sets, ragged rows");
    // large-M plan: lists and statistics do not overlap, one slab per 128 rows
    for (int M : {129, 960, 4096})
        for (int V_act : {1, 127, 128, 129, 32768, 151936}) {
            const GemmPlan g = make_gemm_plan(M, V_act, 10);
            REQUIRE(g.n_slabs == (V_act + 127) / 128 && g.list_len == 16, "gemm slabs");
            REQUIRE(g.stats_off >= (size_t)g.n_slabs * M * g.list_len * 8 && g.total_bytes >= g.stats_off + (size_t)g.n_slabs * M * 8, "gemm layout");
        }
    // small tiles: where they take fewer than some three times the rounds of the large ones
    REQUIRE(use_small_tiles(200, 16384, 4096, 10, 256) && use_small_tiles(129, 1, 64, 1, 256) && use_small_tiles(300, 20000, 2048, 10, 256), "small tiles");
    REQUIRE(!use_small_tiles(960, 32768, 4096, 10, 256) && !use_small_tiles(512, 32768, 4096, 10, 256) && !use_small_tiles(256, 45000, 5120, 10, 256), "large tiles");
    REQUIRE(use_small_tiles(256, 45000, 1024, 10, 256) && use_small_tiles(512, 20011, 2560, 10, 256) && !use_small_tiles(512, 20011, 2560, 1, 256), "three rounds");
    // a bound from other lists: q of each of `sets` lists are k logits, of lists that are there and entries that they have
    for (int k = 1; k <= kKMax; ++k)
        for (int n = 1; n <= 300; ++n) {
            RowBound b;
            choose_bound(&b, n, k);
            REQUIRE(b.k == k && b.n_lists <= n && b.n_lists <= kBoundLists && b.q <= 2 && (b.q == 0 || k <= 16), "k=%d lists=%d", k, n);
            REQUIRE(b.q == 0 || (b.q <= k && b.sets >= 1 && b.sets <= b.n_lists && b.q * b.sets >= k), "k=%d lists=%d q=%d sets=%d", k, n, b.q, b.sets);
        }
    // k past the slabs' own bound: small tiles, but large ones beside extensions that bound the rows, where these take far fewer rounds
    const int32_t full[] = {0, 60, 120, 180, 240, 300, 360, 420, 480, 540, 600, 660, 720, 780, 840, 900, 960};
    for (int packed = 0; packed < 2; ++packed) {
        REQUIRE(tile_route(960, 32768, 4096, 16, 256, true, 0).small && !batch_route(full, 16, 32768, 2048, 4096, 16, 256, packed, 0).small, "16 x 60");
        REQUIRE(batch_route(full, 16, 32768, 2048, 4096, 17, 256, packed, 0).small && batch_route(full, 16, 32768, 300, 4096, 16, 256, packed, 0).small, "no bound");
        REQUIRE(batch_route(full, 5, 32768, 2048, 4096, 16, 256, packed, 0).small == (packed != 0) && batch_route(full, 5, 32768, 2048, 2048, 13, 256, packed, 0).small, "5 x 60");
        REQUIRE(batch_route(full, 16, 8192, 2048, 4096, 16, 256, packed, 0).small, "two rounds");
    }
    // the extensions beside small tiles in twos: where they find places
    REQUIRE(w_in_registers(150, 28000, 4096, 256) && !w_in_registers(200, 16500, 2048, 256) && w_in_registers(200, 22000, 2048, 256) && w_in_registers(200, 17000, 1024, 256), "few with two");
    REQUIRE(!w_in_registers(150, 32768, 4096, 256) && w_in_registers(200, 32768, 4096, 256) && w_in_registers(150, 32768, 2048, 256) && w_in_registers(150, 33000, 4096, 256), "all with two");
    REQUIRE(joint_tiles(150, 26000, 4096, 256, true, 32, 3) && !joint_tiles(150, 30000, 4096, 256, true, 32, 3) && joint_tiles(180, 32768, 4096, 256, true, 32, 3), "packed");
    REQUIRE(joint_tiles(480, 14000, 4096, 256, false, 16, 8) && !joint_tiles(480, 16384, 4096, 256, false, 16, 8) && !joint_tiles(480, 16384, 4096, 256, false, 5, 8) &&
            joint_tiles(367, 15792, 2048, 256, false, 25, 16) && joint_tiles(640, 32768, 4096, 256, false, 32, 11), "row-major");
    REQUIRE(joint_tiles(220, 5225, 4096, 256, false, 3, 11) && joint_tiles(250, 16384, 2048, 256, false, 16, 5) && !joint_tiles(197, 16384, 4096, 256, false, 16, 4), "a compute unit each");
    // 65 to 128 rows in tiles: the lists fit the scratch, whatever the caller's is
    for (int M = 1; M <= 300; ++M)
        for (int k : {1, 4, 7, 8, 10, 12, 13, 16, 17, 64})
            for (int d : {64, 264, 512, 1024, 1088, 4096})
                for (int V_act = k; V_act <= 200000; V_act += V_act / 3 + 7) {
                    const size_t head = workspace_upper_bound(V_act, k), core = core_workspace_bytes(M, d, V_act, k);
                    const TileRoute r = tile_route(M, V_act, d, k, 256, true, head), two = tile_route(M, V_act, d, k, 256, false, core);
                    REQUIRE(r.tiles == two.tiles || (M > kMTile && M < kGemmMinRows), "M=%d", M);
                    if (M <= kMTile) REQUIRE(!r.tiles && !two.tiles, "M=%d", M);
                    REQUIRE(!r.parts || (r.tiles && r.small && M < kGemmMinRows && d >= kTilePartsMinD && k <= 12), "parts M=%d d=%d k=%d", M, d, k);
                    REQUIRE(!two.parts && (!r.tiles || d % 64 == 0) && (!two.tiles || d % 64 == 0), "two sets M=%d d=%d", M, d);
                    const size_t need = make_gemm_plan(M, V_act, k).total_bytes;
                    if (r.tiles && M < kGemmMinRows) REQUIRE(need <= head, "M=%d V_act=%d k=%d", M, V_act, k);
                    if (two.tiles) REQUIRE(need <= core, "M=%d V_act=%d k=%d", M, V_act, k);
                }
    // 65 to 128 rows: one set in parts from 1,024 hidden elements on, where the matrix is large enough for them; two sets always
    const size_t any = ~(size_t)0;
    REQUIRE(use_tiles_early(66, 128, 1024, 10, true, any) && !use_tiles_early(66, 8448, 960, 10, true, any) && use_tiles_early(66, 8448, 960, 10, false, any), "hidden size");
    REQUIRE(use_tiles_early(66, 6144, 4096, 10, true, any) && !use_tiles_early(66, 6016, 4096, 10, true, any) && use_tiles_early(66, 128, 4096, 10, false, any), "small sets");
    // draft rows of few extensions shared out: not where the slabs get taller than by a quarter, or a compute unit two workgroups
    REQUIRE(split_rows(60, 1000, 4096, 10, 256, 4) && split_rows(60, 1024, 4096, 10, 256, 8) && split_rows(33, 1250, 2048, 10, 256, 8), "shared out");
    REQUIRE(!split_rows(32, 1000, 4096, 10, 256, 4) && !split_rows(60, 2048, 4096, 10, 256, 8) && !split_rows(64, 5500, 4096, 10, 256, 4) && !split_rows(60, 1400, 2048, 10, 256, 8) &&
            !split_rows(60, 2048, 4096, 10, 256, 16), "not shared out");
    // the packed tiles' ring: every wait covers the pair of h that is read behind it, whatever the number of pairs
    for (int pairs = 1; pairs <= 40; ++pairs) {
        std::vector<int> flight;                                   // a wavefront's loads in the order of their requests: pair of h, or -1 for W
        std::vector<bool> landed(pairs + 2 * kPRing, false);
        auto request = [&](int what, int n) { flight.insert(flight.end(), n, what); };
        auto wait = [&](int n) {
            while ((int)flight.size() > n) {
                if (flight.front() >= 0) landed[flight.front()] = true;
                flight.erase(flight.begin());
            }
        };
        for (int p = 0; p < kPRing; ++p) { request(p, kRingH); request(-1, p < pairs ? 2 * kRingW : 0); }      // (at least: what nobody reads may not be requested)
        wait(pairs >= kPRing ? ring_first_wait(kPRing) : 0);
        REQUIRE(landed[0], "pairs=%d", pairs);
        int p = 0;
        for (; p < pairs / kPRing * kPRing; ++p) {                 // (whole turns of the ring)
            request(-1, kRingW);
            wait(ring_wait(kPRing));
            REQUIRE(landed[p + 1] || p + 1 >= pairs, "pair %d of %d", p + 1, pairs);
            request(p + kPRing, kRingH);
            request(-1, kRingW);
        }
        wait(0);                                                   // the last pairs request nothing
        for (; p < pairs; ++p) REQUIRE(landed[p], "pair %d of %d", p, pairs);
    }
    REQUIRE(ring_first_wait(kPRing) < 64 && ring_wait(kPRing) < 64, "a wait counts to 63");
    REQUIRE(gemm_list_len(16) == 16 && gemm_list_len(17) == 32 && gemm_list_len(64) == 64, "list_len");
    REQUIRE(use_gemm(129, 4096) && !use_gemm(128, 4096) && !use_gemm(960, 4104), "use_gemm");
    std::printf("ok\n");
    return 0;
}

// Host-side launch planning for the active-vocabulary LM head (no HIP calls here).
//
// The restricted projection of Eq. 1 (EvoSpec paper) streams W_act once.  Rows of
// W_act are cut into slabs of RT = 16 * NW rows; one workgroup of NW wavefronts
// handles one slab and leaves, per draft row, a partial (max, sum-exp, k best keys)
// in the workspace.  This header decides the slab shape for a problem size and lays
// out the workspace; both halves of the head (partials, merge) derive the same plan
// from the same arguments.
#pragma once
#include <cstddef>
#include <cstdint>

namespace evospec {

constexpr int kMTile = 64;          // draft rows per pass over W_act
constexpr int kKMax = 64;           // largest supported k
constexpr int kKC = 256;            // hidden-dimension chunk staged in LDS per step
constexpr int kHStride = kKC;       // LDS row stride of the h chunk (bf16 elements; its pieces are permuted, see slab.hpp)
constexpr int kRowsMinSlab = 64;    // smallest slab any plan uses (workspace upper bound)
constexpr int kLdsLimit = 160 * 1024;
constexpr int kRoundRows = 37;      // fixed cost of a round of workgroups, in slab rows (see make_plan)

// Slab shapes that have a compiled kernel: X(nw, rc, ks4, ks2) with nw tiles of 16 rows per workgroup
// (RT = 16 * nw rows per slab) and a W-operand ring of rc chunks of kKC hidden elements per lane.  (Measured
// on MI355X: more waves per CU beat a deeper ring per wave.)  ks4 / ks2: wavefronts that may share a tile with
// four / two blocks of draft rows.  A workgroup with few tiles has too few wavefronts to hide the operand reads
// and the trips to L2 for h, so several share a tile, up to 16 wavefronts in all (measured at 60 rows, all x
// 4,096 unless said: 8,448 rows 26.8 -> 25.0 us, 18,432 33.9 -> 32.5, 24,000 41.9 -> 39.4, 12,000 x 1,024 16.3 ->
// 13.2; 37 rows, 20,011 x 3,000 41.8 -> 34.8; 20 rows, 16,384 28.5 -> 26.4.  A ring of four chunks instead of
// two: 1 to 12 us slower).  With two blocks of draft rows two workgroups fit a compute unit unless their tiles are
// shared, so that a launch of several rounds goes without (17 rows, 128,105 x 256 26.2 -> 17.1 us for the slabs;
// 24 rows, 51,446 x 512 17.4 -> 14.5; 32 rows, 124,638 x 1,536 72.1 -> 61.3; with four blocks 59,624 x 4,096 119 shared,
// 124 not).
#define EVOSPEC_SLAB_SHAPES(X) \
    X(4, 2, 4, 2) X(5, 2, 2, 2) X(6, 2, 2, 2) X(7, 2, 2, 2) X(8, 2, 2, 2) X(9, 2, 1, 1) X(10, 2, 1, 1) X(12, 2, 1, 1)
struct SlabShape { int nw; int rc; int ks4; int ks2; };
#define EVOSPEC_SHAPE_ENTRY(NW_, RC_, KS4_, KS2_) {NW_, RC_, KS4_, KS2_},
constexpr SlabShape kShapes[] = {EVOSPEC_SLAB_SHAPES(EVOSPEC_SHAPE_ENTRY)};
#undef EVOSPEC_SHAPE_ENTRY
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);
constexpr bool shapes_respect_min_slab() {
    for (int i = 0; i < kNumShapes; ++i)
        if (16 * kShapes[i].nw < kRowsMinSlab) return false;
    return true;
}
static_assert(shapes_respect_min_slab(), "workspace_upper_bound assumes no slab below kRowsMinSlab rows");

// A batch of independent problems handled by one launch (grid.y): chunk i is the draft rows
// [m0, m0 + rows) of h against the rows of sequence `seq` of a per-sequence matrix.  For the
// merge, a_pass / a_slot locate the chunk's rows inside the first partial set.
constexpr int kMaxChunks = 64;
struct ChunkBatch {
    int n = 0;
    int m0[kMaxChunks];
    int rows[kMaxChunks];
    int seq[kMaxChunks];
    int a_pass[kMaxChunks];
    int a_slot[kMaxChunks];
};

// The shared core of a batch, where it rides in the launch of the extensions' slabs: its passes of kMTile draft rows, one after the
// other, `blocks` workgroups in all.
struct CoreSet {
    const void* W = nullptr;
    const int32_t* ids = nullptr;
    void* keys = nullptr;
    void* stats = nullptr;
    size_t pass_keys = 0, pass_stats = 0;     // u64 and float2 between two passes' partials
    int V = 0, M = 0;                         // its rows, and all draft rows
    int n_slabs = 0;                          // slabs of a pass
    int blocks = 0;                           // 0: no core in this launch
    int chunk_slabs = 0;                      // slabs of an extension
};

constexpr size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Operand-tile ("packed") layout of a compact matrix.  The slab kernel hands a wavefront 16 rows and
// feeds them to the matrix cores 32 hidden elements at a time: lane l = 16 g + n supplies the 16
// bytes (row n, elements 32 s + 8 g .. + 8) of k-step s.  The packed layout stores exactly these
// 1 KB operand blocks back to back:
//   piece (row r, 16-byte piece c = element / 8)  ->  piece index
//   (r / 16) * (16 * dp / 8) + (c / 4) * 64 + (c % 4) * 16 + (r % 16),   dp = d rounded up to kKC,
// pieces past d hold zeros, rows are padded to a multiple of 16.  A wavefront then streams one
// contiguous 16 * dp * 2 byte run with fully coalesced 1 KB loads (measured on MI355X: 61 us against
// 71 us for the same head on a row-major matrix, whose wave-loads touch 16 rows x 64 bytes).
constexpr int kPackRows = 16;
constexpr int packed_d(int d) { return (d + kKC - 1) / kKC * kKC; }
constexpr size_t packed_rows(size_t rows) { return align_up(rows, (size_t)kPackRows); }
inline size_t matrix_elems(size_t rows, int d, bool packed) {
    return packed ? packed_rows(rows) * (size_t)packed_d(d) : rows * (size_t)d;
}

// Whether a launch loads its weights past the caches (the slab kernel: of packed matrices whose rows are whole chunks
// only).  A set well below the 256 MB memory-side cache is
// still there when a decode loop comes back to it, and non-temporal loads find it more slowly (7,086 x
// 1,536, 22 MB, 53 rows: 18.0 us with ordinary loads, 18.3 without); a larger one only drags itself through
// (151,936 x 4,096 at one row 207 against 185 us, 36,864 x 4,096 at 60 rows 60.0 against 54.3, and against
// 54.8 -> 53.0 when the same 302 MB are read again at once).  Row-major rows that do not start on
// 128-byte lines share lines between loads, which want the cache (20,011 x 3,000 at 8 rows: 28.3 us
// through it, 31.8 past it).
inline bool streams_once(size_t rows, int d, bool packed) {
    return (packed || d % 64 == 0) && matrix_elems(rows, d, packed) * 2 >= ((size_t)128 << 20);
}

// The slab kernel takes a row-major matrix past the caches only where too little of it is left in the memory-side cache when it is
// read again (another matrix each time, then the same one again, through the caches and past them, x 4,096 at 60 rows: 151,936 rows
// 253 and 244 us; 50,000 rows at 128, two passes, 208 and 198 again; 36,864 rows 67.2 and 64.2, again 63.7 and 65.2; 18,432 rows
// 44.8 and 42.9, again 37.8 and 42.4; 60,000 x 2,048 66.3 and 65.3, again 58.1 and 63.1).
constexpr size_t kSlabOnceMiB = 320;
inline bool slab_streams_once(size_t rows, int d, bool packed) {
    return packed ? streams_once(rows, d, true) : d % kKC == 0 && rows * (size_t)d * 2 >= (kSlabOnceMiB << 20);
}

// One dynamic-buffer update: n rows W_act[slots[i]] <- W_lm[src_ids[i]], act_ids[slots[i]] <- src_ids[i]
// (slots == nullptr: slot i).  Device pointers; row_vec = d / 8.  packed: layout of W_act (W_lm is
// always row-major).
struct GatherArgs {
    const void* W_lm = nullptr;
    int V = 0, row_vec = 0;
    const int32_t* src_ids = nullptr;
    const int32_t* slots = nullptr;
    int n = 0;
    void* W_act = nullptr;
    int32_t* act_ids = nullptr;
    int V_act = 0;
    int packed = 0;
    int past_caches = 0;     // the rows are stored past the caches (update_past_caches)
};

// Whether the rows of an update are stored past the caches.  What matters is what the update adds to the head that
// follows it.  A set that the heads stream past the caches finds nothing of the update there, and lines left dirty
// in L2 are written back in its way (36,864 x 4,096 at 60 rows, added by 32 / 256 / 512 scattered rows: packed 4.1 /
// 17.8 / 20.0 us through the caches, 2.6 / 6.9 / 11.0 past them; row-major, 32 / 256 / 1,024 rows 3.2 / 5.1 / 10.0 and 3.1 / 3.5 / 6.0).  In a packed
// matrix neighbouring rows share lines, which only the caches can put together: from some 700 rows on that is
// worth more (1,024 / 4,096 / 8,192 rows 25 / 48 / 88 us and 22 / 80 / 184; 75,000 x 2,048: 768 rows 10.0 and 10.0,
// 2,048 rows 16.1 and 22.2; 18,000 x 8,192: 512 rows 26 and 21, 1,024 rows 32 and 41).  A smaller set is read
// through the caches, where the rows then are (18,432 x 1,024, packed, 32 / 1,024 rows: 2.6 / 4.0 and 2.9 / 4.7;
// 9,000 x 2,048: 2.0 / 5.2 and 3.0 / 9.4).
constexpr int kDirectUpdateRows = 512;
inline bool update_past_caches(int n, int V_act, int d, bool packed) {
    return streams_once((size_t)V_act, d, packed) && (!packed || n <= kDirectUpdateRows);
}
inline GatherArgs gather_args(const void* W_lm, int V, int d, const int32_t* src_ids, const int32_t* slots, int n, void* W_act,
                              int32_t* act_ids, int V_act, bool packed) {
    return GatherArgs{W_lm, V, d / 8, src_ids, slots, n, W_act, act_ids, V_act, packed ? 1 : 0,
                      update_past_caches(n, V_act, d, packed) ? 1 : 0};
}

// Rows of a small update passed to the kernel by value (see launch_gather_inline).
constexpr int kInlineRows = 32;
struct InlineRows {
    int32_t slot[kInlineRows];
    int32_t id[kInlineRows];
};

struct Plan {
    int nw = 0;              // 16-row tiles per workgroup
    int ks = 1;              // wavefronts that share a tile, each a part of the hidden dimension
    int segs = 1;            // segments of the hidden dimension (see segments_for)
    int mb = 0;              // 16-row blocks of draft rows held in accumulators (1, 2 or 4)
    int rt = 0;              // slab rows
    int n_slabs = 0;
    int gl = 0;              // selection group level of the slab epilogue (see group_level_for)
    size_t lds_bytes = 0;
    // workspace layout (bytes from the workspace base), for one pass of <= 64 draft rows
    size_t keys_off = 0, stats_off = 0, total_bytes = 0;
};

constexpr int mb_for_rows(int rows) { return rows <= 16 ? 1 : (rows <= 32 ? 2 : 4); }

// Granularity of the selection groups in the slab epilogue.  A slab's logits for one draft row
// sit 4 per lane in 4*nw lanes; level 0 takes each lane as a group, level 1 pairs of lanes,
// level 2 whole wavefronts (nw groups).  The k-th largest group maximum is a lower bound of the
// slab's k-th best logit, so only entries at or above it need exact ranking.  Coarser groups cost
// less to rank and filter almost as well: take the coarsest level with at least 1.5 k groups.
inline int group_level_for(int k, int nw) {
    const int want = k + k / 2;
    if (nw >= want) return 2;
    if (2 * nw >= want) return 1;
    return 0;
}

// Row stride, in keys, of the candidate lists of the slab epilogue: two keys of padding make the rows
// start 16 bytes apart modulo the 64 LDS banks, so that accesses of the draft rows of a wavefront to
// the same list position spread over all banks (a stride of rt keys maps every row to two banks).
constexpr int list_stride(int rt) { return rt + 2; }

// Whether the groups of the bound are pairs of a lane's logits: where the 4 * nw lanes that hold a draft row are no more
// than k, so that their maxima bound nothing (or next to nothing: k of k).  Twice as many groups cost four times as
// much to rank, which pays from there on and not before (slab kernel, x 1,024, 60 rows: 9 tiles, k = 34 / 36 / 40 39.4 / 51.0 /
// 56.0 us by lanes, 42.1 / 42.5 / 44.2 by pairs; 12 tiles, k = 36 / 48 37.3 / 66.7 and 51.0 / 54.2; 4 tiles, k = 14 / 16 11.9 /
// 13.8 and 13.0 / 12.7).
constexpr bool fine_groups(int k, int nw) { return k >= 4 * nw; }

// LDS that holds the other segment's sums: an accumulator set of every wavefront.
constexpr size_t slab_level_bytes(int wavefronts, int mb, int segs) { return segs == 2 ? (size_t)wavefronts * mb * 1024 : 0; }

inline size_t lds_bytes_for(int nw, int mb, int k, int ks = 1, int segs = 1) {
    const int rt = 16 * nw;
    const int mrows = 16 * mb;
    size_t hs = 2ull * mrows * kHStride * 2 + slab_level_bytes(nw * ks, mb, segs);   // h chunk, double buffered; segment sums
    size_t list = (size_t)mrows * list_stride(rt) * 8;       // surviving keys per draft row
    size_t u = hs > list ? hs : list;                        // the two never live together
    size_t gm = (size_t)mrows * (fine_groups(k, nw) ? 8 : 4) * nw * 4;   // group maxima
    size_t wsum = (size_t)nw * mrows * 4;                    // per-wave sum-exp
    size_t small = align_up((size_t)rt * 4, 16) + (size_t)mrows * 3 * 4;   // ids, tau, vmax, counters
    return align_up(u, 16) + gm + wsum + small;
}

// Segments of the hidden dimension in the slab kernel.  Rows of a row-major matrix that lie a multiple of 4 KB apart meet at
// the same memory channels while all workgroups are at the same place of their rows; in two segments of alternating
// 2 KB runs, half of the workgroups can take the other run first without a change of any sum (see the kernel).  Measured,
// row-major, 60 draft rows unless said, one segment and two: 151,936 x 4,096 275 and 252 us, 36,864 x 4,096 75.2 and 67.2 (24
// rows 69.0 and 62.5), 32,256 x 2,048 42.6 and 38.0, 60,000 x 2,048 73.4 and 66.3 (12 rows, 48,000 51.5 and 44.4).  Runs
// of 4 KB or of 1 KB gain next to nothing (274, 259).  A packed matrix is summed alike, so that both layouts give the same bits (36,864 x
// 4,096 61.0 and 61.1).  Only where the LDS has room for one set of sums, without costing a second workgroup on the
// compute unit (which four blocks of draft rows have no registers for anyway).  Four wavefronts to a tile gain nothing (8,448 x
// 4,096 35.1 and 35.2) and lose on a packed matrix (26.9 and 27.5).
constexpr int kSegChunks = 4;
constexpr int kSegMaxShare = 2;
inline int segments_for(int nw, int ks, int mb, int d, int k, long rounds) {
    if (d % (2 * kSegChunks * kKC) != 0 || ks > kSegMaxShare) return 1;
    const size_t base = lds_bytes_for(nw, mb, k, ks);
    const size_t limit = rounds > 1 && mb <= 2 && 2 * base <= (size_t)kLdsLimit ? kLdsLimit / 2 : kLdsLimit;
    return lds_bytes_for(nw, mb, k, ks, 2) <= limit ? 2 : 1;
}

// Slab shape for V_act rows of d elements on a device with `num_cu` compute units: the least
// ceil(slabs / CUs) * (RT + kRoundRows), a round of workgroups costing its rows plus a fixed part
// (first loads, epilogue: about what 37 rows of 8 KiB take to stream into one CU); ties go to the
// larger slab (fewer partials to merge).  A slab
// whose bytes are a multiple of 1 MiB is charged one eighth more: all workgroups then walk through
// memory at the same offset within a MiB and meet at the same memory channels (measured on MI355X
// at 32,256 x 4,096: 8 wavefronts = 1 MiB slabs 59 us, 9 wavefronts on fewer CUs 56 us).
// share: several wavefronts may share a tile.  Their parts of a logit's sum are added at the end, another order
// than one wavefront's, so launches whose logits meet in one result must not differ in it: the calls that merge
// two partial sets (a core and an extension) go without.
inline void lay_out(Plan* p, int k) {
    p->keys_off = 0;
    p->stats_off = align_up((size_t)p->n_slabs * kMTile * k * 8, 256);
    p->total_bytes = p->stats_off + align_up((size_t)p->n_slabs * kMTile * 8, 256);
}
inline long round_cost(long rounds, int rt, int d) {
    const long cost = rounds * (rt + kRoundRows) * 8;
    return ((size_t)rt * (size_t)d * 2) % ((size_t)1 << 20) == 0 ? cost + cost / 8 : cost;
}
inline Plan make_plan(int rows /*draft rows in this pass, 1..64*/, int V_act, int d, int k, int num_cu,
                      int replicas = 1 /*chunks that share the launch*/, bool share = true) {
    Plan best;
    long best_cost = -1;
    const int mb = mb_for_rows(rows);
    for (int i = 0; i < kNumShapes; ++i) {
        const int nw = kShapes[i].nw;
        const int rt = 16 * nw;
        const int n_slabs = (V_act + rt - 1) / rt;
        const size_t lds = lds_bytes_for(nw, mb, k);
        if (lds > (size_t)kLdsLimit) continue;
        const long rounds = ((long)n_slabs * replicas + num_cu - 1) / num_cu;
        const long cost = round_cost(rounds, rt, d);
        if (best_cost < 0 || cost < best_cost || (cost == best_cost && rt > best.rt)) {
            best_cost = cost;
            best.nw = nw; best.mb = mb;
            best.ks = !share || mb == 1 || (mb == 2 && rounds > 1) ? 1 : (mb == 2 ? kShapes[i].ks2 : kShapes[i].ks4);
            best.rt = rt; best.n_slabs = n_slabs;
            best.segs = share ? segments_for(nw, best.ks, mb, d, k, rounds) : 1;
            best.gl = group_level_for(k, nw); best.lds_bytes = lds_bytes_for(nw, mb, k, best.ks, best.segs);
        }
    }
    lay_out(&best, k);
    return best;
}

// The plans of a core of V_core rows (M draft rows in passes of kMTile) and of `chunks` extensions of V_arc rows that share one
// launch: one slab shape for both, chosen by the same costs over all their slabs.  No tile is shared and no row in segments (see make_plan).
// A launch of a few slabs is a chain of chunks that leaves the chip idle (4 extensions of 226 rows x 4,096: 16 workgroups, 19 us, row-major
// 38), and so is each pass of a small core: side by side they cost what the longest of them does.  One launch after the other and all
// in one, us for the call: packed, 11,986 + 226 x 4,096, 60 rows of 4 sequences 58 and 39; 32,768 + 2,048, 60 rows of 2 72.6 and 61.7; 5,000 + 200 x
// 2,048, 24 rows of 2 26.1 and 16.4; 30,000 + 1,500 x 2,048, 60 rows of 7 55 and 42; two passes, 20,000 + 1,000, 120 rows of 5, k = 20 115 and 78;
// row-major, 69 rows of 4 over 11,986 + 226, k = 45 136 and 72; 40 rows of 2 over 32,768 + 2,048 97.6 and 75.6.
// (joint_slabs: the threads of a launch are counted in 32 bits.)
constexpr long kJointWorkgroups = 1l << 22;
inline bool joint_slabs(int M, int V_core, int V_arc, int chunks) {
    return ((long)(M + kMTile - 1) / kMTile) * ((V_core + kRowsMinSlab - 1) / kRowsMinSlab) + (long)chunks * ((V_arc + kRowsMinSlab - 1) / kRowsMinSlab) <= kJointWorkgroups;
}
struct JointPlan { Plan core, arc; };
inline JointPlan make_joint_plan(int M, int V_core, int V_arc, int chunks, int d, int k, int num_cu) {
    JointPlan best;
    long best_cost = -1;
    const int mb = mb_for_rows(M < kMTile ? M : kMTile), passes = (M + kMTile - 1) / kMTile;
    for (int i = 0; i < kNumShapes; ++i) {
        Plan c;
        c.nw = kShapes[i].nw; c.mb = mb; c.rt = 16 * c.nw;
        c.gl = group_level_for(k, c.nw);
        c.lds_bytes = lds_bytes_for(c.nw, mb, k);
        if (c.lds_bytes > (size_t)kLdsLimit) continue;
        Plan a = c;
        c.n_slabs = (V_core + c.rt - 1) / c.rt;
        a.n_slabs = (V_arc + a.rt - 1) / a.rt;
        const long rounds = ((long)c.n_slabs * passes + (long)a.n_slabs * chunks + num_cu - 1) / num_cu;
        const long cost = round_cost(rounds, c.rt, d);
        if (best_cost < 0 || cost < best_cost || (cost == best_cost && c.rt > best.core.rt)) {
            best_cost = cost;
            lay_out(&c, k);
            lay_out(&a, k);
            best.core = c;
            best.arc = a;
        }
    }
    return best;
}

// The plan of extensions that share a launch with small tiles, whose workgroups have four wavefronts.
inline Plan make_tile_batch_plan(int max_rows, int V_arc, int k) {
    Plan p;
    p.nw = 4; p.mb = mb_for_rows(max_rows); p.rt = 16 * p.nw;
    p.n_slabs = (V_arc + p.rt - 1) / p.rt;
    p.gl = group_level_for(k, p.nw);
    p.lds_bytes = lds_bytes_for(p.nw, p.mb, k);
    lay_out(&p, k);
    return p;
}

constexpr int kTileRows = 128;           // (tile.hip)

// Whether the extensions' slabs (of make_tile_batch_plan) ride in the launch of the core's small tiles.  Without and with it, us for the call, k = 10:
// packed, 5,225 + 151 x 4,096, 220 rows of 11 52 and 35; 9,276 + 522 x 2,048, 363 of 16 47.6 and 37.5; 14,416 + 332 x 4,096, 477 of 13
// 106 and 93; 16,384 + 1,000 x 4,096, 197 of 4 72 and 69.5; 4,000 + 2,000 x 4,096, 400 of 16 98 and 84.
// More tiles than compute units sit there in twos, in as many places as twice the units; slabs that find none wait for tiles to end, and by themselves they
// would have their rows shared out (split_rows) and leave a bound.  512 places, row-major, whose tiles take over a bound: 440 tiles and 128 slabs 114 and 100; 399 and
// 135 112 and 96; 372 and 400 x 2,048 84 and 76; 1,280 and 352 277 and 259; but 512 and 40 118.6 and 127.9; 512 and 128 118 and 131; 435 and 200 115
// and 122; 483 and 108 x 2,048 68.6 and 70.1; 471 and 256 125 and 127.  Packed, where most tiles do not: 408 and 96 104 and 83; 483 and 108 65 and 61; 512 and 128 109 and 102; 471 and
// 256 117 and 108; 512 and 512 152 and 144; only with little in the second row of tiles and a large hidden dimension not, x 4,096, 150 rows of 3: 470 and 96
// 101.3 and 107.3; 438 and 96 99.5 and 105.4; 512 and 96 104.8 and 111; 138 rows of 12, 498 and 372 122 and 133; 180 of 3, 512 and 96 109 and 109; x 2,048, 150 of 3, 438 and 96 64 and 59.
// Row-major tiles that have a compute unit each have a ring of four stages by themselves and of two beside slabs: all on the chip once (5,225 +
// 151 62 and 39), or beside a few slabs with short rows (16,384 + 1,000 x 2,048, 250 of 5 54 and 51; x 4,096, 197 of 4 82 and 86; 4,906 + 1,764 x 4,096, 293 of 7,
// 117 tiles and 196 slabs, 79 and 91).
inline bool joint_tiles(int M, int V_core, int d, int num_cu, bool packed, int arc_slabs, int chunks) {
    const long tiles = ((V_core + 127l) / 128) * ((M + 127l) / 128), slabs = (long)arc_slabs * chunks;
    if (tiles + slabs > kJointWorkgroups) return false;
    const long places = 2l * num_cu, free = (tiles + places - 1) / places * places - tiles;      // beside the last round of tiles
    if (packed) return d <= 2048 || M > kTileRows + 32 || slabs <= free;         // (few rows in the second row of tiles)
    if (tiles > num_cu) return slabs <= 2 * free || 4 * free >= places;
    return tiles + slabs <= num_cu || (d <= 2048 && 2 * slabs <= tiles);
}

// Whether a batch of chunks gives the draft rows of every chunk to two workgroups, kSplitRows at most to each: where even
// then a compute unit has no more than one, and its slabs are hardly taller for it.  Both read the weights, but with half the
// draft rows a wavefront has half the operand reads and matrix instructions behind every piece of them.  us for the call, without
// and with it (only extensions with a launch of their own: beside large tiles, and beside small ones where joint_tiles says no): row-major, core of 16,384, 4 sequences with 197 rows over 1,000 rows x 4,096 84.7
// and 79.4, 8 with 480 over 500 121.3 and 115.5, over 1,000 123.4 and 117.9, 4 with 240 over 2,048 x 8,192 150 and 141; packed, core of 32,768, 8 with 480 over 500 161.4 and 154.9, over
// 1,000 160.9 and 155.9; core of 30,000, 3 with 150 over 2,048 103.5 and 98.5.  Slabs of 64 and 80 rows: packed, 8 with 480 over 1,250 162.9 and 159.3; row-major 124.2 and 123.9, x 2,048
// 76.8 and 75.7, 2 with 128 over 5,000 93.3 and 95.1.  Taller than that, the extensions filled half of the chip and more by themselves, and the slower streams cost more than that:
// 64 and 96 rows, 2 with 256 over 5,500 95 and 118, 8 with 480 over 1,400 x 2,048 65.0 and 68.9; 64 and 128, 8 with 480 over 2,048 119 and 132.  Two to a compute unit gain no more, and
// lose on long lists (16 x 60 rows 303 and 340).
constexpr int kSplitRows = 32;
inline bool split_rows(int max_rows, int V_act, int d, int k, int num_cu, int chunks) {
    if (max_rows <= kSplitRows) return false;
    const Plan whole = make_plan(max_rows, V_act, d, k, num_cu, chunks, false), half = make_plan(kSplitRows, V_act, d, k, num_cu, 2 * chunks, false);
    return (long)half.n_slabs * 2 * chunks <= num_cu && 4 * half.rt <= 5 * whole.rt;
}

// Few draft rows (narrow.hip): workgroups of kNarrowWaves wavefronts, each a run of 16-row tiles, one
// partial per workgroup and draft row; keys [M][n_slabs][k], stats [M][n_slabs].  One workgroup per
// compute unit, the tiles dealt out evenly (the first rem_tiles workgroups take one more); more rounds
// where the logits of a workgroup would not fit its LDS.
constexpr int kNarrowRows = 16;
constexpr int kNarrowWaves = 8;
constexpr int kNarrowGroup = 8;            // tiles whose partial sums share the LDS
constexpr int kNarrowMaxTiles = 40;        // tiles of a workgroup (logits in LDS: 16 rows x 640 x 4 bytes)
constexpr int kNarrowMaxD = 4096;          // h of a wavefront in registers: 16 k-steps
// Taken for up to 8 rows, one for each wavefront's selection at the end (against the slab kernel at 8 rows: 1,500 to
// 24,000 rows 1.05 to 1.6 times as fast, 48,000 1.0, 100,000 1.0 to 1.4).  From 9 rows on every wavefront selects twice,
// which pays only while a workgroup has a single tile, or where the slab kernel needs more than one round of its
// tallest slabs (16 rows, 768 hidden: 1,500 rows 1.02, 6,000 0.94, 24,000 0.88, 48,000 0.90, 100,000 1.01; 2,048
// hidden, packed: 1.03, 0.93, 0.97, 0.91, 1.00).  The same between those two for hidden sizes that leave wavefronts without
// work, once a workgroup has more than some 6 tiles (256 hidden, 8 rows: 12,000 rows 1.10, 24,000 0.98, 48,000 0.86).
inline bool use_narrow(int M, int d, int V_act, int num_cu) {
    if (M > kNarrowRows || d > kNarrowMaxD) return false;
    const int tiles = (V_act + 15) / 16, tallest = 16 * kShapes[kNumShapes - 1].nw;
    if (tiles <= num_cu || (V_act + tallest - 1) / tallest > num_cu) return true;
    return M <= kNarrowWaves && (d > 256 || tiles <= 6 * num_cu);
}

struct NarrowPlan {
    int n_slabs = 0, base_tiles = 0, rem_tiles = 0;
    int z_stride = 0;                      // logits per draft row in LDS
    size_t lds_bytes = 0;
    size_t keys_off = 0, stats_off = 0, total_bytes = 0;
};
inline NarrowPlan make_narrow_plan(int M, int V_act, int k, int num_cu) {
    NarrowPlan p;
    const int tiles = (V_act + 15) / 16;
    const int rounds = (tiles + num_cu * kNarrowMaxTiles - 1) / (num_cu * kNarrowMaxTiles);
    p.n_slabs = tiles < num_cu * rounds ? tiles : num_cu * rounds;
    p.base_tiles = tiles / p.n_slabs;
    p.rem_tiles = tiles - p.base_tiles * p.n_slabs;
    const int most = p.base_tiles + (p.rem_tiles > 0 ? 1 : 0);
    p.z_stride = most * 16 + 4;
    // partial sums of a group (later the candidate lists), logits, ids
    const size_t red = (size_t)kNarrowGroup * kNarrowWaves * 1024, lists = (size_t)kNarrowWaves * p.z_stride * 8;
    p.lds_bytes = align_up(red > lists ? red : lists, 16) + (size_t)M * p.z_stride * 4 + (size_t)most * 16 * 4;
    p.stats_off = align_up((size_t)p.n_slabs * M * k * 8, 256);
    p.total_bytes = p.stats_off + align_up((size_t)p.n_slabs * M * 8, 256);
    return p;
}
static_assert((size_t)kNarrowWaves * (kNarrowMaxTiles * 16 + 4) * 8 <= (size_t)kNarrowGroup * kNarrowWaves * 1024, "lists fit the group's partial sums");

// Large-M path: 256 x 256 tiles, one partial per 128 active rows and draft row, all M rows in
// one launch.  Taken from kGemmMinRows draft rows on, where the contraction, not the stream of
// W_act, bounds the head.
constexpr int kGemmTile = 256;
constexpr int kGemmSlab = 128;
constexpr int kGemmMinRows = 129;
constexpr int kGemmKChunk = 32;       // hidden elements per MFMA step; the large-M kernel loads two chunks at
                                      // a time and needs d to be a multiple of 64
inline bool use_gemm(int M, int d) { return M >= kGemmMinRows && d % (2 * kGemmKChunk) == 0; }

// Key slots per (slab, draft row) list of the large-M path: the kernel leaves every logit that
// reaches a lower bound of the slab's k-th best, unranked; rarely more than k + a few.
inline int gemm_list_len(int k) { return k <= 16 ? 16 : (k <= 32 ? 32 : 64); }

// Tiles of 128 x 128 (tile.hip) instead of 256 x 256 (gemm.hip); same partials.  A round of one workgroup
// per compute unit costs a large tile some 2.7 times what it costs a small one, and 3.4 times where the hidden
// dimension is short (large and small tiles, measured: 512 x 32,768 x 4,096 in one round of large tiles 138 us, in four
// of small ones 161; one and three rounds: 256 x 45,000 x 5,120 177 and 201, 1,024 x 10,000 x 4,096 132 and 144, 256 x
// 36,864 x 2,048 86 and 89, 256 x 45,000 x 1,024 65 and 58; two and five: 512 x 40,000 x 2,560 183 and 155; 200 x 16,384 x
// 4,096 130 and 52).  A last slab whose rows are too few for the bound (but more than a list holds) sends all its
// draft rows through the selection one by one in large tiles, by halves in small ones (512 x 20,011 x 2,560 138
// and 84 at k = 10; at k = 1, where the bound holds, 90 and 81; 256 x 45,011 x 4,096 145 and 130; 512 x 65,547 x 4,096 378 and 325: the 3.3 is
// from when small tiles selected them one by one as well, and more of these calls would gain).  From k = 13 on most rows have more survivors than a list, which large tiles
// select one by one and small ones by halves: 65,536 x 4,096 at 500 rows, k = 13 336 and 298, k = 16 516 and 304, k = 32 553 and 370;
// 32,768 x 4,096 at 960, k = 64 486 and 368; 32,768 x 1,024 at 512, k = 20 169 and 74; 32,768 x 4,096 at 4,000, k = 16 1,960 and 1,223, x 1,024 1,422 and 472.
// (Below 1,024 hidden elements the rounds decide for these as well, although the small tiles are the faster ones there too: 512 rows, 65,536 x 512, k = 20 320
// and 115, x 960, k = 13 191 and 112.)
// bounded: beside extensions whose lists bound the rows (choose_bound), so that few have.  There the rounds decide again, with more for the small tiles of a packed matrix,
// which share their launch with the extensions (32,768 + 2,048 x 4,096, k = 16, large tiles and small ones: packed, 960 rows of 16, two rounds and eight, 301 and
// 336; 480 of 8, one and four, 177 and 184; 300 of 5, one and three, 160 and 147; 640 of 11, two and five, 282 and 236; row-major 319 and 365, 186
// and 208, 165 and 175, 291 and 259; x 2,048, 24,000 + 1,024, 500 of 16, one and three, 112 and 108).
constexpr int kOwnBoundK = 12;             // largest k whose bound of 32 group maxima (slab_epilogue.hpp) leaves a list of 16 some room
constexpr int kTileMaxD = 1 << 23;         // (rows of a tile within 32-bit offsets)
inline bool slow_last_slab(int V_act, int k) {
    const int last = V_act % kGemmSlab;
    return last > 16 && last / 4 < k + k / 2;
}
inline bool use_small_tiles(int M, int V_act, int d, int k, int num_cu, bool bounded = false, bool packed = false) {
    const bool slow_last = slow_last_slab(V_act, k);
    if (k > kOwnBoundK && d >= 1024 && !bounded) return d <= kTileMaxD;
    const double tile_cost = d < 2048 || slow_last || (bounded && (packed || d <= 2048)) ? 3.3 : 2.9;
    auto rounds = [&](int v, int m) {
        const long n = (long)((V_act + v - 1) / v) * ((M + m - 1) / m);
        return (n + num_cu - 1) / num_cu;
    };
    return d <= kTileMaxD && (double)rounds(kGemmSlab, kTileRows) < tile_cost * (double)rounds(kGemmTile, kGemmTile);
}

// Whether small tiles of a packed matrix that sit in twos on the compute units keep W in registers (lmhead_packed_tile_kernel) or send it through LDS as
// well.  Registers gain 2 to 13 % (x 4,096, us: 28,000 at 150 rows 82.1 and 77.6; 11,000 at 300 68.0 and 60.2; 16,384 at 512 90.4 and 86.1; 32,768 at 250 96.2 and 94.1;
// x 2,048, 28,000 at 200 53.9 and 51.1), but not where only some units have two tiles and the hidden dimension is of the middle (x 2,048, 16,500 at 200 rows
// 38.5 and 40.4, 17,000 at 150 38.6 and 40.3, 8,300 at 512 39.0 and 40.0, 20,000 at 200 42.4 and 42.9; x 1,024 17,000 at 150 28.8 and 29.0; x 4,096 18,000 at 200 77.8 and 76.6),
// nor where all have two, the second row of tiles holds little and the hidden dimension is large (32,768 x 4,096 at 135 rows 88.5 and 92.9, at 170 88.7 and
// 92.0, at 200 90.1 and 88.9; x 8,192 at 150 156 and 168; x 3,072 at 140 72.3 and 74.6; x 2,048 at 135 53.7 and 50.8; 32,400 x 4,096 at 150 88.2 and 88.3).
inline bool w_in_registers(int M, int V_act, int d, int num_cu) {
    const long tiles = ((V_act + kTileRows - 1l) / kTileRows) * ((M + kTileRows - 1l) / kTileRows);
    if (4 * tiles <= 5l * num_cu && d > 1024 && d < 4096) return false;
    return !(tiles > 2l * num_cu - num_cu / 32 && tiles <= 2l * num_cu && M <= kTileRows + 48 && d >= 3072);
}

// The ring of the packed tile kernel (tile.hip): kPRing pairs of k-steps on the way.  A pair is kRingH loads of h to LDS and twice kRingW of W to
// registers, requested in this order; pair p requests half of pair p + S of W in its first k-step, waits for h of pair p + 1, and requests h
// of pair p + S and the other half in its second.  A wait names the loads of a wavefront that may still be under way: those behind
// h of pair 0 at the start, and behind h of pair p + 1 later on, when that was requested by pair p + 1 - S (at the start there are 2 * kRingW more behind it).
constexpr int kPRing = 4, kRingH = 4, kRingW = 2;
constexpr int ring_first_wait(int S) { return 2 * kRingW + (S - 1) * (kRingH + 2 * kRingW); }
constexpr int ring_wait(int S) { return kRingW + (S - 2) * (kRingH + 2 * kRingW) + kRingW; }

// A bound of every draft row for the matrix-tile kernels, from sorted lists of other candidates of the row that
// are there already (the extensions of the batched head): every list's q-th best is reached by q logits, so the
// `sets`-th largest of them is reached by k when q * sets >= k, and no core logit below it can be among the row's k
// best.  The lists of a row lie as the slab kernel leaves them, per chunk of draft rows.
constexpr int kBoundLists = 16;          // lists that are looked at (all lists' bound is hardly better)
constexpr int kBoundK = 16;              // largest k with a bound: longer lists than 16 are more than the tiles stage
struct RowBound {
    const unsigned long long* keys = nullptr;
    size_t chunk_keys = 0;               // keys between two chunks
    int n_lists = 0, q = 0, sets = 0, k = 0;
    int n_chunks = 0;                    // 0: no bound
    int m0[kMaxChunks];                  // first draft row of each chunk
};
// q and sets for n_lists lists, or q = 0 where the bound would be hardly better than the one that a slab finds by itself (reached by some
// 11 of its 128 logits).  With 3 sets to 4 lists of R rows each about 1.4 / R of all logits reach the bound for q = 1, twice
// as many for q = 2.  Without and with the bound, us for the call: 16 x 60 rows, 32,768 + 2,048 rows x 4,096, k = 10 (15 lists) 308
// and 296, k = 16 (q = 2) 333 and 302; 800 rows, 32,768 + 700, k = 4 (11 lists) 267 and 254; row-major small tiles, 197 rows, 16,384 + 1,000 (16) 80.7 and 80.0; 480 rows,
// 16,384 + 512 x 2,048 (8 lists, q = 2) 70.2 and 68.5; 300 rows, 20,000 + 2,048 (16 lists), k = 10 124.6 and 123.4, k = 16 (q = 2) 138 and 127,
// since a slab's own bound leaves more than a list of 16 holds.  Past k = 16 the lists are longer than the tiles stage.
inline void choose_bound(RowBound* b, int n_lists, int k) {
    b->n_lists = n_lists < kBoundLists ? n_lists : kBoundLists;
    b->k = k;
    b->q = 0;
    for (int q = 1; q <= 2 && k <= kBoundK; ++q) {
        const int sets = (k + q - 1) / q;
        if (4 * sets <= 3 * b->n_lists) { b->q = q; b->sets = sets; return; }
    }
}

// Whether the lists of a batch's extensions bound its draft rows: `chunks` of at most max_rows rows in one launch.
inline bool lists_bound(int max_rows, int V_arc, int d, int k, int num_cu, int chunks) {
    if (V_arc <= 0 || chunks < 1 || chunks > kMaxChunks) return false;
    const bool split = split_rows(max_rows, V_arc, d, k, num_cu, chunks);
    RowBound b;
    choose_bound(&b, make_plan(split ? kSplitRows : max_rows, V_arc, d, k, num_cu, split ? 2 * chunks : chunks, false).n_slabs, k);
    return b.q > 0;
}

struct GemmPlan {
    int n_slabs = 0;
    int list_len = 0;
    size_t keys_off = 0, stats_off = 0, total_bytes = 0;
};
inline GemmPlan make_gemm_plan(int M, int V_act, int k) {
    GemmPlan g;
    g.n_slabs = (V_act + kGemmSlab - 1) / kGemmSlab;
    g.list_len = gemm_list_len(k);
    g.stats_off = align_up((size_t)g.n_slabs * M * g.list_len * 8, 256);
    g.total_bytes = g.stats_off + align_up((size_t)g.n_slabs * M * 8, 256);
    return g;
}

// Upper bound of Plan::total_bytes over every slab shape (independent of the device).
inline size_t workspace_upper_bound(int V_act, int k) {
    const size_t n_slabs = ((size_t)V_act + kRowsMinSlab - 1) / kRowsMinSlab;
    return align_up(n_slabs * kMTile * k * 8, 256) + align_up(n_slabs * kMTile * 8, 256);
}

// Heads of 65 to 128 draft rows: the small tiles read the matrix once where passes of 64 rows read it twice.  Only where their
// lists fit the scratch: of one pass for a head (M <= 8 k), of two for the core of the batched call (from k = 8 on).
// Passes and tiles, us: 36,864 x 4,096 at 80 rows, k = 10, 118 and 86; 18,432 x 4,096 at 66 72 and 51; 20,000 x 4,096 at 80 77 and 60; 4,096 x
// 1,024 at 70 28 and 25; 16,384 x 4,096 at 96, k = 12, 74 and 58; full vocabulary row-major at 72 441 and 280; batched, 66 rows, 32,768 + 2,048 121 and
// 83, 128 rows, 4,096 + 128 x 2,048 49 and 39.  k = 13 and more and short last slabs stay with the passes: the tiles selected such rows one by one when these lines
// were drawn.  They are found by halves now, and where the lists fit the scratch the lines could move (passes and tiles, us: 16,384 x 4,096 at 128 rows, k = 16, 82 and 66,
// row-major 80 and 70; at 96, k = 13, 76 and 56; 16,384 x 2,048 at 100, k = 32, 59 and 46; 20,096 x 1,024 at 80, k = 40, 69 and 33; batched, 120 rows over 32,768 + 2,048, k =
// 16, 128 and 89).  A short last slab costs no more than a second pass over a small matrix (4,000 x 1,024 at 70 26.8 and 27.3) and less over a large one (36,896 x 2,048 at 72 75 and
// 54; 30,000 x 4,096 at 66 102 and 60; batched, 120 rows, 30,000 + 1,500 122 and 79).
// parts: the passes would sum the hidden dimension in parts (up to four wavefronts to a tile, eight in the few-row kernel), so the tiles
// sum it in kTileParts parts as well, a few more if d / 64 is no multiple of them.  Relative error of a call's logits against 64 bits in
// passes, in a single chain and in parts, 1e-8: 8,448 x 4,096 at 66 rows 9.9, 34 and 7.2; 20,000 x 4,096 at 80 23, 36 and 7.3;
// 18,432 x 2,048 at 80 16, 24 and 5.9; 4,096 x 1,024 at 70 5.8, 16 and 5.4; 8,192 x 512 at 72 5.0, 12 and 5.2, so that hidden
// sizes below 1,024 stay with the passes.  (Of a call's rows the up to 16 last ones that the few-row kernel would take, in 16 chains, are 7.5
// instead of 5.9 off at 8,448 x 4,096, the first 64 7.3 instead of 10.)
// In parts a tile's chain over a large hidden dimension takes longer than a second pass over a small matrix, above all where that pass
// has only a few rows (passes and tiles at 66 rows, k = 10: x 4,096 1,024 rows 36 and 40, 5,000 40 and 41, 6,144 47 and 45, 8,192 52 and 47; x
// 3,072 500 rows 33 and 35, 4,096 35 and 36, row-major 40 and 36; x 2,048 1,024 rows 29 and 30, 2,048 30 and 30, 3,200 31 and 30; x 1,536 and below
// the tiles from the smallest set on, 128 x 1,024 at 70 27 and 24).  Two sets gain at any size (128 + 200 rows x 4,096 at 66 67 and 51).
constexpr size_t kSlowLastMiB = 96;
constexpr int kTileParts = 8;
constexpr int kTilePartsMinD = 1024;
inline bool use_tiles_early(int M, int V_act, int d, int k, bool parts, size_t scratch) {
    return M > kMTile && M < kGemmMinRows && d % (2 * kGemmKChunk) == 0 && d <= kTileMaxD && (!parts || (d >= kTilePartsMinD && V_act >= 2 * (d - kTilePartsMinD))) && k <= 12 &&
           (!slow_last_slab(V_act, k) || matrix_elems((size_t)V_act, d, false) * 2 >= (kSlowLastMiB << 20)) &&
           make_gemm_plan(M, V_act, k).total_bytes <= scratch;
}

// How M draft rows take a matrix in matrix tiles, if they do.  one_set: no other partial set meets this one in a result.
struct TileRoute {
    bool tiles = false;      // all rows in one launch of matrix tiles
    bool small = false;      // of 128 x 128
    bool parts = false;      // which sum the hidden dimension in parts
};
inline TileRoute tile_route(int M, int V_act, int d, int k, int num_cu, bool one_set, size_t scratch) {
    const bool early = use_tiles_early(M, V_act, d, k, one_set, scratch), tiles = early || use_gemm(M, d);
    return TileRoute{tiles, early || (tiles && use_small_tiles(M, V_act, d, k, num_cu)), early && one_set};
}

// The same for the core of a batch (row_off: the first draft row of every sequence, and M).  Chunks are pieces of at most kMTile rows of one sequence, which
// without tiles end where a pass over the core does.
struct ChunkCount { int n = 0, max_rows = 0; };
inline ChunkCount count_chunks(const int32_t* row_off, int S, bool tiles) {
    ChunkCount c;
    for (int s = 0; s < S; ++s)
        for (int m0 = row_off[s], end = row_off[s + 1]; m0 < end; ++c.n) {
            const int limit = tiles ? m0 + kMTile : (m0 / kMTile + 1) * kMTile, to = end < limit ? end : limit;
            if (to - m0 > c.max_rows) c.max_rows = to - m0;
            m0 = to;
        }
    return c;
}
inline TileRoute batch_route(const int32_t* row_off, int S, int V_core, int V_arc, int d, int k, int num_cu, bool packed, size_t scratch) {
    const int M = row_off[S];
    if (V_core == 0) return TileRoute{};
    TileRoute r = tile_route(M, V_core, d, k, num_cu, V_arc == 0, scratch);
    if (V_arc > 0 && use_gemm(M, d) && k > kOwnBoundK && k <= kBoundK) {
        const ChunkCount c = count_chunks(row_off, S, true);
        if (lists_bound(c.max_rows, V_arc, d, k, num_cu, c.n)) r.small = use_small_tiles(M, V_core, d, k, num_cu, true, packed);
    }
    return r;
}

// Scratch for the shared core of the segmented head: one set of partials per 64-row pass, or
// the large-M layout from kGemmMinRows rows on.
inline size_t core_workspace_bytes(int M, int d, int V_core, int k) {
    if (use_gemm(M, d)) return make_gemm_plan(M, V_core, k).total_bytes;
    const size_t passes = ((size_t)M + kMTile - 1) / kMTile;
    return passes * workspace_upper_bound(V_core, k);
}

}  // namespace evospec

// Device-side work list of the grouped GEMMs: shared by the stand-alone scheduling kernel (moe_gemm.hip) and the
// dispatch kernels that build the work lists in the same launch as the permutation (moe_permute.hip).
#pragma once
#include "moe_internal.h"

// ------------------------------------------------------------------------------------------------
// Device-side work list.  The rows of expert e are cut into ceil(n_e / cap) row tiles of nearly
// equal height (a multiple of 32 rows, at most cap): an expert slightly larger than a multiple of
// the cap does not get a nearly empty extra tile, its rows are spread over its tiles.
//
// The cap itself is chosen per GEMM on the device from the tallest tile and the next five heights down
// (as far as their row tiles fit the work list), from the actual
// loads: a launch runs in ceil(work items / compute units) rounds of roughly one tile time each, so
// when there are only a few rounds (the second expert GEMM has few weight-row tiles) a slightly
// lower cap that fills the last round beats the tallest tile -- the tile-boundary staircase of
// Sec. 3.3.2, seen from the scheduler's side.  Estimated time of a cap, in units of one 32-row
// block of MFMA work: rounds * (mean tile height in blocks + SCHED_TILE_OVERHEAD); a launch with reduction
// splits has that many workgroups per work item.
//
// Order of the work list.  The hardware hands out the workgroups of a launch in index order:
// workgroup b goes to XCD b % 8, and within an XCD to shader engine (b / 8) % 4, whose eight compute
// units take whatever arrives there; the XCD's dispatcher does not move on while the engine whose
// turn it is has no free compute unit (measured with per-workgroup time stamps: an engine that
// keeps receiving workgroups with nothing to do idles, it cannot run ahead of the other three).
// So each XCD's queue -- the entries b = x, x + 8, x + 16, ... of the table -- is dense: real tiles
// only, empty entries follow after the last one.
//
// Which XCD gets which tiles decides how often a byte crosses the fabric.  What misses an XCD's L2 comes at no
// more than about 7 TB/s for all eight together, from HBM or out of the Infinity Cache alike (read-only kernel,
// 64 MB that only that cache holds: 6.9 TB/s), and a single compute unit gets no more than about 60 GB/s of
// misses against 130 GB/s of hits.  So all tiles stand in one row -- expert by expert; an expert of more than
// SCHED_PIECE_MAX row tiles in row ranges of nearly equal length; in a range weight-row tile by weight-row tile;
// the range's row tiles side by side, sharing that weight panel -- and each XCD takes stretches of that row: the
// token rows of an expert are fetched by the few XCDs that its tiles stretch over.  Dealing the weight-row tiles of
// every expert round-robin to the XCDs fetches them up to eight times; bytes past the L2, round-robin against one
// stretch for each XCD: 128 small experts, 8192 tokens 2.31 -> 1.35 and 1.26 -> 0.62 GB (GEMM1, GEMM2), Mixtral shape,
// 4096 tokens, GEMM2 3.39 -> 1.93 GB, 5003 Zipf-distributed rows of 32 experts 2.51 -> 2.23 and 1.16 -> 1.06 GB.
//
// But nothing is stolen between the queues, and an XCD with one stretch of tall tiles ends late.  So the row is dealt
// in laps of eight chunks of 2^SCHED_CHUNK_SHIFT tiles, one round of an XCD's compute units (of half and a quarter of
// that in shorter lists, so that a queue averages over four chunks and more), in the opposite order every other lap:
// on loads that rise or fall along the row the queues then differ by one chunk's difference in height.  Expert GEMMs,
// us, one stretch / laps / weight-row tiles round-robin: Mixtral shape, loads of 300 to 130 rows 734 / 678 / 673, four
// experts of 288 and four of 160 rows 705 / 666 / 666; 16 wide experts, 8192 Zipf-distributed rows 1810 / 1697 /
// 1709; 64 experts, the first half of 288 and the others of 160 rows 1132 / 1065 / 1079, 160 rising to 288
// 1123 / 1074 / 1092; 32 experts, 32768 Zipf-distributed rows 2377 / 2265 / 2290; 128 small experts, half of 288 and
// half of 160 rows 331 / 315 / 375.
// One stretch stays the better one
//  * where all work items run side by side (no more of them than compute units);
//  * where light tiles (below) are more than an eighth: they are bound by the fabric and come last, and it serves
//    them best when the XCDs do not all reach them at once.  Laps without this line: share of 32 of 256 experts, 8192
//    and 12000 tokens, 2 to 3 and 4 % slower; Mixtral shape, 700 to 1300 tokens of which two experts get 60 % each,
//    1 to 2 %; only 16 wide experts with 3001 tokens 2 % faster.  Light ones in among the heavy instead of behind
//    them: 2 to 8 % slower on most loads;
//  * where no expert has more than one block: all tiles cost the same.
//
// The tiles of a light expert are all weights: each streams a panel that nobody shares, while those of a heavy one
// find theirs in the L2.  An XCD whose stretch held light experts only would be bound by its share of the
// fabric while others wait (expert-parallel share, 2048 tokens, one expert with half the rows: 429 us round-robin,
// 446 in stretches).  So where there are both, the heavy experts (SCHED_HEAVY blocks of 32 rows and more, or
// several row tiles, which share their weight panels) are dealt as above and the light ones, whose few token rows
// cost little to fetch eight times, round-robin behind them until every XCD holds an eighth of all tiles: 422 us;
// Zipf-distributed rows 665 -> 652, against 665 with the light ones in stretches too; Mixtral shape, 64 tokens, experts
// of one and two blocks: 381 round-robin, 396 in stretches.  Where no expert has more than one block they are cut into
// stretches (Mixtral shape, 1 token: 124.9 against 122.9 us for the layer, 64 tokens 437 against 430).
// ------------------------------------------------------------------------------------------------
constexpr int SCHED_CU = 256;    // compute units of the device (one workgroup each)
constexpr int SCHED_PIECE_MAX = 8;  // row tiles of a row range, at most
// Per-tile cost that does not scale with the tile's height, in 32-row blocks of MFMA work.  In launches
// where every row tile has the same height and the workgroups run in step the cost is about one block
// (Mixtral shape, tiles forced to 6, 7, 8, 9 blocks: 28 rounds of GEMM1 take 2331, 2656, 2993, 3333 us).
// On ragged loads a tile costs more than that -- its weight panel is shared with fewer neighbours the
// further the workgroups drift apart -- and 3.5 picks caps that are as fast or up to 2 % faster than
// those picked with 1.0 on every benchmark workload.
constexpr float SCHED_TILE_OVERHEAD = 3.5f;
// 32-row blocks from which an expert is heavy: with more than 96 token rows against the 256 weight rows of a work item,
// fetching the token rows eight times shows
constexpr int SCHED_HEAVY = 4;
constexpr int SCHED_CHUNK_SHIFT = 5;  // log2 of the tiles in a chunk of the heavy experts' row, from 2048 tiles on
constexpr int SCHED_CAPS = 6;  // candidate caps: the tallest tile and the next five heights down
static __host__ __device__ inline int sched_min_cap_blocks(int bm) {
    const int h = bm / 32 - (SCHED_CAPS - 1);
    return h < 1 ? 1 : h;
}
// Entries of a work list (= workgroups of the launch) for at most mt row tiles: the eight queues together
// hold (row tiles * weight-row tiles) entries and differ by at most one, which takes up to 8 more entries than tiles
// (64 are kept).  Workgroups past the end of their queue exit at once, but each still has to be placed on a compute
// unit with its full LDS and register allotment (about 0.5 us), so the list follows the bound on the row tiles.
static inline int sched_grid(int mt, int nt) { return mt * nt + 64; }

// inclusive prefix sum over the 64 lanes with data-parallel-primitive moves: a Kogge-Stone scan inside
// each row of 16 lanes, then the row totals are carried into the following rows
static __device__ inline int wave_scan_incl(int v) {
#define DPP_ADD(ctrl, row_mask) v += __builtin_amdgcn_update_dpp(0, v, ctrl, row_mask, 0xf, false);
    DPP_ADD(0x111, 0xf)  // row_shr:1
    DPP_ADD(0x112, 0xf)  // row_shr:2
    DPP_ADD(0x114, 0xf)  // row_shr:4
    DPP_ADD(0x118, 0xf)  // row_shr:8
    DPP_ADD(0x142, 0xa)  // row_bcast:15 into rows 1 and 3
    DPP_ADD(0x143, 0xc)  // row_bcast:31 into rows 2 and 3
#undef DPP_ADD
    return v;
}
// inclusive scan of one int per thread over the 256 threads of the workgroup; part: 4 ints of LDS
// scratch; two barriers
static __device__ inline int block_scan_incl(int v, int32_t* part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_scan_incl(v);
    __syncthreads();  // part[] may still be read from a previous call
    if (lane == 63) part[wave] = v;
    __syncthreads();
    for (int ww = 0; ww < wave; ++ww) v += part[ww];
    return v;
}

// Which tile entry b of a work list is: the light tiles, 0 .. n_light - 1, and the heavy ones, 0 .. total - n_light - 1,
// are numbered apart.  XCD x = b % 8 has an eighth of all tiles in its queue (rounded by where the eighths begin),
// first its heavy ones, then the light ones x, x + 8, ...; the up to seven light ones left over go to the first XCDs
// that have room for one more.  The heavy ones: whole laps of eight chunks of 2^SCHED_CHUNK_SHIFT tiles (less in shorter
// lists), chunk x of the even laps and 7 - x of the odd ones, then a stretch of what is left; the stretch alone where
// one stretch is the better one (see above; alike: no expert has more than one block).  -1: past the end of the queue.
static __host__ __device__ inline int sched_entry(int total, int n_light, int b, bool* light, bool alike = false) {
    const int x = b & 7;
    int j = b >> 3;
    *light = false;
    const int heavy = total - n_light;
    const int shift = heavy >= 2048 ? SCHED_CHUNK_SHIFT : heavy >= 512 ? SCHED_CHUNK_SHIFT - 1 : SCHED_CHUNK_SHIFT - 2;
    const int laps = alike || total <= SCHED_CU || 8 * (long long)n_light > total ? 0 : heavy >> (shift + 3);
    const int dealt = laps << shift;  // tiles each XCD gets in whole laps
    if (j < dealt) {
        const int lap = j >> shift, chunk = 8 * lap + (lap & 1 ? 7 - x : x);
        return (chunk << shift) + (j & ((1 << shift) - 1));
    }
    j -= dealt;
    total -= 8 * dealt;
    auto cut = [&](int y) { return (total >> 3) * y + ((total & 7) * y >> 3); };  // total * y / 8
    const int each = n_light >> 3, left = n_light & 7;
    const int len = cut(x + 1) - cut(x);
    // XCDs before x with room for more than `each` light tiles
    const int rank = (total >> 3) > each ? x : cut(x) - each * x;
    const int lights = each + (len > each && rank < left ? 1 : 0);
    if (j >= len) return -1;
    if (j < len - lights) return 8 * dealt + cut(x) - each * x - (rank < left ? rank : left) + j;
    *light = true;
    const int jl = j - (len - lights);
    return jl < each ? 8 * jl + x : 8 * each + rank;
}

// The tile with index g in the row of tiles of the experts that pre counts (pre[e]: row tiles of those before e,
// pre[E_local] of all; an expert may have none): expert by expert, row range by row range, weight-row tile by weight-row
// tile.  s_off: the exclusive prefix of the experts' rows.  0 <= g < pre[E_local] * nt.
static __host__ __device__ inline TileDesc sched_tile(int g, const int32_t* pre, const int32_t* s_off, int E_local, int nt,
                                                      int bn) {
    // the expert e with pre[e] * nt <= g < pre[e + 1] * nt
    int lo = 0, hi = E_local;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (pre[mid] * nt <= g) lo = mid; else hi = mid;
    }
    const int e = lo;
    const int mte = pre[e + 1] - pre[e];
    // its row ranges: pp of them, the first prem one tile longer
    const int pp = (mte + SCHED_PIECE_MAX - 1) / SCHED_PIECE_MAX, pbase = mte / pp, prem = mte % pp;
    int r = g - pre[e] * nt;
    int range, len;
    if (r < prem * (pbase + 1) * nt) {
        len = pbase + 1;
        range = r / (len * nt);
        r -= range * len * nt;
    } else {
        r -= prem * (pbase + 1) * nt;
        len = pbase;
        range = prem + r / (len * nt);
        r -= (range - prem) * len * nt;
    }
    const int ni = r / len;
    const int mi = range * pbase + (range < prem ? range : prem) + r % len;
    const int e_rows = s_off[e + 1] - s_off[e];
    // 32-row blocks of the expert, dealt evenly to its mte tiles
    const int nblk = (e_rows + 31) / 32;
    const int base = nblk / mte, rem = nblk % mte;
    const int blk0 = mi * base + (mi < rem ? mi : rem);
    const int rows = (base + (mi < rem ? 1 : 0)) * 32, left = e_rows - blk0 * 32;
    TileDesc td;
    td.expert = e;
    td.row0 = s_off[e] + blk0 * 32;
    td.rows = rows < left ? rows : left;
    td.n0 = ni * bn;
    return td;
}

// Whether an expert of nblk 32-row blocks in mte row tiles is heavy
static __host__ __device__ inline bool sched_heavy(int nblk, int mte) { return nblk >= SCHED_HEAVY || mte > 1; }

// The cap of a launch (tallest row tile, in 32-row blocks) among the SCHED_CAPS from hmax down.  tot: 32-row blocks of all
// experts, then their row tiles under each candidate (0: none of that height).
static __host__ __device__ inline int sched_cap(const int* tot, int hmax, int nt, int nsplit, int grid) {
    int cap = hmax;
    float best = 3.0e38f;
#pragma unroll
    for (int c = 0; c < SCHED_CAPS; ++c) {
        const int tiles = tot[c + 1];
        if (tiles > 0 && (long long)tiles * nt + 8 <= grid) {
            const int rounds = (tiles * nt * nsplit + SCHED_CU - 1) / SCHED_CU;
            const float est = (float)rounds * ((float)tot[0] / (float)tiles + SCHED_TILE_OVERHEAD);
            if (est < best) {  // ties keep the taller tile
                best = est;
                cap = hmax - c;
            }
        }
    }
    return cap;
}

// Builds this workgroup's share of the work lists: of `parts` workgroups the first a.parts1 build the first GEMM's
// list, the others the second's (entries tid, + 256 * workgroups of the list, ...).  What bounds a build is the chain
// of dependent integer work in one thread -- cap, scans, then divisions and a binary search per entry -- and
// the two lists have nothing in common but the totals, so no workgroup walks both chains:
// dispatch launch of the layer 10.4 -> 7.1 us (Mixtral shape, 1 token), 11.3 -> 7.6 (128 small experts, 77 tokens),
// 13.6 -> 9.7 (expert-parallel share, 2048 tokens); stand-alone build 11.0 -> 7.6 (16 wide experts, 3001 tokens).
// s_off: the exclusive prefix of the experts' rows, [E_local + 1] entries in SHARED memory, written by the caller and
// published by a barrier before the call.  All 256 threads of the workgroup must call.
static __device__ inline void schedule_tables(const SchedArgs& a, const int32_t* s_off, int part, int parts) {
    __shared__ int32_t s_pre[2][257];  // row tiles of the heavy (0) and light (1) experts before e; [E_local] = all
    __shared__ int32_t s_part[4];
    __shared__ int32_t s_tot[SCHED_CAPS + 1][4];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int E_local = a.E_local;
    int nblk_e = 0;  // 32-row blocks of expert tid
    if (tid < E_local) nblk_e = (s_off[tid + 1] - s_off[tid] + 31) / 32;
    const int hmax = a.bm / 32, hmin = sched_min_cap_blocks(a.bm);
    // totals over the experts: 32-row blocks, row tiles for every candidate cap
    int tot[SCHED_CAPS + 1];
    tot[0] = nblk_e;
#pragma unroll
    for (int c = 0; c < SCHED_CAPS; ++c) {
        const int h = hmax - c;
        tot[c + 1] = (h >= hmin && nblk_e > 0) ? (nblk_e + h - 1) / h : 0;
    }
#pragma unroll
    for (int c = 0; c < SCHED_CAPS + 1; ++c) {
        const int incl = wave_scan_incl(tot[c]);
        if (lane == 63) s_tot[c][wave] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < SCHED_CAPS + 1; ++c) tot[c] = s_tot[c][0] + s_tot[c][1] + s_tot[c][2] + s_tot[c][3];

    const bool which = part >= a.parts1;
    if (which) part -= a.parts1;
    parts = which ? parts - a.parts1 : a.parts1;
    const int nt = which ? a.nt2 : a.nt1;
    const int grid = which ? a.grid2 : a.grid1;
    TileDesc* table = which ? a.t2 : a.t1;
    const int nsplit = which ? a.nsplit2 : a.nsplit1;  // reduction splits: workgroups per table entry
    const int cap = sched_cap(tot, hmax, nt, nsplit, grid);
    // ---- the heavy experts' tiles in one row, the light ones' in another ----------------------
    const int mte_mine = (nblk_e + cap - 1) / cap;
    const bool alike = !__syncthreads_or(nblk_e > 1);  // no expert has more than one block
    const bool heavy_mine = alike || sched_heavy(nblk_e, mte_mine);
    const int incl_h = block_scan_incl(heavy_mine ? mte_mine : 0, s_part);
    const int incl_l = block_scan_incl(heavy_mine ? 0 : mte_mine, s_part);
    s_pre[0][tid + 1] = incl_h;
    s_pre[1][tid + 1] = incl_l;
    if (tid < 2) s_pre[tid][0] = 0;
    __syncthreads();
    const int n_light = s_pre[1][E_local] * nt, total = s_pre[0][E_local] * nt + n_light;
    // Offsets beyond the bound the launches and the buffers were sized for: nothing is scheduled (every
    // entry stays empty, so no kernel touches a row) and the refusal is recorded for the caller.
    const bool refused = a.rows_cap >= 0 && s_off[E_local] > a.rows_cap;
    if (which == 0 && a.refused_out != nullptr && part == 0 && tid == 0) *a.refused_out = refused ? 1 : 0;
    for (int b = part * 256 + tid; b < grid; b += parts * 256) {
        TileDesc td;
        td.expert = 0; td.row0 = 0; td.rows = 0; td.n0 = 0;
        bool light;
        const int g = sched_entry(total, n_light, b, &light, alike);  // index among the heavy, or the light, tiles
        if (!refused && g >= 0) td = sched_tile(g, s_pre[light ? 1 : 0], s_off, E_local, nt, a.bn);
        table[b] = td;
    }
}


// Work split of the tiled GEMM kernels: which output tiles a persistent workgroup computes, in which order.
// Shared by the kernels (device) and the launch code (host); the host can replay the whole schedule
// (batq_debug_tile_schedule) so that it can be checked without a GPU.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace batq {

constexpr int kTile = 256;                 // tile rows
constexpr int kStrip = 64;                 // tile columns come in strips of 64

struct TilePlan {
    int tiles_m;      // row panels of 256
    int strips_n;     // column strips of 64
    int bands;        // column bands (1, 2, 4 or 8)
    int workers;      // workgroups launched, a multiple of 8
    int ksplit;       // parts the K groups are cut into (1: every tile runs over all of K)
    int groups;       // K groups of 256 elements
    int pair;         // 64-column strips per scheduling unit: 1, or 2 when tiles must be an even number of strips
                      // wide (gated output; strips_n then counts units of 128 columns)
    int whole_runs;   // 1: no share reaches from one run (a row panel of a band) into the next, see worker_share
};

struct Tile {
    int m0, n0, nj;
    int part, g0, ng;   // K part, its first K group and its number of K groups
};

// A workgroup's walk through its share [cur, end) of the linear order: K part by K part, inside a part the strip
// order (column bands -> row panels -> strips).  The position is decoded once (divisions) and then advanced tile by
// tile with additions and compares only: the kernels take the next tile between an epilogue and the next main loop,
// where every instruction is on the critical path (the same walk decoded from scratch for every tile cost ~900 cycles
// per tile).
struct TileWalk {
    int cur, end;            // position and end of the share, in scheduling units over all K parts
    int part, at;            // K part of `cur` and position inside it
    int b, bs, width;        // column band of `cur`: index, first unit, units
    int p, sl;               // row panel and unit inside the band's panel row
    int g0, ng;              // K groups of `part`
    int lead;                // narrower tiles still to be put in front of the wider ones (see walk_begin)
};

__host__ __device__ inline void walk_set_band(const TilePlan& pl, TileWalk& w) {
    w.bs = w.b * pl.strips_n / pl.bands;
    w.width = (w.b + 1) * pl.strips_n / pl.bands - w.bs;
}
__host__ __device__ inline void walk_set_part(const TilePlan& pl, TileWalk& w) {
    w.g0 = pl.groups * w.part / pl.ksplit;
    w.ng = pl.groups * (w.part + 1) / pl.ksplit - w.g0;
}
// Tiles a run of `run` units is cut into: at most 4 strips = 4 / pair units each.
__host__ __device__ inline int run_tiles(const TilePlan& pl, int run) {
    const int shift = pl.pair == 2 ? 1 : 2;
    return (run + (1 << shift) - 1) >> shift;
}
// Start of the walk over [cur, end) by workgroup `block`.
// A run of units is cut into tiles of near-equal width, i.e. of two widths one unit apart.  Workgroups whose shares
// are alike would all reach their epilogues at the same moments, and the whole chip would then write its output
// in bursts (the write path, not the compute units, sets the length of such an epilogue) and not at all in
// between.  So the workgroups of an XCD take turns in how many of the narrower tiles of their first run they put in
// front of the wider ones: with 3 narrow tiles of 10 the four classes run a quarter of a tile apart.  Workgroups that
// stream the same weight columns (same place in their row panel, 8 apart inside the XCD) are in the same class.
__host__ __device__ inline void walk_begin(const TilePlan& pl, int block, int cur, int end, TileWalk& w) {
    w.cur = cur;
    w.end = end;
    const int per_part = pl.tiles_m * pl.strips_n;
    w.part = pl.ksplit > 1 ? cur / per_part : 0;
    w.at = cur - w.part * per_part;
    w.b = 0;
    while (w.b + 1 < pl.bands && w.at >= pl.tiles_m * ((w.b + 1) * pl.strips_n / pl.bands)) ++w.b;
    walk_set_band(pl, w);
    const int local = w.at - pl.tiles_m * w.bs;
    w.p = local / w.width;
    w.sl = local - w.p * w.width;
    walk_set_part(pl, w);
    int run = end - cur;
    if (per_part - w.at < run) run = per_part - w.at;
    if (w.width - w.sl < run) run = w.width - w.sl;
    w.lead = 0;
    if (run > 0) {
        const int nt = run_tiles(pl, run);
        const int wide = nt == 1 ? run : (run + nt - 1) / nt;
        const int narrow = nt * wide - run;                 // tiles of width wide - 1 in the run
        w.lead = (block >> 3) & 3;
        while (w.lead > narrow) w.lead -= narrow + 1;
    }
}
// Takes the next tile off the walk: at most 4 strips of what is left of the share in this row panel of the band (a
// tile does not reach into the next panel, band or K part), the run cut into tiles of near-equal width.
__host__ __device__ inline bool next_tile(const TilePlan& pl, TileWalk& w, Tile& t) {
    if (w.cur >= w.end) return false;
    const int per_part = pl.tiles_m * pl.strips_n;
    int run = w.end - w.cur;
    if (per_part - w.at < run) run = per_part - w.at;
    if (w.width - w.sl < run) run = w.width - w.sl;       // units left in this row panel of the band
    const int nt = run_tiles(pl, run);                    // tiles the run is cut into, near-equal widths
    int units = nt == 1 ? run : (run + nt - 1) / nt;
    if (w.lead > 0 && units * nt != run) {                // a narrower tile first
        --units;
        --w.lead;
    }
    t.nj = units * pl.pair;
    t.m0 = w.p * kTile;
    t.n0 = (w.bs + w.sl) * kStrip * pl.pair;
    t.part = w.part;
    t.g0 = w.g0;
    t.ng = w.ng;
    // advance
    w.cur += units;
    w.at += units;
    w.sl += units;
    if (w.sl == w.width) {
        w.sl = 0;
        if (++w.p == pl.tiles_m) {
            w.p = 0;
            if (++w.b == pl.bands) {                      // the part is done (at == per_part)
                w.b = 0;
                w.at = 0;
                ++w.part;
                if (w.cur < w.end) walk_set_part(pl, w);
            }
            if (w.cur < w.end) walk_set_band(pl, w);
        }
    }
    return true;
}

// First of the shares that start at or after unit `pos` when the shares are dealt out run by run: the workgroups in proportion
// to the units in front of `pos`, rounded (total < 2^20, workers <= 2^11).
__host__ __device__ inline int shares_before(const TilePlan& pl, int pos, int total) {
    return (int)(((uint32_t)pos * (uint32_t)pl.workers + (uint32_t)total / 2) / (uint32_t)total);
}

// The share of the linear order that workgroup `block` of `pl.workers` works on: workgroups go to the 8 XCDs
// round-robin, so workgroup b takes share (b % 8) * (workers / 8) + b / 8 and the shares of one XCD are
// contiguous.
// A tile cannot reach into the next run (row panel of a band), so a share that does costs an extra, narrower tile, and its
// workgroup is the one the launch waits for (two tiles of one strip take nearly twice as long as one of two).  Where the
// shares come in two sizes anyway, whole_runs deals the workgroups out run by run and lets each run's workgroups
// share it evenly: the same two sizes, and no share in two runs (graph-replayed, 700 x 4096 x 8192: 25.5 -> 22.4 us,
// with 8-bit codes 42.1 -> 30.3; 2500 x 4096 x 4096 32.4 -> 27.8, 49.6 -> 38.3; 2300 x 4096 x 14336 73.0 -> 68.5, 107.7 -> 94.2).
__host__ __device__ inline void worker_share(const TilePlan& pl, int block, int& cur, int& end) {
    const int per_xcd = pl.workers >> 3;
    const int share = (block & 7) * per_xcd + (block >> 3);
    const int64_t total = (int64_t)pl.tiles_m * pl.strips_n * pl.ksplit;
    if (total < (1 << 20)) {                    // the usual case: 32-bit products and divisions (workers <= 2^11)
        const uint32_t t32 = (uint32_t)total, wk = (uint32_t)pl.workers;
        cur = (int)(t32 * (uint32_t)share / wk);
        if (pl.whole_runs) {
            // the run of an even share is this one's or a neighbour of it
            int b = 0;
            while (b + 1 < pl.bands && cur >= pl.tiles_m * ((b + 1) * pl.strips_n / pl.bands)) ++b;
            int bs = b * pl.strips_n / pl.bands, width = (b + 1) * pl.strips_n / pl.bands - bs;
            int start = pl.tiles_m * bs + (cur - pl.tiles_m * bs) / width * width;
            int first = shares_before(pl, start, (int)t32), last = shares_before(pl, start + width, (int)t32);
            while (share < first || share >= last) {
                if (share < first) {
                    if (start == pl.tiles_m * bs) {                 // into the band before
                        --b;
                        bs = b * pl.strips_n / pl.bands;
                        width = (b + 1) * pl.strips_n / pl.bands - bs;
                    }
                    start -= width;
                } else {
                    start += width;
                    if (start == pl.tiles_m * (bs + width)) {       // into the next band
                        ++b;
                        bs = b * pl.strips_n / pl.bands;
                        width = (b + 1) * pl.strips_n / pl.bands - bs;
                    }
                }
                first = shares_before(pl, start, (int)t32);
                last = shares_before(pl, start + width, (int)t32);
            }
            const uint32_t n = (uint32_t)(last - first), i = (uint32_t)(share - first);
            cur = start + (int)((uint32_t)width * i / n);
            end = start + (int)((uint32_t)width * (i + 1) / n);
            return;
        }
        end = (int)(t32 * (uint32_t)(share + 1) / wk);
        return;
    }
    cur = (int)(total * share / pl.workers);
    end = (int)(total * (share + 1) / pl.workers);
}

// What the ends of the runs mean for a plan's shares: 0 - no share in two runs takes more tiles for it than the largest share does
// alone; 1 - some do, and whole_runs avoids it: the shares come in two sizes, and every run can be made up of the
// workgroups that fall to it with those; 2 - some do, and it cannot.  (More than 64 runs, i.e. 2: not looked into,
// for the host's time.)  Called up to four times per launch: 32-bit divisions, and no further run looked at once the answer is
// 2 (plan of 1536 x 8192: 0.95 -> 0.07 us, 3669 x 9865 0.86 -> 0.55, 4096 x 4096 0.32 -> 0.25).
inline int run_ends(const TilePlan& pl) {
    const int64_t total64 = (int64_t)pl.tiles_m * pl.strips_n, runs = (int64_t)pl.tiles_m * pl.bands;
    if (pl.workers > 2048 || total64 >= (1 << 20) || total64 <= pl.workers) return 0;
    if (runs > 64) return 2;
    const uint32_t total = (uint32_t)total64, wk = (uint32_t)pl.workers;        // products below stay under 2^32
    const int lo = (int)(total / wk), hi = (int)((total + wk - 1) / wk);
    const int hi_tiles = run_tiles(pl, hi);
    bool costly = false, possible = hi > lo;
    int pos = 0, first = 0, start = 0;
    for (int b = 0; b < pl.bands; ++b) {
        const int next = (b + 1) * pl.strips_n / pl.bands, width = next - start;
        start = next;
        for (int p = 0; p < pl.tiles_m; ++p) {
            pos += width;
            if (possible) {
                const int last = shares_before(pl, pos, (int)total), n = last - first;
                if (n * lo > width || n * hi < width) possible = false;
                first = last;
            }
            if (!costly) {
                // the even share that holds unit pos
                const uint32_t s = (((uint32_t)pos + 1) * wk - 1) / total;
                const int cur = (int)(total * s / wk), end = (int)(total * (s + 1) / wk);
                costly = cur < pos && pos < end && run_tiles(pl, pos - cur) + run_tiles(pl, end - pos) > hi_tiles;
            }
            if (costly && !possible) return 2;
        }
    }
    return costly ? 1 : 0;
}

// Column bands: with b bands an XCD's block spans 1/b of N and b/8 of M.  A workgroup walks its strips along N
// inside a row panel, tile round by tile round (a tile is at most 4 strips wide); the workgroups of an XCD do so in
// step, so a round streams the block's A rows once more (they do not survive a round in the 4 MiB L2: measured on
// 8192 x 3584 x 18944 with 4 bands, 10 rounds: 746 MB fetched where one pass over the blocks would be 140 MB)
// and its share of the B columns once.  The bytes all L2s pull are therefore proportional to
// rounds * b * M + (8 / b) * N; take the b that minimises it.
// Where that b leaves shares in two runs (run_ends 2) and another does not, the next cheapest of those serves as long as its
// bytes stay below 1.4 times the least (5293 x 4096 x 6075 at 1.30 times the bytes 73.2 -> 70.5 us with 4-bit, 111.7 -> 104.6
// with 8-bit codes; 3669 x 4096 x 9865 at 1.46 times 90.4 -> 92.2, 135.1 -> 128.2).  With one tile per workgroup the second
// tile costs more than any bytes do: 300 shapes at up to 7 times the bytes, 4 to 15 % gained with 4-bit, 7 to 30 % with 8-bit
// codes (2720 x 4096 x 5802 at 2.2 times 42.5 -> 40.4 and 66.2 -> 58.0 us; 382 x 4096 x 16304 at 6.8 times 28.2 -> 26.3 and
// 45.8 -> 32.6; 262 x 4096 x 16320 at 7.1 times 27.0 -> 23.8).  Not so for shares of three and four strips where the output's
// rows do not start on whole 128-byte lines: their slow stores hide a tile of a short K.  With 8-bit codes below K = 2048 the limit
// stays at 1.4 (1720 x 1024 x 7047 at 2.8 times 26.3 -> 27.8 us, 2093 x 512 x 5556 at 2.4 times 21.3 -> 22.7; but 646 x 2048 x 16524
// at 3.1 times 39.7 -> 37.9, and shares of three, 361 x 1024 x 16551 at 6.8 times 21.7 -> 19.7).  With 4-bit codes it is 2.6 where
// less than an eighth of the workgroups has four, K = 1024 to 5888 (1664 x 4096 x 7120 at 2.9 times 35.7 -> 38.0 us, 656 x 1024 x
// 16668 at 3.1 times 18.8 -> 20.1; but 1520 x 512 x 8202 at 3.3 times 15.1 -> 14.6, 544 x 8192 x 16753 at 3.2 times 67.7 -> 62.2,
// 2188 x 4096 x 5574 at 2.3 times 40.3 -> 38.2).
// Where every b leaves such shares, the cheapest serves after all: more bands are more runs, and more bytes besides (one tile
// each, the costliest b -> the cheapest: 7363 x 4096 x 1607 44.8 -> 34.3 us, with 8-bit codes 74.7 -> 52.7; 20000 x 4096 x 768
// 68.9 -> 37.8, 129.0 -> 58.1).  Except with 8-bit codes, whose tiles take the matrix cores twice as long for less than twice
// the bytes, and shares of up to three strips, where a second tile weighs most: one band, the fewest runs (768 x 4096 x 16384
// 55.3 us with the cheapest, 52.0 with one; 1358 x 4096 x 5401 48.3 and 43.3; 6144 x 4096 x 2048 50.8 and 47.2; shares of four,
// 1412 x 4096 x 10761: 64.1 and 65.6; 4-bit 768 x 4096 x 16384: 34.9 and 36.9).
inline double byte_limit(const TilePlan& pl, long strips, long per_worker, int out_cols, bool a8) {
    constexpr double kAny = 1e100;
    if (per_worker > 4) return 1.4;
    if (out_cols % 64 == 0) return kAny;
    if (per_worker != 4) return kAny;
    if (a8) return pl.groups < 8 ? 1.4 : kAny;
    const bool few = (strips % pl.workers) * 8 < pl.workers;
    return few && pl.groups >= 4 && pl.groups < 24 ? 2.6 : kAny;
}
inline void choose_bands(TilePlan& pl, int M, int N, bool a8) {
    const long strips = (long)pl.tiles_m * pl.strips_n;
    const long per_worker = (strips + pl.workers - 1) / pl.workers;
    const long rounds = per_worker > 4 ? (per_worker + 3) / 4 : 1;
    constexpr double kNever = 1e300;
    double cost[4], limit = kNever;
    for (int i = 0; i < 4; ++i) cost[i] = (1 << i) <= pl.strips_n ? (double)(rounds << i) * M + (8.0 / (1 << i)) * N : kNever;
    int first = 0;
    for (int tries = 0; tries < 4; ++tries) {
        int best = 0;
        for (int i = 1; i < 4; ++i)
            if (cost[i] < cost[best]) best = i;
        if (cost[best] >= limit) break;
        pl.bands = 1 << best;
        const int ends = run_ends(pl);
        pl.whole_runs = ends == 1;
        if (ends != 2) return;
        if (tries == 0) {
            first = best;
            limit = byte_limit(pl, strips, per_worker, N / pl.pair, a8) * cost[best];
        }
        cost[best] = kNever;
    }
    pl.bands = a8 && per_worker <= 3 ? 1 : 1 << first;
    pl.whole_runs = 0;
}

// K parts wanted for a plan without them: fewer strips than half the workgroups (few rows, narrow N) and a
// long K.  A part keeps at least 12 K groups: below that the partial sums' round trip costs more than the
// idle compute units.  `part_bytes` = partial-sum bytes of one part, `scratch_bytes` = what is available.
inline int choose_ksplit(const TilePlan& pl, size_t part_bytes, size_t scratch_bytes) {
    const int strips = pl.tiles_m * pl.strips_n;
    int ksplit = pl.workers / strips;
    if (pl.groups / 12 < ksplit) ksplit = pl.groups / 12;
    if (ksplit > 8) ksplit = 8;
    while (ksplit > 1 && (size_t)ksplit * part_bytes > scratch_bytes) --ksplit;
    return ksplit < 1 ? 1 : ksplit;
}

// Plan of a launch without K parts (ksplit = 1); `glu`: gated output, tiles an even number of strips wide; `a8`: 8-bit
// activation codes.
inline TilePlan make_plan(int M, int N, int nb, int cus, bool glu, bool a8) {
    TilePlan pl;
    pl.pair = glu ? 2 : 1;
    pl.tiles_m = (M + kTile - 1) / kTile;
    pl.strips_n = (N + kStrip * pl.pair - 1) / (kStrip * pl.pair);
    pl.workers = 8 * (cus / 8 > 1 ? cus / 8 : 1);       // one persistent workgroup per compute unit
    pl.bands = 1;
    pl.ksplit = 1;
    pl.groups = (nb + 7) / 8;
    pl.whole_runs = 0;
    choose_bands(pl, M, N, a8);
    return pl;
}

}  // namespace batq

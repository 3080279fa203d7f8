// Rules of the launches that depend on sizes alone, in plain C++ (so that they can be
// checked without a GPU).
#pragma once

#include <cstdint>
#include <initializer_list>

#if defined(__HIPCC__)
#define MV_RULE __host__ __device__ inline
#else
#define MV_RULE inline
#endif

namespace mv {

// HIP refuses a launch of 2^32 threads or more along x; y and z hold at most 65535 blocks.
constexpr int64_t kMaxThreadsX = (int64_t)1 << 32;
constexpr int64_t kMaxGridYZ = 65535;

// ---- beam step on the interleaved grid (kernels_beam.hip) -------------------
constexpr int kBeamGroup = 4;  // beams that one block evaluates its sources on

// Blocks of `spb` sources that one XCD may have to do of a time slot with up to max_m.
MV_RULE int64_t tf_blocks_per_xcd(int64_t max_m, int spb) { return ((max_m + spb - 1) / spb + 7) / 8; }

// Grid of the beam step: x the source blocks (8 XCDs), y the time slots, z the (channel
// group, beam group) pairs, of which one launch takes up to kMaxGridYZ.  As a single x
// dimension the product of the three passed 2^32 threads at sizes that fit the memory
// (128 beams, 3.1 million sources, 11 times of one channel).
struct TfGrid {
    int64_t x, y, z;
};
MV_RULE TfGrid tf_grid(int64_t max_m, int spb, int n_slot, int n_freq, int fg, int n_beam) {
    return TfGrid{8 * tf_blocks_per_xcd(max_m, spb), n_slot,
                  (int64_t)((n_freq + fg - 1) / fg) * ((n_beam + kBeamGroup - 1) / kBeamGroup)};
}

// ---- k-splits of the persistent product launches (k_worklist) ----------------
constexpr int kAntBlock = 128;      // antennas of a block of the product over sources
constexpr int kShortAnts = 96;      // a last block of at most so many has a diagonal launch of its own
constexpr int kMinSplitCols = 64;   // columns that a split keeps at least when splits are added
constexpr int kItemCost = 24480;    // what an item costs beside its columns, in column tiles
constexpr int kFreeCols = 2048;     // splits this short may be fewer than fill the grid
constexpr int kMaxCut = 1024;       // splits of an instance that are considered

// What decides the k-splits of a batch: instance i has K columns and gets n splits of kc
// columns (the last one shorter).
struct SplitRule {
    int64_t ksplit;       // columns of a split at most
    int32_t grid;         // workgroups of the persistent launches; 0: splits of ksplit columns, none added
    int32_t n_st;         // items per split in the item prefix
    int32_t n_bal;        // items per split of the launch that is balanced
    int32_t max_splits;   // splits of an instance that the partials have room for
    int32_t plain_splits; // splits of ksplit columns that the context's columns make
    int32_t n_launch;     // launches over the same splits (0 or 1: n_bal alone counts)
    int32_t items[3];     // their items per split
    int32_t weight[3];    // what a column costs in an item of each (16 x 16 tiles)
    int32_t part_cost;    // what a split's partial costs, in column tiles
};

// The launches of the product over sources as they are cut: full diagonal blocks (136
// tiles an item: two triangles of 36 and a square of 64), a short last one (78 tiles: six
// tile rows), and two items of two 128 x 128 products per block pair (128 tiles, fewer with
// the short block's rows).
// Costs measured on BF16X3 (a column of a diagonal item is 0.09 us): kItemCost an item of
// any launch beside its columns, 17 us (start, end, partial); a split 0.25 us at 200 antennas
// (contention of the partials' writes, and the split sum's read).  Launches and split sum,
// measured and by these: 200 antennas, 64 instances of 1000 columns in 128 / 256 splits
// 205 / 237 and 184 / 200 us; 300 antennas, 6 of 10 000 in 82 / 126 splits 293 / 274 and 294 / 290;
// 160 antennas, 8 of 3000 in 128 / 176 splits 105 / 112 and 103 / 120.
MV_RULE bool short_last_block(int n_ant, int nb) { return n_ant - (nb - 1) * kAntBlock <= kShortAnts; }
MV_RULE void add_launch(SplitRule &r, int items, int weight) {
    r.items[r.n_launch] = items;
    r.weight[r.n_launch++] = weight;
}
MV_RULE void sources_launches(int n_ant, int n_rows_pad, SplitRule &r) {
    const int nb = n_rows_pad / (2 * kAntBlock);
    const bool cut = short_last_block(n_ant, nb);
    const int rows = (n_ant - (nb - 1) * kAntBlock + 15) / 16;  // tile rows of the last block
    r.n_launch = 0;
    if (cut && nb > 1) add_launch(r, nb - 1, 136);
    add_launch(r, cut ? 1 : nb, cut ? 78 : 136);
    if (nb > 1) add_launch(r, nb * (nb - 1), ((nb - 2) * 128 + 2 * 16 * rows) / nb);
    r.part_cost = (int32_t)((int64_t)4 * n_ant * n_ant / 380);
}

// The plan of a batch: splits of at most cols columns where cols > 0, else `share` splits
// more than ceil(K / ksplit) for each instance and one more for the first `rest`; at most
// `cap` an instance.
struct SplitPlan {
    int64_t cols, share, rest;
    int32_t cap;
};
struct Split {
    int32_t n;
    int64_t kc;
};
// (32-bit division is far shorter on the GPU)
MV_RULE int64_t floor_div(int64_t a, int64_t b) {
    if (a < ((int64_t)1 << 31) && b < ((int64_t)1 << 31)) return (uint32_t)a / (uint32_t)b;
    return a / b;
}
MV_RULE int64_t ceil_div(int64_t a, int64_t b) { return floor_div(a + b - 1, b); }
MV_RULE Split split_of(const SplitRule &r, const SplitPlan &p, int64_t K, int i) {
    int64_t n = ceil_div(K, r.ksplit), kc = r.ksplit;
    if (r.grid > 0 && K > 0) {
        int64_t want = p.cols > 0 ? ceil_div(K, p.cols) : n + p.share + (i < p.rest ? 1 : 0);
        const int64_t room = ceil_div(K, kMinSplitCols);
        want = want < p.cap ? want : p.cap;
        want = want < room ? want : room;
        n = want > n ? want : n;
        kc = ceil_div(ceil_div(K, n), 64) * 64;
        n = ceil_div(K, kc);
    }
    return Split{(int32_t)n, kc};
}

// Time of the launches over `units` splits of `cols` columns on average and `longest` at
// most, in column tiles: whole waves of the grid, and the partials.
MV_RULE int64_t split_cost(const SplitRule &r, int64_t units, int64_t cols, int64_t longest) {
    int64_t c = units * r.part_cost;
    for (int l = 0; l < r.n_launch; l++) {
        const int64_t waves = ceil_div(r.items[l] * units, r.grid);
        c += r.weight[l] * ((waves - 1) * cols + longest) + waves * kItemCost;
    }
    return c;
}

// k-splits of a batch of n_slot x nfb instances; cols(slot) is an instance's K.  One
// launch: extra splits until its items fill whole waves of the grid (of n_bal items a
// split; the splits themselves, n_bal = 1, once there is a grid's worth of them).
// Several launches of different item counts: as many splits as fill the grid, which are
// whole waves of each launch, as far as plain_splits allow; or splits of equal length,
// chosen by the summed whole waves of the launches as they are cut, where these take
// less by more than 1/32 -- fewer splits than the former (partials cost too) only of
// kFreeCols columns at most, where a split's rounding is below that of its operands on
// BF16X3 (error against 64 bits on 200 antennas 2.6e-6 in splits of 10 000 columns,
// 3.2e-6 in splits of 20 000).  With the launches counted as one of nb items a split, 200
// antennas and 64 instances of 40 000 columns made 128 splits and took 3.97 ms where 256
// take 2.58; 350 antennas and 48 instances of 20 000 columns took 4.71 ms, 3.42 with the grid
// filled as far as the plain splits went, 2.87 in splits chosen so.
// G: a group of threads (id, size) that all call this, with sum, max and min over them.
template <class G, class Cols>
MV_RULE SplitPlan plan_splits(const SplitRule &r, int n_slot, int nfb, Cols cols, G &g) {
    SplitPlan p{0, 0, 0, r.max_splits};
    if (r.grid <= 0) return p;
    const int n_inst = n_slot * nfb;
    int64_t v = 0;
    for (int s = g.id; s < n_slot; s += g.size) v += nfb * ceil_div(cols(s), r.ksplit);
    const int64_t t = g.sum(v);
    const bool several = r.n_launch > 1;
    const int64_t n = several || (r.n_st == 1 && t >= r.grid) ? 1 : r.n_bal;
    const int64_t extra = floor_div(ceil_div(t * n, r.grid) * r.grid, n) - t;
    if (extra > 0) p.share = floor_div(extra, n_inst), p.rest = extra - p.share * n_inst;
    if (!several || t == 0 || t >= r.grid) return p;

    p.cap = r.plain_splits;
    int64_t units = 0, all = 0, longest = 0, most = 0;
    for (int i = g.id; i < n_inst; i += g.size) {
        const int64_t K = cols(i / nfb);
        const Split s = split_of(r, p, K, i);
        units += s.n;
        all += K;
        if (s.n > 0) longest = longest > s.kc ? longest : s.kc;
        most = most > K ? most : K;
    }
    units = g.sum(units);
    all = g.sum(all);
    longest = g.max(longest);
    most = g.max(most);
    const int64_t now = split_cost(r, units, ceil_div(all, units), longest);
    // candidates: the longest instance in j splits
    constexpr int64_t kNone = (int64_t)1 << 62;
    int64_t best = kNone;
    const int top = r.max_splits < kMaxCut ? r.max_splits : kMaxCut;
    for (int j = 1 + g.id; j <= top; j += g.size) {
        const int64_t len = ceil_div(ceil_div(most, j), 64) * 64;
        if (len > r.ksplit || (j > 1 && len < kMinSplitCols)) continue;
        int64_t u = 0;
        for (int s = 0; s < n_slot; s++) u += nfb * ceil_div(cols(s), len);
        if (u < units && len > kFreeCols) continue;
        const int64_t key = split_cost(r, u, ceil_div(all, u), len) * (2 * kMaxCut) + j;
        best = best < key ? best : key;
    }
    best = g.min(best);
    if (best < kNone && best / (2 * kMaxCut) < now - now / 32) {
        p.cap = r.max_splits;
        p.cols = ceil_div(ceil_div(most, best % (2 * kMaxCut)), 64) * 64;
    }
    return p;
}

// A single thread as plan_splits wants it.
struct OneThread {
    int id = 0, size = 1;
    MV_RULE int64_t sum(int64_t v) { return v; }
    MV_RULE int64_t max(int64_t v) { return v; }
    MV_RULE int64_t min(int64_t v) { return v; }
};

// Splits that a batch of n_slot x nfb instances of K columns or of half of them (half of
// a uniform sky is up) is cut into, of r.max_splits at most.
MV_RULE int32_t splits_wanted(const SplitRule &r, int n_slot, int nfb, int64_t K) {
    int32_t n = 1;
    for (int64_t k : {K, ceil_div(K, 2)}) {
        OneThread g;
        const Split s = split_of(r, plan_splits(r, n_slot, nfb, [&](int) { return k; }, g), k, 0);
        n = n > s.n ? n : s.n;
    }
    return n;
}

}  // namespace mv

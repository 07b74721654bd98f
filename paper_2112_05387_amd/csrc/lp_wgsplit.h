// How a grouped launch of the wide-layer filter-gradient kernel is cut into workgroups and dealt to the chip: which output
// tiles are cut along the pixels, and which workgroup of the grid does which piece.  Plain functions of integers, for the
// launcher, the kernel and the host's own test alike.
#pragma once
#ifdef __HIPCC__
#define LP_WG_HD __host__ __device__ inline
#else
#define LP_WG_HD inline
#endif

namespace lp {

constexpr int kXcds = 8;

// The hardware deals consecutive workgroups round-robin to the 8 XCDs, each with an L2 of its own, and the workgroups of one
// pixel chunk (its filter rows and channel tiles) read the same pixels.  So an XCD gets consecutive pieces of every problem,
// as many as any other: where a problem does not divide by 8 the next one continues with the XCD behind the last that got one
// more.  (Dealt problem by problem, each from XCD 0 and rounded up, five problems of 51 pieces gave seven XCDs 35 pieces for
// 32 compute units: a second round of the whole launch, 589 us instead of 345.)
// piece(i, local) of workgroup `block` of a grid of `blocks(total)` workgroups; false: the workgroup has none.
// count(i): pieces of problem i.
LP_WG_HD int xcd_grid(int total) { return (total + kXcds - 1) / kXcds * kXcds; }
template <class Count>
LP_WG_HD bool xcd_piece(int block, int nprob, Count count, int& prob, int& local) {
    const int x = block & (kXcds - 1);
    int j = block / kXcds, first = 0;              // first: the XCD that gets the first piece of a problem
    for (int i = 0; i < nprob; ++i) {
        const int n = count(i), base = n / kXcds, rem = n - base * kXcds, xr = (x - first) & (kXcds - 1);
        const int mine = base + (xr < rem ? 1 : 0);
        if (j < mine) { prob = i; local = xr * base + (xr < rem ? xr : rem) + j; return true; }
        j -= mine;
        first = (first + rem) & (kXcds - 1);
    }
    return false;
}

// One problem of the plan: `tiles` output tiles of `kt` units each, every one cut into `ksplit` pieces.
struct SplitPart { int tiles, kt, ksplit; };

// Time of a launch in units of the reduction: `slots` workgroups run at once, and what one does besides its units is worth `add`
// of them where partial sums are added with atomics and `store` where its piece is the whole reduction.
struct SplitCost { int slots, add, store; double round(int chunk, bool whole) const { return chunk + (whole ? store : add); } };
// lp_wgrad_fast.hip: units of 32 pixels (0.9 us each), a workgroup has a compute unit to itself (8192 pixels x 640 channels, five
// layers, one and two rounds of 256 and 128 units: 250 us with stores, 282 with atomics, 337 with atomics and half the length).
// Longer pieces are longer chains of fp32 sums.  Six such layers in one launch add up 8192 pixels in one accumulator, where four
// pieces of 2048 met in atomics before `store` was told apart: their gradients are 0.4 to 1.4e-6 (2-norm) from float64 instead of
// 0.3 to 1.05e-6.  The 160-channel layers' pieces of 7712 pixels, as ever, are at 0.5e-6.
// Both costs are of a launch that has the chip to itself, whatever the number of stream lanes.
constexpr SplitCost kFastCost = {256, 52, 16};
// lp_wgrad_tile.hip: units of 64 pixels (1 us each with two workgroups on a compute unit), 64 KB of atomics a workgroup.  Fitted to tiles of
// 128 rows; those of 64 rows, three to a compute unit, are planned with the same 512 slots.  ResNet-50's 14 x 14 layers of 64 samples are
// 0.3 to 0.4e-6 from float64 with these pieces (0.15e-6 with the shorter ones of the general kernel), its 7 x 7
// ones 0.3 to 0.9e-6 (0.15 to 0.5e-6), its 56 x 56 ones 0.13e-6 (0.23e-6).
// A second level of sums in registers every 1024 pixels takes the former to 0.2e-6; its 64 registers cost ResNet-50's step 0.6 %.
constexpr SplitCost kTileCost = {512, 26, 6};

// Pieces of one length for the whole launch, the length that makes rounds x (piece + epilogue) shortest.  Where whole tiles
// are the pieces and the last round would be nearly empty (288 tiles), the tiles of that round -- the last `rest` of the last
// problem -- are cut finer, so that one more, short round holds them.  Returns rest (0: nothing more to cut), cuts in
// `rest_split`.  Of the lengths that make the same pieces the shortest is the cheapest, so the search goes from one number of pieces to the
// next: it runs on the host ahead of every launch, and 10 problems of 3136 units took it 126 us length by length, now 4.  may_cut: the launch has an entry left for that rest; without one the plan is the best that needs none.
inline int plan_wgrad_pieces(SplitPart* p, int n, int& rest_split, const SplitCost& c = kFastCost, int min_chunk = 16, bool may_cut = true) {
    int max_kt = 1, best_chunk = min_chunk, rest = 0;
    double best = 1e300;
    for (int i = 0; i < n; ++i) max_kt = p[i].kt > max_kt ? p[i].kt : max_kt;
    rest_split = 1;
    const int longest = max_kt > min_chunk ? max_kt : min_chunk;
    for (int chunk = min_chunk, next; chunk <= longest; chunk = next) {
        long blocks = 0;
        bool whole = true;
        next = longest + 1;
        for (int i = 0, ks = 0, more = 0; i < n; ++i) {
            if (i == 0 || p[i].kt != p[i - 1].kt) {
                ks = (p[i].kt + chunk - 1) / chunk;
                more = ks > 1 ? (p[i].kt + ks - 2) / (ks - 1) : next;      // the shortest length with fewer pieces
            }
            blocks += (long)p[i].tiles * ks;
            whole = whole && ks == 1;
            next = more < next ? more : next;
        }
        const double cost = (double)((blocks + c.slots - 1) / c.slots) * c.round(chunk, whole);
        if (cost < best) { best = cost; best_chunk = chunk; rest = 0; }
        const int over = (int)(blocks % c.slots), s = over ? c.slots / over : 1;
        const SplitPart& q = p[n - 1];
        if (!may_cut || !whole || blocks < c.slots || s < 2 || over >= q.tiles || q.kt / s < 8) continue;
        const double two = (double)(blocks / c.slots) * c.round(chunk, true) + c.round((q.kt + s - 1) / s, false);
        if (two < best) { best = two; best_chunk = chunk; rest = over; rest_split = s; }
    }
    for (int i = 0; i < n; ++i) p[i].ksplit = (p[i].kt + best_chunk - 1) / best_chunk;
    return rest;
}

}  // namespace lp

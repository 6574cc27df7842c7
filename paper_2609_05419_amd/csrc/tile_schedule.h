// Tile schedule of the int8 GEMM (K3): which workgroup computes which output
// tile.  Shared by the kernel and the host-compiled test of its invariants;
// nothing here touches memory.
//
// Each XCD has a queue of slots, and within a product the slots follow a
// grouped order of the tiles (groups of 8 tile-rows, column-major inside a
// group), cut into windows of 32 tiles (8 tile-rows x 4 tile-columns): the
// tiles resident on one XCD at a time share their A and B stages in that
// XCD's L2.  All XCDs sweep the batch items (one int8 GEMM each) in the same
// order, so at any time the whole chip works on one product.  Products whose
// planes fit in the 256 MB Infinity Cache give each XCD one contiguous chunk
// of the order.  Larger ones (2 x 256 MB at 16384^2) deal the windows
// round-robin (window w -> XCD w % 8), so that all XCDs work in the same
// group of 8 tile-rows at once and its A strip is read once from HBM and
// shared through the Infinity Cache.  Slots beyond a product's tiles idle.
//
// The XCDs of the part do not run at one clock (up to a tenth apart under
// this load), so a fixed share of tiles per XCD would leave the fast ones idle
// while the slowest finishes.  In long launches the first 7/8 of each XCD's
// slots therefore go to workgroups by index, as dispatched (workgroup b runs
// on XCD b % 8 and takes its slot b / 8), and the last 1/8 form a pool that
// workgroups claim at run time: the next slot of the pool of their own XCD,
// and once that is empty, the next slot of the first other pool that still
// has one.  The launch carries spare workgroups for those extra claims; a
// workgroup that finds every pool empty exits.  Only the pool's workgroups
// wait for an atomic round trip before their first stage copy, and the spares
// cost a few microseconds at the end, so short launches (fewer than 128
// k-stages or 256 slots per XCD, where that cost outweighs the balance) keep
// every slot fixed.  Each pool slot is handed out once (atomic counters,
// which start at zero), and every one is claimed: a workgroup only finds all
// pools empty when all their slots are taken, and the pools have more
// workgroups than slots.
//
// Products of fewer than 8 windows (256 tiles) would give an XCD less than one
// window of each, so with a share of every product on every XCD the 32 tiles
// resident there would come from several products and share few stages
// (2 of 16 tiles of a 1024 x 1024 product: 3 operand strips for 2 tiles).
// Those launches are laid out spread instead (gemm_plan): the tiles of all
// products form one sequence, product-major and in the grouped order, and
// each XCD takes one contiguous eighth of it, so that its resident tiles are
// neighbours of one or two products (16 tiles for 8 strips) and every operand
// strip is fetched by one or two XCDs only.  GEMM phase, N = 16, before ->
// after: 1024^3 55 -> 43 us, 2048^3 249 -> 236, 1024 x 1024 x 65536 1702 -> 1448,
// 500 x 333 x 777 26 -> 21; level at 144 and 256 tiles.  A single tile-row or
// tile-column of the 256 x 256 tile (129 to 256 output rows or columns; fewer
// take a smaller tile, always spread) has no such neighbours: its long operand
// is read once either way.  It stays product-major while it fills the XCDs:
// 8192 x 256 x 1024 86 us against 92 spread, 4096 x 200 x 4096 131 against 136,
// 8192 x 200 x 4096 248 against 255.  Past that k spread is the faster one
// (4096 x 250 x 8192 243 against 228, 2500 x 200 x 30000 785 against 650),
// which the plan does not use.
//
// Nor are launches of short k and few tiles spread (kept_flat): there is hardly
// an operand strip to share, the launch is the writing of its outputs, and that
// is faster with every product's rows and columns spread over the XCDs than
// with whole products on one (GEMM phase flat against spread: 1000 x 1000 x 64
// of 16 products 15.7 and 18.6 us, of 32 18.2 and 20.5, 1000 x 1000 x 256 of 16
// 16.1 and 18.8, 700 x 700 x 192 of 16 12.1 and 14.9, 1600 x 1600 x 64 of 8 14.1
// and 18.6, 600 x 2400 x 64 of 16 16.0 and 17.8; of longer k 1000 x 1000 x 384 of
// 16 18.3 and 18.0, 1000 x 1000 x 256 of 32, two rounds, 27.4 and 24.7; of more
// tiles 3000 x 3000 x 64 of 16 52.4 and 50.0; of panels 1000 x 300 x 256 of 16
// 12.2 and 11.5, 4000 x 100 x 256 of 32 16.8 and 15.9).
#pragma once

#ifndef O2M_HD
#define O2M_HD __host__ __device__
#endif

namespace o2m {

constexpr int kXcds = 8;
constexpr int kGroupRows = 8;     // tile-rows per group of the grouped order
constexpr int kWindowTiles = 32;  // tiles per window (8 tile-rows x 4 tile-columns)
constexpr int kSlotBits = 28;     // a claimed slot travels as x << 28 | slot

constexpr int kSpread = 2;        // `deal` of a launch laid out spread

struct TileCoord {
    int p, ti, tj;
    bool valid;
};

// Slot `slot` of XCD x's queue -> product p, tile (ti, tj), or an idle slot.
// deal 0: contiguous chunks of each product, 1: windows dealt round-robin,
// kSpread: slots x chunk + slot of the sequence of all `batch` products' tiles.
O2M_HD inline TileCoord tile_of(int x, int slot, int mt, int nt, int chunk, int deal, int batch = 0) {
    TileCoord c;
    int t;  // index in the grouped order of the product
    if (deal == kSpread) {
        const int g = x * chunk + slot;
        c.p = g / (mt * nt);
        t = g - c.p * (mt * nt);
        c.valid = c.p < batch;
    } else {
        c.p = slot / chunk;
        const int s = slot - c.p * chunk;  // the slot within the product
        t = deal ? (kXcds * (s / kWindowTiles) + x) * kWindowTiles + s % kWindowTiles : x * chunk + s;
        c.valid = t < mt * nt;
    }
    c.ti = c.tj = 0;
    if (!c.valid) return c;  // idle slot (its group arithmetic would divide by zero)
    const int group = t / (kGroupRows * nt);
    const int first = group * kGroupRows;
    const int gsize = mt - first < kGroupRows ? mt - first : kGroupRows;
    const int within = t - group * kGroupRows * nt;
    c.ti = first + within % gsize;
    c.tj = within / gsize;
    return c;
}

// Launch parameters of one batched int8 GEMM.
struct GemmSchedule {
    int deal;    // 1: windows dealt round-robin to the XCDs, kSpread: spread
    int chunk;   // slots per XCD and product (spread: per XCD)
    long slots;  // slots per XCD over the batch
    long fixed;  // of those, taken by workgroup index; the rest are pooled
    long grid;   // workgroups: kXcds * slots plus the spares (0 when nothing to do)
};

// Splits s.slots into fixed and pooled ones and sets the grid: pooled are the
// last 1/8 of each XCD's slots, plus one spare workgroup per 12 slots, so that
// a faster XCD can take slots of a slower one's pool.
O2M_HD inline void pool_slots(GemmSchedule &s, int kblocks) {
    const bool pool = kblocks >= 128 && s.slots >= 256;
    s.fixed = pool ? s.slots - s.slots / 8 : s.slots;
    s.grid = kXcds * (s.slots + (pool ? (s.slots + 11) / 12 : 0));
}

// mt x nt tiles per product, kblocks k-stages of stage_bytes per operand
// tile, batch products.  grid stays 0 for an empty problem; the caller
// rejects grids beyond the launch limit.
O2M_HD inline GemmSchedule gemm_schedule(int mt, int nt, int kblocks, int batch, long stage_bytes) {
    GemmSchedule s = {0, 0, 0, 0, 0};
    const long tiles = (long)mt * nt;
    if (tiles <= 0 || batch <= 0 || kblocks <= 0) return s;
    // deal windows when each XCD gets at least two and one product's operand
    // planes outgrow the 256 MB Infinity Cache
    const long windows = (tiles + kWindowTiles - 1) / kWindowTiles;
    const long plane_bytes = (long)(mt + nt) * stage_bytes * kblocks;
    s.deal = windows >= 2 * kXcds && plane_bytes > (256L << 20) ? 1 : 0;
    s.chunk = (int)(s.deal ? kWindowTiles * ((windows + kXcds - 1) / kXcds) : (tiles + kXcds - 1) / kXcds);
    s.slots = (long)s.chunk * batch;
    pool_slots(s, kblocks);
    return s;
}

// Tile shapes of the GEMM kernels: output rows and columns of a workgroup, and
// workgroups a CU holds.  The time of a launch is estimated as
//   launch + rounds (tile + stage KB) + latency KB   [us]
// over its KB k-stages, rounds = tiles per CU / workgroups per CU, tiles per
// CU rounded up: `tile` is a tile's prologue and epilogue, `stage` a stage
// with the CU full, `latency` what a stage costs however empty the CU is.  The
// constants fit the GEMM phase of 30 shapes from 60^3 to 4096^3 measured with
// each of the four (to 8-11%, narrow panels apart); the estimate's choice is
// the fastest or within 7% of it on all of them.  It has no term for operand
// traffic, which is what a narrow panel costs: of 4096 x 96 x 4096 it says 104,
// 66, 77 and 113 us for the four tiles, measured 129, 113, 116 and 163, in the
// same order.  A launch long enough to be held by its power draw
// pays for the extra data that the smaller tiles move: their stages cost up to
// 16% more (`sustained`, by the large tile's estimate in units of 600 us; 3492
// x 1543 x 16566 at N = 14: 2033 us with the large tile, 2312 with 256 x 128,
// estimated 2021 and 2017 without this; 1100 x 1100 x 8192: 342 and 310).
// Large products take the 256 x 256 tile, which
// moves the least data per MFMA (2048^3: 230 us against 241, 271 and 447);
// short k, ragged sizes and products of fewer tiles than CUs the smaller ones
// (700^3: 34.0, 27.7, 25.2, 28.5; 96 x 80 x 200: 13.0, 10.6, 8.6, 7.2;
// 4096 x 96 x 4096: 129, 113, 116, 163).
struct GemmShape {
    int tm, tn, per_cu;
    double launch, tile, stage, latency;
};
constexpr int kCus = 256;
constexpr int kGemmShapes = 4;
O2M_HD inline GemmShape gemm_shape_of(int i) {
    constexpr GemmShape shapes[kGemmShapes] = {
        {256, 256, 1, 4.0, 6.2, 0.684, 0.0},
        {256, 128, 2, 6.4, 4.75, 0.749, 0.091},
        {128, 128, 3, 6.35, 3.2, 0.662, 0.133},
        {64, 64, 4, 6.4, 1.83, 0.359, 0.077},
    };
    return shapes[i];
}

O2M_HD inline double gemm_estimate(const GemmShape &s, long rows, long cols, int kblocks, int batch,
                                   double sustained = 0.0) {
    const long tiles = (rows + s.tm - 1) / s.tm * ((cols + s.tn - 1) / s.tn) * batch;
    const double rounds = (double)((tiles + kCus - 1) / kCus) / s.per_cu;
    const double stage = s.stage * (1.0 + 0.16 * (sustained < 1.0 ? sustained : 1.0));
    return s.launch + rounds * (s.tile + stage * kblocks) + s.latency * kblocks;
}

// The launch of one batched int8 GEMM: tile shape, tiles and schedule.
struct GemmPlan {
    int shape, tm, tn;
    int mt, nt;
    int chain;       // 1: each workgroup takes every kResident-th slot of its XCD in turn
    GemmSchedule s;
};

// Chained launches of the 256 x 256 tile: one workgroup per CU takes its tiles
// one after another, the next one's first stages on their way during the last
// stages and the epilogue of the one before (measured, GEMM phase: 2048^3 234
// -> 217 us, 4096 x 4096 x 2048 962 -> 877, 1024^3 44.0 -> 40.2, DSYRK 3001 x
// 4999 305 -> 286).  With long k the prologue is a small part of a tile and the
// workgroups of an XCD, which no dispatch lines up again, drift out of the L2
// reuse of their strips: level to 0.5% slower at 64 stages (ZHERK 4096, 4096^3),
// 1024 x 1024 x 65536 1412 -> 1487.
// The ring of four stages needs five.
constexpr int kResident = 32;    // workgroups per XCD
constexpr int kChainMin = 5, kChainMax = 48;

// One k-stage is the writing of the outputs, which the estimate does not know.
// Long outputs, of up to 16 tile-rows or tile-columns of 128, are written faster
// in 256 x 128 tiles than in 128 x 128 ones: 1000 x 30000 of 32 products 309 us
// against 340, 2000 x 20000 424, 447, 20000 x 2000 368, 415, of 52 products 634,
// 730, 1500 x 20000 317, 321; the others not (5000 x 5000 250, 232, 3000 x 10000 of
// 16 147, 142), nor with two stages (500 x 30000 x 128 199, 195), nor where 256
// rows pad an odd few tile-rows of 128 (300 x 60000 321, 260).
constexpr int kLongTiles = 16;

// Launches that are not spread for their short k: up to two k-stages with at
// most three tiles for each place on the chip, up to four with one, of four
// tile-rows and tile-columns or more, where the XCD with the most tiles takes
// no more rounds for it (36 tiles of 40 products, 128 x 128: 200 tiles on an XCD
// of 96 places against 180, 18.6 us against 17.1 spread); 64 x 64 tiles are
// level or up to 10% faster spread (200 x 200 x 256 of 32 products 8.0 and 8.9).
O2M_HD inline bool kept_flat(const GemmShape &sh, int mt, int nt, int kblocks, int batch) {
    const long rounds = kblocks <= 2 ? 3 : kblocks <= 4 ? 1 : 0, tiles = (long)mt * nt;
    if (sh.tm < 128 || mt < 4 || nt < 4 || tiles * batch > rounds * kCus * sh.per_cu) return false;
    const long places = kCus / kXcds * sh.per_cu;
    const long flat = (tiles + kXcds - 1) / kXcds * batch, even = (tiles * batch + kXcds - 1) / kXcds;
    return (flat + places - 1) / places == (even + places - 1) / places;
}

// rows x cols outputs per product, kblocks k-stages of stage_bytes per
// 256-row operand tile, batch products.  A 256 x 256 launch is spread below 8
// windows per product (a single tile-row or tile-column: below one tile per
// XCD) and follows gemm_schedule otherwise; the smaller tiles, of which an XCD
// holds per_cu windows, are spread below 8 of these and never pooled; kept_flat
// excepts some.
O2M_HD inline GemmPlan gemm_plan(int rows, int cols, int kblocks, int batch, long stage_bytes) {
    GemmPlan p = {0, 0, 0, 0, 0, 0, {0, 0, 0, 0, 0}};
    if (rows <= 0 || cols <= 0 || batch <= 0 || kblocks <= 0) return p;
    const double large = gemm_estimate(gemm_shape_of(0), rows, cols, kblocks, batch);
    double best = large;
    for (int i = 1; i < kGemmShapes; ++i) {
        const double t = gemm_estimate(gemm_shape_of(i), rows, cols, kblocks, batch, large / 600.0);
        if (t < best) {
            best = t;
            p.shape = i;
        }
    }
    if (p.shape == 2 && kblocks == 1) {
        const GemmShape s2 = gemm_shape_of(2);
        const long r = ((long)rows - 1) / s2.tm + 1, c = ((long)cols - 1) / s2.tn + 1;
        if (r * c >= kXcds * kWindowTiles * s2.per_cu && (r < c ? r : c) <= kLongTiles && (r % 2 == 0 || r >= kLongTiles))
            p.shape = 1;
    }
    const GemmShape sh = gemm_shape_of(p.shape);
    p.tm = sh.tm;
    p.tn = sh.tn;
    p.mt = (rows - 1) / sh.tm + 1;
    p.nt = (cols - 1) / sh.tn + 1;
    const long tiles = (long)p.mt * p.nt;
    const bool narrow = p.shape == 0 && (p.mt == 1 || p.nt == 1);
    const bool spread = tiles < (narrow ? kXcds : (long)kXcds * kWindowTiles * sh.per_cu) &&
                        !kept_flat(sh, p.mt, p.nt, kblocks, batch);
    if (!spread && p.shape == 0) {
        p.s = gemm_schedule(p.mt, p.nt, kblocks, batch, stage_bytes);
    } else {
        p.s.deal = spread ? kSpread : 0;
        p.s.chunk = (int)(((spread ? tiles * batch : tiles) + kXcds - 1) / kXcds);
        p.s.slots = spread ? p.s.chunk : (long)p.s.chunk * batch;
        p.s.fixed = p.s.slots;
        p.s.grid = kXcds * p.s.slots;
        if (p.shape == 0) pool_slots(p.s, kblocks);
    }
    if (p.shape == 0 && kblocks >= kChainMin && kblocks <= kChainMax && p.s.slots > kResident) {
        p.chain = 1;   // (never pooled: that takes 128 stages)
        p.s.grid = kXcds * kResident;
    }
    return p;
}

}  // namespace o2m

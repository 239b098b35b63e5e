// Which tile shape a linear layer takes, the order in which linear_kernel goes through its tiles, and what its loads may touch
// (internal; no HIP in here, so that CPU tests compile this very code and follow every load of a call against the ends of its
// buffers).
#pragma once

#include <stdint.h>

#if defined(__HIP__) || defined(__HIPCC__)
#define RAGGED_HD __host__ __device__ __attribute__((always_inline))
#else
#define RAGGED_HD
#endif

namespace ragged {

constexpr int kTK = 64;                          // contraction elements per step: 128-byte LDS rows
constexpr int kLdsBytes = 160 * 1024;
constexpr int kLinearXcds = 8;

// Number of LDS stages: as many as fit, up to eight.
constexpr int linear_stages(int NJ, int MT, int PER_CU) {
    const int fit = kLdsBytes / PER_CU / (32 * (NJ + MT) * kTK * 2);
    return fit < 8 ? fit : 8;
}

// Constants of a tile shape: 32 NJ features x 32 MT tokens, PER_CU work-groups (1 or 2) on a CU.
template <int NJ, int MT, int PER_CU>
struct LinearShape {
    static constexpr int TN = 32 * NJ, TM = 32 * MT;           // features x tokens of a tile
    static constexpr int kStages = linear_stages(NJ, MT, PER_CU);
    static_assert(kStages >= 2, "two stages must fit");
    static constexpr bool kTwo = kStages == 2;
    static constexpr bool kRelax = kStages >= 4;
    static constexpr int kAheadX = kTwo ? 2 : (kRelax ? kStages - 1 : kStages);   // step whose x loads go with half B (two stages: A) of step 0
    static constexpr int kAheadW = kTwo ? 2 : kAheadX - 1;                        // ... w loads with half A (two stages: B)
};

// The tiles of one work-group of a call: t_first, t_first + stride, ... < t_end.
struct LinearWalk {
    int rows, m_tiles, n_tiles, panel;                         // rows: 0 where the device's count is negative; panel: feature tiles of a panel
    uint32_t panel_magic, last_magic;                          // div_magic() of panel and of the last panel's width
    int t_first, t_end, stride;

    RAGGED_HD LinearWalk(int rows_, int TM, int n_tiles_, int panel_, uint32_t panel_magic_, uint32_t last_magic_, int block, int grid)
        : rows(rows_ > 0 ? rows_ : 0), m_tiles((rows + TM - 1) / TM), n_tiles(n_tiles_), panel(panel_), panel_magic(panel_magic_), last_magic(last_magic_) {
        const int total = m_tiles * n_tiles;
        const int xcd = block % kLinearXcds;
        const int per_xcd = (total + kLinearXcds - 1) / kLinearXcds;
        t_end = per_xcd * (xcd + 1) < total ? per_xcd * (xcd + 1) : total;
        stride = grid / kLinearXcds;
        t_first = per_xcd * xcd + block / kLinearXcds;
    }

    // tile number -> first row, first feature.  Panels of `panel` feature tiles, one after the other; inside a panel the
    // feature tiles of a token tile come together.
    RAGGED_HD void tile_of(int t, int TM, int TN, int& m0, int& n0) const {
        int first = 0, width = panel;
        while (t >= m_tiles * width) {                         // a few panels at most
            t -= m_tiles * width;
            first += width;
            width = n_tiles - first < panel ? n_tiles - first : panel;
        }
        // t / width, as divmod() does it
        uint32_t mq = (uint32_t)(((uint64_t)(uint32_t)t * (width == panel ? panel_magic : last_magic)) >> 32);
        uint32_t nr = (uint32_t)t - mq * (uint32_t)width;
        if (nr >= (uint32_t)width) { ++mq; nr -= (uint32_t)width; }
        m0 = (int)mq * TM;
        n0 = (first + (int)nr) * TN;
    }
};

// One operand's place in (tile, step), ahead of the arithmetic: the loads of a step read
//     base + first * K elements + soff + [0, bytes - soff)
// and everything further arrives as zeros.  Past the last tile the range is empty, and there the offset stays 0: the range
// check is offset >= bytes - soff in some descriptions of the hardware and offset >= bytes in others, and with bytes == 0
// the two agree only for soff == 0.
struct LinearCursor {
    int tile;
    int first;                                                 // first row (x) or feature (w) of the tile
    uint32_t bytes, soff, step;                                // step: what soff advances by

    template <int TM, int TN, bool X>
    RAGGED_HD void set(const LinearWalk& walk, uint32_t row_bytes) {
        const bool inside = tile < walk.t_end;
        int m0, n0;
        walk.tile_of(inside ? tile : walk.t_first, TM, TN, m0, n0);
        const int live = X ? (walk.rows - m0 < TM ? walk.rows - m0 : TM) : TN;
        first = X ? m0 : n0;
        bytes = inside ? (uint32_t)live * row_bytes : 0u;
        step = inside ? kTK * 2u : 0u;
        soff = 0;
    }
    // true: the tile is done, the next one has to be set
    template <int TM, int TN, bool X>
    RAGGED_HD bool next(const LinearWalk& walk, uint32_t row_bytes) {
        soff += step;
        if (soff != row_bytes) return false;
        tile += walk.stride;
        set<TM, TN, X>(walk, row_bytes);
        return true;
    }
};

// The tile shapes there are, as {NJ, MT, PER_CU}: 32 NJ features x 32 MT tokens, PER_CU work-groups on a CU.  (Pairs of 192 x 128
// fill the LDS of a CU exactly, with two stages each.)
#define LINEAR_SHAPES(X) \
    X(8, 8, 1) X(8, 7, 1) X(8, 6, 1) X(8, 5, 1) X(8, 4, 1) X(6, 4, 1) X(6, 2, 1) X(4, 4, 1) X(4, 3, 1) X(2, 1, 1) \
    X(6, 4, 2) X(6, 3, 2) X(4, 4, 2) X(4, 2, 2) X(2, 4, 2) X(2, 2, 2)

// Tile shape.  The tiles are handed out evenly, n = ceil(tiles / 256) to a CU.  Where one work-group has a CU to itself they
// follow each other,
//     n * (k-steps * step_ns + tile_ns + GELU),
// where two share it, two at a time run in less than twice that, because the epilogue of one overlaps the products of the other,
//     n / 2 * (k-steps * pair_step_ns + pair_tile_ns + GELU) + n % 2 * (k-steps * step_ns + tile_ns + GELU),
// and the shape with the least of it is taken (rows: the caller's estimate, or the capacity).  Large tiles need the fewest
// operand bytes per product and suit long contractions, small ones fill the chip when rows are few, the heights in between
// are there because a round is paid whole (12 608 x 768 x 3072: 51 us in 237 tiles of 160 rows, 66 in 150 of 256), and two
// groups of up to 192 x 128 suit short contractions and GELU, where the epilogue is a large part: 12 608 x 1536 x 384 with
// GELU takes 30.4 us in 256 x 160, 25.6 in pairs of 128 x 128; 25 216 x 3072 x 768 with GELU 145 in 256 x 256, 125 in pairs of
// 192 x 96, 119 in pairs of 192 x 128, which move a sixth fewer operand bytes through LDS (16 000 rows: 90, 82 and 78);
// 12 608 x 768 x 3072 51 in 256 x 160, 66 in pairs of 128 x 128.
// The constants are a least-squares fit to 32 row counts from 20 to 50 432 at the four layers of 768-, 384- and 192-wide blocks
// (per shape; where it is within 40 % of the fastest; constants then moved by up to 3 % a step, 25 % a tile, towards fewer wrong
// picks); the shape taken is 0.4 % slower than the fastest of all on average, 11 % at most (192-wide layers).  Where the capacity
// stands for the rows and few of them are real, the tiles are too large (2521 rows of 25 216 x 384 x 384 6.8 us; with them as
// the estimate 3.9).
constexpr int kCus = 256;
constexpr int kGeluNs = 118, kPairGeluNs = 102;               // per nj * mt of a tile, of a pair of tiles
struct TileShape { int nj, mt, per_cu, step_ns, tile_ns, pair_step_ns, pair_tile_ns; };
constexpr TileShape kTileShapes[] = {
    {8, 8, 1, 1310, 6020, 0, 0}, {8, 7, 1, 1115, 5130, 0, 0}, {8, 6, 1, 970, 4800, 0, 0}, {8, 5, 1, 845, 4530, 0, 0},
    {8, 4, 1, 725, 3670, 0, 0}, {6, 4, 1, 590, 1900, 0, 0}, {6, 2, 1, 370, 1140, 0, 0}, {4, 4, 1, 410, 1850, 0, 0},
    {4, 3, 1, 365, 1180, 0, 0}, {2, 1, 1, 135, 520, 0, 0},
    {6, 4, 2, 705, 1230, 1040, 4080}, {6, 3, 2, 505, 770, 915, 2600}, {4, 4, 2, 485, 760, 805, 2650}, {4, 2, 2, 260, 500, 525, 1260},
    {2, 4, 2, 250, 650, 535, 1640}, {2, 2, 2, 160, 500, 345, 740}};
// Outputs and residual are reached by 32-bit offsets from a tile's first row, so that a tile's rows together may have up to 2^32
// bytes: 256 rows below 2^23 features, 32 rows below 2^26.  Wider rows have a form of the smallest tile with 64-bit addresses.
inline bool linear_offsets_fit(int mt, int N) { return (int64_t)(32 * mt) * N * 2 < (int64_t)1 << 32; }
inline bool linear_is_wide(int N) { return !linear_offsets_fit(1, N); }
// rows: the caller's estimate, or the capacity
inline TileShape pick_linear_shape(int rows, int N, int K, int act) {
    if (linear_is_wide(N)) return TileShape{2, 1, 1, 0, 0, 0, 0};
    TileShape pick{};                                          // N is a multiple of 64: the 64 x 32 one always fits
    int64_t best = INT64_MAX;
    for (const TileShape& c : kTileShapes) {
        if (N % (32 * c.nj) != 0 || !linear_offsets_fit(c.mt, N)) continue;
        const int64_t tiles = (int64_t)((rows + 32 * c.mt - 1) / (32 * c.mt)) * (N / (32 * c.nj));
        const int64_t n = (tiles + kCus - 1) / kCus, pairs = c.per_cu == 2 ? n / 2 : 0;
        const int ksteps = K / kTK, gelu = act == 1 ? c.nj * c.mt : 0;
        const int64_t cost = (n - 2 * pairs) * (ksteps * c.step_ns + c.tile_ns + kGeluNs * gelu) +
                             pairs * (ksteps * c.pair_step_ns + c.pair_tile_ns + kPairGeluNs * gelu);
        if (cost < best) { best = cost; pick = c; }
    }
    return pick;
}
// Feature tiles per panel: the 32 CUs of an XCD then work on a patch of about 6 x 5 tiles, which pulls fewest operand
// bytes into its L2 (12 544 x 3072 x 768: 78 -> 72.5 us against whole rows of tiles; widths of 4 to 6 are alike).
constexpr int kPanel = 6;
// tile_of() passes the panels one by one, so there are not too many of them (up to 24 576 features this changes nothing; 64 rows x
// 151 936 x 768 62 us without the limit and 42 with it, 3 x 4 194 560 x 64 22 ms and 0.37; 1000 x 128 256 x 768 203 and 211 us).
constexpr int kMaxPanels = 64;
struct LinearGrid {
    int n_tiles, panel, last, groups;                          // last: width of the last panel
    LinearGrid(int nj, int mt, int per_cu, int rows_cap, int N) {
        n_tiles = N / (32 * nj);
        const int wanted = (n_tiles + kPanel - 1) / kPanel, panels = wanted < kMaxPanels ? wanted : kMaxPanels;
        panel = (n_tiles + panels - 1) / panels;
        last = n_tiles - (n_tiles - 1) / panel * panel;
        const int64_t tiles = (int64_t)((rows_cap + 32 * mt - 1) / (32 * mt)) * n_tiles;
        groups = (int)(tiles < kCus * per_cu ? (tiles + kLinearXcds - 1) / kLinearXcds * kLinearXcds : kCus * per_cu);
    }
};

}  // namespace ragged

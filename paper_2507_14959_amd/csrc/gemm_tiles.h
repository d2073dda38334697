// Which tile a bf16 product takes (gemm.hip).  Host arithmetic alone, so that the rule can be held without a GPU.
#pragma once

enum { EPI_STORE = 0, EPI_GELU = 1, EPI_RESID = 2 };

struct TiledProduct {
    int n_in, T, Tb, K, N;    // as in GemmArgs: input blocks (1 where the rows run across blocks), rows of one, block length inside such a run or 0
    int RP, r;                // padded rank and rank of the low-rank terms, RP = 0: none
    int mode;                 // EPI_*
    float fan, terms;         // output blocks and low-rank terms per input block, about
    bool sums;                // the terms are summed on one output block
    bool known;               // n_in (T / Tb) blocks or none at all, else a bound of what the device knows
};

// What a product takes on a tile, in us: rounds of as many workgroups as fit the chip, the last one cheaper the fewer workgroups it has (fewer on a CU,
// fewer pulling at the memory).  Per round f + k K for the loop and, per output block, `store` (+ `gelu` or `resid`) for the epilogue.  Where the epilogue
// cannot fetch ahead, `term` (+ `odd` for ranks that fill no 16-byte load) per low-rank term, 16 ranks and block that a wave's region touches, `look` per
// further block, and `late` for a residual.
// Fitted to 3300 products, every tile measured on each (300 to 56000 rows; widths 192 to 768 and their two- to fourfold, 17 to 512 tokens; ranks 0 to 32,
// one to three branches or summed terms): rms 6 to 10 %.  The tile it picks is on average 0.8 % slower than the fastest, more than 10 % on 46 of the 2740
// that the split contraction is not faster on; the rules before (a model of four tiles without the branches' number, thresholds for ranks that are not
// fetched ahead) 7 %, more than 10 % on every third, with the count known or a mean over counts alike.
// us, 256 x 256 / 256 x 128 / 128 x 128 / 128 x 64 / 64 x 64 (blocks x tokens x K -> N): 121 x 197 x 768 -> 2304, three branches 141 / 153 / 133 / 148 / 281;
// 107 x 101 x 768 -> 768 30 / 28 / 19 / 24 / 37; 233 x 17 x 384 -> 1536, rank 4, two branches 63 / 36 / 27 / 25 / 44; 9 x 170 x 1536 -> 768, rank 32, three
// branches 61 / 34 / 28 / 26 / 20; with a residual, 161 x 50 x 768 -> 768, two summed terms of rank 4 63 / 37 / 43 / 43 / 43, on four waves of 64 x 32 33.
struct TileCost {
    int bm, bn, per_cu, rows;                              // workgroups per CU, rows of a wave's region
    bool ahead, ahead_resid;                               // an epilogue that fetches ahead, also with a residual
    float start, f, k, store, gelu, resid, term, odd, look, late, last1, last2, q;   // last1, last2: share of a round with one / two workgroups per CU in it
};
enum { TILE_128x64, TILE_128x128, TILE_256x128, TILE_256x256, TILE_64x64, TILE_128x64_TALL, TILE_128x128_TALL, N_TILES };   // (TALL: four waves of 64 rows)
inline const TileCost &tile_costs(int tile)
{
    static const TileCost cost[N_TILES] = {
        {128, 64, 3, 32, true, true, 3.38f, 0.607f, 0.0129f, 2.32f, 1.01f, 3.99f, 0.944f, 1.49f, 0.405f, 4.f, 0.544f, 0.752f, 0.131f},
        {128, 128, 2, 32, true, true, 3.79f, 0.643f, 0.0147f, 2.76f, 1.45f, 8.95f, 1.04f, 1.53f, 0.441f, 3.28f, 0.592f, 0.f, 0.21f},
        {256, 128, 1, 64, true, true, 1.92f, 3.27f, 0.0117f, 3.15f, 1.84f, 5.49f, 1.11f, 1.73f, 0.339f, 3.31f, 0.f, 0.f, 0.329f},
        {256, 256, 1, 128, true, true, 2.02f, 3.15f, 0.0231f, 5.51f, 3.84f, 13.f, 1.62f, 2.41f, 0.162f, 3.f, 0.f, 0.f, 0.3f},
        {64, 64, 2, 32, false, false, 3.47f, 1.1f, 0.00542f, 1.43f, 0.444f, 1.55f, 0.547f, 0.499f, 0.719f, 0.f, 0.72f, 0.f, 0.178f},
        {128, 64, 3, 64, false, false, 3.67f, 0.66f, 0.0128f, 3.1f, 1.03f, 4.69f, 0.889f, 0.902f, 0.648f, 0.f, 0.588f, 0.773f, 0.126f},
        {128, 128, 2, 64, true, true, 3.14f, 0.944f, 0.0136f, 3.17f, 1.78f, 5.76f, 1.14f, 1.88f, 0.401f, 3.58f, 0.72f, 0.f, 0.199f}};
    return cost[tile];
}

// Tiles of 256 rows leave a last round in which few CUs have one (22655 rows x 768: 534 of 256 x 128).  Where MAX_TAIL tiles of 128 x 128, one to a CU,
// are enough for the rows past the full rounds, they are cut into those by the same launch: rows that stay in large tiles, all of them where not.
// us without / with: 22064 rows x 768 -> 2304 on 256 x 256 (6 + 768 tiles) 113 / 101, 43734 rows 194 / 184, 22064 rows x 768 -> 768 52.5 / 47.8; with a
// residual on 256 x 128, 11032 rows x 3072 -> 768 and x 768 -> 768 together 120 / 106, 12608 rows 126 / 110.  Twice as many small tiles gain nothing
// (a second round of them, with its start, takes what a round of 256 x 256 with half the CUs does), and 256 x 128 without a residual has a cheap last round
// already (11032 rows x 768 -> 3072 80.5 / 79.3, 12608 rows 84.0 / 86.3).
constexpr int MAX_TAIL = 256;
constexpr bool has_tail(int bm, int bn, int mode, bool ahead) { return bm == 256 && (mode == EPI_RESID ? ahead : bn == 256); }
constexpr long tail_tiles(int rows, int N) { return (long)((rows + 127) / 128) * ((N + 127) / 128); }
constexpr int large_tile_rows(int rows, int N, int bm, int bn)
{
    const int tiles_n = (N + bn - 1) / bn;
    const long tiles = (long)((rows + bm - 1) / bm) * tiles_n;
    if (tiles < 256 || tiles % 256 == 0) return rows;
    const int large = (int)(tiles / 256 * 256 / tiles_n) * bm;
    return tail_tiles(rows - large, N) <= MAX_TAIL ? large : rows;
}

// ---- which workgroup takes which tile
constexpr int panel_tiles(int bn) { return 768 / bn; }     // column tiles per L2 panel (1.2 MB of W at K = 768)

// The j-th of the tiles of one of eight runs: all tiles in the order (panel of `panel` column tiles, row tile, column tile inside the panel) are cut
// into eight equal runs, one per XCD: a run covers one or two W panels and a contiguous range of row tiles, and no XCD has more than one tile more than
// another.  False, and j less the run's tiles, if the run has no such tile: with a tail, j is then its place in the XCD's run of the 128 x 128 tiles.  (Inlined before the optimiser looks at the kernel: later, the kernel of two tiles spills ten times the registers.)
__attribute__((always_inline)) constexpr bool xcd_tile(int xcd, int &j, int tiles_mtot, int tiles_n, int panel, int &mt, int &tn)
{
    const long total = (long)tiles_mtot * tiles_n;
    const long lo = total * xcd / 8, hi = total * (xcd + 1) / 8;
    const long L = lo + j;
    if (L >= hi) { j -= (int)(hi - lo); return false; }
    const long full = (long)tiles_mtot * panel;            // tiles per full panel
    const int pn = (int)(L / full);
    const int rem = (int)(L - pn * full);
    const int n_lo = pn * panel;
    const int width = panel < tiles_n - n_lo ? panel : tiles_n - n_lo;
    mt = rem / width;
    tn = n_lo + rem - mt * width;
    return true;
}

// Workgroups of an XCD in a grid of `tiles` large tiles or, with a tail, of `rows` rows; known: the number of rows is no bound
constexpr long xcd_workgroups(long tiles, bool tail, bool known, int rows, int N, int bm, int bn)
{
    if (!tail) return (tiles + 7) / 8;
    if (!known) return (tiles + 7) / 8 + (MAX_TAIL + 7) / 8;   // (fewer blocks than the bound may have a tail where the bound has none)
    const int large = large_tile_rows(rows, N, bm, bn);
    return ((long)((large + bm - 1) / bm) * ((N + bn - 1) / bn) + 7) / 8 + (tail_tiles(rows - large, N) + 7) / 8;
}

inline long product_tiles(int n_in, int T, int N, int bm, int bn) { return (long)n_in * ((T + bm - 1) / bm) * ((N + bn - 1) / bn); }

inline bool fetches_ahead(const TileCost &c, const TiledProduct &p)
{
    return (p.mode == EPI_RESID ? c.ahead_resid : c.ahead) && (!p.Tb || p.Tb >= c.rows) && !p.sums && (!p.RP || (p.RP == 16 && p.r % 8 == 0));
}

inline float round_cost(const TileCost &c, const TiledProduct &p)
{
    const bool resid = p.mode == EPI_RESID;
    float round = c.f + c.k * p.K + p.fan * (c.store + (p.mode == EPI_GELU ? c.gelu : resid ? c.resid : 0.f));
    if (!fetches_ahead(c, p)) {
        const float more = p.Tb ? (float)(c.rows - 1) / p.Tb : 0.f;    // blocks a region touches beyond the first, on average
        round += (c.term + (p.r % 8 != 0 ? c.odd : 0.f)) * p.terms * (p.RP / 16) * (1.f + more) + p.fan * (c.look * more + (resid ? c.late : 0.f));
    }
    return round;
}

inline float tile_cost(const TileCost &c, const TiledProduct &p, long n)
{
    const float round = round_cost(c, p);
    const long slots = 256L * c.per_cu, rest = n % slots, small = rest * (c.bn / 64);
    float rounds = (float)(n / slots);
    if (has_tail(c.bm, c.bn, p.mode, fetches_ahead(c, p)) && p.Tb && n >= slots && rest && small <= MAX_TAIL) {
        const TileCost &t = tile_costs(TILE_128x128);
        return c.start + round * rounds + 4.f + round_cost(t, p) * (t.last1 - t.q * (1.f - small / 256.f));
    }
    if (rest) {
        const int per_cu = (int)((rest + 255) / 256);
        rounds += (per_cu == c.per_cu ? 1.f : per_cu == 1 ? c.last1 : c.last2) - c.q * (per_cu - rest / 256.f);
    }
    return c.start + round * rounds;
}

// Where the count is known, the cheapest tile at it.  Where the device alone knows how many blocks there are, the smallest mean of a tile's time over
// the fastest's at half to all of the bound, all of it three times: which round ends well at the bound says nothing of fewer blocks (64 frames
// with one to three adapters each have 115 blocks of a bound of 192), and the mean of the times alone misses the bound by a round (5555 rows of
// 3072 -> 768 on 264 tiles of 128 x 128 80 us, 128 x 64 44).
inline int cheapest_tile(const TiledProduct &p)
{
    float worse[N_TILES] = {};
    for (int part = p.known ? 16 : 8; part <= 16; ++part) {
        float us[N_TILES], least = 1e30f;
        for (int i = 0; i < N_TILES; ++i) {
            const TileCost &c = tile_costs(i);
            us[i] = tile_cost(c, p, (product_tiles(p.n_in, p.T, p.N, c.bm, c.bn) * part + 15) / 16);
            least = us[i] < least ? us[i] : least;
        }
        for (int i = 0; i < N_TILES; ++i) worse[i] += us[i] / least * (part == 16 ? 3.f : 1.f);
    }
    int best = 0;
    for (int i = 1; i < N_TILES; ++i)
        if (worse[i] < worse[best]) best = i;
    return best;
}

// Where the input blocks are one row each and have low-rank terms: on tiles whose contraction is split over the waves (gemm_ks.hip) instead of the shared-ring
// kernel, whose epilogue goes through the blocks of a tile one by one, a chain of loads for each.  On many rows the larger tiles win all the same.  us,
// shared ring / split (n blocks, K -> N):
//   rows that fan out (the isolated linear; two terms of rank 64 each): 192 -> 576 300 137 / 107, 2000 181 / 157, 4000 253 / 288; 768 -> 768 1100 206 / 154, 2000 280 / 291; 768 -> 2304
//     300 152 / 126, 700 242 / 248, 4000 780 / 1132; a round of 64 x 64 tiles is the line (384 -> 1152 896 rows, 252 tiles, 167 / 130, 1024, 288 tiles, 163 / 231), two of them up to a
//     contraction of 256, whose tiles leave a CU room for a second one (192 -> 768 1664 172 / 148, 2368, 444 tiles, 223 / 159, 2752, 516, 230 / 251; of rank 20, one each,
//     1664 96 / 93, 2368 132 / 97; two of rank 32 5 % slower
//     to 7 % faster); of rank 16, one each, slower at every count: 768 -> 2304 300 46 / 51, 4000 143 / 453, 768 -> 3072 4000 139 / 588
//   one term a block, the whole call (two layers 768 wide, adapters on all linears of the second): rank 16 128 blocks 197 / 178, 1200 627 / 525, 2400 1037 / 1000,
//     4000 1650 / 1671; rank 64 2400 1548 / 1569, 4000 2378 / 2509, 8000 4547 / 4956; 192 wide 2400 357 / 288, 8000 891 / 850
//   a block's terms summed: 768 wide rank 64 200 569 / 550, 300 647 / 629, 400 787 / 800, 4000 4255 / 5153; rank 16 150 336 / 336, 400 483 / 539; 192 wide 300 271 / 251, 2000
//     488 / 473, 4000 798 / 802
// Where the terms are summed one round of 64 x 64 tiles of a contraction of 768, where a block has one term eight times that.
inline bool one_row_split(long rows, int N, int K, int RP, bool fans_out, bool summed)
{
    const double products = (double)rows * N * K;
    if (fans_out) return RP > 16 && (rows + 63) / 64 * ((N + 63) / 64) <= (K <= 256 ? 512 : 256);
    return products <= (summed ? 1. : 8.) * 256 * 64 * 64 * 768;
}

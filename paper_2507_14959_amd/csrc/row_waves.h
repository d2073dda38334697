// Which kernel takes the row-wise part of a layer 192 wide: tiles of 64 rows (rowlayer.hip) or 32 rows in the registers of each of four or eight waves
// (rowreg.hip).  Host arithmetic alone, so that the rule can be held without a GPU.
#pragma once

#include <initializer_list>

constexpr int RR_D = 192;           // model width
constexpr int RR_MAX_DM = 768;

// (frame, adapter) pairs that only the device knows: between one a frame and the bound, and the choice may fall on one each however much room there is: the row
// kernels for many rows are taken only where they are no slower there either.  us per call, 64 rows a tile / many rows, a bound of four a frame, the last two
// layers of twelve adapted, one / two / three adapters on every frame: 34 frames 461 / 492, 515 / 497, 531 / 513, 64 frames 495 / 512, 561 / 531,
// 622 / 631; a bound of five, every layer, 32 frames: 472 / 672, 553 / 696, 877 / 786.
// Room for up to three a frame is mostly half used: a tenth slower at one each is taken (100 frames, a bound of three, 1.8 each, every layer: 1288 / 1050;
// the 128-row tiles, no slower at one each, 1398.  One each, a bound of three: 80 frames 810 / 712, 90 880 / 945, 100 898 / 951, 120 994 / 797).
struct PairCount {
    int usual, least;
    float slack;
};
inline PairCount pair_count(int F, int R) { return {(F + R) / 2, F, R > 3 * F ? 1.f : 1.1f}; }
inline PairCount known_count(int blocks) { return {blocks, blocks, 1.f}; }

// Full rounds of 256-row tiles and the rows past them on tiles of 128, in a launch of their own (a lone tile of 128 rows has a wave per SIMD and takes 36 us, one of 256 rows, or a
// third round of 128, as long or longer).  Only where the count is what the host knows, or at most that.  Twelve layers of DeiT-tiny, ten of them shared, us, before / now: 333 frames of 197
// tokens 1737 / 1640, 400 1853 / 1721, 498 (one and a half rounds) 1992 / 1854, 700 2981 / 2890; of 113 tokens 581 1708 / 1614, 860 1956 / 1814; of 50 1700 1916 / 1775.
constexpr int ROWREG_BOTH = 12;
inline long rowreg_full(long rows) { return rows / 65536 * 65536; }

// us of the row-wise part of a layer of DeiT-tiny on n workgroups, a CU each at a time: a round takes `c`, and up to `d` more the more CUs are at work (they share the
// memory and the power).  waves 0: tiles of 64 rows; 4, 8: of 128 / 256 rows (rowreg.hip).  Twelve layers and everything else of a forward: 12214 rows 486 / 610 /
// 772 us, 18912 817 / 678 / 839, 32702 941 / 808 / 941, 37430 1255 / 1247 / 1039, 57130 1656 / 1424 / 1212, 65601 (a row in a round of its own) 1956 / 1875 /
// 1834, but see above; with adapters 14184 rows (288 tiles that end with their block) 809 / 714 / 891, 28368 1257 / 897 / 1047, 42552 1665 / 1482 / 1171.
inline float row_layer_us(int waves, int T, int r, bool by_block, int blocks)
{
    auto rounds = [](long n, float c, float d) { return (float)(n / 256) * (c + d) + (n % 256 ? c + d * (float)(n % 256) / 256.f : 0.f); };
    const long rows = (long)blocks * T;
    if (waves == 0) return rounds(by_block ? (long)blocks * ((T + 63) / 64) : (rows + 63) / 64, r ? 31.f : 27.5f, 0.f);
    const float few = r ? 46.f : 36.f;
    if (waves == ROWREG_BOTH) return rounds(rowreg_full(rows) / 256, r ? 58.f : 48.f, 30.f) + rounds((rows - rowreg_full(rows) + 127) / 128, few, 8.f) + 2.f;
    return waves == 4 ? rounds((rows + 127) / 128, few, 8.f) : rounds((rows + 255) / 256, r ? 58.f : 48.f, 30.f);
}

// Waves per workgroup of rowreg.hip (or ROWREG_BOTH) where `n.usual` blocks of T rows are that many that it is faster, and on `n.least` blocks, where there may be as few, no slower
// than `n.slack` times; 0 where they are not or it does not apply.  r: rank of the adapters in the launch, 0 without; by_block: adapters or a map.
inline int rowreg_waves(int T, int D, int Dm, int r, bool by_block, const PairCount &n)
{
    if (D != RR_D || Dm < 128 || Dm % 64 || Dm > RR_MAX_DM || (r && r != 8 && r != 16) || (by_block && T < 32)) return 0;
    auto us = [&](int waves, int blocks) { return row_layer_us(waves, T, r, by_block, blocks); };
    int best = 0;
    for (int waves : {4, 8, ROWREG_BOTH}) {
        if (waves == ROWREG_BOTH && (n.usual != n.least || (long)n.usual * T <= 65536 || (long)n.usual * T % 65536 == 0)) continue;
        if (us(waves, n.usual) < us(best, n.usual) && us(waves, n.least) <= us(0, n.least) * n.slack) best = waves;
    }
    return best;
}

// Rows of a tile where layers 192 wide run as tiles that stay on their CUs (rowrun.hip), 64 or 32; 0 where two launches a layer are faster.  The tiles take a round of 256
// at a time through all layers, the row-wise part and attention together: 64 rows 26.5 us a layer, 32 rows, which pull the same weights, 20.5 (197 tokens; shorter blocks
// have less attention).  Two launches a layer: the row-wise part as above and attention, 4.5 us and what its rows take.  Twelve layers of DeiT-tiny and everything
// else of a forward, us, two launches a layer / tiles of 64 / of 32 rows: every layer adapted, 16 blocks of 197 tokens (64 and 112 tiles) 440 / 338 / 270, 36 (252 of 32) 461 /
// 346 / 276, 40 463 / 340 / 528, 64 (256 of 64) 484 / 347 / 535, 72 685 / 635 / 787, 96 753 / 647, 128 781 / 699, 160 (640 of 64) 820 / 1015; ten layers shared, 64 frames
// 507 / 402, 72 506 / 647, 84 615 / 630, 87 651 / 632, 102 661 / 638; 113 tokens, a bound of three a frame, 1.8 each: 24 frames 424 / 331 / 250, 64 487 / 339 / 495, 96 784 / 646, 160 968 / 971; 17 tokens: 128 375 / 305 / 243, 256
// 397 / 308 / 245.
constexpr int RN_MAX_TILES = 512;   // of the usual count: two rounds
// Four where the other way is tiles of 64 rows too (a bound far above the frames, of which one each may have an adapter; ranks and blocks that rowreg.hip does not take): it takes as
// many rounds of 27.5 to 31 us.  64 frames of 197 tokens, a bound of four each, 2.5 there: every layer adapted 1131 / 952 us, two of twelve 431 / 411, in the lagged loop one / two / three
// each 363 / 345, 408 / 401, 450 / 448; 120 of 113 1116 / 950; 17 tokens: 333, a bound of four, 983 / 727, 520, one each, 944 / 725.
constexpr int RN_MOST_TILES = 1024;
// Rounds that `blocks` of so many tiles take: the tiles of a block run side by side, so of each queue's 32 CUs (rowrun.hip) a round fills what is a multiple of them, unless
// all there is fits at once (36 blocks of seven tiles 295 us, 64 547, 72 808)
inline int rowrun_rounds(int blocks, int tiles)
{
    const int at_once = 8 * (32 / tiles);
    return (long)blocks * tiles <= 256 ? 1 : (blocks + at_once - 1) / at_once;
}
// Where a block has the sum of several adapters' terms (tiles of 32 rows alone), the other way is the small tasks up to 270 tiles of 32 rows and two launches for each linear
// beyond: up to four rounds.  Twelve layers, up to three terms on a block, us, the other way / tiles: 8 blocks of 197 tokens 330 / 317, 24 541 / 314, 36 739 / 318, 64 1022 / 573, 128 (four
// rounds) 1538 / 1114; 64 of 113 712 / 303; 256 of 17 713 / 295.  (333 of 197: eleven rounds would be 2970, the other way 2895.)
constexpr int RN_SUM_ROUNDS = 4;

inline float rowrun_us(int rows, int T, int blocks, int most = RN_MAX_TILES)
{
    const int tiles = (T + rows - 1) / rows;
    return (long)blocks * tiles > most ? 1e9f : (rows == 64 ? 24.5f + (float)T / 100.f : 18.f + (float)T / 80.f) * (float)rowrun_rounds(blocks, tiles);
}
inline float two_launches_us(int T, int D, int Dm, int r, bool by_block, const PairCount &n)
{
    const float second = T > 192 && n.usual == n.least && n.usual * (D / 64) > 256 ? 3.f : 0.f;      // (of attention, where CUs have a second workgroup)
    return row_layer_us(rowreg_waves(T, D, Dm, r, by_block, n), T, r, by_block, n.usual) + 4.5f + (float)n.usual * T / 2700.f + second;
}
inline int rowrun_rows(int T, int D, int Dm, int r, bool by_block, const PairCount &n)
{
    const int most = rowreg_waves(T, D, Dm, r, by_block, n) ? RN_MAX_TILES : RN_MOST_TILES;
    const int rows = rowrun_us(32, T, n.usual, most) < rowrun_us(64, T, n.usual, most) ? 32 : 64;
    return rowrun_us(rows, T, n.usual, most) < two_launches_us(T, D, Dm, r, by_block, n) ? rows : 0;
}

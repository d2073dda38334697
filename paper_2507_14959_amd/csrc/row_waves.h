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

// us of the row-wise part of a layer of DeiT-tiny on n workgroups, a CU each at a time: a round takes `c`, and up to `d` more the more CUs are at work (they share the
// memory and the power).  waves 0: tiles of 64 rows; 4, 8: of 128 / 256 rows (rowreg.hip).  Twelve layers and everything else of a forward: 12214 rows 486 / 610 /
// 772 us, 18912 817 / 678 / 839, 32702 941 / 808 / 941, 37430 1255 / 1247 / 1039, 57130 1656 / 1424 / 1212, 65601 (a row in a round of its own) 1956 / 1875 /
// 1834; with adapters 14184 rows (288 tiles that end with their block) 809 / 714 / 891, 28368 1257 / 897 / 1047, 42552 1665 / 1482 / 1171.
inline float row_layer_us(int waves, int T, int r, bool by_block, int blocks)
{
    auto rounds = [](long n, float c, float d) { return (float)(n / 256) * (c + d) + (n % 256 ? c + d * (float)(n % 256) / 256.f : 0.f); };
    const long rows = (long)blocks * T;
    if (waves == 0) return rounds(by_block ? (long)blocks * ((T + 63) / 64) : (rows + 63) / 64, r ? 31.f : 27.5f, 0.f);
    return waves == 4 ? rounds((rows + 127) / 128, r ? 46.f : 36.f, 8.f) : rounds((rows + 255) / 256, r ? 58.f : 48.f, 30.f);
}

// Waves per workgroup of rowreg.hip where `n.usual` blocks of T rows are that many that it is faster, and on `n.least` blocks, where there may be as few, no slower
// than `n.slack` times; 0 where they are not or it does not apply.  r: rank of the adapters in the launch, 0 without; by_block: adapters or a map.
inline int rowreg_waves(int T, int D, int Dm, int r, bool by_block, const PairCount &n)
{
    if (D != RR_D || Dm < 128 || Dm % 64 || Dm > RR_MAX_DM || (r && r != 8 && r != 16) || (by_block && T < 32)) return 0;
    auto us = [&](int waves, int blocks) { return row_layer_us(waves, T, r, by_block, blocks); };
    int best = 0;
    for (int waves : {4, 8})
        if (us(waves, n.usual) < us(best, n.usual) && us(waves, n.least) <= us(0, n.least) * n.slack) best = waves;
    return best;
}

// Whether layers 192 wide run as tiles that stay on their CUs (rowrun.hip), which take a round of 256 at a time through all layers, 26.5 us each with attention
// in it, rather than in two launches a layer: the row-wise part as above and attention, 4.5 us and what its rows take.  Twelve layers of DeiT-tiny and everything
// else of a forward, us, two launches a layer / tiles: every layer adapted, 16 blocks of 197 tokens (64 tiles) 440 / 335, 64 (256) 484 / 347, 72 (288) 685 / 635, 96 (384)
// 753 / 647, 128 (512) 781 / 699, 160 (640) 820 / 1015; ten layers shared, 64 frames 507 / 402, 72 506 / 647; 113 tokens, a bound of three a frame, 1.8 each: 64
// frames 487 / 339, 96 784 / 646, 128 819 / 672, 160 968 / 971; 17 tokens: 128 375 / 307, 256 397 / 313.
constexpr int RN_MAX_TILES = 512;   // of the usual count: two rounds
inline bool rowrun_faster(int T, int D, int Dm, int r, bool by_block, const PairCount &n)
{
    const long tiles = (long)n.usual * ((T + 63) / 64);
    if (tiles > RN_MAX_TILES) return false;
    const float attention = 4.5f + (float)n.usual * T / 2700.f;
    return 26.5f * (float)((tiles + 255) / 256) < row_layer_us(rowreg_waves(T, D, Dm, r, by_block, n), T, r, by_block, n.usual) + attention;
}

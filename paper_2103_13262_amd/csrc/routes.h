// Which kernels a bf16 product runs in (internal; compiled for the host as well).  The host decides from sizes alone, since it does not know
// the experts' row counts; a "round" below is one 256 x 256 tile for each of 256 workgroups.
// Product: anything with the fields M (rows), E (experts), K (reduction), Nout (columns), stream_out, accumulate, out_f32 and wide_gather of
// GemmArgs.
#pragma once
#include <algorithm>
#include <cmath>

namespace moe {

// Whether a lane's place in a block of an operand fits 32 bits (setup_offsets): a block spans at most kMaxTileRows rows of the operand, so
// it does for all but rows of millions of values (512 rows of 2^22 values are 4 GB).  Gathered rows lie anywhere in X.
constexpr int kMaxTileRows = 512;
template <class Product> constexpr bool offsets_fit(const Product& a) { return a.K < (1 << 22) && a.Nout < (1 << 22) && !a.wide_gather; }

// Many small experts: the rows kinds that are not in the small tiles run in 64 x 256 tiles, otherwise in two size classes (GemmArgs::cls).
template <class Product> constexpr bool few_rows(const Product& a) { return a.M < 96L * a.E; }

// Columns of 256, and about how many 256 x 256 tiles the rows make.
template <class Product> constexpr long wide_columns(const Product& a) { return (a.Nout + 255) / 256; }
template <class Product> constexpr long wide_tiles(const Product& a) { return (a.M / 256 + a.E / 2) * wide_columns(a); }

constexpr int kMinSplitDepth = 16 * 64;         // a stream-K piece is at least this deep (16 blocks of 64): handing a partial sum on costs
                                                // about as much time as 6 such blocks, and the hand-overs of one tile form a chain
// Reductions that are never cut into pieces: few last pieces in 128 x 128 tiles with 128-deep blocks (ggemm_classes).
template <class Product> constexpr bool shallow(const Product& a) { return a.K < 2 * kMinSplitDepth; }

constexpr int kTileCols = 128;                  // columns of a small tile

// At most so many small tiles of BM rows.
template <class Product> constexpr long most_tiles(const Product& a, int BM)
{
    const long touched = std::min<long>(a.E, a.M);
    return (a.M + touched * (BM - 1)) / BM * ((a.Nout + kTileCols - 1) / kTileCols);
}

// One or two experts whose rows, at their mean, are whole blocks of 256 (or nearly: a last piece above 128 rows counts as a block): the big tiles have
// no last pieces behind them then.
template <class Product> constexpr bool whole_blocks(const Product& a)
{
    const long last = a.M / a.E % 256;
    return a.E <= 2 && (last == 0 || last > 128);
}
// A fraction of the columns that 256-wide tiles compute is not there: a sixth, or nearly a quarter.
template <class Product> constexpr bool sixth_missing(const Product& a) { return wide_columns(a) * 256 * 5 >= (long)a.Nout * 6; }
template <class Product> constexpr bool quarter_missing(const Product& a) { return wide_columns(a) * 256 * 10 >= (long)a.Nout * 13; }

// Whether a forward product is better off in the small tiles (ggemm_bf16_tile.h) than in the persistent kernels'.  The lines come from both
// sides' times of FC1 and FC2 of 130 drawn layers (1 to 32000 tokens, 2 to 254 experts, d 256 to 2048, h 512 to 8192, launch included) and, above
// 96 rows per expert, of 630 more (96 to 32000 tokens, 1 to 256 experts, d 256 to 4096):
//   * up to 96 rows per expert: 1.1 to 2 times as fast (64 rows, 256 experts, d 512, h 1024: FC1 96 -> 83, FC2 74 -> 68 us; 64 experts,
//     d 1024, h 2048: 80 -> 66 and 72 -> 55; 8 tokens, 16 experts, d 1024, h 4096: 25 -> 23 and 33 -> 24; 7 tokens: 26 -> 13);
//   * more rows, but less than half a round of 256 x 256 tiles, or less than a whole one with a shallow reduction, where the big
//     tiles leave compute units idle and the last pieces' phase is as long as the tiles' (250 rows, 8 experts, d 768, h 3072: 55 -> 33
//     and 59 -> 42 us; beyond: 1024 rows, 4 experts, K 1024, 4096 columns: 72 -> 82);
//   * widths that fill 256-wide tiles badly, up to three rounds of them: a sixth of the columns not there up to K 3000 (290 rows, 222 experts, K
//     1088, 384 columns: 125 -> 107 us; 1498 rows, 9 experts, K 5056, 800 columns: 151 -> 187), nearly a quarter up to 6000 (476 rows, 64
//     experts, K 4512, 288 columns: 223 -> 192; 1630 rows, 18 experts, K 7584, 352 columns: 214 -> 348).
// Not so: reductions of 5000 and more with more than 250 small tiles, whose weights all row tiles read again (226 rows, 6 experts, K 7712, 3712 columns:
// 127 -> 175 us), but for one expert with a last piece (5223 rows, K 7104, 896 columns: 163 -> 123); and one or two experts of whole blocks, where
// the big tiles are at their best, from one round of small tiles on (512: 8192 rows, K 512, 2048 columns: 38 -> 48; K 4096, 1024 columns: 81 -> 93;
// 2 experts, 1705 rows, K 896, 3488 columns: 35 -> 44).
// Of those 630 layers' products 12 are slower by 5 to 21 % than in the kernels before the small tiles (without the last two rules 51, by up to
// 67 %), and all of them take 0.76 of the time.
template <class Product> constexpr bool tile_pays(const Product& a)
{
    if (few_rows(a)) return true;
    const long big = wide_tiles(a), small = most_tiles(a, 128);
    if (whole_blocks(a) && !sixth_missing(a) && (small > 512 || (small >= 400 && a.K >= 4096))) return false;
    const bool one_last_piece = a.E == 1 && !whole_blocks(a);
    if (big <= 128 && (a.K < 5000 || small <= 250 || one_last_piece)) return true;
    if ((big <= 192 && a.K <= 1536) || (big <= 256 && a.K <= 512)) return true;
    return big <= 768 && ((sixth_missing(a) && a.K <= 3000 && a.M < 6000L * a.E) || (quarter_missing(a) && a.K <= 6000));
}

// Backward products: whether a rows kind in small tiles, with the weight gradient in a launch of its own, beats
// the launch that holds both.  The shared launch keeps all compute units busy to its end and hides the fp32 gradients' reads; the
// small tiles read every expert's weights once where 64-row tiles read them twice, do not compute columns that do not exist, and
// have a deep reduction done by many workgroups instead of few.  Both sides' times of 26 drawn layers and, for the last line, of 630 more:
//   * 56 to 96 rows per expert, K above 1024: 61 rows, 111 experts, d 1408, h 2144: 372 -> 330 (dZ with dW2) and 441 -> 345 us (dXs with
//     dW1); 64 rows, 64 experts, d 1024, h 2048: 157 -> 139; K 1024, 256 experts, d 512: 137 -> 140.  Accumulating in fp32: 198 -> 213.
//   * widths that fill 256-wide tiles badly: 34 rows, 97 experts, 544 columns: 81 -> 67; 16 rows, 65 experts, 800 columns: 115 -> 92.
//   * a quarter of a round of big tiles with a deep reduction: 250 rows, 8 experts, d 768, h 3072: 105 -> 95; 90 rows, 7 experts, d 320,
//     h 2432: 39 -> 29; a whole round and more: 174 -> 239 (512 rows, 16 experts, d 1024, h 4096); 2500 rows per expert and more, or half a round
//     of small tiles and K below 4096: 88 -> 135 (4096 rows, one expert, K 4096, 1024 columns), 60 -> 86 (2 experts, 2048 rows, K 2048, 1024 columns).
template <class Product> constexpr bool tile_beats_pair(const Product& a)
{
    if (a.M <= 0) return false;
    if (!few_rows(a)) return wide_tiles(a) <= 64 && a.K >= 2048 && a.M < 2500L * a.E && (most_tiles(a, 128) < 256 || a.K >= 4096);
    if (wide_tiles(a) <= 64 && a.K >= 2048) return true;
    if (!a.stream_out || (a.accumulate && a.out_f32)) return false;   // (up to 48 MB of weights a launch more costs what it saves)
    return (a.M > 56L * a.E && a.K > 1024) || wide_columns(a) * 256 * 4 >= (long)a.Nout * 5;
}

// Backward products: whether a rows kind and a weight gradient share a launch.  With few tiles per workgroup the ragged end of a rows-kind launch
// (a quarter to half a tile per workgroup) and the launch gap are worth more than the counter's round trips; measured, the pair wins up to
// about 8 tiles per workgroup (4096 tokens, 16 experts, d 1024, h 4096: -3 % per step, 8192 tokens, 64 experts: -1.4 %) and loses 0.5 % at
// 34 (32768 tokens, 32 experts, d 2048, h 8192).  (64-bit offsets: no pairs, whose tiles are never cut; a reduction over 2^22 and more has to be,
// and that many columns are more than 8 tiles per workgroup.)
template <class Product> constexpr bool pair_pays(const Product& rows, int workgroups)
{
    return offsets_fit(rows) && !tile_beats_pair(rows) && wide_tiles(rows) <= 8L * workgroups;
}

// A weight gradient that follows a rows product in one launch: whether its tiles are so few that half as high ones still make a single round, over
// reductions long enough to matter.  Both sides' times of the launch, 153 drawn products with at most 256 of the smaller tiles: 0.67 to 1.0 with 1024 rows
// per expert and more and up to 224 of them, with a few up to 1.13 (0.84 on average; one expert, 9768 rows, K 1408, 384 columns: 178 -> 119 us; 10 experts,
// 3079 rows, K 448, 960 columns: 118 -> 102); 0.93 to 1.06 with fewer rows; 0.89 to 1.18 with more tiles.  Of 237 more inside the line (rows not cut, see
// below) 22 are slower by over 2 %, by up to 22 % (1429 rows, one expert, K 5088, 800 columns: 50 -> 62; the whole step 0.99), 0.84 on average: mostly even loads
// where the larger tiles just fit the workgroups that the rows product's last round leaves free and the smaller do not.  Skewed loads of such sizes take 0.66 to
// 0.75, and the host does not know which it has.
template <class Product> constexpr bool half_round(const Product& a)
{
    return a.M >= 1024L * a.E && a.E * wide_columns(a) * ((a.K + 127) / 128) <= 224;
}

// Into how many ranges those tiles' rows are cut (at most eight, and one range for each of 256 workgroups), from an estimate of the launch in
// microseconds, by the experts' mean rows: the rows product's tiles (1.7 a block of 64, and 12) leave `free` workgroups of their last round to start on
// the ranges at once (0.37 a block of 32 rows, and 8), the others come when it ends; a tile's last workgroup adds its ranges' sums up (3 each, and 6).  Cut
// only where that is 5 % better.  Against no cuts, 65 drawn launches (1100 to 12600 rows per expert, 18 to 128 tiles) cut once into as many ranges as a
// rule without the rows product gave: the 26 where this estimate is better took 0.44 to 0.98 of the time (one expert, 9768 rows, K 384, 1408 columns: 122
// -> 54 us; 5948 rows, 3 experts: 110 -> 75), the others 0.82 to 1.25.  With the ranges that it gives now the 88 launches of that sweep take 0.92 of the
// time on average, the slowest of them 1.05.  Skewed loads, where the largest expert gets fewer ranges than its rows would want (51 layers of 2 to 12
// experts, up to nearly all rows in one), against 256 x 256 tiles without ranges: 0.25 to 1.01.
template <class Product> inline int half_round_slices(const Product& rows, const Product& cols)
{
    const long tiles = cols.E * wide_columns(cols) * ((cols.K + 127) / 128), big = wide_tiles(rows), rounds = std::max(1L, (big + 255) / 256);
    const long free = 256 * rounds - big;
    const double blocks = cols.M / cols.E / 32.0, round = rows.K / 64 * 1.7 + 12, begin = (rounds - 1) * round, end = rounds * round;
    auto estimate = [&](int s) {
        const double each = blocks * 0.37 / s + 8;
        auto done = [&](double t) {        // ranges that are through by then
            return (t > begin ? free * (long)((t - begin) / each + 1e-9) : 0) + (t > end ? (256 - free) * (long)((t - end) / each + 1e-9) : 0);
        };
        double best = end + 256 * each;    // (one workgroup a range: always enough)
        for (int n = 1; n <= 32; ++n) {
            if (done(begin + n * each) >= tiles * s) best = std::min(best, begin + n * each);
            if (done(end + n * each) >= tiles * s) best = std::min(best, end + n * each);
        }
        return std::max(best, end) + (s > 1 ? 6 + 3 * s : 0);
    };
    int slices = 1;
    double least = 0.95 * estimate(1);
    for (int s = 2; s <= 8 && tiles * s <= 256; ++s) {
        const double t = estimate(s);
        if (t < least) { least = t; slices = s; }
    }
    return slices;
}

// A weight gradient in a launch of its own: whether tiles of 128 x 256 beat those of 256 x 256.  A tile's time is mostly that of its gradient's way to
// memory, so what counts is how much of the last round of tiles (256 at a time) is empty; but a tile half as high reads nearly as much.
// Both sides' times (1 to 200 experts, 2 to 2900 rows each, K 256 to 5700, 500 to 6100 columns), rounds of either in brackets:
//   * a single round of the smaller ones: 0.68 to 0.88 of the time (88 and 132 tiles, added up in fp32: 66 -> 45 us; 105 and 189: 17 -> 14);
//   * as many rounds of either, up to 1000 rows per expert: 91 products, 0.90 on average, 0.69 to 1.09; three with more rows 0.77 to 1.20;
//   * a third more rounds of the smaller ones (3 and 4), up to 500 rows, an expert's tiles a multiple of eight, so that every XCD gets as many: 11
//     products, 0.91, 0.84 to 1.0; 85 others 0.96, up to 1.11 (16 experts, K 544, 2752 columns: 24 -> 26); added up in fp32 whatever the tiles: 10, 0.86;
//   * half as many more (2 and 3, 4 and 6) where fp32 gradients are added to, which is read as well, up to 500 rows: 49, 0.94, 0.84 to 1.04; with more
//     rows 54, 1.0, up to 1.2 (822 rows, 5 experts, K 672, 5024 columns: 65 -> 77).
// Beyond: 0.97 to 1.26.
template <class Product> constexpr bool half_tiles_pay(const Product& a)
{
    const long columns = a.E * wide_columns(a), high = (a.K + 127) / 128, whole = (columns * ((a.K + 255) / 256) + 255) / 256, half = (columns * high + 255) / 256;
    if (half <= 1) return true;
    if (half == whole) return a.M < 1000L * a.E;
    if (a.M >= 500L * a.E) return false;
    if (a.accumulate && a.out_f32) return half * 2 <= whole * 3;
    return half * 3 <= whole * 4 && wide_columns(a) * high % 8 == 0;
}

// 64-bit offsets, 96 rows per expert and more: whether the two size classes beat 64 x 256 tiles.  Millions of columns: always (one expert, 100 to
// 3000 rows, 32 to 512 deep: 0.57 to 0.87 of the time).  A reduction over millions with few big tiles: no, since a tile is cut among the workgroups of one XCD only and
// 64-row tiles are more (300 rows, 128 columns: FC2 1.8 ms against 14, dXs 2.4 against 13; 1000 rows, 256 columns, 3 tiles: 4.4 against 7.2 and
// 6.8 against 7.2; 512 columns, 6 tiles: 8.7 against 7.1 and 12.5 against 7.4; 3000 rows, 256 columns: 13.2 against 13.9 and 20.7 against 13.7).
template <class Product> constexpr bool wide_classes_pay(const Product& a) { return a.Nout >= (1 << 22) || wide_tiles(a) >= 6; }

// The kernel of a product that has a launch of its own, and of the first one of a pair (kTiles64 or kClasses).
enum class Route { kSmallTiles, kTiles64, kClasses, kWideTiles64, kWideClasses };
template <class Product> constexpr Route route(const Product& a, bool forward)
{
    if (!offsets_fit(a)) return few_rows(a) || !wide_classes_pay(a) ? Route::kWideTiles64 : Route::kWideClasses;
    if (forward ? tile_pays(a) : tile_beats_pair(a)) return Route::kSmallTiles;
    return few_rows(a) ? Route::kTiles64 : Route::kClasses;      // (forward products never run in 64 x 256 tiles: tile_pays)
}

// Whether a forward product's small tiles request weights that one tile alone reads as streaming loads, which leave nothing of them in the
// memory-side cache (256 MB).  Streaming is the faster way to read them (8 tokens, 16 experts, d 1024, h 4096: 53.8 us a pass, ordinary loads 58.9), but
// what it leaves out is missing where it is read again soon: the second layer's weights first of all, with which the backward pass begins.  Few
// enough to stay there beside those of other layers or steps, they come as ordinary loads.  Over 130 drawn layers below 96 rows per expert, three of
// them in turn, against both streaming (us):
//   * up to 40 MB touched per layer neither streams: a forward pass 0.90 to 1.0, a training step 0.86 to 1.04 (6 tokens, 13 experts, d 1600, h 1472,
//     22 MB: 115 -> 99); one layer by itself: dXs with dW1 69 -> 49 (4 tokens, 31 experts, d 1248, h 2944, 27 MB);
//   * up to 80 MB the first alone: 0.91 to 1.0 and 0.93 to 1.02 (32 tokens, 3 experts, d 1536, h 6208, 55 MB: 54 -> 51 and 143 -> 136);
//   * beyond, the first alone makes a forward pass 1.0 to 1.11 times as long for a step of 0.94 to 1.04 (1024 tokens, 64 experts, d 1024, h 2048, 256
//     MB: 142 -> 158 and 380 -> 395; 412 tokens, 32 experts, d 1312, h 1696, 136 MB: 78 -> 83 and 246 -> 236): both stream.
// touched: bytes of one layer's experts that the tokens reach, if they choose evenly.
inline double touched_weights(long tokens, int k, int E, double bytes) { return bytes * (1.0 - std::pow(1.0 - (double)k / E, (double)tokens)); }
constexpr bool stream_weights(bool second_layer, double touched) { return touched > (second_layer ? 80.0 : 40.0) * (1 << 20); }

// The small tile's height: an expert's rows in one tile, or its weights are read once more for each (with a mean of 56 rows a tile of 64 still
// holds most experts'); 32 rows only for a handful, where more workgroups fit a compute unit (3 rows, 96 experts, d 480, h 2080: 42 and
// 41 us against 46 and 42 in tiles of 64; 34 rows: 33 and 31 against 28 and 26; 82 rows, 13 experts, d 1984, h 3392: 82 and 68 in
// tiles of 32, 65 and 63 of 64, 55 and 60 of 128).  Fewer tiles than compute units: smaller ones as well, since a slice of a
// reduction costs its sums' way through memory (63 rows, 4 experts, d 1728, h 2016: 24 and 22 us in tiles of 64, 16 and 15 of 32).
template <class Product> constexpr int small_tile_height(const Product& a)
{
    const long avg = a.M / std::min<long>(a.E, a.M);
    int BM = avg <= 8 ? 32 : avg <= 56 ? 64 : 128;
    while (BM > 32 && most_tiles(a, BM) < 200) BM /= 2;
    return BM;
}

}  // namespace moe

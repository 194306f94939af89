// Rules by which a launcher chooses between kernels, apart from these so that they can be checked without a GPU.
#pragma once

namespace snip {

// ---- gemm_paper.hip / gemm_paper_wide.hip ----
// The kernel of gemm_paper.hip (tiles of 128 x 128) or that of gemm_paper_wide.hip (256 x 128), whichever is estimated to be
// faster,
//     start + full rounds * turn + stages * slow * (full rounds * full + idle + (full - idle) * load of the last round)
// in microseconds: a round is a tile on every compute unit, a stage 256 contraction elements for FP4 x FP4 and 128 else; a stage
// of a last round takes `idle` on a nearly empty chip (`alone` if it is the only round, else `tail`) and `full` with a tile on
// every compute unit.  `slow`: the wide kernel copies the scales of four slabs at once where a row's lie on 16 bytes, else one
// by one, 8 ... 14 % more per stage.
// Fitted to 21564 problems (128 ... 16384 rows, contractions of 384 ... 8192: random, around whole rounds, multiples of 256 ... 1024;
// FP8 x FP8 and FP4 x FP4, B in blocks and in tiles, operands in the caches and from memory, which differ by less than the
// fit).  On 5632 others the pick is on average 0.15 % slower than the faster kernel, 10 % at worst, and 128 x 128 alone 3.9 %; on
// 10408 more, mixed formats among them, 0.6 % are more than 3 % slower than with 128 x 128 alone, 11 % at worst, which is what the 2 %
// are for by which the wide kernel has to be ahead.  An earlier estimate without `slow` and with `alone` for every last round took
// it for long contractions with a little more than whole rounds, up to 25 % slower than the other ([4992 x 1792 x 7040] FP8 97 us ->
// 122, B in tiles 114 -> 151; [3200 x 7640 x 3840] FP4 86 -> 95).
struct PaperCost { int rows; double start, turn, alone, full, tail, slow; };
constexpr PaperCost kPaperCosts[2][2][2] = {           // [FP4 x FP4][B in tiles][kernel]
    {{{128, 4.841, 1.769, 0.483, 0.611, 0.436, 0.}, {256, 5.002, 2.250, 0.730, 1.014, 0.657, 0.104}},
     {{128, 5.212, 1.797, 0.564, 0.694, 0.506, 0.}, {256, 5.371, 2.275, 1.024, 1.298, 0.916, 0.082}}},
    {{{128, 5.237, 1.866, 0.719, 0.797, 0.701, 0.}, {256, 5.156, 1.777, 1.078, 1.352, 1.035, 0.139}},
     {{128, 5.763, 1.771, 0.911, 0.997, 0.900, 0.}, {256, 5.566, 1.558, 1.605, 1.873, 1.524, 0.119}}},
};

// I x J output, contraction R > 0; `scales16`: every row's scales start on 16 bytes (both operands); `ncu` compute units.
inline bool paper_wide_pays(long long I, long long J, long long R, bool both4, bool b_tiles, bool scales16, long long ncu)
{
    const double stages = (double)((R + (both4 ? 255 : 127)) / (both4 ? 256 : 128));
    double t[2];
    for (int k = 0; k < 2; ++k) {
        const PaperCost& c = kPaperCosts[both4][b_tiles][k];
        const long long tiles = (I + c.rows - 1) / c.rows * ((J + 127) / 128), rounds = (tiles - 1) / ncu;
        const double load = (double)(tiles - rounds * ncu) / (double)ncu, idle = rounds > 0 ? c.tail : c.alone;
        t[k] = c.start + (double)rounds * c.turn +
               stages * (scales16 ? 1.0 : 1.0 + c.slow) * ((double)rounds * c.full + idle + (c.full - idle) * load);
    }
    return t[1] < 0.98 * t[0];
}

// ---- gemm_small.hip, tiles of 64 x 32 and 32 x 32: stages per barrier ----
// Two where operands are likely `cached` (up to kColdBytes): from memory the larger steps cost 64 x 32 2-4 %, and 16 % with more tiles
// than compute units ([9 x 21120 x 7936] FP8 42.4 us -> 49.2), 32 x 32 up to 1 %.  And from four stages on: pairs wait for two stages
// before they begin and multiply a stage of zeros where the number is odd.  Pairs against single stages, averages over 368
// problems, either tile: one stage 3.5 % slower (0.1-0.2 us of 3.0: [126 x 224 x 128] FP8 3.14 -> 3.38), two 0.7 % faster, three 1.5 %
// slower ([98 x 832 x 320] FP8 3.59 -> 3.87), four 2.3 % faster, five the same, seven 1.8 %, eight 5 % and more than that 11 % faster.
constexpr int small_stages_per_barrier(bool cached, long long stages) { return cached && stages >= 4 ? 2 : 1; }

}  // namespace snip

// Rules by which a launcher chooses between kernels, apart from these so that they can be checked without a GPU.
#pragma once
#include "copy_ranges.h"      // SNIP_HD

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
// 20066 more, mixed formats among them, 0.5 % are more than 3 % slower than with 128 x 128 alone, 11 % at worst, which is what the 2 %
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

// ---- gemm_small.hip, tile of 32 x 32: stages per barrier ----
// Two where operands are likely `cached` (up to kColdBytes): from memory the larger steps cost up to 3 %.  And from four stages on:
// pairs wait for two stages before they begin and multiply a stage of zeros where the number is odd.  Single stages against pairs,
// mean of 2600 calls with operands of up to 10 MB, in the caches: up to three stages 1.6 % faster ([126 x 224 x 128] FP8 3.26 us and
// 3.38), four to seven 0.6 % slower, eight to fifteen 2.8 %, sixteen to 31 6.6 %, beyond that 10 %.
constexpr int small_stages_per_barrier(bool cached, long long stages) { return cached && stages >= 4 ? 2 : 1; }

// ---- GEMMs: whether the result is stored streaming (store16 in gemm_common.h) ----
// Result at address `at`, rows `ldc` elements apart.  Rows that do not all start on 64 bytes leave parts of 64-byte pieces at the edges
// of every tile, which memory takes singly: plain stores there.  Streaming against plain, operands from memory, us: pitch off 64 bytes (paper
// recipe) [7040 x 5200 x 256] FP4 32.5 and 27.9, 63 calls +2 %; rows on 64 bytes, 9 calls, -3 %, whole lines, 27 calls above 1 M elements,
// -7 %.  Pitch on 64 bytes, start 16 or 32 bytes past that: [4096 x 2048 x 2048] FP4, fp32, 28.6 and 21.8, [8192 x 3072 x 3072] 94.6 and 73.2,
// [4096 x 4096 x 4096] bf16 42.7 and 39.9, [1024 x 1024 x 1024] 4.64 and 4.23, paper recipe [4096 x 8192 x 2048] FP8 99.5 and 91.9; 44 random calls with
// bf16 results, 512 ... 12288 rows, the same on average, 19 % slower ([1472 x 12576 x 512]) to 25 % faster ([1952 x 1408 x 4096] FP8).
// No limit of size: whoever reads a result at once takes back a part of what streaming it gains, or more than that, as it then comes from memory,
// but a step gains.  GEMM alone, followed by a quantize call and by an elementwise pass that read the result, operands from memory, plain ->
// streaming, us: [64 x 4096 x 4096] FP4, 0.5 MB, 4.65 -> 4.67, 8.15 -> 8.41 and 6.85 -> 6.90; [512 x 2048 x 2048] 2 MB 4.88 -> 4.92, 8.75 -> 9.27 and
// 7.30 -> 7.54; [4096 x 2048 x 2048] 17 MB 15.7 -> 13.2, 23.5 -> 23.0 and 21.9 -> 22.2, fp32 17.5 -> 16.9 and (elementwise) 28.1 -> 32.0; [8192 x 8192 x
// 3072] 134 MB 107.2 -> 105.9, 133 -> 147 and 157 -> 160; [16384 x 11008 x 4096] 368 -> 350, 460 -> 442 and 470 -> 461.  Training steps of one to four blocks in
// which elementwise passes read every Y and dX as soon as it is there, 64 ... 16384 tokens, hidden 1024 ... 8192, take 0.2 ... 5 % less
// (21 steps, mean 2.5), with every dW read at once too 0.1 % (twelve, -1.6 ... +1.6), with fp32 dW that wait 1 ... 9 % less (eight), with no reader 2 ... 11 %.
// Limits tried: plain below 1 MB, 1 % less for 64 tokens of hidden 2048 with readers, 1 % more for forwards of 64 tokens without; below 4 MB up to 3 %
// more without readers; plain from 56 MB or 200 MB on, 1 % less to 1.5 % more.
constexpr bool streams_result(unsigned long long at, long long ldc, bool f32) { return ((at | (unsigned long long)ldc * (f32 ? 4 : 2)) & 63) == 0; }

// ---- gemm_small.hip: whether the codes of B are streamed ----
// Where one row of tiles reads them, once (few tokens through a weight); other tile rows would find them in L2 ([65 x 11008 x 4096] FP4, two rows
// of 64 x 64, four weights in turn 9.2 us -> 12.5, 24 of them, from memory, 11.3 -> 13.1).  From 20 MB on: a block with such weights has 90 MB
// of them, so the memory-side cache (256 MB) keeps them for no second use, and streamed they come faster and leave it to the smaller ones.
// What that is worth follows from how much is read in turn, which a call does not see.  Plain -> streaming, [1 x 11008 x 4096] and [64 x 11008 x 4096]
// FP4 (22.5 MB), us: one weight again and again 5.13 -> 5.14 and 6.16 -> 6.24, four 5.95 -> 6.11 and 6.50 -> 8.16, eight 5.95 -> 6.30 and 6.51 -> 8.34, sixteen
// (361 MB) 6.78 -> 6.40 and 8.77 -> 8.45; FP8 (45 MB) four 9.16 -> 10.2 and 10.1 -> 14.0, sixteen 11.8 -> 10.6 and 14.8 -> 14.3.  Forwards of blocks, four shapes of
// 7B to 13B, one and 64 tokens: one block again and again 3 ... 21 % slower (7B-shaped FP4 47.6 -> 49.1 and 52.9 -> 59.8), three in turn 1 ... 14 %
// faster (52.9 -> 48.5 and 62.9 -> 56.4), eight 0 ... 7 % (53.5 -> 53.1 and 64.4 -> 64.4).  A program has all blocks of a model in turn.
// Smaller weights may be in that cache, and streaming would bring them from memory again (8 tokens, hidden 3584, FP4, three blocks
// in turn: 47.8 us and 56.9; streamed from 8 MB on 64 tokens through 7B-shaped blocks took 60.7).
constexpr bool small_streams_b(bool one_row, long long bytes) { return one_row && bytes >= 20ll << 20; }

// ---- quant_kernels.hip, quantize for both orientations: the order of the units among the XCDs ----
// A unit is a row unit (RBU tiles of 32 rows) of a column group (128 columns).  Workgroup ids go to the XCDs in turn (id mod 8); units
// go to them in turns of eight consecutive ones or, if `eighth` is not 0, `eighth` units each.  Consecutive units walk pairs of row units
// column group by column group (a turn is two row units by four column groups), so that the two halves of a 128-byte line (FP4
// codes of a row: 64 bytes per unit; FP4 codes of a column, likewise) and the scale bytes of neighbours meet in one L2.  Dealt one by
// one, 37 % more bytes reached memory than there are for [16384 x 11008] FP4.  (Turns of any length would take a division in qb_unit: 0.1
// us of the 4.0 us of a small call.)
// In turns, what row units the pairs leave over, and a last one with fewer tiles, are walked by themselves behind all others: where
// there are a few more units than fit at once, whole ones at the end are a round of their own (all statistics, [1344 x 11264] FP4 28.6 us
// instead of 24.2, [2912 x 5632] 29.0 instead of 26.0, [800 x 27392] 36.2 instead of 32.9).  With eighths one XCD would have nearly all
// the short ones ([160 x 25984] FP4 7.1 instead of 6.4): they stay in their pairs.
// Where the stored columns are no whole number of 128-byte lines, every row unit shares lines of every column with the next one, and
// bands of four row units instead of two (a turn of four by two) leave fewer of them to two L2s: FP4 columns beside FP8 rows, pairs
// -> four, [86080 x 2048] 155 -> 129, [52000 x 2048] 96.7 -> 81.1, [28608 x 6144] 159 -> 137, [8160 x 11008] 90.4 -> 84.2, [25760 x 1984] 49.2 ->
// 43.7; on average 2 % below 64 M elements and 6 % above, at worst 6.5 % slower.  Not where the last column group is a part of one:
// the rows' lines run on into the next group, and a turn of four by two splits more of these ([22624 x 8288] FP4 161 -> 174), unless
// bands of four bring the same columns to the same XCD again (16 groups or an odd multiple).  Nor at a multiple of 32 groups or near
// one, where pairs do that already ([8160 x 8160] FP4 54.3 -> 60.9, [2624 x 16000] 36.1 -> 38.5).
struct QbPlace { int ru, cg; };
SNIP_HD constexpr int qb_unit(int v, int eighth) { return eighth ? (v & 7) * eighth + (v >> 3) : (v & ~63) + (v & 7) * 8 + (v >> 3 & 7); }
SNIP_HD constexpr int qb_bands(int whole_row_units, int row_units, int eighth, int log2) { return (eighth ? row_units : whole_row_units) >> log2; }
SNIP_HD constexpr QbPlace qb_place(int u, int bands, int log2, int ncg)
{
    const int banded = (bands * ncg) << log2;
    const bool in_band = u < banded;
    const int band = in_band ? ncg << log2 : ncg, from = in_band ? u : u - banded, k = from / band, rem = from - k * band;
    return in_band ? QbPlace{(k << log2) + (rem & ((1 << log2) - 1)), rem >> log2} : QbPlace{(bands << log2) + k, rem};
}
constexpr int qb_band_log2(long long cols, long long column_bytes)
{
    const long long phase = (cols + 127) / 128 % 32;
    return column_bytes % 128 != 0 && (phase == 16 || (cols % 128 == 0 && phase >= 4 && phase <= 28)) ? 2 : 1;
}
// An eighth of the tensor each (true) or turns of eight units.  us per call, dealt one by one / turns of eight / eighths:
//   - below 8 M elements the tensor fits the L2s: eighths, which lead by a little ([1504 x 2080] FP4 6.4 / 5.9 / 5.8, FP8 6.6 / 6.3 /
//     6.1), up to 24 M where rows hold no whole number of four blocks, so that scale bytes share dwords and lines with the
//     neighbours' at odd places ([2432 x 4896] FP4 13.0 / 12.7 / 12.9, FP8 15.4 / 15.6 / 15.3, with all statistics 22.6 / 21.8 / 21.6).
//   - larger tensors: turns of eight; far apart, the eighths meet in few memory channels.  [16384 x 11008] FP4 131 / 128 / 133, [32768 x
//     4096] 100.5 / 87.9 / 103 and FP8 116 / 107 / 131, [16384 x 8192] 97.5 / 89.8 / 99.8, [8160 x 8160] 72.7 / 54.2 / 69.4 and 98.8 / 82.3 / 89.6,
//     [2048 x 22016] 37.9 / 35.8 / 38.8 and 42.6 / 42.2 / 46.4, [6144 x 22016] 104 / 100 / 104 and 119 / 118 / 124; with all statistics
//     [11008 x 4096] 52.4 / 50.4 / 50.6, [4096 x 4096] 23.3 / 23.7 / 27.7.
//   - but where the stored columns lie whole multiples of 4096 bytes apart, the column groups of a turn meet in few channels too:
//     for more than 16384 columns eighths again, without statistics, where rows start on whole lines.  [8192 x 28672] FP4 181 / 166 /
//     168, FP8 214 / 206 / 198, [8192 x 32768] 218 / 200 / 186 and 254 / 262 / 223, [4096 x 28672] FP8 107 / 104 / 103, beside FP4 rows
//     103 / 100 / 98.  (FP8 with 16384 columns and less also gains, 2-4 % from 8192 rows on; FP4 loses 2 %.)
//   - and for such rows with FP8 columns of whole 128-byte lines from 160 M elements on, where row units share no line of a column:
//     turns / eighths [10496 x 23808] FP8 227 / 212, [12544 x 21504] beside FP4 rows 224 / 210; 111 calls of 192 ... 420 M 3.5 % on average,
//     17 of 160 ... 192 M 1.5 %.  Below 144 M turns lead by 3 % ([4224 x 30080] FP8 107 / 114).  Columns that are no whole lines gain
//     7 % from turns (77 calls), FP4 ones that are 1 %.
constexpr bool qb_eighths(long long rows, long long cols, long long ld, long long column_bytes, bool stats)
{
    const bool fp8_columns = column_bytes == rows;
    return rows * cols < (cols % 128 != 0 ? 24ll << 20 : 8ll << 20) ||
           (!stats && cols > 16384 && ld % 128 == 0 &&
            (column_bytes % 4096 == 0 || (fp8_columns && column_bytes % 128 == 0 && rows * cols >= 160ll << 20)));
}

// ---- ... whether its tiles go through LDS, without statistics ----
// As soon as a compute unit has more than two units: rows and columns of a tile both fetched it, which is what bound the kernel
// (without the rows' share [8192 x 3072] FP4 took 15.7 us of 23.3).  Direct -> LDS: [16384 x 11008] FP4 140 -> 127, FP8 162 -> 160, [32768 x
// 4096] 101 -> 88 and 112 -> 106, FP8 rows beside FP4 columns 106 -> 98, [8192 x 28672] 191 -> 169 and 215 -> 199, FP4 rows beside FP8
// 207 -> 186, [8160 x 8160] 59.8 -> 55.1 and 81.8 -> 80.6, [3072 x 3072] 12.5 -> 11.4 and 15.0 -> 13.1.  With up to two units the two more
// barriers cost 0.3-0.45 us ([2048 x 2048] FP4 5.9 against 6.3, FP8 6.9 against 7.3), and with more than three and up to four, of
// which a compute unit takes three at once, up to 8 % ([3200 x 4096] 14.4 against 15.2, mixed 15.9 against 17.2; [4096 x 4096] 16.2
// against 16.3).  Half a column group and less is too little to fetch for that: [140800 x 32] FP4 9.2 against 10.2, [68736 x 64] 7.1
// against 7.8, [262144 x 32] 14.5 against 15.5; with 96 columns they are even (8.9 and 8.8 on [68736 x 96]).
// Where the line lies is decided on tensors that come from memory and results that go there, as in a step of a model; mean of 1200 calls of
// 1.6 ... 9 units per compute unit, LDS against direct: up to two units 1.0 % slower, three 10.6 % faster ([2432 x 4224] FP8 12.3 us and 11.2,
// [1536 x 5760] FP4 14.9 and 11.8), four 1.9 % faster (10 % slower ... 14 % faster), beyond that 3.8-5.5 % faster.  On one buffer again and
// again, all in the caches, the direct form is faster throughout, by 8.5 % up to two units and 4-5 % beyond (8.3 and 8.9, 9.1 and 9.9).
constexpr bool qb_through_lds(long long cols, long long units, long long ncu)
{
    return cols > 64 && units > 2 * ncu && !(units > 3 * ncu && units <= 4 * ncu);
}

// ---- ... whether the waves of rows leave the columns' stores to those of columns, without statistics or LDS ----
// With up to one unit per compute unit, where a call is one tile's chain: [256 x 512] FP4 3.7 us -> 3.45, [1024 x 1024] 4.2 -> 3.95, FP8 4.3 ->
// 4.0, [1504 x 2080] 5.8 -> 5.5, [2048 x 2048] 6.5 -> 6.3 and 7.56 -> 7.53; six launches of a 256 x 512 x 512 step 20.8 -> 20.0.  Beyond that half of
// the waves store 16 KB of FP8 columns too slowly ([4096 x 2048] 10.8 -> 11.4, [2048 x 5632] 11.4 -> 12.2, FP4 9.5 -> 9.6 and 10.1 -> 9.9;
// through LDS [8192 x 3072] 21.9 -> 23.3).
constexpr bool qb_rows_apart(long long units, long long ncu) { return units <= ncu; }

// ---- ... whether the forms for large tensors (through LDS; a wave per unit) stream their codes past the caches ----
// From 128 MB of codes in both orientations on, half of the memory-side cache (256 MB), and of FP4 codes alone from 256 MB on: they would
// not be there any more when a GEMM wants them, and leave their place to those of smaller tensors and to what the GEMMs read.  Plain ->
// streaming, us: steps of one linear, gradients of [16384 x 4096] FP8 (128 MB) 294 -> 278, [4096 x 16384] 301 -> 285, [16384 x 11008] FP8 rows and FP4
// columns (258 MB) 1050 -> 1013; but [8192 x 8192] FP8 395 -> 413.  Steps of blocks, 7B-shaped, 16384 tokens, FP8 7937 -> 7912 (9788 -> 9706 with readers of
// every Y and dX), rows and columns of both formats 7163 -> 7155 (9054 -> 8992), 70B-shaped FP8 15783 -> 15725; FP4, tensors of 256 MB ([32768 x 8192])
// 3606 -> 3572.  Less is slower: FP4 gradients of [16384 x 4096] (64 MB) 184 -> 193, in both formats (96 MB) 247 -> 262, blocks in FP4 with tensors of 172 MB
// 4638 -> 4675 and with 224 MB 8966 -> 9021; streamed from 16 M elements on, 40 steps of one linear lose 1.8 % on average (14 % at worst, [2176 x 8960 x
// 1024] 102 us -> 117).
// With statistics the codes come more slowly, and it pays from 64 M elements on: steps of one linear with gradients of 64 M ... 172 M elements, FP8
// 2.4 % less on average (eight, 0.6 ... 6.7), both formats 1.0 % (sixteen, 4.3 ... -1.8), FP4 the same (eight, 1.6 ... -2.2); [4096 x 16384] FP8 336 -> 313, FP4 rows and FP8
// columns 302 -> 290.
// And where every stored row starts on 64 bytes, by pitch and by address: pieces of 64 bytes reach memory by themselves ([12384 x 10656]
// FP4, rows of 5328 bytes, 161 us -> 196).
constexpr bool qb_streams(long long rows, long long cols, bool fp8_rows, bool fp8_columns, bool stats, unsigned long long at_rows = 0, unsigned long long at_columns = 0)
{
    const long long row = fp8_rows ? cols : cols / 2, column = fp8_columns ? rows : rows / 2;        // bytes
    if (((at_rows | at_columns | (unsigned long long)row | (unsigned long long)column) & 63) != 0) return false;
    if (stats) return rows * cols >= 64ll << 20;
    return rows * row + cols * column >= (fp8_rows || fp8_columns ? 128ll << 20 : 256ll << 20);
}

}  // namespace snip

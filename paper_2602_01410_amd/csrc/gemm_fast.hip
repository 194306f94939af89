// Large-tile variant of the block-scaled GEMM, used when both operands carry the grouped scale copy
// (scales_g4) and the contraction extent is longer than a stage.
//
//   workgroup tile 256 x 256, 8 waves (2 x 4), wave tile 128 (A rows) x 64 (B rows), fp32
//   accumulators in registers (128 per lane); for outputs that would leave compute units without a
//   tile, 256 x 128 with 4 x 2 waves of 64 x 64 (same code, other template argument).
//   256 x 256 has two stage buffers (68 KB each, FP8 66), 256 x 128 three (51 KB, FP8 50; two for few stages): a copy then has
//   1.75-2 stages to arrive instead of 0.75-1, which memory needs under load (a stage is 0.9-1.1 us).
//   A pipeline stage is 128 code bytes of every tile row for an FP8 operand and for FP4 x FP4
//   (256 contraction elements there), so every 128-byte line that is fetched is used whole.
//   Codes and scale dwords go global -> LDS through the load unit (global_load_lds), never through
//   VGPRs.
//   The eight waves run a ping-pong schedule: the two waves of a SIMD alternate between reading
//   their operands of a phase from LDS and issuing that phase's MFMAs, one phase apart, separated by
//   workgroup barriers, so that the matrix core of every SIMD always has a wave with operands ready.
//   A wave issues its global -> LDS copies between the MFMAs of one of its MFMA phases, where issue
//   slots are free (an MFMA occupies the matrix core for 32 or 64 cycles, a copy instruction costs the
//   wave about 40); issued in front of the LDS reads they made that phase the longest of the four.
//   LDS rows are unpadded; the 16-byte chunks of a row are XOR-swizzled on the global-address side
//   of the copy so that the 16 lanes served together by a ds_read_b128 hit 16 different bank groups.
//   The result tile leaves through LDS as well: each wave transposes its 128 x 64 block so that the
//   global stores are 16 bytes per lane and 128 contiguous bytes per row.
//   The kernel is persistent: one workgroup per compute unit walks its tiles (dispatch ids blockIdx.x,
//   blockIdx.x + gridDim.x, ...) and treats their pipeline stages as one sequence, so the first stage of the
//   next tile is copied into the free stage buffer during the last stage of the current one and a tile's
//   start-up latency is paid once per workgroup, not once per tile.  The result tile is staged in the other
//   stage buffer (the one the last stage was read from), 64 KB at a time.
//
// What bounds it (hardware counters and variants of this kernel with one part removed, 16384 x 4096 x 4096 and
// 4096 x 4096 x 16384 on Gaussian data): the matrix cores are busy for 0.62-0.64 of the compute units' busy cycles
// and the shader clock (GRBM_GUI_ACTIVE over the launch duration) is 1.83 GHz (FP4) to 1.95 GHz (FP8) instead of 2.4;
// a loop of nothing but MFMAs on random operands runs at 1.64 / 2.03 GHz.  LDS is active a third of the time with
// 2 % bank-conflict cycles.  Leaving out the workgroup barriers changes nothing.  Leaving out the global -> LDS
// copies gains 20 % on random codes but 7 % on all-zero codes, half of the copies 8.5 %, and copies that always
// hit one L2-resident stage 5 %: what the copies cost is mostly clock (the chip slows down as more random bytes
// move through a compute unit), not latency and not misses.  Plain result stores cost 10 % at contraction extent
// 4096 (streaming ones less, see store16): all workgroups finish a tile together, 32 MB per round, and the next tile's
// copies queue behind them in the wave's memory counter.
// Time stamps in a launch of one tile per workgroup ([4096 x 2048 x 2048] FP4, 256 x 128, operands from memory): 1.5 us after the
// launch before it, 1.9 until the first stage is there, eight stages of 0.72 (the first) to 1.0 us, 2.4 for the result; the shader
// clock falls from 2.4 GHz to 1.65 within the first 4 us of stages.
//
// Registers: 256 vector registers (256 x 256), 200-246 (256 x 128; 193-215 with two buffers).  Scalar registers run out and spill to
// lanes of vector registers: 23-25 for bf16 outputs and 58-65 for fp32 (256 x 256; 256 x 128 20-26 and 60-65, with two buffers 17-19
// and 57-59), 50-62 and 84-97 with TAIL (63-71 and 93-102, 50-62 and 85-96), of which a stage restores up to six.
//
// See gemm.hip for the register layout of v_mfma_scale_f32_32x32x64_f8f6f4.
#include "gemm_common.h"
#include <algorithm>
#include <type_traits>

namespace snip {
namespace {

constexpr int NWAVE = 8, NT = NWAVE * 64;

// Workgroup tile TM (A rows) x TN (B rows), split over the eight waves as (TM / WTM) x (TN / WTN) wave tiles.
template <int TM_, int TN_, int WTM_, int WTN_, int NST_, int PH_> struct TileCfg {
    static constexpr int TM = TM_, TN = TN_, WTM = WTM_, WTN = WTN_, NST = NST_, PH = PH_;      // stage buffers, phases of a stage
    static constexpr int WGN = TN / WTN;                   // waves along the B rows
    static constexpr int MB = WTM / 32, NB = WTN / 32;     // 32 x 32 MFMA blocks of a wave tile
    static_assert(TM == 256 && (TN == 256 || TN == 128), "copy shares and scale areas are laid out for these tiles");
    static_assert((TM / WTM) * (TN / WTN) == NWAVE, "eight waves");
};
// 256 x 256, 2 x 4 waves of 128 x 64: the largest tile the register file allows (fewest operand bytes per FLOP).
using TileBig = TileCfg<256, 256, 128, 64, 2, 2>;
// 256 x 128, 4 x 2 waves of 64 x 64: twice as many tiles for outputs that would leave compute units without one.  us per call on
// operands from memory with two stage buffers (and operand lines pulled into L2 four stages ahead) -> with three: [4096 x 2048 x
// 8192] FP4 48.5 -> 43.0, FP8 74.6 -> 69.3, [4096 x 2048 x 2048] 19.6 -> 18.0, 25.4 -> 23.3, [8192 x 3072 x 3072] FP8 89 -> 81.5,
// [2048 x 4096 x 4096] FP8 41.6 -> 39.0.  Pulling lines ahead of three buffers as well costs 1-8 %.  A stage is one phase here (its
// operands take 64 registers), which halves the barriers and the LDS latencies of a stage; two phases -> one: [4096 x 2048 x 2048]
// FP4 18.5 -> 17.4, FP8 24.4 -> 23.2, [4096 x 2048 x 8192] 44.8 -> 43.0 and 68.6 -> 65.5, [8192 x 3072 x 3072] 59.0 -> 55.8 and 84.8 -> 82.9,
// [3072 x 8192 x 8192] 118 -> 112 and 186 -> 175; operands in the caches 2-9 %.
using TileWide = TileCfg<256, 128, 64, 64, 3, 1>;
// The same tile for contractions of two stages, which three buffers do not take, and of three whole ones, where the result's two
// passes cost more than the third buffer gives.  Two stages against the best other tile: [15616 x 384 x 512] FP4 11.3 -> 8.3 us,
// [10304 x 672 x 384] 11.8 -> 9.2, [2048 x 3456 x 512] 10.3 -> 8.1.  Three against three buffers, 10 outputs in all formats: -3.3 %
// (cached) and 0 (memory) over several rounds, -1.2 and -2.2 % in one; three stages of which the last is cut +5 ... +7 %, four +3 ... +8 %.
using TileShort = TileCfg<256, 128, 64, 64, 2, 2>;

template <int FA, int FB, class T> struct FCfg {
    static constexpr int TM = T::TM, TN = T::TN;
    static constexpr bool BOTH4 = FA == kFP4 && FB == kFP4;
    static constexpr int KE = BOTH4 ? 256 : 128;                 // contraction elements per stage
    static constexpr int SBA = FA == kFP8 ? KE : KE / 2;         // code bytes per row per stage (128, or 64 for FP4 next to FP8)
    static constexpr int SBB = FB == kFP8 ? KE : KE / 2;
    static constexpr int KS = KE / 64;                           // MFMA steps per stage
    static constexpr int NG = KE / 128;                          // scale dwords (groups of 4 blocks) per row per stage
    static constexpr int NST = T::NST;
    static constexpr int A_BYTES = TM * SBA, B_BYTES = TN * SBB;
    // Scale dwords of one stage, [group][256 rows] of A and [group][TN rows] of B, in copies of 1 KB: NSA of A, then B's (two groups
    // of a 128-row B tile are one copy, a single one is half of one)
    static constexpr int NSA = NG, NSB = (TN * NG * 4 + 1023) / 1024, NSC = NSA + NSB;
    static constexpr int SLOT = A_BYTES + B_BYTES + NSC * 1024;
    // Stage buffers lie STRIDE apart.  The result staging area is part of the LDS array that covers the buffer of the tile's
    // last stage and never reaches into the other buffers, which already receive the next tile: with two buffers (one at
    // the start of the array, one at its end) the first or the last 64 KB, with three the first 32 KB of that buffer.
    static constexpr int LDS_BYTES = NST == 2 ? 159 * 1024 : NST * SLOT;
    static constexpr int STRIDE = NST == 2 ? LDS_BYTES - SLOT : SLOT;
    static constexpr int EPI_BYTES = NST == 2 ? 64 * 1024 : 32 * 1024;
    static constexpr int epi_base(int last) { return NST == 2 ? (last ? LDS_BYTES - EPI_BYTES : 0) : last * STRIDE; }
    static constexpr int LA = A_BYTES / 1024 / NWAVE;            // 1 KB copies of codes per wave per stage
    static constexpr int LB = B_BYTES / 1024 / NWAVE;
    static constexpr int L = LA + LB;                            // (and one of scales in the waves of group 0, in front of them)
    static_assert(NSC <= NWAVE / 2, "the waves of group 0 copy the scales");
    static_assert(STRIDE % 1024 == 0 && SLOT <= STRIDE && (NST - 1) * STRIDE + SLOT <= LDS_BYTES, "stage buffers must not overlap");
    static_assert(EPI_BYTES <= (NST == 2 ? STRIDE : SLOT), "the result staging area must stay clear of the other stage buffers");
    static_assert(L * (NST - 1) <= 60, "copies in flight must be countable");
    static_assert(LDS_BYTES + 64 <= 160 * 1024, "LDS budget");
};

// TAIL: the contraction extent does not end with a stage.  Copies then go through buffer descriptors, which deliver zeros
// for chunks past the end of a row, and the scale bytes past the last block are masked.  It is a variant of its own
// because descriptors and masks cost the whole-stage form 10-14 % (16384 x 4096 x 4096, FP4 134 -> 147 us, FP8 202 -> 233;
// scalar registers spill); against the general kernel it is 3.5-4 times as fast (4096 x 4096 x 4128, FP4 190 -> 46 us).
// STREAM: result stores (store16).  Kernels of their own too: with both kinds in one, whole tiles of fp32 results had to share the
// stores of ragged ones where they are plain, for want of scalar registers (rows off 64 bytes, operands from memory: [4096 x 2048 x 2048]
// FP4 21.6 us -> 19.5, FP8 27.0 -> 26.1, [8192 x 3072 x 3072] FP4 71.8 -> 70.1).
template <int FA, int FB, bool OUT_F32, class T, bool TAIL, bool STREAM>
__global__ __launch_bounds__(NT) void gemm_fast_kernel(const uint8_t* __restrict__ a_codes,
                                                       const uint8_t* __restrict__ a_g4,
                                                       const uint8_t* __restrict__ b_codes,
                                                       const uint8_t* __restrict__ b_g4,
                                                       int I, int J, int R, void* __restrict__ c_out, int64_t ldc,
                                                       int tiles_i, int tiles_j, float* __restrict__ norm_partials)
{
    using C = FCfg<FA, FB, T>;
    constexpr int TM = T::TM, TN = T::TN, WTM = T::WTM, WTN = T::WTN, WGN = T::WGN, MB = T::MB, NB = T::NB;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[C::LDS_BYTES];
    // stage buffer layout: [A codes][B codes][A scale dwords: group-major, 256 rows][B scale dwords]

    const int nblk = tiles_i * tiles_j;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int r32 = lane & 31, g = lane >> 5;

    const int64_t a_row_bytes = FA == kFP8 ? R : R / 2;
    const int64_t b_row_bytes = FB == kFP8 ? R : R / 2;
    const int nstage = (R + C::KE - 1) / C::KE;                       // >= NST (launch_gemm_fast)
    const int ngrp = (R + 127) / 128;                                 // scale groups of a row
    const int64_t a_pitch = g4_pitch(I), b_pitch = g4_pitch(J);      // dwords per scale group

    // ---- source addresses of the global->LDS copies of ONE tile (the tile the wave's copies currently belong
    //      to, which runs ahead of the tile being multiplied): wave-uniform base + per-lane 32-bit offset.
    //      Rows past the end of an operand re-read its last row (their products are never stored). ----
    unsigned oa[C::LA], ob[C::LB];
    const uint8_t* abase;
    const uint8_t* bbase;
    // TAIL: descriptors over the tile's rows (rows past the end of an operand lie past their end) and over the grouped
    // scale copy.
    v4i ra, rb, rs;
    // Scales: a wave of group 0 makes one 1 KB copy per stage, 16 bytes per lane: four rows of a scale group of A, or of B (of a 128-row
    // B tile: half of the lanes each group, or both halves the same one).  Where there are fewer than four copies the other waves
    // repeat them.  With copies of a dword per lane in every wave it was 20 copy instructions of a stage's two waves of a SIMD
    // instead of 17 (256 x 256, FP4); the GEMMs of a step, FP4: 70B-shaped block 6547 -> 6471 us, 7B 2929 -> 2904, FP8 the same; [16384 x
    // 4096 x 4096] FP4 256 x 256 138.0 -> 137.3, 256 x 128 159.6 -> 158.2, [16384 x 4096 x 11008] 326.7 -> 323.0 and 383.4 -> 378.7.
    const int sq = wave % C::NSC;
    const bool sop = sq >= C::NSA;
    const int sgrp = sop ? (TN == 256 ? sq - C::NSA : 0) : sq;
    const unsigned spitch = (unsigned)(sop ? b_pitch : a_pitch) * 4;
    const uint8_t* sbase;
    const unsigned os = TN == 128 && sop ? scale_lane(C::NG == 2 ? lane / 32 : 0, lane % 32 * 4, spitch) : scale_lane(TAIL ? sgrp : 0, lane * 4, spitch);
    auto chunk_a = [&](int j) { constexpr int CPR = C::SBA / 16, RPI = 1024 / C::SBA; return (lane % CPR) ^ swz<C::SBA>((wave * C::LA + j) * RPI + lane / CPR); };
    auto chunk_b = [&](int j) { constexpr int CPR = C::SBB / 16, RPI = 1024 / C::SBB; return (lane % CPR) ^ swz<C::SBB>((wave * C::LB + j) * RPI + lane / CPR); };
    auto set_copy_tile = [&](int u) {
        int ti, tj;
        tile_of(u, nblk, tiles_i, tiles_j, ti, tj);
        const int i0 = ti * TM, j0 = tj * TN;
#pragma unroll
        for (int j = 0; j < C::LA; ++j) {
            constexpr int CPR = C::SBA / 16, RPI = 1024 / C::SBA;
            const int row = (wave * C::LA + j) * RPI + lane / CPR;
            oa[j] = (unsigned)((TAIL ? row : min(row, I - 1 - i0)) * a_row_bytes + chunk_a(j) * 16);
        }
#pragma unroll
        for (int j = 0; j < C::LB; ++j) {
            constexpr int CPR = C::SBB / 16, RPI = 1024 / C::SBB;
            const int row = (wave * C::LB + j) * RPI + lane / CPR;
            ob[j] = (unsigned)((TAIL ? row : min(row, J - 1 - j0)) * b_row_bytes + chunk_b(j) * 16);
        }
        if (TAIL) {
            const unsigned row4 = (unsigned)(sop ? j0 : i0) * 4;
            ra = buffer_desc(a_codes + (int64_t)i0 * a_row_bytes, (unsigned)(min(TM, I - i0) * a_row_bytes));
            rb = buffer_desc(b_codes + (int64_t)j0 * b_row_bytes, (unsigned)(min(TN, J - j0) * b_row_bytes));
            rs = buffer_desc((sop ? b_g4 : a_g4) + row4, scale_size(ngrp, spitch, row4));
            return;
        }
        // (the padded pitch of the grouped copy covers whole tiles)
        sbase = (sop ? b_g4 : a_g4) + (int64_t)sgrp * (sop ? b_pitch : a_pitch) * 4 + (int64_t)(sop ? j0 : i0) * 4;
        abase = a_codes + (int64_t)i0 * a_row_bytes;
        bbase = b_codes + (int64_t)j0 * b_row_bytes;
    };
    // A workgroup's last copies, which nobody reads, all from one place: they are waited for before the result is stored, and take L2
    // and power beside the last MFMAs.  From memory, graphs: 3B-shaped block 2146 us -> 2133, backward of 8192 x 8192 x 3072 283.8 -> 281.3.
    // (Not where fp32 results leave no scalar registers: of a cut contraction, 35 spilled ones fetched between MFMAs, of FP8 times FP4 in
    // 256 x 128, 28.)
    constexpr bool QUIET = !(OUT_F32 && (TAIL || (FA == kFP8 && FB == kFP4 && TN == 128)));
    auto copy_nothing = [&]() {
#pragma unroll
        for (int j = 0; j < C::LA; ++j) oa[j] = TAIL ? kNoSource : 0u;
#pragma unroll
        for (int j = 0; j < C::LB; ++j) ob[j] = TAIL ? kNoSource : 0u;
    };
    // TAIL, before the copies of the last stage: lanes whose chunk lies past the end of the row lose their source until the
    // next set_copy_tile.
    auto cut_tail = [&](int stage) {
        if (!TAIL || stage != nstage - 1) return;
#pragma unroll
        for (int j = 0; j < C::LA; ++j) oa[j] = chunk_a(j) * 16 < (int)a_row_bytes - stage * C::SBA ? oa[j] : kNoSource;
#pragma unroll
        for (int j = 0; j < C::LB; ++j) ob[j] = chunk_b(j) * 16 < (int)b_row_bytes - stage * C::SBB ? ob[j] : kNoSource;
    };
    const unsigned lds0 = lds_addr(lds);

    // Where this wave's share of the codes lies in stage buffer `slot`.  The empty statements keep it in one scalar register (two for
    // unequal shares): the compiler would otherwise form the place of every copy ahead of all loops, spill these, and fetch each
    // back with a vector instruction between the MFMAs, which hold such up for about 20 cycles.  Formed in front of the operand
    // reads; behind the barrier in front of the MFMAs FP8 took 1-4 % longer.  Cached operands, fp32 results, cut last stage, us: FP4
    // [5376 x 1152 x 11648] 52.2 -> 49.2, [407 x 14080 x 14976] 67.5 -> 62.5, FP8 [2784 x 2368 x 10560] 77.1 -> 73.5; mean of 24 problems FP4
    // 2.5 % (bf16 results 0.5 %), FP8 1 % (0.4 %), FP8 x FP4 0.2 % (1 %); from memory the same.  Kernels of whole stages with bf16
    // results have a third of the spills and nothing to gain, and with 256 x 256 and FP4 lost three lane registers of the result
    // store's ragged path to scratch ([4960 x 1760 x 512] 10.9 -> 11.8 us, [6944 x 2016 x 512] 12.0 -> 13.0).
    constexpr bool HELD = TAIL || OUT_F32;
    struct Share { unsigned a, b; };
    auto share = [&](int slot) {
        Share d;
        if constexpr (!HELD) {
            d.a = lds0 + slot * C::STRIDE;
            d.b = d.a + C::A_BYTES;
            return d;
        }
        d.a = lds0 + wave * C::LA * 1024 + slot * C::STRIDE;
        asm volatile("" : "+s"(d.a));
        if (C::LA == C::LB) {
            d.b = d.a + C::A_BYTES;
        } else {
            d.b = lds0 + C::A_BYTES + wave * C::LB * 1024 + slot * C::STRIDE;
            asm volatile("" : "+s"(d.b));
        }
        return d;
    };
    // copy instruction j (0 .. L-1) of this wave's share of the codes of `stage` (of the copy tile)
    auto issue_one = [&](int j, int stage, Share to) {
        if constexpr (!HELD) to = Share{to.a + wave * C::LA * 1024, to.b + wave * C::LB * 1024};
        if (j < C::LA) {
            if constexpr (TAIL) blds16(ra, oa[j], stage * C::SBA, to.a + j * 1024);
            else glds16(abase + (int64_t)stage * C::SBA, oa[j], to.a + j * 1024);
        } else {
            const int k = j - C::LA;
            if constexpr (TAIL) blds16(rb, ob[k], stage * C::SBB, to.b + k * 1024);
            else glds16(bbase + (int64_t)stage * C::SBB, ob[k], to.b + k * 1024);
        }
    };
    auto issue_scale = [&](int stage, int slot) {
        const unsigned dst = lds0 + slot * C::STRIDE + C::A_BYTES + C::B_BYTES + sq * 1024;
        if constexpr (TAIL) blds16(rs, os, scale_uniform(stage, C::NG, spitch), dst);
        else glds16(sbase + (int64_t)stage * C::NG * (sop ? b_pitch : a_pitch) * 4, os, dst);
    };
    auto issue = [&](int stage, int slot) {
        const Share to = share(slot);
#pragma unroll
        for (int j = 0; j < C::L; ++j) issue_one(j, stage, to);
    };

    // ---- per-lane LDS read offsets ----
    constexpr int NCA = FA == kFP8 ? 2 * C::KS : C::KS, NCB = FB == kFP8 ? 2 * C::KS : C::KS;
    int offa[NCA], offb[NCB];
    frag_offsets<FA, C::SBA, C::KS>(r32, g, offa);
    frag_offsets<FB, C::SBB, C::KS>(r32, g, offb);
    const int sca_off = C::A_BYTES + C::B_BYTES + (wm * WTM + r32) * 4;
    const int scb_off = C::A_BYTES + C::B_BYTES + TM * C::NG * 4 + (wn * WTN + r32) * 4;

    v16f acc[MB][NB];

    // ---- ping-pong schedule.  The two waves that share a SIMD (wave w and w + 4) belong to different
    //      groups.  A stage is PH phases (two below); in every phase a wave either reads its operands of that phase
    //      from LDS into registers (R) or issues that phase's MFMAs (M).  Workgroup barriers separate the
    //      phases and group 1 runs one phase behind group 0, so while one wave of a SIMD feeds the matrix
    //      core the other one fetches:
    //          barrier    b0      b1      b2      b3      b4      b5 ...
    //          group 0        R0(0)   M0(0)   R1(0)   M1(0)   R0(1)   M0(1)
    //          group 1        -       R0(0)   M0(0)   R1(0)   M1(0)   R0(1)
    //      (256 x 128, one phase: R(0) M(0) R(1) ..., b(4s) and b(4s+1) only; M0 and M1 below are the same then, and b(4s+4) is the
    //      barrier behind b(4s+1).)
    //      Stage s of a tile is complete in LDS before b(4s): every wave waits for its own copies before that
    //      barrier.  The buffer of stage s is free after b(4s+4): group 1, the last reader, waits for its R1(s)
    //      data before that barrier, so no read of the buffer is in flight when the first copy into it is issued.
    //      The NST buffers are used in turn across tiles as well: stage s of a tile uses buffer (s + par) mod NST, par
    //      being the number of stages of all earlier tiles.
    //      At the end of a tile (S stages): group 0 has issued its share of the next tile's stages 0 .. NST-2 during
    //      M0(S-NST+1) .. M0(S-1) and group 1 during M1(S-NST) .. M1(S-2), each into the buffer that the stage of
    //      the same number past S would use.  After b(4S) group 0
    //      stores its result block through the staging area (which covers the last stage's buffer, free since
    //      b(4S)) while group 1 still issues M1(S-1), then group 1 stores its block; the next tile's b(0) follows.
    //      Group 1's share of the next tile's stage NST-1, which goes into the buffer under the staging area, is
    //      issued after that barrier (where the first tile issues it, too). ----
    constexpr int PH = T::PH, KP = C::KS / PH;         // phases of a stage, k-steps per phase
    constexpr int NQ = (KP + 1) / 2;                   // scale dwords per row and phase
    v8i fa[KP][MB], fb[KP][NB];
    unsigned sa[NQ][MB], sb[NQ][NB];
    auto RD = [&](int slot, int p, int stage) {
        const uint8_t* base = lds + slot * C::STRIDE;
        const uint8_t* ta = base + wm * WTM * C::SBA;
        const uint8_t* tb = base + C::A_BYTES + wn * WTN * C::SBB;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int q = C::NG == 2 ? p * NQ + i : 0;
#pragma unroll
            for (int m = 0; m < MB; ++m) sa[i][m] = *reinterpret_cast<const unsigned*>(base + sca_off + q * TM * 4 + m * 128) >> (8 * g);
#pragma unroll
            for (int n = 0; n < NB; ++n) sb[i][n] = *reinterpret_cast<const unsigned*>(base + scb_off + q * TN * 4 + n * 128) >> (8 * g);
            // scale bytes past the last block are unspecified (a group past the last one was delivered as zeros)
            if (TAIL && (R & 127) != 0 && stage * C::NG + q == ngrp - 1) {
                const unsigned mask = ((1u << (8 * ((R & 127) / kBlock))) - 1u) >> (8 * g);
#pragma unroll
                for (int m = 0; m < MB; ++m) sa[i][m] &= mask;
#pragma unroll
                for (int n = 0; n < NB; ++n) sb[i][n] &= mask;
            }
        }
#pragma unroll
        for (int k = 0; k < KP; ++k) {
#pragma unroll
            for (int m = 0; m < MB; ++m) fa[k][m] = read_frag<FA>(ta, m * 32 * C::SBA, offa, p * KP + k);
#pragma unroll
            for (int n = 0; n < NB; ++n) fb[k][n] = read_frag<FB>(tb, n * 32 * C::SBB, offb, p * KP + k);
        }
    };
    // The MFMAs of phase p.  With COPY the wave's copy instructions of stage `nxt` (of the copy tile) into
    // buffer `nslot` are spread evenly between the phase's NM MFMAs (the sched_barriers keep them there).
    constexpr int NM = KP * MB * NB;
    auto MM = [&](auto copy_tag, int p, int nxt, int nslot, Share to) {
        constexpr bool COPY = decltype(copy_tag)::value != 0, SCALES = decltype(copy_tag)::value == 2;
        constexpr int ca = FB == kFP8 ? 0 : 4, cb = FA == kFP8 ? 0 : 4;
        __builtin_amdgcn_s_setprio(1);
        int idx = 0;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            const int ks = p * KP + k;
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    if ((ks & 1) == 0)
                        acc[m][n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[k][n], fa[k][m], acc[m][n], ca, cb, 0, (int)sb[k / 2][n], 0, (int)sa[k / 2][m]);
                    else
                        acc[m][n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[k][n], fa[k][m], acc[m][n], ca, cb, 2, (int)sb[k / 2][n], 2, (int)sa[k / 2][m]);
                    if (COPY) {
                        __builtin_amdgcn_sched_barrier(0);
                        if (SCALES && idx == 0) issue_scale(nxt, nslot);
#pragma unroll
                        for (int j = 0; j < C::L; ++j)
                            if ((SCALES ? (j + 1) * NM / (C::L + 1) : j * NM / C::L) == idx) issue_one(j, nxt, to);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    ++idx;
                }
        }
        __builtin_amdgcn_s_setprio(0);
    };
    const std::integral_constant<int, 0> no_copy{};
    const std::integral_constant<int, 1> with_copy{};
    const std::integral_constant<int, 2> with_scales{};          // group 0

    // ---- result of tile u: optional sum of squares, then every wave transposes its block through its
    //      own part of the staging area at byte `ebase` of the LDS array ----
    auto store_tile = [&](int u, int ebase) {
        int ti, tj;
        tile_of(u, nblk, tiles_i, tiles_j, ti, tj);
        const int i0 = ti * TM, j0 = tj * TN;
        const bool interior = i0 + TM <= I && j0 + TN <= J;
        // optional: sum of squares of the tile as it will be stored (rounded to the output type), elements
        // outside the matrix excluded; one partial per tile, combined by a second kernel.  Interior tiles take
        // the short path: bf16 pairs are squared and added by v_dot2c_f32_bf16.
        if (norm_partials) {
            __shared__ float wave_ss[NWAVE];
            float ss = 0.f;
            if (interior) {
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int n = 0; n < NB; ++n)
#pragma unroll
                        for (int k = 0; k < 16; k += 2) {
                            if (OUT_F32) {
                                ss = fmaf(acc[m][n][k], acc[m][n][k], ss);
                                ss = fmaf(acc[m][n][k + 1], acc[m][n][k + 1], ss);
                            } else {
                                const float2_t pr = {acc[m][n][k], acc[m][n][k + 1]};
                                const bf16x2 r = __builtin_convertvector(pr, bf16x2);
                                const unsigned rb = __builtin_bit_cast(unsigned, r);
                                asm("v_dot2c_f32_bf16 %0, %1, %1" : "+v"(ss) : "v"(rb));       // ss += r.x * r.x + r.y * r.y
                            }
                        }
            } else {
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const bool row_ok = i0 + wm * WTM + m * 32 + r32 < I;
#pragma unroll
                    for (int n = 0; n < NB; ++n)
#pragma unroll
                        for (int k = 0; k < 16; ++k) {
                            const int col = j0 + wn * WTN + n * 32 + 8 * (k >> 2) + 4 * g + (k & 3);
                            float v = acc[m][n][k];
                            if (!OUT_F32) v = (float)(__bf16)v;
                            ss = (row_ok && col < J) ? fmaf(v, v, ss) : ss;
                        }
                }
            }
            ss = wave_sum(ss);
            if (lane == 0) wave_ss[wave] = ss;
            __syncthreads();
            if (threadIdx.x == 0) {
                float t = 0.f;
                for (int w = 0; w < NWAVE; ++w) t += wave_ss[w];
                norm_partials[u] = t;
            }
        }
        // In registers, lane (r32, g) of block (m, n) holds C[32m + r32][32n + 8q + 4g + t] in acc[m][n][4q + t].
        // In LDS a row is ROWB bytes of 16-byte chunks, chunk c of row r stored at position c ^ f(r).
        constexpr int ESZ = OUT_F32 ? 4 : 2;
        constexpr int REGION = C::EPI_BYTES / NWAVE;     // LDS bytes a wave may use
        constexpr int NBP = 32 * WTN * ESZ <= REGION ? NB : 1;         // column blocks of a pass
        constexpr int ROWB = NBP * 32 * ESZ;             // 128 or 256 bytes per row
        constexpr int CPR = ROWB / 16;                   // 8 or 16 chunks per row
        constexpr int ROWS_PER_PASS = REGION / ROWB < WTM ? REGION / ROWB : WTM;
        constexpr int MB_PER_PASS = ROWS_PER_PASS / 32;
        static_assert(MB_PER_PASS >= 1 && MB % MB_PER_PASS == 0 && NB % NBP == 0 && (CPR == 8 || CPR == 16), "staging passes must be whole 32-row blocks");
        auto spread = [](int row) { return CPR == 16 ? row & 15 : (row >> 1) & 7; };
        uint8_t* reg = lds + ebase + wave * REGION;
#pragma unroll
        for (int pass = 0; pass < MB / MB_PER_PASS * (NB / NBP); ++pass) {
            const int pm = pass / (NB / NBP), pn = pass % (NB / NBP) * NBP;          // row pass, first column block
#pragma unroll
            for (int mm = 0; mm < MB_PER_PASS; ++mm) {
                const int m = pm * MB_PER_PASS + mm;
                const int row = mm * 32 + r32;
                const int f = spread(row);
#pragma unroll
                for (int nn = 0; nn < NBP; ++nn)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int n = pn + nn;
                        const float v0 = acc[m][n][4 * q + 0], v1 = acc[m][n][4 * q + 1];
                        const float v2 = acc[m][n][4 * q + 2], v3 = acc[m][n][4 * q + 3];
                        if (OUT_F32) {
                            const int c = nn * 8 + q * 2 + g;            // 4 floats = one chunk
                            *reinterpret_cast<float4*>(reg + row * ROWB + ((c ^ f) * 16)) = make_float4(v0, v1, v2, v3);
                        } else {
                            const int c = nn * 4 + q;                    // 4 bf16 = half a chunk
                            const float2_t lo = {v0, v1}, hi = {v2, v3};
                            const bf16x2 blo = __builtin_convertvector(lo, bf16x2), bhi = __builtin_convertvector(hi, bf16x2);
                            *reinterpret_cast<uint2*>(reg + row * ROWB + ((c ^ f) * 16) + 8 * g) =
                                make_uint2(__builtin_bit_cast(unsigned, blo), __builtin_bit_cast(unsigned, bhi));
                        }
                    }
            }
            // read back row-contiguous: 64 lanes cover 64 / CPR rows per instruction (stores: store16)
            constexpr int RPI = 64 / CPR;
            if (interior) {
                // whole tile inside the matrix (wave-uniform): no per-lane tests, one wave-uniform base per
                // instruction plus a 32-bit lane offset
                const unsigned lane_off = (unsigned)((lane / CPR) * (int)ldc * ESZ + (lane % CPR) * 16);
                const uint8_t* cb = reinterpret_cast<const uint8_t*>(c_out) +
                                    ((int64_t)(i0 + wm * WTM + pm * ROWS_PER_PASS) * ldc + j0 + wn * WTN + pn * 32) * ESZ;
#pragma unroll
                for (int it = 0; it < ROWS_PER_PASS / RPI; ++it) {
                    const int row = it * RPI + lane / CPR;
                    const int c = lane % CPR;
                    const int f = spread(row);
                    const v4u v = *reinterpret_cast<const v4u*>(reg + row * ROWB + ((c ^ f) * 16));
                    store16(v, const_cast<uint8_t*>(cb) + (int64_t)(it * RPI) * ldc * ESZ + lane_off, STREAM);
                }
            } else {
                for (int it = 0; it < ROWS_PER_PASS / RPI; ++it) {
                    const int row = it * RPI + lane / CPR;
                    const int c = lane % CPR;
                    const int f = spread(row);
                    const uint4 v = *reinterpret_cast<const uint4*>(reg + row * ROWB + ((c ^ f) * 16));
                    const int i = i0 + wm * WTM + pm * ROWS_PER_PASS + row;
                    const int j = j0 + wn * WTN + pn * 32 + c * (16 / ESZ);
                    if (i < I) {
                        uint8_t* p = reinterpret_cast<uint8_t*>(c_out) + ((int64_t)i * ldc + j) * ESZ;
                        if (j + 16 / ESZ <= J) {
                            store16(v4u{v.x, v.y, v.z, v.w}, p, STREAM);
                        // (lanes past the last column would walk through the tests below: 1 us of a tile with two passes; cached
                        // operands, [7936 x 544 x 640] FP8 10.3 -> 8.9 us, [416 x 9440 x 1152] 12.0 -> 10.7)
                        } else if (j < J) {
                            const unsigned w[4] = {v.x, v.y, v.z, v.w};
                            for (int e = 0; e < 16 / ESZ; ++e)
                                if (j + e < J) {
                                    if (OUT_F32) reinterpret_cast<unsigned*>(p)[e] = w[e];
                                    else reinterpret_cast<uint16_t*>(p)[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                                }
                        }
                    }
                }
            }
        }
    };

    constexpr int NST = C::NST;
    auto after = [](int slot) { return slot == NST - 1 ? 0 : slot + 1; };
    auto before = [](int slot) { return slot == 0 ? NST - 1 : slot - 1; };
    int u = blockIdx.x;                  // dispatch id of the tile being multiplied
    int par = 0;                         // buffer of its stage 0
    bool first = true;
    set_copy_tile(u);
#pragma unroll
    for (int k = 0; k < NST - 1; ++k) {
        if (wave < NWAVE / 2) issue_scale(k, k);
        issue(k, k);
    }
    for (;;) {
        const int un = u + (int)gridDim.x;
        const bool has_next = un < nblk;
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int k = 0; k < 16; ++k) acc[a][b][k] = 0.f;
        // Buffer of stage s.  With two buffers it follows from s; this and what comes of it below keeps the forms that two buffers
        // need, without those for more: fewer scalar instructions in a stage.  256 x 256 is 0.6 % faster so from memory (18 shapes,
        // all formats) and 1.8 % on operands in the caches ([3072 x 3072 x 8192] FP8 75.6 -> 73.0 us).
        int ring = par;
        auto slot_of = [&](int s) { return NST == 2 ? (s + par) & 1 : ring; };
        const int ebase2 = NST == 2 ? C::epi_base((nstage - 1 + par) & 1) : 0;
        if (wave < NWAVE / 2) {
            // group 0 issues its copies of stage s + NST - 1 during M0(s), between b(4s+1) and b(4s+2); during the last
            // NST - 1 stages these are the copies of the next tile's first stages
            auto stage0 = [&](auto copy_tag, int s, int cstage) {
                const int slot = slot_of(s);
                // the first NST - 1 stages of a later tile were waited for before the previous tile's result was stored;
                // waiting for them here again would wait for those stores
                if (first || s >= NST - 1) SNIP_WAIT_VM((NST - 2) * (C::L + 1));
                SNIP_BAR();                                         // b(4s)
                const int to = NST == 2 ? slot ^ 1 : before(slot);
                const Share at = share(to);
                RD(slot, 0, s); SNIP_BAR();      // b(4s+1)
                MM(copy_tag, 0, cstage, to, at);
                if (PH == 2) {
                    SNIP_BAR();                                     // b(4s+2)
                    RD(slot, 1, s); SNIP_BAR();  // b(4s+3)
                    MM(no_copy, 1, 0, 0, Share());
                }
            };
            // Every stage carries copies, so that the MFMA code exists once (two variants of it merging in front
            // of the result store cost the register allocator its in-place accumulators).  Without a next tile the
            // last stages' copies go into free buffers, where nobody reads them (copy_nothing).
            for (int s = 0; s < nstage; ++s) {
                const int c = s + NST - 1;
                const bool past = NST == 2 ? s == nstage - 1 : c >= nstage;
                const int cs = past ? (NST == 2 ? 0 : c - nstage) : c;
                if constexpr (QUIET) {
                    if (NST == 2 ? past : c == nstage) {
                        if (has_next) set_copy_tile(un); else copy_nothing();
                    }
                } else if ((NST == 2 ? past : c == nstage) && has_next) {
                    set_copy_tile(un);
                }
                cut_tail(cs);
                stage0(with_scales, s, cs);
                if (NST > 2) ring = after(ring);
            }
            SNIP_BAR();                                             // b(4S)
            SNIP_WAIT_VM(0);                                        // own shares of the next tile's first stages
        } else {
            // group 1 issues its copies of stage s + NST during M1(s), between b(4s+4) and b(4s+5) (during M1(S-NST) and
            // later those of the next tile's first stages, during M1(S-1) none); those of stage NST - 1 while it idles
            // through the tile's first phase
            auto stage1 = [&](auto copy_tag, int s, int cstage) {
                const int slot = slot_of(s);
                SNIP_BAR();                                         // b(4s+1)
                if (PH == 2) {
                    RD(slot, 0, s);
                    SNIP_BAR();                  // b(4s+2)
                    MM(no_copy, 0, 0, 0, Share()); SNIP_BAR();      // b(4s+3)
                }
                const Share at = decltype(copy_tag)::value ? share(slot) : Share();
                RD(slot, PH - 1, s);
                if (NST == 2) {
                    __builtin_amdgcn_s_waitcnt(0x0070);             // vmcnt(0) and lgkmcnt(0)
                } else {
                    if (first || s >= NST - 2) SNIP_WAIT_VM((NST - 2) * C::L);              // stage s + 1 (see stage0)
                    __builtin_amdgcn_s_waitcnt(0xC07F);             // lgkmcnt(0)
                }
                SNIP_BAR();                                         // b(4s+4)
                MM(copy_tag, PH - 1, cstage, slot, at);
            };
            if (first) SNIP_WAIT_VM((NST - 2) * C::L);
            SNIP_BAR();                                             // b(0)
            cut_tail(NST - 1);
            issue(NST - 1, NST == 2 ? (1 + par) & 1 : before(par));
            // (without a next tile the last copies go into free buffers)
            for (int s = 0; s < nstage - 1; ++s) {
                const int c = s + NST;
                const bool past = NST == 2 ? s == nstage - 2 : c >= nstage;
                const int cs = past ? (NST == 2 ? 0 : c - nstage) : c;
                if constexpr (QUIET) {
                    if (NST == 2 ? past : c == nstage) {
                        if (has_next) set_copy_tile(un); else copy_nothing();
                    }
                } else if ((NST == 2 ? past : c == nstage) && has_next) {
                    set_copy_tile(un);
                }
                cut_tail(cs);
                stage1(with_copy, s, cs);
                if (NST > 2) ring = after(ring);
            }
            stage1(no_copy, nstage - 1, 0);
            if (NST > 2) ring = after(ring);
            if (NST > 2) SNIP_WAIT_VM(0);                           // (nothing may land in LDS after the workgroup's end either)
        }
        store_tile(u, NST == 2 ? ebase2 : C::epi_base(before(ring)));
        if (!has_next) break;
        u = un;
        par = NST == 2 ? (par + nstage) & 1 : ring;
        first = false;
    }
}

template <int FA, int FB, bool OUT_F32, class T, bool TAIL>
hipError_t launch_fast_t(const GemmArgs& a, hipStream_t s)
{
    const int ti = (int)((a.I + T::TM - 1) / T::TM), tj = (int)((a.J + T::TN - 1) / T::TN);
    // one workgroup per compute unit (the LDS array admits no second one), each walking its share of the tiles
    const int ncu = gemm_compute_units();
    const dim3 grid((unsigned)(ti * tj < ncu ? ti * tj : ncu)), block(NT);
    auto* const kernel = gemm_streams(a) ? gemm_fast_kernel<FA, FB, OUT_F32, T, TAIL, true> : gemm_fast_kernel<FA, FB, OUT_F32, T, TAIL, false>;
    hipLaunchKernelGGL(kernel, grid, block, 0, s, a.a_codes, a.a_scales_g4, a.b_codes, a.b_scales_g4,
                       (int)a.I, (int)a.J, (int)a.R, a.c, a.ldc, ti, tj, a.norm_partials);
    return hipGetLastError();
}
template <int FA, int FB, class T>
hipError_t launch_fast_f(const GemmArgs& a, hipStream_t s)
{
    if (a.R % FCfg<FA, FB, T>::KE == 0) return a.out_fp32 ? launch_fast_t<FA, FB, true, T, false>(a, s) : launch_fast_t<FA, FB, false, T, false>(a, s);
    return a.out_fp32 ? launch_fast_t<FA, FB, true, T, true>(a, s) : launch_fast_t<FA, FB, false, T, true>(a, s);
}

template <class T>
hipError_t launch_fast_tile(const GemmArgs& a, hipStream_t s)
{
    if (a.fmt_a == kFP8 && a.fmt_b == kFP8) return launch_fast_f<kFP8, kFP8, T>(a, s);
    if (a.fmt_a == kFP8 && a.fmt_b == kFP4) return launch_fast_f<kFP8, kFP4, T>(a, s);
    if (a.fmt_a == kFP4 && a.fmt_b == kFP8) return launch_fast_f<kFP4, kFP8, T>(a, s);
    return launch_fast_f<kFP4, kFP4, T>(a, s);
}

}  // namespace

static int stage_extent(const GemmArgs& a) { return a.fmt_a == kFP4 && a.fmt_b == kFP4 ? 256 : 128; }

bool gemm_fast_eligible(const GemmArgs& a)
{
    const int ke = stage_extent(a);
    // 32-bit source offsets: 256 rows of codes and, where the last stage is not whole, a grouped scale copy within a descriptor
    if (a.R > (1 << 22)) return false;
    const int64_t groups = (a.R + 127) / 128, most = std::max(g4_pitch(a.I), g4_pitch(a.J)) * 4 * groups;
    if (a.R % ke != 0 && !descriptor_covers(most)) return false;
    return a.a_scales_g4 && a.b_scales_g4 && a.R > ke && a.I > 128 && a.J > 128;      // at least two stages
}

hipError_t launch_gemm_fast(const GemmArgs& a, GemmTile tile, hipStream_t s)
{
    if (tile == GemmTile::kBig) return launch_fast_tile<TileBig>(a, s);
    const int64_t ke = stage_extent(a);
    return a.R > 2 * ke && a.R != 3 * ke ? launch_fast_tile<TileWide>(a, s) : launch_fast_tile<TileShort>(a, s);
}

}  // namespace snip

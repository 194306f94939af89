// GEMM on operands quantized with the paper's own recipe (see gemm_paper.hip: what is computed, and the arithmetic), for
// outputs with enough tiles of 256 x 128.  The results agree bit for bit with gemm_paper.hip: same products, same factors,
// folded slab by slab in the same order.
//
//   What bounds the 128 x 128 tile of gemm_paper.hip is its copies (32 KB per 4.2 MFLOP) and one compute wave per SIMD, whose
//   LDS latencies and barrier nothing covers.  Here eight waves of 64 x 64 (4 x 2) share a tile of 256 x 128 (24 KB per 4.2
//   MFLOP) and alternate, as in gemm_fast.hip: of the two waves of a SIMD one reads its operands of a stage from LDS while the
//   other issues its MFMAs and folds the products of the blocks before, one phase apart, workgroup barriers between:
//       b(4s)    group 0 (waves 0-3) R(s)    group 1 M(s - 1)
//       b(4s+1)  group 0 M(s)                group 1 R(s)             b(4s+4) follows
//   Three stage buffers of 128 code bytes per row.  In R(s) a wave issues its global->LDS copies of stage s + 2 behind its operand
//   reads, into the buffer of stage s - 1: that was read last in group 1's R(s - 1), which waits for its reads before b(4s).  (Here
//   the MFMA phase is full of vector instructions: with the copies between the MFMAs, as in gemm_fast.hip, FP4 with B in blocks took
//   3-7 % longer, FP8 the same.)  Stage s + 1 has landed at b(4s+4): group 0 waits in front of that barrier for all but its copies
//   of stage s + 2, group 1 behind its own issue of them.
//   The fold takes 16 (B in 128 x 128 blocks: one factor per lane and slab) or 32 (a factor per column) vector instructions
//   per 32 x 32 block beside 2 x 64 (FP8) or 2 x 32 (FP4) cycles of MFMA; an instruction takes 4.3 cycles and an MFMA blocks
//   their issue for about 20, so that with a factor per column the vector instructions are what bounds it.
//   Scales: the waves of group 0 copy those of four slabs (a "chunk": two or four stages) at a time, a row's four adjacent
//   ones with one 16-byte copy.  A row's reciprocal is formed by one lane of each wave that needs it while its operands are on
//   their way; the reciprocals of B's columns, 32 per lane and slab, come from LDS, where group 0 leaves them a stage ahead.
//   (All reciprocals through LDS, by group 0: a chain of read, division, write and wait in front of a barrier, 10 % of the
//   kernel.)
// us per call against the 128 x 128 tile, A in tiles, B in blocks / in tiles: [4096 x 2048 x 8192] FP8 89.0 -> 73.9 / 100 -> 89, FP4
// 58.3 -> 47.6 / 74 -> 66; [4096 x 8192 x 2048] FP8 98.5 -> 81.9, FP4 65.8 -> 52.9; [8192 x 2048 x 4096] in tiles FP8 103 -> 93, FP4 78.0
// -> 68.7; [8192 x 8192 x 8192] in tiles FP8 790 -> 685.  The plain GEMM with this tile takes 66 (FP8) and 38 us for [4096 x 2048 x 8192].
#include "gemm_common.h"
#include <type_traits>

namespace snip {
namespace {

constexpr int TM = 256, TN = 128, WTM = 64, WTN = 64, MB = 2, NB = 2;
constexpr int NWAVE = 8, NT = NWAVE * 64, NST = 3;
constexpr int kSlab = 128;                                      // contraction elements of a scaling group
constexpr int kChunk = 4;                                       // slabs whose scales are fetched together
constexpr unsigned kUnitScale = 0x7F7F7F7Fu;                    // E8M0 127 = 2^0 in every byte

template <int FA, int FB> struct WideCfg {
    static constexpr int NG = FA == kFP4 && FB == kFP4 ? 2 : 1;          // slabs per stage
    static constexpr int KE = NG * kSlab, KS = KE / 64;
    static constexpr int SBA = FA == kFP8 ? KE : KE / 2, SBB = FB == kFP8 ? KE : KE / 2;
    static constexpr int A_BYTES = TM * SBA, B_BYTES = TN * SBB, SLOT = A_BYTES + B_BYTES;
    static constexpr int LA = A_BYTES / 1024 / NWAVE, LB = B_BYTES / 1024 / NWAVE, L = LA + LB;      // 1 KB copies per wave and stage
    static constexpr int SPC = kChunk / NG;                               // stages per chunk
    // Scales of a chunk as they are copied, in blocks of 1 KB ([64 rows][slab] if 16 bytes at a time, else [slab][64 rows]): two
    // buffers of A's four; B's four of 32 rows each (the lanes' second half repeats the first) or, in 128 x 128 blocks, one.
    // Without blocks two buffers of B's reciprocals, [slab][128 rows].
    static constexpr int SCL = 64 * kChunk * 4, OFF_SA = NST * SLOT, OFF_SB = OFF_SA + 2 * 4 * SCL;
    static constexpr int OFF_F = OFF_SB + 4 * SCL, FBUF = kChunk * TN * 4, LDS_BYTES = OFF_F + 2 * FBUF;
    static constexpr int EPI = 4096;                                      // result staging per wave, in the last stage's buffer
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
    static_assert(NWAVE * EPI <= SLOT, "the result staging area must stay clear of the other stage buffers");
    static_assert(SPC >= 2, "a chunk's scales are turned into factors a stage after they were requested, at the earliest");
};

template <int FA, int FB, bool OUT_F32, bool B_BLOCK>
__global__ __launch_bounds__(NT) void gemm_paper_wide_kernel(const uint8_t* __restrict__ a_codes, const float* __restrict__ a_scales, int a_shift,
                                                             const uint8_t* __restrict__ b_codes, const float* __restrict__ b_scales,
                                                             int I, int J, int R, void* __restrict__ c_out, int64_t ldc, int tiles_i, int tiles_j, int stream_out)
{
    using C = WideCfg<FA, FB>;
    constexpr int NG = C::NG, KS = C::KS, SPC = C::SPC;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[C::LDS_BYTES];

    const int nblk = tiles_i * tiles_j;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int r32 = lane & 31, g = lane >> 5;
    const int64_t a_row_bytes = FA == kFP8 ? R : R / 2, b_row_bytes = FB == kFP8 ? R : R / 2;
    const int nslab = R / kSlab, nstage = (nslab + NG - 1) / NG;         // nstage >= NST (the launcher)
    const unsigned lds0 = lds_addr(lds);

    // ---- code copies of the tile they currently belong to.  Rows past the end of an operand read its last row again (their
    // products are never stored).
    unsigned oa[C::LA], ob[C::LB];
    const uint8_t *abase, *bbase;
    auto chunk_a = [&](int j) { constexpr int CPR = C::SBA / 16, RPI = 1024 / C::SBA; return (lane % CPR) ^ swz<C::SBA>((wave * C::LA + j) * RPI + lane / CPR); };
    auto chunk_b = [&](int j) { constexpr int CPR = C::SBB / 16, RPI = 1024 / C::SBB; return (lane % CPR) ^ swz<C::SBB>((wave * C::LB + j) * RPI + lane / CPR); };
    auto set_copy_tile = [&](int i0, int j0) {
#pragma unroll
        for (int j = 0; j < C::LA; ++j) {
            constexpr int CPR = C::SBA / 16, RPI = 1024 / C::SBA;
            oa[j] = (unsigned)(min((wave * C::LA + j) * RPI + lane / CPR, I - 1 - i0) * a_row_bytes + chunk_a(j) * 16);
        }
#pragma unroll
        for (int j = 0; j < C::LB; ++j) {
            constexpr int CPR = C::SBB / 16, RPI = 1024 / C::SBB;
            ob[j] = (unsigned)(min((wave * C::LB + j) * RPI + lane / CPR, J - 1 - j0) * b_row_bytes + chunk_b(j) * 16);
        }
        abase = a_codes + (int64_t)i0 * a_row_bytes;
        bbase = b_codes + (int64_t)j0 * b_row_bytes;
    };
    // FP4 x FP4, odd number of slabs: the last stage's second half repeats its first (its factors are zero).  Once per tile, before
    // the copies of its last stage.
    auto cut_tail = [&](int stage) {
        if (NG == 1 || (nslab & 1) == 0 || stage != nstage - 1) return;
#pragma unroll
        for (int j = 0; j < C::LA; ++j) oa[j] -= chunk_a(j) >= 4 ? 64 : 0;
#pragma unroll
        for (int j = 0; j < C::LB; ++j) ob[j] -= chunk_b(j) >= 4 ? 64 : 0;
    };
    auto issue_one = [&](int j, int stage, int slot) {
        const unsigned base = lds0 + slot * C::SLOT;
        if (j < C::LA) glds16(abase + (int64_t)stage * C::SBA, oa[j], base + (wave * C::LA + j) * 1024);
        else glds16(bbase + (int64_t)stage * C::SBB, ob[j - C::LA], base + C::A_BYTES + (wave * C::LB + j - C::LA) * 1024);
    };
    auto issue = [&](int stage, int slot) {
#pragma unroll
        for (int j = 0; j < C::L; ++j) issue_one(j, stage, slot);
    };

    // ---- scales, copied by the waves of group 0
    const bool vec = (nslab & 3) == 0 && (((uintptr_t)a_scales | (uintptr_t)b_scales) & 15) == 0;
    auto issue_scales = [&](int i0, int j0, int chunk, int buf) {
        auto copy = [&](const float* first_row, int row, unsigned d) {
            const uint8_t* p = reinterpret_cast<const uint8_t*>(first_row + chunk * kChunk);
            const unsigned off = (unsigned)(row * nslab * 4);
            if (vec) {
                glds16(p, off, d);
            } else {
#pragma unroll
                for (int k = 0; k < kChunk; ++k) glds4(p + min(k, nslab - 1 - chunk * kChunk) * 4, off, d + k * 256);
            }
        };
        copy(a_scales + (int64_t)(i0 >> a_shift) * nslab, min(wave * 64 + lane, I - 1 - i0) >> a_shift, lds0 + C::OFF_SA + (buf * 4 + wave) * C::SCL);
        if (!B_BLOCK) copy(b_scales + (int64_t)j0 * nslab, min(wave * 32 + lane % 32, J - 1 - j0), lds0 + C::OFF_SB + wave * C::SCL);
        else if (wave == 0) copy(b_scales + (int64_t)(j0 >> 7) * nslab, 0, lds0 + C::OFF_SB + buf * C::SCL);
    };
    // offset of (row of a block, slab of a chunk) among copied scales
    auto scale_at = [&](int row, int slab) { return vec ? row * 16 + slab * 4 : slab * 256 + row * 4; };
    // B's scales that this wave copied -> reciprocals, two slabs per lane
    auto convert = [&](int buf) __attribute__((always_inline)) {
        if (B_BLOCK) return;
        const int k0 = lane / 32 * 2, r = lane % 32;
        const uint8_t* p = lds + C::OFF_SB + wave * C::SCL;
        float v[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) v[k] = *reinterpret_cast<const float*>(p + scale_at(r, k0 + k));
#pragma unroll
        for (int k = 0; k < 2; ++k) *reinterpret_cast<float*>(lds + C::OFF_F + buf * C::FBUF + ((k0 + k) * TN + wave * 32 + r) * 4) = __fdiv_rn(1.f, v[k]);
        __builtin_amdgcn_s_waitcnt(0xC07F);                     // lgkmcnt(0)
    };

    // ---- operands of a stage
    constexpr int NCA = FA == kFP8 ? 2 * KS : KS, NCB = FB == kFP8 ? 2 * KS : KS;
    int offa[NCA], offb[NCB];
    frag_offsets<FA, C::SBA, KS>(r32, g, offa);
    frag_offsets<FB, C::SBB, KS>(r32, g, offb);
    v8i fa[KS][MB], fb[KS][NB];
    float da[NG][MB], db[NG];                                    // factors: A's rows; B's block
    const uint8_t* facs = lds + C::OFF_F + wn * WTN * 4;         // B's factors of the current stage's first slab
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 1> c1{};
    float cols[NB][16];                                          // factors of the columns of block n, of one slab
    auto read_cols = [&](auto n_, int q) __attribute__((always_inline)) {
        constexpr int n = n_;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 v = *reinterpret_cast<const float4*>(facs + (q * TN + n * 32 + 8 * k + 4 * g) * 4);
            cols[n][4 * k] = v.x; cols[n][4 * k + 1] = v.y; cols[n][4 * k + 2] = v.z; cols[n][4 * k + 3] = v.w;
        }
    };
    auto RD = [&](int slot, int s, int buf, int nxt, int nslot) __attribute__((always_inline)) {
        const int k0 = s % SPC * NG;                             // first slab in the chunk
        const uint8_t* sa = lds + C::OFF_SA + (buf * 4 + wm) * C::SCL;
        facs = lds + C::OFF_F + buf * C::FBUF + (k0 * TN + wn * WTN) * 4;
        float ra[NG], rb;                                        // a lane fetches one row's scale of A and one slab's of a block of B
#pragma unroll
        for (int q = 0; q < NG; ++q) ra[q] = *reinterpret_cast<const float*>(sa + scale_at(lane, k0 + q));
        if (B_BLOCK) rb = *reinterpret_cast<const float*>(lds + C::OFF_SB + buf * C::SCL + scale_at(0, k0 + (NG == 2 ? g : 0)));
        __builtin_amdgcn_sched_barrier(0);
        const uint8_t* ta = lds + slot * C::SLOT + wm * WTM * C::SBA;
        const uint8_t* tb = lds + slot * C::SLOT + C::A_BYTES + wn * WTN * C::SBB;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
#pragma unroll
            for (int n = 0; n < NB; ++n) fb[k][n] = read_frag<FB>(tb, n * 32 * C::SBB, offb, k);
#pragma unroll
            for (int m = 0; m < MB; ++m) fa[k][m] = read_frag<FA>(ta, m * 32 * C::SBA, offa, k);
        }
        __builtin_amdgcn_sched_barrier(0);
        issue(nxt, nslot);
        if (!B_BLOCK) read_cols(c0, 0);
        // The scales were read first: their reciprocals while the operands are on their way, each row's by one lane; the halves of
        // the wave then exchange theirs.  (A slab past the last one: zeros.)
        auto halves = [](float v, float& lo, float& hi) {        // lo: the value of lane r32 in lanes r32 and 32 + r32, hi: of lane 32 + r32
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
            lo = __uint_as_float(r[0]);
            hi = __uint_as_float(r[1]);
        };
#pragma unroll
        for (int q = 0; q < NG; ++q)
            halves(NG == 2 && s * NG + q >= nslab ? 0.f : __fdiv_rn(1.f, ra[q]), da[q][0], da[q][1]);
        if (B_BLOCK) {
            rb = NG == 2 && s * NG + g >= nslab ? 0.f : __fdiv_rn(1.f, rb);
            if constexpr (NG == 2) halves(rb, db[0], db[1]);
            else db[0] = rb;
        }
    };

    // ---- products and fold.  The products of what was worked on last wait in `pend` until the next MFMAs are under way (those of
    // the end of a stage: of the next stage), pend_a: the factors of their rows (B_BLOCK: their whole factor).
    // B_BLOCK: pairs of blocks, (0, n) and (1, n) of a slab: four MFMAs, behind each of them half a block of the pair before is
    // folded, 8 vector instructions.  (Behind the two MFMAs of one block the products of the block just before would not be
    // ready: up to 16 idle cycles.)  Else one block, two MFMAs, 16 instructions behind each; a pair more of products would not
    // fit the registers.
    v16f acc[MB][NB], pend[NB][MB];
    float pend_a[MB];
    constexpr int ca = FB == kFP8 ? 0 : 4, cb = FA == kFP8 ? 0 : 4;              // first operand = B tile
    auto pair = [&](auto q_, auto n_) __attribute__((always_inline)) {
        constexpr int q = q_, n = n_;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ks = i >> 1, m = i & 1;
            if (ks == 0)
#pragma unroll
                for (int k = 0; k < 16; ++k) pend[n][m][k] = 0.f;
            pend[n][m] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[2 * q + ks][n], fa[2 * q + ks][m], pend[n][m], ca, cb, 0, (int)kUnitScale, 0, (int)kUnitScale);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 8 * (i & 1); k < 8 * (i & 1) + 8; ++k)
                acc[i >> 1][1 - n][k] = fmaf(pend[1 - n][i >> 1][k], pend_a[i >> 1], acc[i >> 1][1 - n][k]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < MB; ++m) pend_a[m] = __fmul_rn(da[q][m], db[q]);
    };
    auto fold_block = [&](auto m_, auto n_, int k0, int k1) __attribute__((always_inline)) {
        constexpr int m = m_, n = n_;
#pragma unroll
        for (int k = k0; k < k1; ++k) acc[m][n][k] = fmaf(pend[0][0][k], __fmul_rn(pend_a[0], cols[n][k]), acc[m][n][k]);
    };
    auto block = [&](auto q_, auto n_, auto m_) __attribute__((always_inline)) {
        constexpr int q = q_, n = n_, m = m_;
        v16f t;
#pragma unroll
        for (int k = 0; k < 16; ++k) t[k] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            t = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[2 * q + ks][n], fa[2 * q + ks][m], t, ca, cb, 0, (int)kUnitScale, 0, (int)kUnitScale);
            __builtin_amdgcn_sched_barrier(0);
            fold_block(std::integral_constant<int, 1 - m>{}, std::integral_constant<int, m == 0 ? 1 - n : n>{}, 8 * ks, 8 * ks + 8);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the columns of 1 - n are done with this slab (n == 0: with the slab before)
        if constexpr (m == 0 && n == 0) read_cols(c1, q);
        if constexpr (m == 0 && n == 1 && q + 1 < NG) read_cols(c0, q + 1);
        __builtin_amdgcn_sched_barrier(0);
        pend[0][0] = t;
        pend_a[0] = da[q][m];
    };
    auto slab = [&](auto q) __attribute__((always_inline)) {
        if constexpr (B_BLOCK) {
            pair(q, c0);
            pair(q, c1);
        } else {
            block(q, c0, c0);
            block(q, c0, c1);
            block(q, c1, c0);
            block(q, c1, c1);
        }
    };
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < MB; ++m) {
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int k = 0; k < 16; ++k) acc[m][n][k] = 0.f;
            // nothing is pending: the tile's first fold adds 0 * 0.  (The factors too: the last tile's may be NaN.)
#pragma unroll
            for (int k = 0; k < 16; ++k) pend[B_BLOCK ? 1 : 0][B_BLOCK ? m : 0][k] = 0.f;
            pend_a[m] = 0.f;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) cols[1][k] = 0.f;
    };
    auto fold_rest = [&]() __attribute__((always_inline)) {
        if constexpr (B_BLOCK) {
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int k = 0; k < 16; ++k) acc[m][1][k] = fmaf(pend[1][m][k], pend_a[m], acc[m][1][k]);
        } else {
            fold_block(c1, c1, 0, 16);
        }
    };
    // The MFMAs of a stage and, between them, the fold.
    auto MM = [&]() __attribute__((always_inline)) {
        if (!B_BLOCK) __builtin_amdgcn_s_setprio(1);             // (with a block's single factor it slows the other wave's divisions down: FP4 50.1 -> 54.8 us)
        slab(c0);
        if constexpr (NG == 2) slab(c1);
        if (!B_BLOCK) __builtin_amdgcn_s_setprio(0);
    };

    // ---- result of a tile, staged in the last stage's buffer
    auto store_tile = [&](int ti0, int tj0, int slot) __attribute__((always_inline)) {
        uint8_t* const reg = lds + slot * C::SLOT + wave * C::EPI;
        const int ti = ti0 + wm * WTM, tj = tj0 + wn * WTN;
        const bool interior = ti0 + TM <= I && tj0 + TN <= J;
        if (stream_out) store_block64<OUT_F32, true>(acc, reg, lane, c_out, ldc, ti, tj, I, J, interior);
        else store_block64<OUT_F32, false>(acc, reg, lane, c_out, ldc, ti, tj, I, J, interior);
    };

    auto after = [](int slot) { return slot == NST - 1 ? 0 : slot + 1; };
    auto before = [](int slot) { return slot == 0 ? NST - 1 : slot - 1; };
    int u = blockIdx.x;                  // dispatch id of the tile being multiplied
    int ti, tj;
    tile_of(u, nblk, tiles_i, tiles_j, ti, tj);
    int i0 = ti * TM, j0 = tj * TN;
    int ring = 0, cbuf = 0;              // buffers of the current stage and chunk
    bool first = true;
    set_copy_tile(i0, j0);
    if (wave < NWAVE / 2) issue_scales(i0, j0, 0, 0);
#pragma unroll
    for (int k = 0; k < NST - 1; ++k) issue(k, k);
    if (wave < NWAVE / 2) {
        SNIP_WAIT_VM((NST - 1) * C::L);
        convert(0);
    }
    for (;;) {
        const int un = u + (int)gridDim.x;
        const bool has_next = un < nblk;
        // without a next tile the copies past the last stage re-fetch what this tile began with into free buffers
        int ni0 = i0, nj0 = j0;
        if (has_next) {
            tile_of(un, nblk, tiles_i, tiles_j, ti, tj);
            ni0 = ti * TM;
            nj0 = tj * TN;
        }
        clear();
        if (wave < NWAVE / 2) {
            // group 0 issues its code copies of stage s + 2 in R(s), and the scale copies of the next chunk (or of the next tile's
            // first one) in front of M(s) of a chunk's first stage s.  These are its newest copies at the wait of stage s + 1, which
            // may leave them in flight; that of stage s + 2 (the first that can read them), the one before `convert` and the one
            // behind the last stage do not.
            for (int s = 0; s < nstage; ++s) {
                const int c = s + NST - 1, cs = c >= nstage ? c - nstage : c;
                const int in_chunk = s & (SPC - 1);
                if (c == nstage && has_next) set_copy_tile(ni0, nj0);
                cut_tail(cs);
                // (the first two stages of a later tile were waited for before the previous tile's result was stored)
                if (first || s >= NST - 1) SNIP_WAIT_VM(C::L);
                SNIP_BAR();                                         // b(4s)
                RD(ring, s, cbuf, cs, before(ring));
                if (!B_BLOCK && in_chunk == SPC - 1 && s != nstage - 1) {
                    SNIP_WAIT_VM(C::L);
                    convert(cbuf ^ 1);
                }
                SNIP_BAR();                                         // b(4s+1)
                if (in_chunk == 0) {
                    const bool same = s + SPC < nstage;
                    issue_scales(same ? i0 : ni0, same ? j0 : nj0, same ? s / SPC + 1 : 0, cbuf ^ 1);
                }
                MM();
                ring = after(ring);
                if (in_chunk == SPC - 1 || s == nstage - 1) cbuf ^= 1;
            }
            SNIP_BAR();                                             // b(4S)
            SNIP_WAIT_VM(0);                                        // own shares of the next tile's first stages and scales
            convert(cbuf);
        } else {
            // group 1 issues its copies of stage s + 2 in R(s), a phase after group 0, and none in the tile's first phase
            auto stage1 = [&](int s, int cstage) {
                SNIP_BAR();                                         // b(4s+1)
                RD(ring, s, cbuf, cstage, before(ring));
                if (first || s >= NST - 2) SNIP_WAIT_VM(C::L);      // stage s + 1 (as above)
                __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0)
                SNIP_BAR();                                         // b(4s+4)
                MM();
                ring = after(ring);
                if ((s & (SPC - 1)) == SPC - 1 || s == nstage - 1) cbuf ^= 1;
            };
            if (first) SNIP_WAIT_VM(C::L);
            SNIP_BAR();                                             // b(0)
            for (int s = 0; s < nstage; ++s) {
                const int c = s + NST - 1, cs = c >= nstage ? c - nstage : c;
                if (c == nstage && has_next) set_copy_tile(ni0, nj0);
                cut_tail(cs);
                stage1(s, cs);
            }
            SNIP_WAIT_VM(0);                                        // (nothing may land in LDS after the workgroup's end either)
        }
        fold_rest();
        store_tile(i0, j0, before(ring));
        if (!has_next) break;
        u = un;
        i0 = ni0;
        j0 = nj0;
        first = false;
    }
}

template <int FA, int FB, bool OUT_F32>
hipError_t launch_t(const GemmPaperArgs& a, hipStream_t s)
{
    const int ti = (int)((a.I + TM - 1) / TM), tj = (int)((a.J + TN - 1) / TN);
    const int ncu = gemm_compute_units();
    const dim3 grid((unsigned)(ti * tj < ncu ? ti * tj : ncu)), block(NT);
    const int a_shift = a.a_group == 1 ? 0 : 7, stream_out = gemm_streams(a);
    if (a.b_group != 1)
        hipLaunchKernelGGL((gemm_paper_wide_kernel<FA, FB, OUT_F32, true>), grid, block, 0, s, a.a_codes, a.a_scales, a_shift, a.b_codes, a.b_scales,
                           (int)a.I, (int)a.J, (int)a.R, a.c, a.ldc, ti, tj, stream_out);
    else
        hipLaunchKernelGGL((gemm_paper_wide_kernel<FA, FB, OUT_F32, false>), grid, block, 0, s, a.a_codes, a.a_scales, a_shift, a.b_codes, a.b_scales,
                           (int)a.I, (int)a.J, (int)a.R, a.c, a.ldc, ti, tj, stream_out);
    return hipGetLastError();
}

template <int FA, int FB>
hipError_t launch_f(const GemmPaperArgs& a, hipStream_t s)
{
    return a.out_fp32 ? launch_t<FA, FB, true>(a, s) : launch_t<FA, FB, false>(a, s);
}

}  // namespace

bool gemm_paper_wide_eligible(const GemmPaperArgs& a)
{
    // three stages at least, 32-bit source offsets inside 256 rows of codes
    const int64_t ke = a.fmt_a == kFP4 && a.fmt_b == kFP4 ? 2 * kSlab : kSlab;
    return a.R > 2 * ke && a.R <= (1 << 22);
}

hipError_t launch_gemm_paper_wide(const GemmPaperArgs& a, hipStream_t s)
{
    if (a.fmt_a == kFP8 && a.fmt_b == kFP8) return launch_f<kFP8, kFP8>(a, s);
    if (a.fmt_a == kFP8 && a.fmt_b == kFP4) return launch_f<kFP8, kFP4>(a, s);
    if (a.fmt_a == kFP4 && a.fmt_b == kFP8) return launch_f<kFP4, kFP8>(a, s);
    return launch_f<kFP4, kFP4>(a, s);
}

}  // namespace snip

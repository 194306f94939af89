// Block-scaled GEMM for outputs that 256-wide tiles do not serve: few rows (a short micro-batch against a weight), few
// tiles, contraction extents that end inside a pipeline stage.  Same operands (grouped scale copies), instruction and
// summation order as gemm_fast.hip, so the results agree bit for bit.
//
//   One workgroup per tile, tiles of 128 x 128 (four waves of 64 x 64) down to 32 x 32 (one wave), so that a launch
//   has enough workgroups whatever the output's shape.  A ring of NST stage buffers is filled by global->LDS copies
//   NST - 1 stages ahead (128 code bytes per row and stage as in gemm_fast.hip).  Copies and arithmetic belong to
//   different waves: with one or two waves per SIMD a wave retires an instruction every 4-5 cycles, and the copy
//   instructions with their address arithmetic took half of the time of a stage when every wave did both.  One barrier per
//   stage: behind that of stage s, stage s + 1 is complete in LDS and is read into registers while the MFMAs of stage s,
//   whose operands were read a stage earlier, are issued; the buffer of stage s is refilled with stage s + NST.
//   Measured (us per call, back to back in a graph; before: the general kernel): [64 x 4096 x 4096] FP4 23.6 -> 5.2, FP8
//   33 -> 7.0; [64 x 4096 x 11008] FP4 53 -> 8.9; [64 x 11008 x 4096] FP4 24.5 -> 6.3; [1504 x 2080 x 1568] FP4 25.3 -> 9.4,
//   FP8 31.5 -> 11.9; [256 x 512 x 512] FP8 6.5 (256 x 128 tile) -> 3.45.
//   Waves with one 32 x 32 block have one chain of dependent MFMAs, 160 cycles of a stage's 300; the rest was the LDS latency behind
//   the last of them and the barrier.  The 32 x 32 tile therefore takes two stages per barrier (G) on operands of up to 10 MB, from
//   four stages on (picks.h), and asks for the next two during the first five of eight MFMAs (FP4 x FP4; else two of four): operands
//   in the caches [64 x 4096 x 4096] FP4 5.40 -> 4.95, FP8 7.24 -> 6.76, [64 x 4096 x 11008] 9.02 -> 7.94 and 14.4 -> 13.8, [1 x 2048 x 2048] FP8
//   4.84 -> 4.63; from memory the same (6.15 and 6.22).  64 x 32 keeps one: with two it gained 3-6 % from the caches ([224 x 1696 x 4224]
//   FP8 8.01 -> 7.75) and lost 2-10 % from memory (10.5 -> 11.0, FP8 x FP4 9.6 -> 10.4).  With four stages, or a ring of 12 or 16, slower
//   (the rings' fill and LDS cost more than they hide), the 64 x 64 tile too (12.3 -> 16.7 on [1504 x 2080 x 1568]: one workgroup per
//   compute unit instead of two).  What is left is the chain and 3 us of launch, first fill and result.
//   Copies go through buffer descriptors: rows past the end of an operand and chunks past the end of a row deliver
//   zeros, and the scale bytes past the last block are masked, so any contraction extent that is a multiple of 32 runs.
#include "gemm_common.h"
#include <type_traits>
#include "picks.h"

namespace snip {
namespace {

// BM x BN tile, one compute wave per WTM x WTN part, NP copy waves, NST stage buffers, a barrier every G stages.
template <int BM_, int BN_, int WTM_, int WTN_, int NST_, int NP_, int G_> struct SmallTile {
    static constexpr int BM = BM_, BN = BN_, WTM = WTM_, WTN = WTN_, NST = NST_, NP = NP_, G = G_;
    static_assert(NST % G == 0 && NST >= 2 * G, "the ring holds whole groups of stages");
    static constexpr int NC = (BM / WTM) * (BN / WTN), NT = (NC + NP) * 64;
    static constexpr int WGN = BN / WTN;
    static constexpr int MB = WTM / 32, NB = WTN / 32;
};

template <int FA, int FB, class T> struct SmallCfg {
    static constexpr int KE = (FA == kFP4 && FB == kFP4) ? 256 : 128;    // contraction elements per stage
    static constexpr int SBA = FA == kFP8 ? KE : KE / 2, SBB = FB == kFP8 ? KE : KE / 2;
    static constexpr int KS = KE / 64, NG = KE / 128;
    // copy instructions of a stage: 1 KB of codes or 64 scale dwords each; a wave takes LA + LB + LS of them (where they do
    // not divide evenly some are issued twice, with the same bytes)
    static constexpr int NA = T::BM * SBA / 1024, NBC = T::BN * SBB / 1024;
    static constexpr int NSA = (T::BM * NG + 63) / 64, NSB = (T::BN * NG + 63) / 64;
    static constexpr int LA = (NA + T::NP - 1) / T::NP, LB = (NBC + T::NP - 1) / T::NP, LS = (NSA + NSB + T::NP - 1) / T::NP;
    static constexpr int L = LA + LB + LS;
    // stage buffer: [A codes][B codes][A scale dwords: group-major][B scale dwords: group-major]
    static constexpr int OFF_B = NA * 1024, OFF_SA = OFF_B + NBC * 1024, OFF_SB = OFF_SA + NSA * 256, SLOT = OFF_SB + NSB * 256;
    // (the result tile is staged in the stage buffers)
    static constexpr int LDS_BYTES = T::NST * SLOT > T::BM * T::BN * 4 ? T::NST * SLOT : T::BM * T::BN * 4;
    static_assert(L * (T::NST - 1) <= 63, "copies in flight must be countable");
    static_assert(LDS_BYTES <= 159 * 1024, "LDS budget");
};

template <int FA, int FB, bool OUT_F32, class T, bool STREAM_B>
__global__ __launch_bounds__(T::NT) void gemm_small_kernel(const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_g4,
                                                           const uint8_t* __restrict__ b_codes, const uint8_t* __restrict__ b_g4,
                                                           int I, int J, int R, void* __restrict__ c_out, int64_t ldc,
                                                           int tiles_i, int tiles_j, float* __restrict__ norm_partials, int stream_out)
{
    using C = SmallCfg<FA, FB, T>;
    constexpr int BM = T::BM, BN = T::BN, WTM = T::WTM, WTN = T::WTN, MB = T::MB, NB = T::NB, NST = T::NST, NP = T::NP, G = T::G;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[C::LDS_BYTES];

    int ti, tj;
    tile_of(blockIdx.x, tiles_i * tiles_j, tiles_i, tiles_j, ti, tj);
    const int i0 = ti * BM, j0 = tj * BN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nkb = R / kBlock, ngrp = (nkb + 3) / 4;
    const int nstage = (R + C::KE - 1) / C::KE;

    if (wave >= T::NC) {
        // ---- a copy wave.  Copy instruction q of an operand fills 1 KB of its LDS tile.
        const int p = wave - T::NC;
        const int a_row_bytes = FA == kFP8 ? R : R / 2, b_row_bytes = FB == kFP8 ? R : R / 2;
        const unsigned a_bytes = min(BM, I - i0) * a_row_bytes, b_bytes = min(BN, J - j0) * b_row_bytes;
        v4i ra = buffer_desc(a_codes + (int64_t)i0 * a_row_bytes, a_bytes);
        v4i rb = buffer_desc(b_codes + (int64_t)j0 * b_row_bytes, b_bytes);
        auto qa = [&](int j) { return (p + NP * j) % C::NA; };
        auto qb = [&](int j) { return (p + NP * j) % C::NBC; };
        auto row_a = [&](int j) { return qa(j) * (1024 / C::SBA) + lane / (C::SBA / 16); };
        auto row_b = [&](int j) { return qb(j) * (1024 / C::SBB) + lane / (C::SBB / 16); };
        auto chunk_a = [&](int j) { return (lane % (C::SBA / 16)) ^ swz<C::SBA>(row_a(j)); };
        auto chunk_b = [&](int j) { return (lane % (C::SBB / 16)) ^ swz<C::SBB>(row_b(j)); };
        unsigned oa[C::LA], ob[C::LB], os[C::LS];
#pragma unroll
        for (int j = 0; j < C::LA; ++j) oa[j] = (unsigned)(row_a(j) * a_row_bytes + chunk_a(j) * 16);
#pragma unroll
        for (int j = 0; j < C::LB; ++j) ob[j] = (unsigned)(row_b(j) * b_row_bytes + chunk_b(j) * 16);
        // scale dword f of an operand's area: scale group f / rows inside the stage, row f % rows.  Rows past the end lie in
        // the padded pitch, groups past the last one past the end of the descriptor.
        const unsigned pa = (unsigned)g4_pitch(I) * 4, pb = (unsigned)g4_pitch(J) * 4;       // bytes per scale group
        v4i rs[C::LS];
        unsigned spitch[C::LS], srow0[C::LS], sdst[C::LS];
#pragma unroll
        for (int j = 0; j < C::LS; ++j) {
            const int q = (p + NP * j) % (C::NSA + C::NSB);
            const bool isa = q < C::NSA;
            const int f = (isa ? q : q - C::NSA) * 64 + lane;
            const int grp = isa ? f / BM : f / BN, row = isa ? f % BM : f % BN;
            spitch[j] = isa ? pa : pb;
            srow0[j] = (unsigned)(isa ? i0 : j0) * 4;
            os[j] = grp < C::NG ? scale_lane(grp, row, spitch[j]) : kNoSource;
            rs[j] = buffer_desc((isa ? a_g4 : b_g4) + srow0[j], scale_size(ngrp, spitch[j], srow0[j]));
            sdst[j] = C::OFF_SA + q * 256;
        }
        const unsigned lds0 = lds_addr(lds);
        const int tail_stage = R % C::KE != 0 ? nstage - 1 : -1;
        // This wave's share of stage st into stage buffer `slot`.  Every stage issues the same number of copies, so that
        // the waits count in stages.  In a last stage that is not whole, lanes whose chunk lies past the end of the row
        // lose their source for good; past the last stage the descriptors are empty and the offsets zero (no memory is read).
        auto issue = [&](int st, int slot) {
            if (st == tail_stage) {
                // a branch and not selects in every stage: a copy waits until the copies before it have read the offsets that a
                // select is to write (64 x 32, [123 x 2240 x 17024] FP8 24.3 us -> 28.9, [163 x 1792 x 11136] FP8 x FP4 18.1 -> 20.1)
                asm volatile("");
#pragma unroll
                for (int j = 0; j < C::LA; ++j) oa[j] = chunk_a(j) * 16 < a_row_bytes - st * C::SBA ? oa[j] : kNoSource;
#pragma unroll
                for (int j = 0; j < C::LB; ++j) ob[j] = chunk_b(j) * 16 < b_row_bytes - st * C::SBB ? ob[j] : kNoSource;
            }
            const unsigned base = lds0 + slot * C::SLOT;
            const CopyRange ca = code_range(st, nstage, a_bytes, C::SBA), cb = code_range(st, nstage, b_bytes, C::SBB);
            ra[2] = ca.size;
            rb[2] = cb.size;
#pragma unroll
            for (int j = 0; j < C::LA; ++j) blds16(ra, oa[j], ca.uniform, base + qa(j) * 1024);
#pragma unroll
            for (int j = 0; j < C::LB; ++j) blds16<STREAM_B>(rb, ob[j], cb.uniform, base + C::OFF_B + qb(j) * 1024);
#pragma unroll
            for (int j = 0; j < C::LS; ++j) {
                const CopyRange cs = scale_range(st, nstage, ngrp, C::NG, spitch[j], srow0[j]);
                rs[j][2] = cs.size;
                blds4(rs[j], os[j], cs.uniform, base + sdst[j]);
            }
        };
#pragma unroll
        for (int st = 0; st < NST; ++st) issue(st, st);
        SNIP_WAIT_VM(C::L * (NST - G));                          // the first G stages
        SNIP_BAR();
        int slot = 0;
        for (int s = 0; s < nstage; s += G) {
            SNIP_WAIT_VM(C::L * (NST - 2 * G));                  // stages s + G ... s + 2 G - 1 have landed
            SNIP_BAR();                                          // the compute waves have read stages s ... s + G - 1
#pragma unroll
            for (int j = 0; j < G; ++j) issue(s + NST + j, slot + j);
            slot = slot == NST - G ? 0 : slot + G;
        }
        SNIP_WAIT_VM(0);                                         // the empty copies past the last stage write zeros
        SNIP_BAR();
        if (norm_partials) __syncthreads();
        return;
    }

    // ---- a compute wave
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    const int r32 = lane & 31, g = lane >> 5;
    constexpr int NCA = FA == kFP8 ? 2 * C::KS : C::KS, NCB = FB == kFP8 ? 2 * C::KS : C::KS;
    int offa[NCA], offb[NCB];
    frag_offsets<FA, C::SBA, C::KS>(r32, g, offa);
    frag_offsets<FB, C::SBB, C::KS>(r32, g, offb);
    const int sca_off = C::OFF_SA + (wm * WTM + r32) * 4;
    const int scb_off = C::OFF_SB + (wn * WTN + r32) * 4;

    v16f acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int k = 0; k < 16; ++k) acc[a][b][k] = 0.f;

    // Operands of G stages: codes of their KS MFMA steps and scale dwords.
    constexpr int KG = G * C::KS, QG = G * C::NG;
    struct Operands { v8i fa[KG][MB], fb[KG][NB]; unsigned sa[QG][MB], sb[QG][NB]; } op0, op1;
    auto read_scales = [&](Operands& o, int slot) {
#pragma unroll
        for (int q = 0; q < QG; ++q) {
            const uint8_t* base = lds + (slot + q / C::NG) * C::SLOT;
#pragma unroll
            for (int m = 0; m < MB; ++m) o.sa[q][m] = *reinterpret_cast<const unsigned*>(base + sca_off + q % C::NG * BM * 4 + m * 128);
#pragma unroll
            for (int n = 0; n < NB; ++n) o.sb[q][n] = *reinterpret_cast<const unsigned*>(base + scb_off + q % C::NG * BN * 4 + n * 128);
        }
    };
    constexpr int NR = KG * (MB + NB);                           // operand blocks of G stages
    auto read_block = [&](Operands& o, int slot, int r) {
        const int k = r / (MB + NB), i = r % (MB + NB), ks = k % C::KS;
        const uint8_t* base = lds + (slot + k / C::KS) * C::SLOT;
        if (i < MB) o.fa[k][i] = read_frag<FA>(base + wm * WTM * C::SBA, i * 32 * C::SBA, offa, ks);
        else        o.fb[k][i - MB] = read_frag<FB>(base + C::OFF_B + wn * WTN * C::SBB, (i - MB) * 32 * C::SBB, offb, ks);
    };
    constexpr int ca = FB == kFP8 ? 0 : 4, cb = FA == kFP8 ? 0 : 4;              // first operand = B tile
    // Stages s ... s + G - 1: their operands are in `cur`; those of the next G are read meanwhile.
    auto step = [&](Operands& cur, Operands& nxt, int s, int slot1) {
        SNIP_BAR();                                              // the next G stages are complete
        read_scales(nxt, slot1);
        __builtin_amdgcn_sched_barrier(0);
        // scale bytes past the last block are unspecified: masked (whole groups past the end were delivered as zeros)
        if ((nkb & 3) != 0 && s + G >= nstage) {
#pragma unroll
            for (int q = 0; q < QG; ++q) {
                const unsigned mask = s * C::NG + q == ngrp - 1 ? (1u << (8 * (nkb & 3))) - 1u : 0xFFFFFFFFu;
#pragma unroll
                for (int m = 0; m < MB; ++m) cur.sa[q][m] &= mask;
#pragma unroll
                for (int n = 0; n < NB; ++n) cur.sb[q][n] &= mask;
            }
        }
        // lane group g looks at bytes g and 2 + g of its rows' dwords
#pragma unroll
        for (int q = 0; q < QG; ++q) {
#pragma unroll
            for (int m = 0; m < MB; ++m) cur.sa[q][m] >>= 8 * g;
#pragma unroll
            for (int n = 0; n < NB; ++n) cur.sb[q][n] >>= 8 * g;
        }
        // the next stages' operands are requested between the MFMAs: all at once they would fill the LDS queue and hold
        // the MFMAs back for the time of all waves' reads.  (A stage past the last one multiplies the zeros it was filled with.)
        constexpr int NM = KG * MB * NB, NI = G == 1 ? NM : NM * 5 / 8;      // (G > 1: the last ones arrive while the chain goes on)
        int idx = 0;
#pragma unroll
        for (int k = 0; k < KG; ++k)
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    if ((k & 1) == 0)
                        acc[m][n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cur.fb[k][n], cur.fa[k][m], acc[m][n], ca, cb, 0, (int)cur.sb[k >> 1][n], 0, (int)cur.sa[k >> 1][m]);
                    else
                        acc[m][n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cur.fb[k][n], cur.fa[k][m], acc[m][n], ca, cb, 2, (int)cur.sb[k >> 1][n], 2, (int)cur.sa[k >> 1][m]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        if (r * NI / NR == idx) read_block(nxt, slot1, r);
                    __builtin_amdgcn_sched_barrier(0);
                    ++idx;
                }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);                      // lgkmcnt(0): they are read before the next barrier
    };
    SNIP_BAR();                                                  // the first G stages are complete
    read_scales(op0, 0);
#pragma unroll
    for (int r = 0; r < NR; ++r) read_block(op0, 0, r);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    int slot1 = G;
    for (int s = 0;;) {
        step(op0, op1, s, slot1);
        slot1 = slot1 == NST - G ? 0 : slot1 + G;
        if ((s += G) >= nstage) break;
        step(op1, op0, s, slot1);
        slot1 = slot1 == NST - G ? 0 : slot1 + G;
        if ((s += G) >= nstage) break;
    }
    SNIP_BAR();                                                  // nothing writes to the stage buffers any more

    // Optional: sum of squares of the tile as it will be stored, elements outside the matrix excluded.
    if (norm_partials) {
        __shared__ float wave_ss[T::NC];
        float ss = 0.f;
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
        ss = wave_sum(ss);
        if (lane == 0) wave_ss[wave] = ss;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
            for (int w = 0; w < T::NC; ++w) t += wave_ss[w];
            norm_partials[blockIdx.x] = t;
        }
    }

    // Result: every compute wave transposes its block through its own part of the stage buffers.  In registers, lane
    // (r32, g) of block (m, n) holds C[32m + r32][32n + 8q + 4g + t] in acc[m][n][4q + t].
    constexpr int ESZ = OUT_F32 ? 4 : 2;
    constexpr int ROWB = WTN * ESZ, CPR = ROWB / 16, RPI = 64 / CPR;
    uint8_t* reg = lds + wave * WTM * ROWB;
    auto spread = [](int row) { return CPR >= 16 ? row & (CPR - 1) : CPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3; };
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int row = m * 32 + r32;
        const int f = spread(row);
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float v0 = acc[m][n][4 * q + 0], v1 = acc[m][n][4 * q + 1];
                const float v2 = acc[m][n][4 * q + 2], v3 = acc[m][n][4 * q + 3];
                if (OUT_F32) {
                    *reinterpret_cast<float4*>(reg + row * ROWB + (((n * 8 + q * 2 + g) ^ f) * 16)) = make_float4(v0, v1, v2, v3);
                } else {
                    const float2_t lo = {v0, v1}, hi = {v2, v3};
                    const bf16x2 blo = __builtin_convertvector(lo, bf16x2), bhi = __builtin_convertvector(hi, bf16x2);
                    *reinterpret_cast<uint2*>(reg + row * ROWB + (((n * 4 + q) ^ f) * 16) + 8 * g) =
                        make_uint2(__builtin_bit_cast(unsigned, blo), __builtin_bit_cast(unsigned, bhi));
                }
            }
    }
    // (a branch around all stores, not one at each: 1504 x 2080 x 1568 0.2 us a GEMM)
    auto store = [&](auto stream) {
#pragma unroll
        for (int it = 0; it < WTM / RPI; ++it) {
            const int row = it * RPI + lane / CPR, c = lane % CPR;
            const uint4 v = *reinterpret_cast<const uint4*>(reg + row * ROWB + ((c ^ spread(row)) * 16));
            const int i = i0 + wm * WTM + row, j = j0 + wn * WTN + c * (16 / ESZ);
            if (i < I) {
                uint8_t* p = reinterpret_cast<uint8_t*>(c_out) + ((int64_t)i * ldc + j) * ESZ;
                if (j + 16 / ESZ <= J) {
                    store16(v4u{v.x, v.y, v.z, v.w}, p, stream);
                } else {
                    const unsigned w[4] = {v.x, v.y, v.z, v.w};
                    for (int e = 0; e < 16 / ESZ; ++e)
                        if (j + e < J) {
                            if (OUT_F32) reinterpret_cast<unsigned*>(p)[e] = w[e];
                            else reinterpret_cast<uint16_t*>(p)[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                        }
                }
            }
        }
    };
    if (stream_out) store(std::true_type()); else store(std::false_type());
}

template <int FA, int FB, class T, bool STREAM_B>
hipError_t launch_small_s(const GemmArgs& a, hipStream_t s)
{
    const int ti = (int)((a.I + T::BM - 1) / T::BM), tj = (int)((a.J + T::BN - 1) / T::BN);
    const dim3 grid((unsigned)(ti * tj)), block(T::NT);
    if (a.out_fp32)
        hipLaunchKernelGGL((gemm_small_kernel<FA, FB, true, T, STREAM_B>), grid, block, 0, s, a.a_codes, a.a_scales_g4, a.b_codes, a.b_scales_g4,
                           (int)a.I, (int)a.J, (int)a.R, a.c, a.ldc, ti, tj, a.norm_partials, (int)gemm_streams(a));
    else
        hipLaunchKernelGGL((gemm_small_kernel<FA, FB, false, T, STREAM_B>), grid, block, 0, s, a.a_codes, a.a_scales_g4, a.b_codes, a.b_scales_g4,
                           (int)a.I, (int)a.J, (int)a.R, a.c, a.ldc, ti, tj, a.norm_partials, (int)gemm_streams(a));
    return hipGetLastError();
}
template <int FA, int FB, class T>
hipError_t launch_small_t(const GemmArgs& a, hipStream_t s)
{
    if constexpr (T::BM <= 64 && T::G == 1)
        if (small_streams_b(a.I <= T::BM, a.J * a.R / (FB == kFP8 ? 1 : 2))) return launch_small_s<FA, FB, T, true>(a, s);
    return launch_small_s<FA, FB, T, false>(a, s);
}

template <class T>
hipError_t launch_small_tile(const GemmArgs& a, hipStream_t s)
{
    if (a.fmt_a == kFP8 && a.fmt_b == kFP8) return launch_small_t<kFP8, kFP8, T>(a, s);
    if (a.fmt_a == kFP8 && a.fmt_b == kFP4) return launch_small_t<kFP8, kFP4, T>(a, s);
    if (a.fmt_a == kFP4 && a.fmt_b == kFP8) return launch_small_t<kFP4, kFP8, T>(a, s);
    return launch_small_t<kFP4, kFP4, T>(a, s);
}

}  // namespace

bool gemm_small_eligible(const GemmArgs& a)
{
    // 32-bit source offsets inside the buffer descriptors: 128 rows of codes and a whole grouped scale copy
    const int64_t groups = (a.R + 127) / 128;
    return a.a_scales_g4 && a.b_scales_g4 && a.R <= (1 << 22) && descriptor_covers(g4_pitch(a.I) * 4 * groups) &&
           descriptor_covers(g4_pitch(a.J) * 4 * groups) && (a.I + 31) / 32 * ((a.J + 31) / 32) < ((int64_t)1 << 31);
}

hipError_t launch_gemm_small(const GemmArgs& a, GemmTile tile, hipStream_t s)
{
    const bool both4 = a.fmt_a == kFP4 && a.fmt_b == kFP4;
    const bool pairs = small_stages_per_barrier(gemm_operand_bytes(a) <= kColdBytes, (a.R + (both4 ? 255 : 127)) / (both4 ? 256 : 128)) == 2;
    switch (tile) {
        case GemmTile::k128x128: return launch_small_tile<SmallTile<128, 128, 64, 64, 4, 4, 1>>(a, s);
        case GemmTile::k64x64:
            // Up to 32 rows: half of the tile's rows would be copied from nowhere, and the room goes to two more stages instead.  Few
            // tokens through weights wider than a round of 32 x 32.  64 x 64 -> 32 x 64, us, operands from memory: [1 x 11008 x 4096] FP4 8.9 ->
            // 7.25, FP8 14.7 -> 11.8, 32 rows 9.5 -> 8.6 and 15.3 -> 13.8, [1 x 13824 x 5120] 10.4 -> 9.3 and 16.4 -> 14.5; 96 calls from the caches and from
            // memory 6 % on average, none slower ([1 ... 32 x 8224 x 128] the same).  Rings of eight and eleven stages are 1-5 % slower.
            if (a.I <= 32) return launch_small_tile<SmallTile<32, 64, 32, 32, 6, 4, 1>>(a, s);
            return launch_small_tile<SmallTile<64, 64, 32, 32, 4, 4, 1>>(a, s);
        case GemmTile::k64x32:   return launch_small_tile<SmallTile<64, 32, 32, 32, 6, 4, 1>>(a, s);
        default:
            return pairs ? launch_small_tile<SmallTile<32, 32, 32, 32, 8, 4, 2>>(a, s) : launch_small_tile<SmallTile<32, 32, 32, 32, 8, 4, 1>>(a, s);
    }
}

}  // namespace snip

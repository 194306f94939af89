// GEMM on operands quantized with the paper's own recipe (SNIP Sec. 2.3 / 5.1: real-valued scale per
// 1x128 tile or 128x128 block): C[I][J] = sum_r (A[i][r] / sa) * (B[j][r] / sb).
//
// The matrix instruction applies only power-of-two scales to 32-element blocks, so the real-valued scales
// are applied in software: the contraction runs in slabs of 128 elements (one scaling group of either
// operand); the codes of a slab are multiplied on the matrix cores with unit scales into a fresh fp32
// accumulator, which is then folded into the running result with the factor (1/sa) * (1/sb) of that slab.
//
// 128 x 128 tile, organised as in gemm_small.hip: four compute waves of 64 x 64, three copy waves that fill a ring of
// NST stage buffers with global->LDS copies NST - 1 stages ahead (128 code bytes per row and stage, two slabs for
// FP4 x FP4), one barrier per stage.  Another wave fetches the scales and leaves their reciprocals in LDS, so that the
// compute waves read ready factors.  A compute wave folds the previous 32 x 32 block while the matrix core works on the current one (two
// accumulators of 16 registers in turn): beside 2 x 64 (FP8) or 2 x 32 (FP4) cycles of MFMA per block that takes 16
// fused multiply-adds of 4 cycles, and 16 products more where B has a factor per column (weight gradients).  With B in
// 128 x 128 blocks the factor is one value per lane and slab (B_BLOCK).
// The kernel is persistent: the stages of a workgroup's tiles form one sequence, the copy waves are already in the next
// tile while the result of the last one is stored (through 4 KB of LDS per wave, whole 128-byte runs).
// Measured against a 128 x 128 tile of four waves staged through registers, results bit-identical (us per call, A in tiles, B
// in blocks / in tiles): [4096 x 2048 x 8192] FP8 158 -> 80 / 93, [4096 x 8192 x 2048] FP8 168 -> 108 / 112 (20 us of it the
// output rows 16 KB apart: 89 / 101 with padded rows), [4096 x 4096 x 4096] FP4 58 / 72.  1.7 (FP8) and 2.4 (FP4) PFLOP/s with
// B in blocks; without the copies it would be 2.3 and 3.1, without the fold 5 % more, and of the rest the matrix cores'
// clock under random operands takes most.  Outputs with enough tiles go to gemm_paper_wide.hip (picks.h).
// Register layout of the instruction: see gemm.hip.
#include "gemm_common.h"
#include "picks.h"
#include <cstdlib>
#include <cstring>

namespace snip {
namespace {

constexpr int BM = 128, BN = 128, WTM = 64, WTN = 64, MB = 2, NB = 2;
constexpr int NC = 4, NP = 3, NT = (NC + NP + 1) * 64;          // compute waves, copy waves, one wave for the scales
constexpr int NST = 4;                                          // stage buffers
constexpr int NFS = 3;                                          // factor slots: two stages are read while a third is written
constexpr int kSlab = 128;                                      // contraction elements of a scaling group
constexpr unsigned kUnitScale = 0x7F7F7F7Fu;                    // E8M0 127 = 2^0 in every byte

template <int FA, int FB> struct PaperCfg {
    static constexpr int NG = FA == kFP4 && FB == kFP4 ? 2 : 1;          // slabs per stage
    static constexpr int KE = NG * kSlab, KS = KE / 64;
    static constexpr int SBA = FA == kFP8 ? KE : KE / 2, SBB = FB == kFP8 ? KE : KE / 2;
    static constexpr int NA = BM * SBA / 1024, NQ = NA + BN * SBB / 1024;    // 1 KB copies of a stage: A's, all
    static constexpr int L = (NQ + NP - 1) / NP;                          // per copy wave (where they do not divide evenly some are issued twice)
    static constexpr int OFF_B = BM * SBA, SLOT = OFF_B + BN * SBB;
    static constexpr int FSLOT = NG * (BM + BN) * 4;                      // factors of a stage: [slab][A rows, B rows]
    static constexpr int OFF_F = NST * SLOT, OFF_E = OFF_F + NFS * FSLOT;
    static constexpr int EPI = 4096;                                      // result staging per compute wave
    static constexpr int LDS_BYTES = OFF_E + NC * EPI;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
    static_assert(L * (NST - 1) <= 63, "copies in flight must be countable");
};

// As glds16 (gemm_common.h) with a 64-bit source address per lane: a row of codes may be longer than 2^24 bytes.
__device__ __forceinline__ void glds16_at(uint64_t src, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds) : "memory", "m0");
}
template <int FA, int FB, bool OUT_F32, bool B_BLOCK>
__global__ __launch_bounds__(NT) void gemm_paper_kernel(const uint8_t* __restrict__ a_codes, const float* __restrict__ a_scales, int a_group,
                                                        const uint8_t* __restrict__ b_codes, const float* __restrict__ b_scales, int b_group,
                                                        int I, int J, int R, void* __restrict__ c_out, int64_t ldc, int tiles_i, int tiles_j, int stream_out)
{
    using C = PaperCfg<FA, FB>;
    constexpr int NG = C::NG, KS = C::KS;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[C::LDS_BYTES];

    const int ntile = tiles_i * tiles_j;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nslab = R / kSlab, nstage = (nslab + NG - 1) / NG;
    const int mine = (ntile - 1 - (int)blockIdx.x) / (int)gridDim.x + 1;          // tiles of this workgroup
    const int64_t total = (int64_t)mine * nstage;                                 // stages of all of them

    if (wave < NC + NP && wave >= NC) {
        // ---- a copy wave.  Copy q of a stage fills 1 KB of A's or B's LDS tile; rows past the end of an operand read its
        // last row again (their products are never stored).
        const int p = wave - NC;
        __builtin_amdgcn_s_setprio(2);                      // (its instructions start the copies everything else waits for: 1-3 %)
        auto unit = [&](int j) { return min(p + NP * j, C::NQ - 1); };
        uint64_t src[C::L];
        int ct = blockIdx.x, cs = 0;                        // tile and stage the next copies belong to
        auto set_tile = [&]() {
            int ti, tj;
            tile_of(ct, ntile, tiles_i, tiles_j, ti, tj);
#pragma unroll
            for (int j = 0; j < C::L; ++j) {
                const int q = unit(j);
                if (q < C::NA) {
                    const int row = q * (1024 / C::SBA) + lane / (C::SBA / 16), chunk = (lane % (C::SBA / 16)) ^ swz<C::SBA>(row);
                    src[j] = (uint64_t)a_codes + (uint64_t)(min(ti * BM + row, I - 1) * (int64_t)(FA == kFP8 ? R : R / 2) + chunk * 16);
                } else {
                    const int row = (q - C::NA) * (1024 / C::SBB) + lane / (C::SBB / 16), chunk = (lane % (C::SBB / 16)) ^ swz<C::SBB>(row);
                    src[j] = (uint64_t)b_codes + (uint64_t)(min(tj * BN + row, J - 1) * (int64_t)(FB == kFP8 ? R : R / 2) + chunk * 16);
                }
            }
        };
        const unsigned lds0 = lds_addr(lds);
        auto issue = [&](int slot) {
            const unsigned base = lds0 + slot * C::SLOT;
            if (NG == 2 && cs == nstage - 1 && (nslab & 1)) {
                // FP4 x FP4, odd number of slabs: the last stage's second half repeats its first (its factors are zero)
#pragma unroll
                for (int j = 0; j < C::L; ++j)
                    if (((lane % 8) ^ swz<128>(unit(j) * 8 + lane / 8)) >= 4) src[j] -= 64;
            }
#pragma unroll
            for (int j = 0; j < C::L; ++j) {
                glds16_at(src[j], base + unit(j) * 1024);
                src[j] += C::SBA == C::SBB ? C::SBA : unit(j) < C::NA ? C::SBA : C::SBB;
            }
            if (++cs == nstage) {
                cs = 0;
                ct += gridDim.x;
                if (ct < ntile) set_tile();
            }
        };
        auto wait_in_flight = [&](int64_t n) {              // at most n stages still in flight
            if (n >= 3) SNIP_WAIT_VM(C::L * 3);
            else if (n == 2) SNIP_WAIT_VM(C::L * 2);
            else if (n == 1) SNIP_WAIT_VM(C::L);
            else SNIP_WAIT_VM(0);
        };
        static_assert(NST == 4, "waits above");
        set_tile();
        int64_t issued = 0;
        int islot = 0;
        for (; issued < NST && issued < total; ++issued) issue((int)issued);
        wait_in_flight(issued - 1);
        SNIP_BAR();                                          // stage 0 is complete
        for (int64_t s = 0; s < total; ++s) {
            wait_in_flight(issued - s - 2);                  // stage s + 1 has landed
            SNIP_BAR();                                      // the compute waves have read the codes of stage s
            if (issued < total) {
                issue(islot);
                islot = islot == NST - 1 ? 0 : islot + 1;
                ++issued;
            }
        }
        return;
    }
    if (wave == NC + NP) {
        // ---- the scale wave: the reciprocals of a stage's scales into LDS, one stage ahead.  A lane serves rows lane and 64 +
        // lane of both operands and fetches four slabs of a row at a time (a row's scales of consecutive slabs are adjacent:
        // one line then serves four slabs; a dword per row and slab cost a quarter of the kernel), four slabs ahead of their use.
        const bool wide = (nslab & 3) == 0 && (((uintptr_t)a_scales | (uintptr_t)b_scales) & 15) == 0;
        float cur[4][4], nxt[4][4];
        int ft = blockIdx.x, fc = 0;                         // tile and first slab of the next fetch
        auto fetch = [&]() {
            if (ft >= ntile) return;
            int ti, tj;
            tile_of(ft, ntile, tiles_i, tiles_j, ti, tj);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const int row = h < 2 ? min(ti * BM + h * 64 + lane, I - 1) : min(tj * BN + (h - 2) * 64 + lane, J - 1);
                const float* p = (h < 2 ? a_scales : b_scales) + (int64_t)((h < 2 ? a_group : b_group) == 1 ? row : row >> 7) * nslab;
                if (wide) {
                    const float4 v = *reinterpret_cast<const float4*>(p + fc);
                    nxt[h][0] = v.x; nxt[h][1] = v.y; nxt[h][2] = v.z; nxt[h][3] = v.w;
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) nxt[h][k] = p[min(fc + k, nslab - 1)];
                }
            }
            fc += 4;
            if (fc >= nslab) { fc = 0; ft += gridDim.x; }
        };
        float* const fac = reinterpret_cast<float*>(lds + C::OFF_F) + lane;
        int fslot = 0;
        fetch();
        for (int u = blockIdx.x; u < ntile; u += gridDim.x)
            for (int c0 = 0; c0 < nslab; c0 += 4) {
#pragma unroll
                for (int h = 0; h < 4; ++h)
#pragma unroll
                    for (int k = 0; k < 4; ++k) cur[h][k] = nxt[h][k];
                fetch();
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int q = NG == 2 ? k & 1 : 0;
                    if (c0 + k - q >= nslab) break;          // (the second slab of a last stage may be missing: zero factors)
#pragma unroll
                    for (int h = 0; h < 4; ++h)
                        fac[fslot * (C::FSLOT / 4) + q * (BM + BN) + h * 64] = NG == 2 && c0 + k >= nslab ? 0.f : __fdiv_rn(1.f, cur[h][k]);
                    if (q == NG - 1) {
                        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
                        SNIP_BAR();
                        fslot = fslot == NFS - 1 ? 0 : fslot + 1;
                    }
                }
            }
        SNIP_BAR();
        return;
    }

    // ---- a compute wave
    const int wm = wave >> 1, wn = wave & 1;
    const int r32 = lane & 31, g = lane >> 5;
    constexpr int NCA = FA == kFP8 ? 2 * KS : KS, NCB = FB == kFP8 ? 2 * KS : KS;
    int offa[NCA], offb[NCB];
    frag_offsets<FA, C::SBA, KS>(r32, g, offa);
    frag_offsets<FB, C::SBB, KS>(r32, g, offb);

    // Operands of a slab, one set: a block of 32 rows is reloaded with the next slab's as soon as its last products are issued.
    v8i fa[2][MB], fb[2][NB];
    auto read_a = [&](int ks, int m, int slot, int q) {
        fa[ks][m] = read_frag<FA>(lds + slot * C::SLOT + wm * WTM * C::SBA, m * 32 * C::SBA, offa, 2 * q + ks);
    };
    auto read_b = [&](int ks, int n, int slot, int q) {
        fb[ks][n] = read_frag<FB>(lds + slot * C::SLOT + C::OFF_B + wn * WTN * C::SBB, n * 32 * C::SBB, offb, 2 * q + ks);
    };
    constexpr int ca = FB == kFP8 ? 0 : 4, cb = FA == kFP8 ? 0 : 4;              // first operand = B tile

    v16f acc[MB][NB];
    auto clear = [&]() {
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int k = 0; k < 16; ++k) acc[a][b][k] = 0.f;
    };
    // Products of the block worked on last, not yet folded, and its factors: B_BLOCK one value, else A's value and the 16
    // of B's columns (lane (r32, g) holds C[row r32][column 8q + 4g + t] in register 4q + t of a 32 x 32 block).
    v16f pend;
    float pend_a, dbn[16];
    auto fold = [&](v16f& c, int k0, int k1) {
#pragma unroll
        for (int k = k0; k < k1; ++k)
            c[k] = fmaf(pend[k], B_BLOCK ? pend_a : __fmul_rn(pend_a, dbn[k]), c[k]);
    };
    // A stage.  Of its first slab the blocks b0 and a0 are in registers already; a1 and b1 are read during the first two of the
    // four products of a slab, the next slab's b0 and a0 during the last two.  With its last slab's b1 a wave has read the
    // stage: there, behind the first MFMA that needs it, is the barrier that frees the buffer and says that the next stage
    // is complete.
    auto step = [&](int slot, int slot1, int fslot) {
        const float* fac = reinterpret_cast<const float*>(lds + C::OFF_F + fslot * C::FSLOT);
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            const bool last = q == NG - 1;
            float da[MB], db = 0.f;
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    v16f& prev = acc[1 - m][m == 0 ? 1 - n : n];               // the block before this one
                    v16f t;
#pragma unroll
                    for (int k = 0; k < 16; ++k) t[k] = 0.f;
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        t = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[ks][n], fa[ks][m], t, ca, cb, 0, (int)kUnitScale, 0, (int)kUnitScale);
                        __builtin_amdgcn_sched_barrier(0);
                        if (last && n == 1 && m == 0 && ks == 0) {
                            __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0)
                            SNIP_BAR();
                        }
                        if (n == 0 && m == 0 && ks == 0) {
#pragma unroll
                            for (int i = 0; i < MB; ++i) da[i] = fac[q * (BM + BN) + wm * WTM + i * 32 + r32];
                            if (B_BLOCK) db = fac[q * (BM + BN) + BM];
                        }
                        if (n == 0 && m == 0) read_a(ks, 1, slot, q);
                        if (n == 0 && m == 1) read_b(ks, 1, slot, q);
                        if (n == 1 && m == 0) read_b(ks, 0, last ? slot1 : slot, last ? 0 : q + 1);
                        if (n == 1 && m == 1) read_a(ks, 0, last ? slot1 : slot, last ? 0 : q + 1);
                        fold(prev, 8 * ks, 8 * ks + 8);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (!B_BLOCK && m == 0) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float4 v = *reinterpret_cast<const float4*>(fac + q * (BM + BN) + BM + wn * WTN + n * 32 + 8 * k + 4 * g);
                            dbn[4 * k] = v.x; dbn[4 * k + 1] = v.y; dbn[4 * k + 2] = v.z; dbn[4 * k + 3] = v.w;
                        }
                    }
                    pend = t;
                    pend_a = B_BLOCK ? __fmul_rn(da[m], db) : da[m];
                }
        }
    };

    uint8_t* const reg = lds + C::OFF_E + wave * C::EPI;         // result staging of the wave
    auto store_tile = [&](int u) {
        int ti, tj;
        tile_of(u, ntile, tiles_i, tiles_j, ti, tj);
        const int i0 = ti * BM + wm * WTM, j0 = tj * BN + wn * WTN;
        if (stream_out) store_block64<OUT_F32, true>(acc, reg, lane, c_out, ldc, i0, j0, I, J, false);
        else store_block64<OUT_F32, false>(acc, reg, lane, c_out, ldc, i0, j0, I, J, false);
    };

    SNIP_BAR();                                              // stage 0 is complete
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) { read_b(ks, 0, 0, 0); read_a(ks, 0, 0, 0); }
    int slot = 0, fslot = 0;
    for (int u = blockIdx.x; u < ntile; u += gridDim.x) {
        clear();
        // nothing is pending: the tile's first fold adds 0 * 0.  (The factors too: the last tile's may be NaN.)
#pragma unroll
        for (int k = 0; k < 16; ++k) { pend[k] = 0.f; dbn[k] = 0.f; }
        pend_a = 0.f;
        for (int s = 0; s < nstage; ++s) {
            const int slot1 = slot == NST - 1 ? 0 : slot + 1;
            step(slot, slot1, fslot);
            slot = slot1;
            fslot = fslot == NFS - 1 ? 0 : fslot + 1;
        }
        fold(acc[MB - 1][NB - 1], 0, 16);
        store_tile(u);
    }
}

template <int FA, int FB, bool OUT_F32>
hipError_t launch_t(const GemmPaperArgs& a, hipStream_t s)
{
    const int ti = (int)((a.I + BM - 1) / BM), tj = (int)((a.J + BN - 1) / BN);
    const int ncu = gemm_compute_units();
    const dim3 grid((unsigned)(ti * tj < ncu ? ti * tj : ncu)), block(NT);
    // Small results plain too: at the end of a short kernel memory answers later than the caches ([832 x 768 x 256] FP4 5.3 us and 5.6; 1 %
    // on average below 1 M elements, above 4-6 % the other way).
    const int stream_out = gemm_streams(a) && a.I * a.J >= 1 << 20;
    if (a.b_group != 1)
        hipLaunchKernelGGL((gemm_paper_kernel<FA, FB, OUT_F32, true>), grid, block, 0, s, a.a_codes, a.a_scales, a.a_group, a.b_codes,
                           a.b_scales, a.b_group, (int)a.I, (int)a.J, (int)a.R, a.c, a.ldc, ti, tj, stream_out);
    else
        hipLaunchKernelGGL((gemm_paper_kernel<FA, FB, OUT_F32, false>), grid, block, 0, s, a.a_codes, a.a_scales, a.a_group, a.b_codes,
                           a.b_scales, a.b_group, (int)a.I, (int)a.J, (int)a.R, a.c, a.ldc, ti, tj, stream_out);
    return hipGetLastError();
}

template <int FA, int FB>
hipError_t launch_f(const GemmPaperArgs& a, hipStream_t s)
{
    return a.out_fp32 ? launch_t<FA, FB, true>(a, s) : launch_t<FA, FB, false>(a, s);
}

// This kernel or that of gemm_paper_wide.hip (picks.h).  SNIP_GEMM_PAPER_TILE=128x128|256x128 in the environment, read at every
// call, fixes the kernel where it can serve the call; for tests and measurements.
bool use_wide(const GemmPaperArgs& a)
{
    if (!gemm_paper_wide_eligible(a)) return false;
    if (const char* e = getenv("SNIP_GEMM_PAPER_TILE")) {
        if (!strcmp(e, "256x128")) return true;
        if (!strcmp(e, "128x128")) return false;
    }
    return paper_wide_pays(a.I, a.J, a.R, a.fmt_a == kFP4 && a.fmt_b == kFP4, a.b_group == 1, gemm_paper_scales16(a), gemm_compute_units());
}

}  // namespace

hipError_t launch_gemm_paper(const GemmPaperArgs& a, hipStream_t s)
{
    if (a.I == 0 || a.J == 0) return hipSuccess;
    if (use_wide(a)) return launch_gemm_paper_wide(a, s);
    if (a.fmt_a == kFP8 && a.fmt_b == kFP8) return launch_f<kFP8, kFP8>(a, s);
    if (a.fmt_a == kFP8 && a.fmt_b == kFP4) return launch_f<kFP8, kFP4>(a, s);
    if (a.fmt_a == kFP4 && a.fmt_b == kFP8) return launch_f<kFP4, kFP8>(a, s);
    return launch_f<kFP4, kFP4>(a, s);
}

}  // namespace snip

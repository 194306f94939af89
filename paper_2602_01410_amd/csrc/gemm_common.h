// What the two global->LDS GEMM kernels (gemm_fast.hip: large tiles, persistent; gemm_small.hip: small tiles) share:
// the copy instructions, the LDS swizzle, the operand fragments of v_mfma_scale_f32_32x32x64_f8f6f4 and the order in
// which tiles are dealt to the chip.  Register layout of the instruction: see gemm.hip.
#pragma once
#include "snip_internal.h"
#include "copy_ranges.h"

namespace snip {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Global -> LDS copy issued by the load unit: lane i's 16 (or 4) bytes land at lds + 16*i (4*i); `lds` is
// wave-uniform and travels in M0.  Written as inline assembly on purpose: the compiler then keeps no
// scoreboard entry for these copies and never adds its own (conservative, count-zero) wait in front of LDS
// reads; completion is enforced by explicit SNIP_WAIT_VM + barrier in the kernels.  The "memory"
// clobber tells the compiler that LDS contents change here.
__device__ __forceinline__ unsigned lds_addr(const void* p)
{
    return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
// The source address is a wave-uniform 64-bit base (SGPR pair) plus a 32-bit per-lane byte offset.
// A memory instruction may read a scalar register five wait states after a vector instruction wrote it.  The compiler does
// not keep that distance in front of inline assembly, and where it runs out of scalar registers (gemm_fast.hip) it fetches
// an address with v_readlane right there: s_mov and s_nop 3 are the five (tests/test_wait_states.py reads the built code).
// The wait costs 0.1-0.5 % of a training step, measured against s_mov_b64 of the base to a register of the assembly's own
// (not kept: eight copies had that register written by v_mad_u64_u32 just before); four wait states more cost 1-2 %.
__device__ __forceinline__ void glds16(const uint8_t* base, unsigned lane_off, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_off), "s"(base), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void glds4(const uint8_t* base, unsigned lane_off, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dword %0, %1" : : "v"(lane_off), "s"(base), "s"(lds) : "memory", "m0");
}
// The same with a buffer descriptor as source, per-lane offset `lane_off` + wave-uniform `soff`: a lane whose offset lies at
// or past the descriptor's size - soff delivers zeros (kNoSource is past every size used here; soff: see copy_ranges.h).
constexpr unsigned kNoSource = 0x80000000u;
template <bool STREAM = false>
__device__ __forceinline__ void blds16(v4i rsrc, unsigned lane_off, unsigned soff, unsigned lds)
{
    if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 3\n\tbuffer_load_dwordx4 %0, %1, %2 offen nt lds"
                     : : "v"(lane_off), "s"(rsrc), "s"(soff), "s"(lds) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 3\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                     : : "v"(lane_off), "s"(rsrc), "s"(soff), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void blds4(v4i rsrc, unsigned lane_off, unsigned soff, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 3\n\tbuffer_load_dword %0, %1, %2 offen lds"
                 : : "v"(lane_off), "s"(rsrc), "s"(soff), "s"(lds) : "memory", "m0");
}
// Raw buffer descriptor (stride 0, 32-bit data format) of `bytes` < 2^31 bytes at `p`; both wave-uniform.
__device__ __forceinline__ v4i buffer_desc(const uint8_t* p, unsigned bytes)
{
    const uint64_t a = (uint64_t)p;
    v4i r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)((unsigned)(a >> 32) & 0xFFFFu));
    r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    r[3] = 0x00020000;
    return r;
}
// s_waitcnt vmcnt(n), other counters untouched (gfx9 encoding: vmcnt[3:0], expcnt[6:4], lgkmcnt[11:8], vmcnt[5:4] in [15:14])
#define SNIP_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | ((((n) >> 4) & 3) << 14))
#define SNIP_BAR() do { __builtin_amdgcn_sched_barrier(0); __builtin_amdgcn_s_barrier(); __builtin_amdgcn_sched_barrier(0); } while (0)

// Swizzle: chunk position p of `row` holds logical chunk p ^ f(row); f makes the 16/CPR rows that share
// a 256-byte bank span use different positions.
template <int SB> __device__ __forceinline__ int swz(int row)
{
    constexpr int CPR = SB / 16;
    return (row / (16 / CPR)) % CPR;
}

// Chunk offsets (bytes inside a row block) a lane reads for MFMA step ks: FP8 two 16-byte chunks
// (bytes [16g,16g+16) and [32+16g, ...) of the step's 64-byte slab), FP4 one (bytes [16g, 16g+16) of
// the step's 32-byte slab).
template <int F, int SB, int KS>
__device__ __forceinline__ void frag_offsets(int r32, int g, int* off)
{
    const int f = swz<SB>(r32);          // row-block bases are multiples of 32 rows: f depends on r32 only
    constexpr int NC = F == kFP8 ? 2 * KS : KS;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        const int c = F == kFP8 ? ((k >> 1) * 4 + (k & 1) * 2 + g) : (k * 2 + g);
        off[k] = r32 * SB + ((c ^ f) * 16);
    }
}

template <int F>
__device__ __forceinline__ v8i read_frag(const uint8_t* tile, int rowblock_off, const int* off, int ks)
{
    v8i f = {0, 0, 0, 0, 0, 0, 0, 0};
    if (F == kFP8) {
        const uint4 a = *reinterpret_cast<const uint4*>(tile + rowblock_off + off[ks * 2 + 0]);
        const uint4 b = *reinterpret_cast<const uint4*>(tile + rowblock_off + off[ks * 2 + 1]);
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    } else {
        const uint4 a = *reinterpret_cast<const uint4*>(tile + rowblock_off + off[ks]);
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    }
    return f;
}

// Dispatch id -> tile.  Workgroups are dealt round-robin to the 8 XCDs, so ids u, u + 8, u + 16, ... share an L2:
// each XCD gets a contiguous run of the tile sequence, and the sequence walks bands of 4 tile rows column by
// column, so that the 32 tiles an XCD works on at a time are a 4 x 8 patch (4 + 8 operand slabs for 32 tiles).
__device__ __forceinline__ void tile_of(int u, int nblk, int tiles_i, int tiles_j, int& ti, int& tj)
{
    int bid = u;
    const int per = nblk / 8;
    if (bid < per * 8) bid = (bid % 8) * per + bid / 8;
    const int band = 4;
    const int band_sz = band * tiles_j;
    const int b0 = bid / band_sz;
    const int rem = bid - b0 * band_sz;
    const int rows_in_band = min(band, tiles_i - b0 * band);
    ti = b0 * band + rem % rows_in_band;
    tj = rem / rows_in_band;
}

// 16 bytes of a result, streaming ("nt") or plain.  Plain stores take room in the memory-side cache (256 MB) from the quantized
// operands of the GEMMs that follow and leave the L2s dirty lines, which the end of a kernel writes out with the chip idle: from the last
// store of a launch (17 MB) to the first instruction of the next one it was 3.4 us with plain stores and is 1.5 with these.  Plain ->
// streaming, GEMMs alone, us: [4096 x 2048 x 2048] FP4 16.0 -> 13.7, FP8 22.4 -> 18.8, [8192 x 3072 x 3072] FP4 58.5 -> 51.9, [2048 x 4096 x 4096]
// FP8 39.7 -> 36.2, fp32 42.2 -> 36.8; random calls on operands from memory 7 % on average (30 % ... -3 %), on one buffer again and again 2 %.
// Write-through besides ("sc1 nt") shortens the gap to 1.3 us, but tiles that follow each other wait for it (blocks of the 70B and 7B
// shapes 0.4 % slower, 1B 0.4 % faster).  Which results, and what their readers pay: streams_result (picks.h).
// (The empty statements keep the compiler from making one plain store of the two kinds.)
__device__ __forceinline__ void store16(v4u v, uint8_t* p, bool stream = true)
{
    if (stream) {
        __builtin_nontemporal_store(v, reinterpret_cast<v4u*>(p));
    } else {
        asm volatile("");
        *reinterpret_cast<v4u*>(p) = v;
        asm volatile("");
    }
}

// Result of a wave's 64 x 64 block with its corner at (i0, j0), of a kernel whose first MFMA operand is the B tile: turned through
// 4 KB of LDS of the wave's own, 32 rows x 128 bytes at a time.  16-byte piece c of row r sits at position c ^ (r / 2 % 8) (bf16: a
// piece is written in two halves).  `interior`: no row or column lies outside; STREAM: see store16.
template <bool OUT_F32, bool STREAM>
__device__ __forceinline__ void store_block64(const v16f (&acc)[2][2], uint8_t* reg, int lane, void* c_out, int64_t ldc, int i0, int j0,
                                              int I, int J, bool interior)
{
    constexpr int ESZ = OUT_F32 ? 4 : 2;
    const int r32 = lane & 31, g = lane >> 5, f = (r32 >> 1) & 7;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int h = 0; h < (OUT_F32 ? 2 : 1); ++h) {
            if (OUT_F32) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4*>(reg + r32 * 128 + (((q * 2 + g) ^ f) * 16)) =
                        make_float4(acc[m][h][4 * q], acc[m][h][4 * q + 1], acc[m][h][4 * q + 2], acc[m][h][4 * q + 3]);
            } else {
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float2_t lo = {acc[m][n][4 * q], acc[m][n][4 * q + 1]}, hi = {acc[m][n][4 * q + 2], acc[m][n][4 * q + 3]};
                        const bf16x2 blo = __builtin_convertvector(lo, bf16x2), bhi = __builtin_convertvector(hi, bf16x2);
                        *reinterpret_cast<uint2*>(reg + r32 * 128 + (((n * 4 + q) ^ f) * 16) + 8 * g) =
                            make_uint2(__builtin_bit_cast(unsigned, blo), __builtin_bit_cast(unsigned, bhi));
                    }
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int row = it * 8 + lane / 8, c = lane % 8;
                const v4u v = *reinterpret_cast<const v4u*>(reg + row * 128 + ((c ^ ((row >> 1) & 7)) * 16));
                const int i = i0 + m * 32 + row, j = j0 + h * 32 + c * (16 / ESZ);
                uint8_t* p = reinterpret_cast<uint8_t*>(c_out) + ((int64_t)i * ldc + j) * ESZ;
                if (interior) {
                    store16(v, p, STREAM);
                } else if (i < I) {
                    if (j + 16 / ESZ <= J) {
                        store16(v, p, STREAM);
                    } else if (j < J) {
                        for (int e = 0; e < 16 / ESZ; ++e)
                            if (j + e < J) {
                                if (OUT_F32) reinterpret_cast<unsigned*>(p)[e] = v[e];
                                else reinterpret_cast<uint16_t*>(p)[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
                            }
                    }
                }
            }
        }
}

}  // namespace
}  // namespace snip

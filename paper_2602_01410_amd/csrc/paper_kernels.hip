// The paper's own quantization recipe (SNIP Sec. 2.3 and Sec. 5.1): a real-valued scale
// s = FPX_MAX / max|x| per scaling group, codes = RNE_FPX(x * s), value seen by the GEMM = code / s;
// groups are 1x128 tiles (activations, gradients) or 128x128 blocks (weights), both in the STORED
// orientation (blocks along rows, or down columns with the result stored transposed).
//
// Unlike the power-of-two block scales of the main path, s and x * s are not exact, so their precision is
// part of the definition: fp32, one correctly rounded division and one correctly rounded product, which is
// what these kernels compute (v_div_* sequence, v_mul_f32) before gfx950's v_cvt_scalef32_pk_{fp8,fp4}_f32
// rounds to the element format (scale operand 1.0; the FP8 form does not saturate, so x * s is clamped to
// +-448 first: the product can exceed 448 by one rounding).
//
// Kernels: quantize along rows (tile maxima by a 16-lane DPP reduction inside the pass), quantize down
// columns (a lane owns two columns; the four waves of a workgroup exchange their maxima), 128x128 blocks along rows (a workgroup
// owns a block), and the matching statistics kernels (both formats from one read).  All are streaming kernels bound by HBM bandwidth or VALU rate.
#include "snip_internal.h"

namespace snip {
namespace {

typedef short short2_t __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Streaming (non-temporal) loads for sources that are read once.
__device__ __forceinline__ uint4 ld16_stream(const void* p)
{
    const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ unsigned ld4_stream(const void* p) { return __builtin_nontemporal_load(reinterpret_cast<const unsigned*>(p)); }

constexpr int kGroup = 128;              // scaling-group extent along the blocked dimension
constexpr int kSeg = 512;                // elements of a row one wave handles per load
constexpr int kUnroll = 4;               // rows in flight per wave (row kernels)
constexpr int kColsPerWave = 128;        // columns per unit (column kernels)

template <int FMT> __device__ __forceinline__ float fmt_max() { return FMT == kFP8 ? 448.f : 6.f; }

__device__ __forceinline__ unsigned pk_max_u16(unsigned a, unsigned b)
{
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a),
                                                                  __builtin_bit_cast(ushort2_t, b)));
}
__device__ __forceinline__ unsigned umax(unsigned a, unsigned b) { return a > b ? a : b; }

// Scale of a group from the 15 magnitude bits of its bf16 maximum: MAX / amax in fp32, 1 for an all-zero
// group, capped at 2^126 (a group of denormal-sized values would overflow it), NaN for a group that holds
// an infinity or a NaN.
template <int FMT>
__device__ __forceinline__ float group_scale(unsigned amax_bits)
{
    if (amax_bits >= 0x7F80u) return __builtin_nanf("");
    if (amax_bits == 0u) return 1.f;
    const float s = __fdiv_rn(fmt_max<FMT>(), __uint_as_float(amax_bits << 16));
    return s <= 0x1p126f ? s : 0x1p126f;
}

// Magnitude bits of the largest of the 8 bf16 values of one 16-byte load.
__device__ __forceinline__ unsigned amax8(const uint4& v)
{
    const unsigned m = pk_max_u16(pk_max_u16(v.x & 0x7FFF7FFFu, v.y & 0x7FFF7FFFu),
                                  pk_max_u16(v.z & 0x7FFF7FFFu, v.w & 0x7FFF7FFFu));
    return umax(m & 0xFFFFu, m >> 16);
}
// Maximum over the 16 lanes of a DPP row: quad permutes, then rotations by 4 and 8 inside the row.
__device__ __forceinline__ unsigned row16_max(unsigned m)
{
    m = umax(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, true));     // quad_perm [1,0,3,2]
    m = umax(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, true));     // quad_perm [2,3,0,1]
    m = umax(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x124, 0xF, 0xF, true));    // row_ror:4
    m = umax(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x128, 0xF, 0xF, true));    // row_ror:8
    return m;
}

// x * s for the two bf16 halves of a word.
__device__ __forceinline__ void scaled2(unsigned w, float s, float& lo, float& hi)
{
    lo = __fmul_rn(__uint_as_float(w << 16), s);
    hi = __fmul_rn(__uint_as_float(w & 0xFFFF0000u), s);
}
__device__ __forceinline__ float clamp448(float t) { return fminf(fmaxf(t, -448.f), 448.f); }

// Four words (8 consecutive elements) -> 8 FP8 bytes (c0, c1) or 8 FP4 nibbles (c0).
template <int FMT>
__device__ __forceinline__ void encode8(const unsigned* w, float s, unsigned& c0, unsigned& c1)
{
    float t[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) scaled2(w[i], s, t[2 * i], t[2 * i + 1]);
    if (FMT == kFP8) {
        short2_t a = {0, 0}, b = {0, 0};
        a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(a, clamp448(t[0]), clamp448(t[1]), 1.0f, false);
        a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(a, clamp448(t[2]), clamp448(t[3]), 1.0f, true);
        b = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(b, clamp448(t[4]), clamp448(t[5]), 1.0f, false);
        b = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(b, clamp448(t[6]), clamp448(t[7]), 1.0f, true);
        c0 = __builtin_bit_cast(unsigned, a);
        c1 = __builtin_bit_cast(unsigned, b);
    } else {
        unsigned r = 0;
        r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[0], t[1], 1.0f, 0);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[2], t[3], 1.0f, 1);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[4], t[5], 1.0f, 2);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[6], t[7], 1.0f, 3);
        c0 = r;
        c1 = 0;
    }
}

// Error sums of 8 elements for one format: (code / s - x)^2 with code = RNE(x * s); also sum x^2 if asked.
template <int FMT>
__device__ __forceinline__ void err8(const unsigned* w, float s, float inv_s, float& s0, float& se, bool want_s0)
{
    unsigned c0, c1;
    encode8<FMT>(w, s, c0, c1);
    float2_t qq[4];
    if (FMT == kFP8) {
        qq[0] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c0, 1.0f, false);
        qq[1] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c0, 1.0f, true);
        qq[2] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c1, 1.0f, false);
        qq[3] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c1, 1.0f, true);
    } else {
        qq[0] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c0, 1.0f, 0);
        qq[1] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c0, 1.0f, 1);
        qq[2] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c0, 1.0f, 2);
        qq[3] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c0, 1.0f, 3);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float2_t q = qq[i];
        const float xl = __uint_as_float(w[i] << 16), xh = __uint_as_float(w[i] & 0xFFFF0000u);
        const float dl = q[0] * inv_s - xl, dh = q[1] * inv_s - xh;
        se = fmaf(dl, dl, se);
        se = fmaf(dh, dh, se);
        if (want_s0) { s0 = fmaf(xl, xl, s0); s0 = fmaf(xh, xh, s0); }
    }
}

// Unit of workgroup b.  Workgroups b, b + 8, ... run on one XCD: of every 8 * kAdjacent units each XCD takes kAdjacent in a row.
constexpr int kAdjacent = 4;
__device__ __forceinline__ int unit_of(int b, int units)
{
    const int b0 = b / (8 * kAdjacent) * (8 * kAdjacent);
    return b0 + 8 * kAdjacent <= units ? b0 + (b & 7) * kAdjacent + ((b - b0) >> 3) : b;
}

// ------------------------------------------------------------------------------------------
// 128x128 blocks, codes along rows.  A workgroup owns a block, its four waves 32 rows each; 16 lanes hold a row's 128 columns,
// eight 16-byte loads are in flight.  The block stays in registers while the waves exchange their maxima, so the source is read
// once.  Against a pass for the maxima and a pass for the codes, us per call on sources in memory: [8192 x 2048] FP8 20.7 -> 11.6,
// [4096 x 8192] 36 -> 22, FP4 31 -> 19, [16384 x 11008] 173 -> 106 and 145 -> 80; statistics (with one second stage for the three
// sums instead of three) [8192 x 2048] 29 -> 14.5, [16384 x 11008] 158 -> 98.
// MODE as below; scales [row / 128][col / 128].
// ------------------------------------------------------------------------------------------
template <int FMT, int MODE>
__global__ __launch_bounds__(256) void paper_block_kernel(const uint16_t* __restrict__ x, int rows, int cols, int64_t ld,
                                                          uint8_t* __restrict__ codes, float* __restrict__ scales,
                                                          float* __restrict__ partials)
{
    __shared__ unsigned maxima[2][kWavesPerBlock];
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ncb = cols / kGroup, units = (rows + kGroup - 1) / kGroup * ncb;
    float s0 = 0.f, e4 = 0.f, e8 = 0.f;
    int turn = 0;
    for (int b = blockIdx.x; b < units; b += gridDim.x, turn ^= 1) {
        const int u = unit_of(b, units);
        const int br = u / ncb, bc = u - br * ncb;
        const int col = bc * kGroup + (lane & 15) * 8, row0 = br * kGroup + wib * 32 + (lane >> 4);
        // rows past the end re-read the last row: a maximum does not mind, and nothing else comes of them
        uint4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = ld16_stream(x + (int64_t)min(row0 + 4 * j, rows - 1) * ld + col);
        unsigned m = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) m = umax(m, amax8(v[j]));
        m = row16_max(m);
        m = umax(m, (unsigned)__shfl_xor((int)m, 16, 64));
        m = umax(m, (unsigned)__shfl_xor((int)m, 32, 64));
        if (lane == 0) maxima[turn][wib] = m;
        __syncthreads();                                 // (two sets: the next block's maxima do not wait for readers of this one's)
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) m = umax(m, maxima[turn][w]);
        const float s8 = MODE == 1 || FMT == kFP8 ? group_scale<kFP8>(m) : 1.f, s4 = MODE == 1 || FMT == kFP4 ? group_scale<kFP4>(m) : 1.f;
        if (MODE == 0) {
            const float s = FMT == kFP8 ? s8 : s4;
            const bool bad = s != s;
            if (threadIdx.x == 0) scales[u] = s;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const unsigned w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
                unsigned c0, c1;
                encode8<FMT>(w, s, c0, c1);
                if (bad) { c0 = 0; c1 = 0; }
                const int64_t e0 = (int64_t)(row0 + 4 * j) * cols + col;
                if (row0 + 4 * j < rows) {
                    if (FMT == kFP8) *reinterpret_cast<uint2*>(codes + e0) = make_uint2(c0, c1);
                    else             *reinterpret_cast<unsigned*>(codes + (e0 >> 1)) = c0;
                }
            }
        } else {
            const float i8 = __fdiv_rn(1.f, s8), i4 = __fdiv_rn(1.f, s4);
            // (at most 16 elements are added one by one before their sums meet those of the rows before: the rounding of a long
            // chain leans one way)
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                float t0 = 0.f, t4 = 0.f, t8 = 0.f;
#pragma unroll
                for (int j = 2 * h; j < 2 * h + 2; ++j) {
                    const unsigned w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
                    float dummy = 0.f;
                    if (row0 + 4 * j < rows) {
                        err8<kFP8>(w, s8, i8, t0, t8, true);
                        err8<kFP4>(w, s4, i4, dummy, t4, false);
                    }
                }
                s0 += t0; e4 += t4; e8 += t8;
            }
        }
    }
    if (MODE == 1) {
        const int wave = blockIdx.x * kWavesPerBlock + wib;
        s0 = wave_sum(s0); e4 = wave_sum(e4); e8 = wave_sum(e8);
        if (lane == 0) { partials[wave] = s0; partials[kStreamWaves + wave] = e4; partials[2 * kStreamWaves + wave] = e8; }
    }
}

// ------------------------------------------------------------------------------------------
// 1x128 tiles along rows.  A lane owns 8 consecutive elements, 16 lanes own a tile; its scale goes to scales [row][col / 128].
// MODE 0: write codes (+ tile scales).  MODE 1: statistics of both formats, nothing written but partials.
// ------------------------------------------------------------------------------------------
template <int FMT, int MODE>
__global__ __launch_bounds__(256) void paper_row_kernel(const uint16_t* __restrict__ x, int rows, int cols, int64_t ld,
                                                        uint8_t* __restrict__ codes, float* __restrict__ scales,
                                                        float* __restrict__ partials)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
    const int nwaves = gridDim.x * kWavesPerBlock;
    const int spr = (cols + kSeg - 1) / kSeg;
    const int units = ((rows + kUnroll - 1) / kUnroll) * spr;
    const int ng = cols / kGroup;
    float s0 = 0.f, e4 = 0.f, e8 = 0.f;
    for (int u = wave; u < units; u += nwaves) {
        const int rg = u / spr;
        const int col = (u - rg * spr) * kSeg + lane * 8;
        uint4 v[kUnroll];
        bool act[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            const int row = rg * kUnroll + j;
            act[j] = row < rows && col < cols;
            v[j] = make_uint4(0, 0, 0, 0);
            if (act[j]) v[j] = ld16_stream(x + (int64_t)row * ld + col);
        }
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            const int row = rg * kUnroll + j;
            const unsigned w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
            const int gidx = row * ng + (col >> 7);
            float s8 = 1.f, s4 = 1.f;
            const unsigned am = row16_max(amax8(v[j]));
            if (MODE == 1 || FMT == kFP8) s8 = group_scale<kFP8>(am);
            if (MODE == 1 || FMT == kFP4) s4 = group_scale<kFP4>(am);
            if (MODE == 0) {
                const float s = FMT == kFP8 ? s8 : s4;
                const bool bad = s != s;
                unsigned c0, c1;
                encode8<FMT>(w, s, c0, c1);
                if (bad) { c0 = 0; c1 = 0; }
                const int64_t e0 = (int64_t)row * cols + col;
                if (act[j]) {
                    if (FMT == kFP8) *reinterpret_cast<uint2*>(codes + e0) = make_uint2(c0, c1);
                    else             *reinterpret_cast<unsigned*>(codes + (e0 >> 1)) = c0;
                    if ((lane & 15) == 0) scales[gidx] = s;
                }
            } else if (act[j]) {
                float dummy = 0.f;
                err8<kFP8>(w, s8, __fdiv_rn(1.f, s8), s0, e8, true);
                err8<kFP4>(w, s4, __fdiv_rn(1.f, s4), dummy, e4, false);
            }
        }
    }
    if (MODE == 1) {
        s0 = wave_sum(s0); e4 = wave_sum(e4); e8 = wave_sum(e8);
        if (lane == 0) { partials[wave] = s0; partials[kStreamWaves + wave] = e4; partials[2 * kStreamWaves + wave] = e8; }
    }
}

// ------------------------------------------------------------------------------------------
// Blocks down columns, result stored transposed.  A workgroup owns 128 columns x 128 rows (one tile per column), its four
// waves 32 rows each; a lane owns two adjacent columns.  The rows stay in registers: one read serves the column maxima,
// which the waves exchange through LDS, and the encoding.  The codes are staged in LDS as a
// [128 stored rows][ROWB] image (ROWB = 128 bytes FP8, 64 bytes FP4) whose 16-byte chunks are XOR-swizzled,
// then stored with 16 bytes per lane so that whole 128- / 64-byte runs are written.
// A wave per unit, which held its 128 rows in 128 registers, left half of the SIMDs without a wave on a [4096 x 2048] tensor:
// 11.7 -> 8.1 us; [8192 x 2048] in blocks 15.2 -> 11.8, [4096 x 8192] 27.4 -> 23.1 (FP8, kernel trace).  Four column groups in a
// row go to one XCD, 1 KB of a source row: dealt one by one (the same calls, us: a wave per unit / one by one / four) [16384 x
// 4096] FP4 32.8 / 35.6 / 32.9, [4096 x 28672] FP4 55.7 / 60.5 / 57.6, [12288 x 8192] FP8 63.8 / 56.8 / 54.9.  A wave per unit
// is still the faster one with FP4 codes of very large tensors of some pitches ([24576 x 4096] 48.3 against 51.9, [8192 x 28672]
// 117 against 137; not so [16384 x 11008], 101 against 93).
// ------------------------------------------------------------------------------------------
template <int FMT>
__device__ __forceinline__ void encode_column(const unsigned* v, int half, float s, uint8_t* __restrict__ lds_row,
                                              int k, int swz)
{
    // rows 2j, 2j+1 of this column are adjacent in the stored row
    float t[32];
#pragma unroll
    for (int i = 0; i < 32; ++i)
        t[i] = __fmul_rn(half ? __uint_as_float(v[i] & 0xFFFF0000u) : __uint_as_float(v[i] << 16), s);
    const bool bad = s != s;
    if (FMT == kFP8) {
        unsigned c[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            short2_t a = {0, 0};
            a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(a, clamp448(t[4 * q]), clamp448(t[4 * q + 1]), 1.0f, false);
            a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(a, clamp448(t[4 * q + 2]), clamp448(t[4 * q + 3]), 1.0f, true);
            c[q] = bad ? 0u : __builtin_bit_cast(unsigned, a);
        }
        *reinterpret_cast<uint4*>(lds_row + (((k * 2 + 0) ^ swz) * 16)) = make_uint4(c[0], c[1], c[2], c[3]);
        *reinterpret_cast<uint4*>(lds_row + (((k * 2 + 1) ^ swz) * 16)) = make_uint4(c[4], c[5], c[6], c[7]);
    } else {
        unsigned c[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            unsigned r = 0;
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[8 * q], t[8 * q + 1], 1.0f, 0);
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[8 * q + 2], t[8 * q + 3], 1.0f, 1);
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[8 * q + 4], t[8 * q + 5], 1.0f, 2);
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[8 * q + 6], t[8 * q + 7], 1.0f, 3);
            c[q] = bad ? 0u : r;
        }
        *reinterpret_cast<uint4*>(lds_row + ((k ^ swz) * 16)) = make_uint4(c[0], c[1], c[2], c[3]);
    }
}

// Error sums of one column's 32 rows for one format.
template <int FMT>
__device__ __forceinline__ void err_column(const unsigned* v, int half, float s, float inv_s, float& s0, float& se, bool want_s0)
{
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        float x[4], t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[i] = half ? __uint_as_float(v[4 * q + i] & 0xFFFF0000u) : __uint_as_float(v[4 * q + i] << 16);
            t[i] = __fmul_rn(x[i], s);
        }
        float2_t q01, q23;
        if (FMT == kFP8) {
            short2_t a = {0, 0};
            a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(a, clamp448(t[0]), clamp448(t[1]), 1.0f, false);
            a = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(a, clamp448(t[2]), clamp448(t[3]), 1.0f, true);
            const unsigned c = __builtin_bit_cast(unsigned, a);
            q01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c, 1.0f, false);
            q23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c, 1.0f, true);
        } else {
            unsigned r = 0;
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[0], t[1], 1.0f, 0);
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, t[2], t[3], 1.0f, 1);
            q01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(r, 1.0f, 0);
            q23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(r, 1.0f, 1);
        }
        const float d0 = q01[0] * inv_s - x[0], d1 = q01[1] * inv_s - x[1];
        const float d2 = q23[0] * inv_s - x[2], d3 = q23[1] * inv_s - x[3];
        se = fmaf(d0, d0, se); se = fmaf(d1, d1, se); se = fmaf(d2, d2, se); se = fmaf(d3, d3, se);
        if (want_s0) { s0 = fmaf(x[0], x[0], s0); s0 = fmaf(x[1], x[1], s0); s0 = fmaf(x[2], x[2], s0); s0 = fmaf(x[3], x[3], s0); }
    }
}

template <int FMT, bool BLOCKS, int MODE>
__global__ __launch_bounds__(256) void paper_col_kernel(const uint16_t* __restrict__ x, int rows, int cols, int64_t ld,
                                                        uint8_t* __restrict__ codes, float* __restrict__ scales,
                                                        float* __restrict__ partials)
{
    constexpr int ROWB = FMT == kFP8 ? 128 : 64;
    constexpr int CPR = ROWB / 16;
    __shared__ __attribute__((aligned(16))) uint8_t reg[MODE == 0 ? kColsPerWave * ROWB : 16];
    __shared__ unsigned maxima[kWavesPerBlock][64];
    const int lane = threadIdx.x & 63;
    const int k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // this wave's rows: 32 k ... 32 k + 31 of the unit
    const int wave = blockIdx.x * kWavesPerBlock + k;
    const int ncg = (cols + kColsPerWave - 1) / kColsPerWave;
    const int nru = rows / kGroup;                       // rows is a multiple of 128
    const int units = ncg * nru;
    const int64_t out_row_bytes = FMT == kFP8 ? rows : rows / 2;
    float s0 = 0.f, e4 = 0.f, e8 = 0.f;
    for (int b = blockIdx.x; b < units; b += gridDim.x) {
        const int u = unit_of(b, units);
        const int ru = u / ncg, cg = u - ru * ncg;
        const int c = cg * kColsPerWave + lane * 2;
        const bool act = c < cols;
        // The loads carry no condition (a lane past the last column reads column 0 of the same rows and is zeroed under
        // a wave-uniform test), so that all of them are in flight together.
        const uint16_t* const base = x + ((int64_t)ru * kGroup + k * 32) * ld + (act ? c : 0);
        unsigned v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = ld4_stream(base + (int64_t)i * ld);
        if ((cg + 1) * kColsPerWave > cols) {
#pragma unroll
            for (int i = 0; i < 32; ++i) v[i] = act ? v[i] : 0u;
        }
        unsigned m = 0;
#pragma unroll
        for (int i = 0; i < 32; ++i) m = pk_max_u16(m, v[i] & 0x7FFF7FFFu);
        maxima[k][lane] = m;
        __syncthreads();                                 // (the staging area is free again, too)
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) m = pk_max_u16(m, maxima[w][lane]);
        float s8[2] = {1.f, 1.f}, s4[2] = {1.f, 1.f};
        if (BLOCKS) {
            // the unit is one 128 x 128 block: its maximum is the maximum over the lanes
            unsigned bm = umax(m & 0xFFFFu, m >> 16);
            for (int off = 32; off > 0; off >>= 1) bm = umax(bm, (unsigned)__shfl_xor((int)bm, off, 64));
            if (MODE == 1 || FMT == kFP8) s8[0] = s8[1] = group_scale<kFP8>(bm);
            if (MODE == 1 || FMT == kFP4) s4[0] = s4[1] = group_scale<kFP4>(bm);
            if (MODE == 0 && threadIdx.x == 0) scales[cg * nru + ru] = FMT == kFP8 ? s8[0] : s4[0];   // stored orientation: [column group][row group]
        } else {
            const unsigned am[2] = {m & 0xFFFFu, m >> 16};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (MODE == 1 || FMT == kFP8) s8[h] = group_scale<kFP8>(am[h]);
                if (MODE == 1 || FMT == kFP4) s4[h] = group_scale<kFP4>(am[h]);
            }
            if (MODE == 0 && act && k == 0) {
                scales[(int64_t)c * nru + ru] = FMT == kFP8 ? s8[0] : s4[0];
                scales[(int64_t)(c + 1) * nru + ru] = FMT == kFP8 ? s8[1] : s4[1];
            }
        }
        const int swz = lane & (CPR - 1);
        if (MODE == 0) {
            encode_column<FMT>(v, 0, FMT == kFP8 ? s8[0] : s4[0], reg + (2 * lane) * ROWB, k, swz);
            encode_column<FMT>(v, 1, FMT == kFP8 ? s8[1] : s4[1], reg + (2 * lane + 1) * ROWB, k, swz);
        } else if (act) {
            float dummy = 0.f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                err_column<kFP8>(v, h, s8[h], __fdiv_rn(1.f, s8[h]), s0, e8, true);
                err_column<kFP4>(v, h, s4[h], __fdiv_rn(1.f, s4[h]), dummy, e4, false);
            }
        }
        __syncthreads();                                 // the codes are staged; everyone has read the maxima
        if (MODE == 0) {
#pragma unroll
            for (int it = k; it < kColsPerWave * CPR / 64; it += kWavesPerBlock) {
                const int idx = it * 64 + lane;
                const int row = idx / CPR, chunk = idx % CPR;
                const uint4 val = *reinterpret_cast<const uint4*>(reg + row * ROWB + ((chunk ^ ((row >> 1) & (CPR - 1))) * 16));
                const int cc = cg * kColsPerWave + row;
                if (cc < cols)
                    *reinterpret_cast<uint4*>(codes + (int64_t)cc * out_row_bytes + (int64_t)ru * ROWB + chunk * 16) = val;
            }
        }
    }
    if (MODE == 1) {
        s0 = wave_sum(s0); e4 = wave_sum(e4); e8 = wave_sum(e8);
        if (lane == 0) { partials[wave] = s0; partials[kStreamWaves + wave] = e4; partials[2 * kStreamWaves + wave] = e8; }
    }
}

// Workgroups for `units` units of a workgroup each: one per unit, as long as a launch takes them.  Statistics need four
// partial-sum slots per workgroup: equal shares then.
int blocks_for(int64_t units, bool stats)
{
    const int64_t most = stats ? kStreamBlocks : kMostBlocks, share = (units + most - 1) / most;
    return units <= 0 ? 1 : (int)((units + share - 1) / share);
}

template <int FMT, bool BLOCKS, int MODE>
int launch_one(const PaperArgs& a, float* partials, hipStream_t s)
{
    const int64_t groups = ((a.rows + kGroup - 1) / kGroup) * ((a.cols + kGroup - 1) / kGroup);
    int blocks;
    if (a.axis != 0) {
        blocks = blocks_for(groups, MODE == 1);
        hipLaunchKernelGGL((paper_col_kernel<FMT, BLOCKS, MODE>), dim3(blocks), dim3(256), 0, s,
                           a.x, (int)a.rows, (int)a.cols, a.ld, a.codes, a.scales, partials);
    } else if (BLOCKS) {
        blocks = blocks_for(groups, MODE == 1);
        hipLaunchKernelGGL((paper_block_kernel<FMT, MODE>), dim3(blocks), dim3(256), 0, s,
                           a.x, (int)a.rows, (int)a.cols, a.ld, a.codes, a.scales, partials);
    } else {
        const int64_t units = ((a.rows + kUnroll - 1) / kUnroll) * ((a.cols + kSeg - 1) / kSeg);
        blocks = blocks_for((units + kWavesPerBlock - 1) / kWavesPerBlock, MODE == 1);
        hipLaunchKernelGGL((paper_row_kernel<FMT, MODE>), dim3(blocks), dim3(256), 0, s,
                           a.x, (int)a.rows, (int)a.cols, a.ld, a.codes, a.scales, partials);
    }
    return blocks;
}

}  // namespace

// (room for two scales per group as well: earlier forms of the statistics kept them there, and callers have allocated it)
size_t paper_workspace_bytes(int64_t rows, int64_t cols)
{
    const size_t nblocks = (size_t)((rows + kGroup - 1) / kGroup) * (size_t)((cols + kGroup - 1) / kGroup);
    return 3 * (size_t)kStreamWaves * sizeof(float) + 2 * nblocks * sizeof(float);
}

// Workspace layout: [3][kStreamWaves] float partial sums.
hipError_t launch_paper(const PaperArgs& a, hipStream_t s)
{
    const bool stats = a.stats != nullptr;
    float* partials = (float*)a.workspace;
    int blocks = 0;
    if (a.rows != 0 && a.cols != 0) {
        if (stats) {
            blocks = a.blocks ? launch_one<kFP8, true, 1>(a, partials, s) : launch_one<kFP8, false, 1>(a, partials, s);
        } else if (a.fmt == kFP8) {
            blocks = a.blocks ? launch_one<kFP8, true, 0>(a, partials, s) : launch_one<kFP8, false, 0>(a, partials, s);
        } else {
            blocks = a.blocks ? launch_one<kFP4, true, 0>(a, partials, s) : launch_one<kFP4, false, 0>(a, partials, s);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return stats ? launch_sum_partials(partials, (int64_t)blocks * kWavesPerBlock, a.stats, s, 3, kStreamWaves) : hipSuccess;
}

}  // namespace snip

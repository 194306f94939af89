// Streaming kernels: bf16 -> block-scaled FP8/FP4 quantization (SNIP Sec. 2.3, applied to
// the tensors Sec. 2.2 names) and the quantization-error statistics of Sec. 3.1 Step 1
// (row-wise form: Sec. 5.3).  All of them are bound by HBM bandwidth: one 2-byte read per
// element, 0.53 / 1.03 bytes written (FP4 / FP8), and a handful of VALU ops per element.
//
// A block of 32 elements is handled as follows.
//   amax    : integer maximum of the bf16 magnitude bits (order-preserving for non-negative
//             floats), packed 2 x u16 per VGPR.
//   scale   : integer function of amax's exponent and mantissa fields (no log2).
//   cast    : gfx950's v_cvt_scalef32_pk_{fp8,fp4}_bf16, which divides by the power of two
//             in the scale operand's exponent field and rounds to nearest even.  The FP4
//             form saturates; the FP8 form does not, so under the floor rule magnitudes are
//             clamped to 448 * 2^e first (the no-overflow rule never exceeds it).
//   error   : v_cvt_scalef32_pk_f32_{fp8,fp4} gives q(x) exactly in fp32; the difference to x
//             (exact in fp32) is squared and summed in fp32 per lane, then per wave, and the
//             per-wave partials are summed in double by a single-block kernel in fixed order.
#include "snip_internal.h"
#include "picks.h"
#include <cstdlib>
#include <cstring>

namespace snip {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

template <int FMT> struct Fmt;
template <> struct Fmt<kFP8> { static constexpr int emax = 8; static constexpr unsigned mmax = 0x60; };  // 448 = 1.75 * 2^8
template <> struct Fmt<kFP4> { static constexpr int emax = 2; static constexpr unsigned mmax = 0x40; };  // 6   = 1.5  * 2^2

// Source loads.  A source line is read once and never again, so its load carries the streaming hint (measured:
// quantize ROW 4.7 -> 5.8 TB/s, COL 4.0 -> 4.75 TB/s of algorithmic bytes on a 361 MB tensor).  Where the one-pass kernel
// for both orientations reads every line twice, the second time out of cache, both of its reads are plain loads
// (with the hint on either one the kernel got 4-6 % slower).
typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld16(const uint16_t* p)
{
    const v4u_t v = __builtin_nontemporal_load(reinterpret_cast<const v4u_t*>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ unsigned ld4(const uint16_t* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const unsigned*>(p));
}

__device__ __forceinline__ unsigned pk_max_u16(unsigned a, unsigned b)
{
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a),
                                                                  __builtin_bit_cast(ushort2_t, b)));
}
__device__ __forceinline__ unsigned pk_min_u16(unsigned a, unsigned b)
{
    return __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(ushort2_t, a),
                                                                  __builtin_bit_cast(ushort2_t, b)));
}

// Maximum over the four lanes of a quad (DPP quad_perm [1,0,3,2] then [2,3,0,1]).
__device__ __forceinline__ unsigned quad_max(unsigned m)
{
    unsigned t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, true);
    m = m > t ? m : t;
    t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, true);
    return m > t ? m : t;
}

// E8M0 byte from the 15 magnitude bits of the block maximum; 0xFF for Inf/NaN.
template <int FMT, int RULE>
__device__ __forceinline__ unsigned scale_byte(unsigned amax_bits)
{
    // (rule 0: adding 0x7F - mmax carries into the exponent where the mantissa exceeds mmax)
    int b = (int)amax_bits + ((RULE == 0 ? 0x7F - (int)Fmt<FMT>::mmax : 0) - (Fmt<FMT>::emax << 7));
    b = b < 0 ? 0 : b;
    return amax_bits >= 0x7F80u ? 0xFFu : (unsigned)b >> 7;
}

// The conversion instructions read only the exponent field of their scale operand; the
// mantissa bit set here keeps byte 0 (2^-127) from being an all-zero word.
__device__ __forceinline__ float scale_operand(unsigned byte)
{
    return __uint_as_float((byte << 23) | 0x00400000u);
}

// Clamp both bf16 halves of w to magnitude <= 448 * 2^(byte-127) (floor rule, FP8 only).
__device__ __forceinline__ unsigned clamp_fp8(unsigned w, unsigned byte)
{
    const unsigned lim = ((byte + 8u) << 7) | 0x60u;
    const unsigned mag = pk_min_u16(w & 0x7FFF7FFFu, lim | (lim << 16));
    return mag | (w & 0x80008000u);
}

// A register with unspecified content, at no cost: the packing conversions below replace their destination piece by
// piece (two halves for FP8, four bytes for FP4) and keep the rest, so the value they start from never survives;
// starting from zero would cost a move per destination.
__device__ __forceinline__ unsigned any_value()
{
    unsigned r;
    asm volatile("" : "=v"(r));
    return r;
}

// Two bf16 pairs (4 elements) -> 4 FP8 bytes.
template <int RULE>
__device__ __forceinline__ unsigned enc8(unsigned w0, unsigned w1, float sc, unsigned byte)
{
    if (RULE == 1) { w0 = clamp_fp8(w0, byte); w1 = clamp_fp8(w1, byte); }
    short2_t r = __builtin_bit_cast(short2_t, any_value());
    r = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, __builtin_bit_cast(bf16x2, w0), sc, false);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, __builtin_bit_cast(bf16x2, w1), sc, true);
    return __builtin_bit_cast(unsigned, r);
}

// Four bf16 pairs (8 elements) -> 8 FP4 nibbles, element 0 in the lowest nibble.
__device__ __forceinline__ unsigned enc4(unsigned w0, unsigned w1, unsigned w2, unsigned w3, float sc)
{
    unsigned r = any_value();
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(r, __builtin_bit_cast(bf16x2, w0), sc, 0);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(r, __builtin_bit_cast(bf16x2, w1), sc, 1);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(r, __builtin_bit_cast(bf16x2, w2), sc, 2);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(r, __builtin_bit_cast(bf16x2, w3), sc, 3);
    return r;
}

// ---- stochastic rounding to FP4 (Sec. 5.1: FP4 output gradients are rounded probabilistically to the two
//      nearest values).  Definition: with lo <= |v| <= hi the neighbouring grid magnitudes of the scaled
//      element and p = (|v| - lo) / (hi - lo), the magnitude goes up iff rnd < floor(256 p), rnd being the
//      element's random byte: byte (i mod 8) of Threefry-2x32-20(counter = i div 8, key = seed), i the
//      element's row-major position in the stored matrix. ----

// Threefry-2x32, 20 rounds (Salmon et al., SC'11): adds, rotates and XORs only, which suits a VALU whose
// 32-bit multiplies run at quarter rate.
__device__ __forceinline__ unsigned rotl32(unsigned v, int r) { return (v << r) | (v >> (32 - r)); }
__device__ __forceinline__ void threefry2x32_20(unsigned c0, unsigned c1, unsigned k0, unsigned k1,
                                                unsigned& o0, unsigned& o1)
{
    constexpr int R[8] = {13, 15, 26, 6, 17, 29, 16, 24};
    const unsigned ks[3] = {k0, k1, 0x1BD11BDAu ^ k0 ^ k1};
    unsigned x0 = c0 + ks[0], x1 = c1 + ks[1];
#pragma unroll
    for (int r = 0; r < 20; ++r) {
        x0 += x1;
        x1 = rotl32(x1, R[r % 8]) ^ x0;
        if (r % 4 == 3) {
            const int inj = r / 4 + 1;
            x0 += ks[inj % 3];
            x1 += ks[(inj + 1) % 3] + (unsigned)inj;
        }
    }
    o0 = x0; o1 = x1;
}

// The rule is carried out by gfx950's stochastic-rounding conversion v_cvt_scalef32_sr_pk_fp4_f32.  What that
// instruction does was established on the hardware for every bf16 magnitude from 2^-12 to 6 (both signs)
// against 256 seeds per operand slot: for the first element of its pair it adds bits [31:10] of the seed
// to the 22 mantissa bits that FP4 drops (denormalised below 1) and rounds up on a carry, so with a seed
// R << 24 it rounds up iff floor(256 p) + R >= 256 -- the rule above with R = 255 - rnd.  The second
// element of a pair takes the seed shifted by one bit, which would tie its random number to the first
// one's; every element therefore goes through the first slot of its own instruction, and what the second slot makes
// of whatever its register holds is masked away (a zero there costs a move per element: 17.8 vector instructions per element along
// rows and 17.1 along columns then, 16.1 and 15.5 now, which is what bounds these kernels: us per call along rows [8192 x
// 8192] 43.0 -> 38.7, [4096 x 8192] 24.6 -> 21.8, [2048 x 4096] 8.2 -> 7.5; along columns 44.6 -> 42.1, 23.0 -> 22.8, 9.1 -> 8.6).
// Bits below the top eight of the seed must be zero, or they could carry into the comparison.  The form that takes
// packed bf16 would save the unpacking, but it drops bits of p between 1/4 and 1.
// The instruction is written as inline assembly: it replaces one byte of its destination and keeps the
// other three, and the compiler's builtin for it does not tie the destination to the previous value.
typedef float float2_t_sr __attribute__((ext_vector_type(2)));
#define SNIP_SR_CVT(dst, src, seed, sc, OPSEL) \
    asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3" OPSEL : "+v"(dst) : "v"(float2_t_sr{src, __uint_as_float(any_value())}), "v"(seed), "v"(sc))

// 8 consecutive stored elements -> 8 FP4 nibbles with stochastic rounding; r0 holds the
// random bytes of elements 0-3, r1 those of elements 4-7; sc is the block scale operand.
__device__ __forceinline__ unsigned enc4_sr(const float (&e)[8], float sc, unsigned r0, unsigned r1)
{
    const unsigned n[2] = {~r0, ~r1};                       // 255 - rnd in every byte
    unsigned even = any_value(), odd = any_value();         // byte i: code of element 2i / 2i+1 in its low nibble
    unsigned s[8];                                          // byte i % 4 of n moved to the top byte, zeros below
#pragma unroll
    for (int i = 0; i < 8; ++i)
        s[i] = i % 4 == 0 ? n[i / 4] << 24 : i % 4 == 3 ? n[i / 4] & 0xFF000000u
                          : __builtin_amdgcn_perm(n[i / 4], 0u, i % 4 == 1 ? 0x050C0C0Cu : 0x060C0C0Cu);
    SNIP_SR_CVT(even, e[0], s[0], sc, "");
    SNIP_SR_CVT(odd, e[1], s[1], sc, "");
    SNIP_SR_CVT(even, e[2], s[2], sc, " op_sel:[0,0,1,0]");
    SNIP_SR_CVT(odd, e[3], s[3], sc, " op_sel:[0,0,1,0]");
    SNIP_SR_CVT(even, e[4], s[4], sc, " op_sel:[0,0,0,1]");
    SNIP_SR_CVT(odd, e[5], s[5], sc, " op_sel:[0,0,0,1]");
    SNIP_SR_CVT(even, e[6], s[6], sc, " op_sel:[0,0,1,1]");
    SNIP_SR_CVT(odd, e[7], s[7], sc, " op_sel:[0,0,1,1]");
    return (even & 0x0F0F0F0Fu) | ((odd << 4) & 0xF0F0F0F0u);
}
#undef SNIP_SR_CVT

// Codes of the 8 consecutive stored elements that start at stored position 8 * grp.
__device__ __forceinline__ unsigned enc4_sr_at(const float (&e)[8], float sc, uint64_t grp, uint2 seed)
{
    unsigned r0, r1;
    threefry2x32_20((unsigned)grp, (unsigned)(grp >> 32), seed.x, seed.y, r0, r1);
    return enc4_sr(e, sc, r0, r1);
}

// s0 += x_lo^2 + x_hi^2 for a bf16 pair (one instruction: the products are exact, the sum is rounded once)
__device__ __forceinline__ void acc_sq(unsigned w, float& s0)
{
    asm("v_dot2c_f32_bf16 %0, %1, %1" : "+v"(s0) : "v"(w));
}
__device__ __forceinline__ void acc_err(float2_t q, unsigned w, float& s0, float& se)
{
    const float xl = __uint_as_float(w << 16), xh = __uint_as_float(w & 0xFFFF0000u);
    const float dl = q[0] - xl, dh = q[1] - xh;
    se = fmaf(dl, dl, se);
    se = fmaf(dh, dh, se);
    acc_sq(w, s0);
}

// Error sums of 8 source elements w[0..3] against their FP8 codes c[0..1].
__device__ __forceinline__ void err8(const unsigned* w, unsigned c0, unsigned c1, float sc,
                                     float& s0, float& se)
{
    acc_err(__builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c0, sc, false), w[0], s0, se);
    acc_err(__builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c0, sc, true),  w[1], s0, se);
    acc_err(__builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c1, sc, false), w[2], s0, se);
    acc_err(__builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c1, sc, true),  w[3], s0, se);
}
__device__ __forceinline__ void err4(const unsigned* w, unsigned c, float sc,
                                     float& s0, float& se)
{
    acc_err(__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, sc, 0), w[0], s0, se);
    acc_err(__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, sc, 1), w[1], s0, se);
    acc_err(__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, sc, 2), w[2], s0, se);
    acc_err(__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, sc, 3), w[3], s0, se);
}

// The same on elements unpacked to fp32, which is what the statistics work on: unpacked once, an element serves the block's
// maximum, the conversions to both formats and both errors, and nothing has to be re-paired.  Against packed pairs (masked for
// the maximum, re-paired for the conversions, unpacked for the errors) quant_both_kernel with all sums takes 1361 vector
// instructions per tile instead of 1483 (FP4), and us per call: statistics of both directions [16384 x 11008] 134.7 -> 121.4, [16384 x
// 4096] 49.1 -> 44.8, of rows 83 -> 78; quantize with all sums [16384 x 11008] FP4 174 -> 169, FP8 197 -> 194, [8192 x 4096] 41.3 ->
// 39.6 and 43.6 -> 42.
__device__ __forceinline__ void unpack2(unsigned w, float& lo, float& hi)
{
    lo = __uint_as_float(w << 16);
    hi = __uint_as_float(w & 0xFFFF0000u);
}
// max(m, |a|, |b|); a NaN stays a NaN
__device__ __forceinline__ float max3_abs(float m, float a, float b)
{
    float r;
    asm("v_maximum3_f32 %0, %1, |%2|, |%3|" : "=v"(r) : "v"(m), "v"(a), "v"(b));
    return r;
}
template <int N> __device__ __forceinline__ float max_abs(const float* x)
{
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < N; i += 2) m = max3_abs(m, x[i], x[i + 1]);
    return m;
}
// 4 elements -> 4 FP8 bytes, 8 elements -> 8 FP4 nibbles (`byte`: the scale; floor rule: magnitudes clamped to 448 * 2^(byte-127))
template <int RULE>
__device__ __forceinline__ unsigned enc8x4(const float* x, float sc, unsigned byte)
{
    float t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float lim = __uint_as_float(((byte + 8u) << 23) | 0x600000u);
        t[i] = RULE == 1 ? __builtin_amdgcn_fmed3f(x[i], -lim, lim) : x[i];
    }
    short2_t r = __builtin_bit_cast(short2_t, any_value());
    r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, t[0], t[1], sc, false);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, t[2], t[3], sc, true);
    return __builtin_bit_cast(unsigned, r);
}
__device__ __forceinline__ unsigned enc4x8(const float* x, float sc)
{
    unsigned r = any_value();
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, x[0], x[1], sc, 0);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, x[2], x[3], sc, 1);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, x[4], x[5], sc, 2);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, x[6], x[7], sc, 3);
    return r;
}
__device__ __forceinline__ void acc_err2(float2_t q, const float* x, float& se)
{
    const float d0 = q[0] - x[0], d1 = q[1] - x[1];
    se = fmaf(d0, d0, se);
    se = fmaf(d1, d1, se);
}
__device__ __forceinline__ void err8x4(const float* x, unsigned c, float sc, float& se)
{
    acc_err2(__builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c, sc, false), x, se);
    acc_err2(__builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c, sc, true), x + 2, se);
}
__device__ __forceinline__ void err4x8(const float* x, unsigned c, float sc, float& se)
{
    acc_err2(__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, sc, 0), x, se);
    acc_err2(__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, sc, 1), x + 2, se);
    acc_err2(__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, sc, 2), x + 4, se);
    acc_err2(__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c, sc, 3), x + 6, se);
}
// Error sums of N elements (a multiple of 8) of one block under both formats, am: magnitude bits of the block's maximum.
template <int N, int RULE>
__device__ __forceinline__ void both_errors(const float* x, unsigned am, float& se4, float& se8)
{
    const unsigned b8 = scale_byte<kFP8, RULE>(am), b4 = scale_byte<kFP4, RULE>(am);
    const float sc8 = scale_operand(b8), sc4 = scale_operand(b4);
#pragma unroll
    for (int k = 0; k < N; k += 8) {
        err8x4(x + k, enc8x4<RULE>(x + k, sc8, b8), sc8, se8);
        err8x4(x + k + 4, enc8x4<RULE>(x + k + 4, sc8, b8), sc8, se8);
        err4x8(x + k, enc4x8(x + k, sc4), sc4, se4);
    }
}
__device__ __forceinline__ unsigned magnitude_bits(float m) { return __float_as_uint(m) >> 16; }

// Magnitude bits of the largest of the 8 bf16 values in v (one lane's share of a block).
__device__ __forceinline__ unsigned amax8(const uint4& v)
{
    unsigned m = pk_max_u16(pk_max_u16(v.x & 0x7FFF7FFFu, v.y & 0x7FFF7FFFu),
                            pk_max_u16(v.z & 0x7FFF7FFFu, v.w & 0x7FFF7FFFu));
    const unsigned lo = m & 0xFFFFu, hi = m >> 16;
    return lo > hi ? lo : hi;
}

// ------------------------------------------------------------------------------------------
// Row blocks.  A lane owns 8 consecutive elements (one 16-byte load), a quad owns a block, a
// wave owns 512 consecutive elements of a row ("segment").  Four segments are in flight per
// wave.  Loads and code stores are fully coalesced; the 16 scale bytes of a segment are
// written by the first lane of each quad to 16 consecutive addresses.
// ------------------------------------------------------------------------------------------
constexpr int kSeg = 512;
constexpr int kUnroll = 4;
constexpr int kStatUnroll = 8;         // loads in flight per lane in the row statistics kernel

template <int FMT, int RULE, bool STATS, bool SR = false>
__global__ __launch_bounds__(256) void quant_row_kernel(const uint16_t* __restrict__ x, int rows,
                                                        int cols, int64_t ld,
                                                        uint8_t* __restrict__ codes,
                                                        uint8_t* __restrict__ scales,
                                                        uint8_t* __restrict__ scales_g4, int64_t kpitch,
                                                        float* __restrict__ partials, uint2 seed)
{
    static_assert(!SR || (FMT == kFP4 && !STATS), "stochastic rounding: FP4, no fused statistics");
    // unit = (group of 4 consecutive rows, 512-element segment); the wave's four loads in flight
    // are the four rows, so that the block-major scale copy gets one dword (4 rows) per block.
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
    const int nwaves = gridDim.x * kWavesPerBlock;
    const int spr = (cols + kSeg - 1) / kSeg;
    const int units = ((rows + kUnroll - 1) / kUnroll) * spr;
    float s0 = 0.f, se = 0.f;

    for (int u = wave; u < units; u += nwaves) {
        const int rg = u / spr;
        const int col = (u - rg * spr) * kSeg + lane * 8;
        // Loads carry no condition: lanes past the last column read column 0 and rows past the last one that row; with
        // statistics they count as zeros, otherwise only their scale bytes are cleared (they reach the grouped copy).
        const bool in = col < cols;
        const unsigned ucol = in ? (unsigned)col : 0u;
        uint4 v[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) v[j] = ld16(x + (int64_t)min(rg * kUnroll + j, rows - 1) * ld + ucol);
        // stored position of the unit's first row / 8, stepped in scalar registers out of the compiler's sight (it would multiply
        // anew for every address, in 64 bits on the vector unit)
        const int64_t step = cols >> 3;
        int64_t at0 = (int64_t)(rg * kUnroll) * step;
        asm volatile("" : "+s"(at0));
        int64_t at = at0;
        unsigned packed = 0, c0[kUnroll], c1[kUnroll];
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            const int row = rg * kUnroll + j;
            const bool act = in && row < rows;
            if (STATS && !act) v[j] = make_uint4(0, 0, 0, 0);
            const unsigned am = quad_max(amax8(v[j]));
            const unsigned byte = scale_byte<FMT, RULE>(am);
            const float sc = scale_operand(byte);
            const bool bad = byte == 0xFFu;
            const unsigned w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
            if (FMT == kFP8) {
                c0[j] = enc8<RULE>(w[0], w[1], sc, byte); c1[j] = enc8<RULE>(w[2], w[3], sc, byte);
                if (bad) { c0[j] = 0; c1[j] = 0; }
                if (STATS) err8(w, c0[j], c1[j], sc, s0, se);
            } else if (SR) {
                float e[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) unpack2(w[i], e[2 * i], e[2 * i + 1]);
                c0[j] = enc4_sr_at(e, sc, (uint64_t)at + ucol / 8, seed);
                at += step;
                if (bad) c0[j] = 0;
            } else {
                c0[j] = enc4(w[0], w[1], w[2], w[3], sc);
                if (bad) c0[j] = 0;
                if (STATS) err4(w, c0[j], sc, s0, se);
            }
            packed |= (act ? byte : 0u) << (8 * j);
        }
        if (in) {
            at = at0;
#pragma unroll
            for (int j = 0; j < kUnroll; ++j, at += step) {
                if (rg * kUnroll + j >= rows) break;                 // wave-uniform
                if (FMT == kFP8) *reinterpret_cast<uint2*>(codes + at * 8 + ucol) = make_uint2(c0[j], c1[j]);
                else             *reinterpret_cast<unsigned*>(codes + at * 4 + ucol / 2) = c0[j];
            }
            at = at0;
            if ((lane & 3) == 0)
#pragma unroll
                for (int j = 0; j < kUnroll; ++j, at += step) {
                    if (rg * kUnroll + j >= rows) break;
                    scales[(at >> 2) + ucol / kBlock] = (uint8_t)(packed >> (8 * j));
                }
        }
        // Grouped copy: `packed` holds this block's byte for each of the 4 rows.  Fetch the same
        // word from the next three quads (the next three blocks of the same 128-element group),
        // transpose the 4x4 bytes, and let the first lane of every 16 store the four rows' dwords
        // (16 contiguous bytes).  Rows past the end fall inside the padded pitch.
        if (scales_g4) {
            const unsigned p0 = packed;
            const unsigned p1 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)packed, 0x104, 0xF, 0xF, true);   // lane + 4
            const unsigned p2 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)packed, 0x108, 0xF, 0xF, true);   // lane + 8
            const unsigned p3 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)packed, 0x10C, 0xF, 0xF, true);   // lane + 12
            const unsigned a_lo = __builtin_amdgcn_perm(p1, p0, 0x05010400u), a_hi = __builtin_amdgcn_perm(p1, p0, 0x07030602u);
            const unsigned b_lo = __builtin_amdgcn_perm(p3, p2, 0x05010400u), b_hi = __builtin_amdgcn_perm(p3, p2, 0x07030602u);
            const uint4 d = make_uint4(__builtin_amdgcn_perm(b_lo, a_lo, 0x05040100u), __builtin_amdgcn_perm(b_lo, a_lo, 0x07060302u),
                                       __builtin_amdgcn_perm(b_hi, a_hi, 0x05040100u), __builtin_amdgcn_perm(b_hi, a_hi, 0x07060302u));
            if (col < cols && (lane & 15) == 0)
                *reinterpret_cast<uint4*>(scales_g4 + ((int64_t)(col >> 7) * kpitch + rg * kUnroll) * 4) = d;
        }
    }
    if (STATS) {
        s0 = wave_sum(s0);
        se = wave_sum(se);
        if (lane == 0) { partials[wave * 3 + 0] = s0; partials[wave * 3 + 1] = se; partials[wave * 3 + 2] = 0.f; }
    }
}

// Statistics only, both formats, row blocks.  One wave walks whole rows so that the per-row
// sums of Sec. 5.3 come out of the same pass.
template <int RULE>
__global__ __launch_bounds__(256) void stats_row_kernel(const uint16_t* __restrict__ x, int rows,
                                                        int cols, int64_t ld,
                                                        float* __restrict__ partials,
                                                        float* __restrict__ per_line)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
    const int nwaves = gridDim.x * kWavesPerBlock;
    float t0 = 0.f, t4 = 0.f, t8 = 0.f;
    for (int row = wave; row < rows; row += nwaves) {
        const uint16_t* xr = x + (int64_t)row * ld;
        float s0 = 0.f, s4 = 0.f, s8 = 0.f;
        for (int c0 = 0; c0 < cols; c0 += kSeg * kStatUnroll) {
            uint4 v[kStatUnroll];
#pragma unroll
            for (int j = 0; j < kStatUnroll; ++j) {
                const int col = c0 + j * kSeg + lane * 8;
                v[j] = make_uint4(0, 0, 0, 0);     // zeros quantize to zero: no contribution
                if (col < cols) v[j] = ld16(xr + col);
            }
#pragma unroll
            for (int j = 0; j < kStatUnroll; ++j) {
                if (c0 + j * kSeg >= cols) break;                    // wave-uniform: the row has no such segment
                const unsigned w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
                float x8[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) { unpack2(w[i], x8[2 * i], x8[2 * i + 1]); acc_sq(w[i], s0); }
                const unsigned am = quad_max(__float_as_uint(max_abs<8>(x8))) >> 16;
                both_errors<8, RULE>(x8, am, s4, s8);
                if (am >= 0x7F80u) { s4 = __builtin_nanf(""); s8 = __builtin_nanf(""); }
            }
        }
        s0 = wave_sum(s0); s4 = wave_sum(s4); s8 = wave_sum(s8);
        if (per_line && lane == 0) {
            per_line[(int64_t)row * 3 + 0] = s0; per_line[(int64_t)row * 3 + 1] = s4; per_line[(int64_t)row * 3 + 2] = s8;
        }
        t0 += s0; t4 += s4; t8 += s8;
    }
    if (lane == 0) { partials[wave * 3 + 0] = t0; partials[wave * 3 + 1] = t4; partials[wave * 3 + 2] = t8; }
}

// ------------------------------------------------------------------------------------------
// Column blocks.  A lane owns two adjacent columns and reads them one dword per row: a wave
// reads 256 contiguous bytes of each of 32 rows (one block per column), 32 independent loads
// in flight.  The block maximum of a column never leaves the lane.  Rows are re-paired with
// v_perm so that the conversion instructions pack elements that are adjacent in the
// transposed output; each lane then stores 32 (FP8) or 16 (FP4) contiguous bytes per column.
// A wave processes four (FP8) or eight (FP4) vertically adjacent blocks back to back, i.e. exactly one
// 128-byte line of every stored row, so that no line of the output is written in two pieces.
// ------------------------------------------------------------------------------------------
constexpr int kColsPerWave = 128;
constexpr int kRowBlocksPerUnit = 4;

struct ColBlock {
    unsigned lo[16], hi[16];   // bf16 pairs (row 2k, row 2k+1) of the lane's two columns
    unsigned am_lo, am_hi;     // magnitude bits of each column's block maximum
};

// Magnitude bits of both columns' maxima, the first column's in the low half.
__device__ __forceinline__ unsigned col_maxima(const unsigned (&v)[32])
{
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < 32; ++i) m = pk_max_u16(m, v[i] & 0x7FFF7FFFu);
    return m;
}

__device__ __forceinline__ void pair_col_block(const unsigned (&v)[32], ColBlock& b)
{
    const unsigned m = col_maxima(v);
    b.am_lo = m & 0xFFFFu;
    b.am_hi = m >> 16;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        b.lo[k] = __builtin_amdgcn_perm(v[2 * k + 1], v[2 * k], 0x05040100u);
        b.hi[k] = __builtin_amdgcn_perm(v[2 * k + 1], v[2 * k], 0x07060302u);
    }
}

// Two adjacent columns (c0 + 2 * lane) of 32 rows from `row` on, streaming; zeros past the last column.  `row` is
// wave-uniform and stepped in scalar registers, out of the compiler's sight: left alone it computes the 32 row addresses
// ahead, runs out of scalar registers and keeps them in lanes of vector registers, which cost the statistics kernel 118
// vector instructions per tile of 1360.  One condition around all loads and only where the tile is not whole: a branch
// around each would keep them from being in flight together.
__device__ __forceinline__ void load_col_tile(const uint16_t* __restrict__ row, int c0, int lane, int cols, int64_t ld, unsigned (&v)[32])
{
    typedef const __attribute__((address_space(1))) uint8_t* gbyte;
    if (c0 + kColsPerWave <= cols) {
        gbyte p = (gbyte)(uintptr_t)(row + c0);
        // (The offset's 32 bits are made known here: a load then takes base and offset as they are; with the widening hoisted out of the
        // caller's loop each load had a 64-bit sum of its own and a wait state behind it, 64 of 250-900 issue slots per tile.  us per call,
        // statistics of both directions [16384 x 11008] 107.3 -> 103.7, [4096 x 8192] 26.3 -> 25.4.)
        unsigned off = (unsigned)lane * 4;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            v[i] = __builtin_nontemporal_load((const __attribute__((address_space(1))) unsigned*)(p + off));
            p += ld * 2;
            asm volatile("" : "+s"(p));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = 0u;
        if (c0 + 2 * lane < cols) {
            const uint16_t* p = row + c0 + 2 * lane;
#pragma unroll
            for (int i = 0; i < 32; ++i, p += ld) v[i] = ld4(p);
        }
    }
}

// Codes of one column's block (32 rows) -> the wave's LDS staging area; returns the scale byte.
// In LDS the wave keeps a [128 stored rows][ROWB bytes] image of its unit's output (ROWB = 128: 128 source
// rows of FP8 codes or 256 of FP4 codes); 16-byte chunk c of row r sits at position c ^ ((r >> 1) & (CPR-1)).
template <int FMT, int RULE, bool STATS>
__device__ __forceinline__ unsigned quant_one_column(const unsigned* w, unsigned am, uint8_t* __restrict__ lds_row,
                                                     int rb_local, int swz, float& s0, float& se)
{
    const unsigned byte = scale_byte<FMT, RULE>(am);
    const float sc = scale_operand(byte);
    const bool bad = byte == 0xFFu;
    if (FMT == kFP8) {
        unsigned c[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            c[k] = enc8<RULE>(w[2 * k], w[2 * k + 1], sc, byte);
        }
        if (__builtin_amdgcn_ballot_w64(bad) != 0)                       // wave-uniform
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] = bad ? 0u : c[k];
        *reinterpret_cast<uint4*>(lds_row + (((rb_local * 2 + 0) ^ swz) * 16)) = make_uint4(c[0], c[1], c[2], c[3]);
        *reinterpret_cast<uint4*>(lds_row + (((rb_local * 2 + 1) ^ swz) * 16)) = make_uint4(c[4], c[5], c[6], c[7]);
        if (STATS) {
#pragma unroll
            for (int k = 0; k < 4; ++k) err8(w + 4 * k, c[2 * k], c[2 * k + 1], sc, s0, se);
        }
    } else {
        unsigned c[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            c[k] = enc4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3], sc);
        }
        if (__builtin_amdgcn_ballot_w64(bad) != 0)                       // wave-uniform
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] = bad ? 0u : c[k];
        *reinterpret_cast<uint4*>(lds_row + ((rb_local ^ swz) * 16)) = make_uint4(c[0], c[1], c[2], c[3]);
        if (STATS) {
#pragma unroll
            for (int k = 0; k < 4; ++k) err4(w + 4 * k, c[k], sc, s0, se);
        }
    }
    return byte;
}

// The same with stochastic rounding, of the column in the low (HI: high) halves of v; grp: stored position of its first
// element / 8, a multiple of 4.
template <int RULE, bool HI>
__device__ __forceinline__ unsigned quant_sr_column(const unsigned (&v)[32], unsigned am, uint8_t* __restrict__ lds_row, int rb_local,
                                                    int swz, uint64_t grp, uint2 seed)
{
    const unsigned byte = scale_byte<kFP4, RULE>(am);
    const float sc = scale_operand(byte);
    const bool bad = byte == 0xFFu;
    unsigned c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = __uint_as_float(HI ? v[8 * k + i] & 0xFFFF0000u : v[8 * k + i] << 16);
        c[k] = enc4_sr_at(e, sc, grp | (unsigned)k, seed);
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0)                           // wave-uniform
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = bad ? 0u : c[k];
    *reinterpret_cast<uint4*>(lds_row + ((rb_local ^ swz) * 16)) = make_uint4(c[0], c[1], c[2], c[3]);
    return byte;
}

// COOP: the four waves of a workgroup share one unit (wave w takes its row blocks w, w + 4) and one staging area, so
// that a workgroup needs 17 KB of LDS instead of 64 KB and more waves are resident; the scale bytes of the four row
// blocks of a dword meet in LDS.  Same bytes out.
template <int FMT, int RULE, bool STATS, bool SR = false, bool COOP = false>
__global__ __launch_bounds__(256) void quant_col_kernel(const uint16_t* __restrict__ x, int rows,
                                                        int cols, int64_t ld,
                                                        uint8_t* __restrict__ codes,
                                                        uint8_t* __restrict__ scales,
                                                        uint8_t* __restrict__ scales_g4, int64_t kpitch,
                                                        float* __restrict__ partials, uint2 seed)
{
    static_assert(!SR || (FMT == kFP4 && !STATS), "stochastic rounding: FP4, no fused statistics");
    // row blocks per unit: one full 128-byte line of every stored row (128 FP8 / 256 FP4 source rows); the
    // stochastic variant, bound by VALU work and register count rather than by stores, keeps half lines
    constexpr int RBU = FMT == kFP8 ? 4 : (SR ? 4 : 8);
    constexpr int ROWB = RBU * (FMT == kFP8 ? 32 : 16);   // staged output bytes per stored row
    constexpr int CPR = ROWB / 16;
    __shared__ __attribute__((aligned(16))) uint8_t stage[COOP ? 1 : kWavesPerBlock][kColsPerWave * ROWB];
    __shared__ __attribute__((aligned(4))) uint8_t scale_stage[COOP ? RBU * kColsPerWave : 4];   // COOP: scale byte of (row block, column)
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* const reg = stage[COOP ? 0 : wib];
    const int wave = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + wib);
    const int nwaves = gridDim.x * kWavesPerBlock;
    const int ncg = (cols + kColsPerWave - 1) / kColsPerWave;
    const int nrb = rows / kBlock;
    const int nru = (nrb + RBU - 1) / RBU;
    const int units = ncg * nru;
    const int64_t out_row_bytes = FMT == kFP8 ? rows : rows / 2;
    float s0 = 0.f, se = 0.f;
    for (int u = COOP ? (int)blockIdx.x : wave; u < units; u += COOP ? (int)gridDim.x : nwaves) {
        const int ru = u / ncg, cg = u - ru * ncg;
        const int c = cg * kColsPerWave + lane * 2;
        const bool act = c < cols;
        const int rb0 = ru * RBU;
        const int nb = min(nrb - rb0, RBU);
        const int swz_lo = lane & (CPR - 1);          // ((2 * lane) >> 1) & (CPR - 1); the odd row shares it
        // row block kk of the unit: codes into the staging area, returns the two columns' scale bytes
        auto one_block = [&](int kk, unsigned& y0, unsigned& y1) {
            unsigned v[32];
            load_col_tile(x + (int64_t)(rb0 + kk) * kBlock * ld, cg * kColsPerWave, lane, cols, ld, v);
            uint8_t* const r0 = reg + (2 * lane) * ROWB;
            if (SR) {
                const unsigned m = col_maxima(v);
                const uint64_t grp = (uint64_t)c * (unsigned)(rows >> 3) + (unsigned)((rb0 + kk) * 4);         // stored row = source column
                y0 = quant_sr_column<RULE, false>(v, m & 0xFFFFu, r0, kk, swz_lo, grp, seed);
                y1 = quant_sr_column<RULE, true>(v, m >> 16, r0 + ROWB, kk, swz_lo, grp + (unsigned)(rows >> 3), seed);
            } else {
                ColBlock b;
                pair_col_block(v, b);
                y0 = quant_one_column<FMT, RULE, STATS>(b.lo, b.am_lo, r0, kk, swz_lo, s0, se);
                y1 = quant_one_column<FMT, RULE, STATS>(b.hi, b.am_hi, r0 + ROWB, kk, swz_lo, s0, se);
            }
        };
        // Four row blocks at a time (blocks 0 .. last of the group starting at rbh): their scale bytes of a column
        // form one dword of the row-major array (when the row length allows it) and exactly one dword of the
        // grouped copy.
        auto store_scales = [&](int rbh, int last, unsigned lo, unsigned hi) {
            if (act) {
                uint8_t* s_lo = scales + (int64_t)c * nrb + rbh;
                if ((nrb & 3) == 0) {
                    *reinterpret_cast<unsigned*>(s_lo) = lo;
                    *reinterpret_cast<unsigned*>(s_lo + nrb) = hi;
                } else if (!COOP) {
                    for (int k = 0; k <= last; ++k) { s_lo[k] = (uint8_t)(lo >> (8 * k)); s_lo[nrb + k] = (uint8_t)(hi >> (8 * k)); }
                }
                if (scales_g4)
                    *reinterpret_cast<uint2*>(scales_g4 + ((int64_t)(rbh / kRowBlocksPerUnit) * kpitch + c) * 4) = make_uint2(lo, hi);
            }
        };
        if (COOP) {
            for (int kk = wib; kk < nb; kk += kWavesPerBlock) {
                unsigned y0, y1;
                one_block(kk, y0, y1);
                *reinterpret_cast<uint16_t*>(scale_stage + kk * kColsPerWave + 2 * lane) = (uint16_t)(y0 | (y1 << 8));
            }
            __syncthreads();                                   // all row blocks of the unit are staged
            for (int h = wib; h * kRowBlocksPerUnit < nb; h += kWavesPerBlock) {
                const int last = min(kRowBlocksPerUnit - 1, nb - 1 - h * kRowBlocksPerUnit);
                unsigned lo = 0, hi = 0;
                for (int k = 0; k <= last; ++k) {
                    const unsigned v = *reinterpret_cast<const uint16_t*>(scale_stage + (h * kRowBlocksPerUnit + k) * kColsPerWave + 2 * lane);
                    lo |= (v & 0xFFu) << (8 * k);
                    hi |= (v >> 8) << (8 * k);
                }
                store_scales(rb0 + h * kRowBlocksPerUnit, last, lo, hi);
            }
            // (as in quant_both_kernel)
            if ((nrb & 3) != 0)
                for (int p = wib; p < (nb + 3) / 4 * 8; p += kWavesPerBlock) {
                    int l = lane;
                    asm volatile("" : "+v"(l));
                    const int blk = p / 8 * 4 + (l & 3), col = p % 8 * 16 + (l >> 2), to = cg * kColsPerWave + col;
                    if (blk < nb && to < cols) scales[(int64_t)to * nrb + rb0 + blk] = scale_stage[blk * kColsPerWave + col];
                }
        } else {
            for (int h = 0; h < RBU / kRowBlocksPerUnit; ++h) {
                const int nbh = min(nb - h * kRowBlocksPerUnit, kRowBlocksPerUnit);
                if (nbh <= 0) break;
                unsigned g4_lo = 0, g4_hi = 0;
                for (int k = 0; k < nbh; ++k) {
                    unsigned y0, y1;
                    one_block(h * kRowBlocksPerUnit + k, y0, y1);
                    g4_lo |= y0 << (8 * k);
                    g4_hi |= y1 << (8 * k);
                }
                store_scales(rb0 + h * kRowBlocksPerUnit, nbh - 1, g4_lo, g4_hi);
            }
        }
        // Codes: read the staged image back row-contiguous and store 16 bytes per lane, so that every store
        // instruction writes whole ROWB-byte runs of 64 / CPR stored rows.
#pragma unroll
        for (int it = COOP ? wib : 0; it < kColsPerWave * CPR / 64; it += COOP ? kWavesPerBlock : 1) {
            const int idx = it * 64 + lane;
            const int row = idx / CPR, chunk = idx % CPR;
            const uint4 v = *reinterpret_cast<const uint4*>(reg + row * ROWB + ((chunk ^ ((row >> 1) & (CPR - 1))) * 16));
            const int cc = cg * kColsPerWave + row;
            const int blk = FMT == kFP8 ? chunk >> 1 : chunk;        // row block this chunk belongs to
            if (cc < cols && blk < nb)
                *reinterpret_cast<uint4*>(codes + (int64_t)cc * out_row_bytes + (int64_t)ru * ROWB + chunk * 16) = v;
        }
        if (COOP) __syncthreads();                             // the staging areas go to the next unit
    }
    if (STATS) {
        s0 = wave_sum(s0);
        se = wave_sum(se);
        if (lane == 0) { partials[wave * 3 + 0] = s0; partials[wave * 3 + 1] = se; partials[wave * 3 + 2] = 0.f; }
    }
}

// The six sums of a workgroup's waves, added in wave order in double, to partials[workgroup][6].
template <int WPB>
__device__ __forceinline__ void store_wave_sums(const float (&sums)[6], int wib, int lane, double* __restrict__ partials)
{
    __shared__ float wave_sums[WPB][6];
    if (lane == 0)
#pragma unroll
        for (int j = 0; j < 6; ++j) wave_sums[wib][j] = sums[j];
    __syncthreads();
    if (threadIdx.x < 6) {
        double t = 0.0;
        for (int w = 0; w < WPB; ++w) t += (double)wave_sums[w][threadIdx.x];
        partials[(size_t)blockIdx.x * 6 + threadIdx.x] = t;
    }
}

// Both orientations of one tensor from one pass over HBM (Sec. 2.2: X feeds the forward GEMM with blocks along
// its rows and the weight-gradient GEMM with blocks down its columns; W and dY likewise).  A wave owns the same
// units as in quant_col_kernel.  A 32-row x 128-column tile goes through the column-block path above and, read with the row
// kernel's lane layout (a lane = 8 consecutive elements, a quad = one block, 16 lanes = the tile's 128 columns of one
// row, 4 rows per load), through the row path: from LDS, or from cache, the lines having just been fetched by the same wave or
// workgroup.  Results are bit-identical to the two single-orientation kernels.
// One column's block in quant_both_kernel's statistics forms: quant_one_column on unpacked elements, with the error of the
// other format too if STATS == 2.
template <int FMT, int RULE, int STATS>
__device__ __forceinline__ unsigned quant_column_stats(const float* x, uint8_t* __restrict__ lds_row, int rb_local, int swz, float& se, float& so)
{
    const unsigned am = magnitude_bits(max_abs<32>(x));
    const unsigned byte = scale_byte<FMT, RULE>(am), other = scale_byte<1 - FMT, RULE>(am);
    const float sc = scale_operand(byte), sco = scale_operand(other);
    const bool bad = byte == 0xFFu;
    unsigned c[FMT == kFP8 ? 8 : 4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float* y = x + 8 * k;
        if (FMT == kFP8) { c[2 * k] = enc8x4<RULE>(y, sc, byte); c[2 * k + 1] = enc8x4<RULE>(y + 4, sc, byte); }
        else c[k] = enc4x8(y, sc);
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0)                           // wave-uniform
#pragma unroll
        for (int k = 0; k < (FMT == kFP8 ? 8 : 4); ++k) c[k] = bad ? 0u : c[k];
    if (FMT == kFP8) {
        *reinterpret_cast<uint4*>(lds_row + (((rb_local * 2 + 0) ^ swz) * 16)) = make_uint4(c[0], c[1], c[2], c[3]);
        *reinterpret_cast<uint4*>(lds_row + (((rb_local * 2 + 1) ^ swz) * 16)) = make_uint4(c[4 % (FMT == kFP8 ? 8 : 4)], c[5 % (FMT == kFP8 ? 8 : 4)], c[6 % (FMT == kFP8 ? 8 : 4)], c[7 % (FMT == kFP8 ? 8 : 4)]);
    } else {
        *reinterpret_cast<uint4*>(lds_row + ((rb_local ^ swz) * 16)) = make_uint4(c[0], c[1], c[2], c[3]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float* y = x + 8 * k;
        if (FMT == kFP8) {
            err8x4(y, c[(2 * k) % (FMT == kFP8 ? 8 : 4)], sc, se);
            err8x4(y + 4, c[(2 * k + 1) % (FMT == kFP8 ? 8 : 4)], sc, se);
            if (STATS == 2) err4x8(y, enc4x8(y, sco), sco, so);
        } else {
            err4x8(y, c[k], sc, se);
            if (STATS == 2) {
                err8x4(y, enc8x4<RULE>(y, sco, other), sco, so);
                err8x4(y + 4, enc8x4<RULE>(y + 4, sco, other), sco, so);
            }
        }
    }
    return byte;
}

// Memory access of quant_both_kernel: buffer descriptors with a wave-uniform base per tile, a lane offset that is the same for
// every row of the tile and the row's offset in a scalar register, so that a load or store costs no vector instruction for its
// address; a lane that has nothing to load or store takes an offset past the descriptor's end (loads deliver zeros, stores
// are dropped) instead of a branch.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef unsigned v2u_t __attribute__((ext_vector_type(2)));
// A 16-byte store takes its whole offset in the lane: with a scalar register for the offset the hardware was seen to store the
// first dword of a vector register that the next instruction overwrote, and the compiler puts no wait state there (it does
// where the scalar offset is a constant); stores of 4 and 8 bytes do not read late.
constexpr int kPast = (int)0x80000000u;                // past the end of every descriptor
__device__ __forceinline__ rsrc_t tile_rsrc(const void* p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7FFFFFFF, 0x00020000); }
// Copy of 16 bytes per lane straight into LDS: lane i's land at lds + 16 i (lanes past the descriptor's end: zeros).
template <int POLICY>
__device__ __forceinline__ void copy_to_lds(rsrc_t r, uint8_t* lds, int voff, int soff)
{
#ifdef __HIP_DEVICE_COMPILE__          // (the host pass knows neither the builtin's size of 16 nor the address space)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voff, soff, 0, POLICY);
#endif
}
__device__ __forceinline__ void step(int& soff, int by)
{
    soff += by;
    asm volatile("" : "+s"(soff));                      // stepped, not computed ahead: 32 offsets at once would not fit the scalar registers
}

// NW != 0: the NW waves of a workgroup share a unit of RBU tiles (wave w takes tiles w, w + NW, ...) and one staging area.
// RAW_LDS: the tiles of a unit are copied straight into LDS, once, and the waves of rows and columns take them from there.
// Without statistics NW more waves take the rows of the tiles (SPLIT), and the first NW the columns: 60-67 registers instead
// of 96 put seven waves on a SIMD instead of four or five, and the two chains of a tile run side by side.  With statistics
// a workgroup would wait for its column waves, whose work is the longer: [8192 x 4096] FP4 54 us against 41.
// APART: a row takes its wave 1.0 us of work where a column takes 0.4 (time stamps, [2048 x 2048] FP4), and the waves of rows stand in
// front of the barrier behind which the columns' codes are stored.  They meet it on their way, after three of their eight
// steps, when the columns are done, and leave the columns' stores to the others (qb_rows_apart, picks.h).
// NW == 0 (with statistics): a wave per unit, four of them in a workgroup.  Same bytes out.
// Without statistics bound by memory (and by launch and one tile's chain below 4 M elements), with them by vector arithmetic.
// Vector instructions per tile of 4096 elements, FP4: 765 -> 464 without statistics, 1800 -> 1480 with all of them, when
// addresses and conditions moved into descriptors and scalar registers.  Both changes, us per call on sources in memory,
// before -> now: [256 x 512] FP8 5.2 -> 4.0, [2048 x 2048] FP4 7.7 -> 6.2, [4096 x 8192] FP4 34.8 -> 29.9, FP8 39.1 -> 34.0, [16384 x
// 11008] FP4 141 -> 133, FP8 177 -> 165; with all statistics [4096 x 4096] FP4 27.0 -> 24.8, [16384 x 4096] 77 -> 68, FP8 81.5 -> 76,
// [16384 x 11008] FP4 195 -> 174, FP8 214 -> 197.
// Offsets inside a tile are 32-bit: launch_quantize_both keeps to tensors whose rows are short enough (qb_offsets_fit).
// Cache policies of buffer instructions: streaming ("nt") and write-through ("sc1").  A tile that goes through LDS is read once and
// streamed, so that sources leave the memory-side cache to the codes: alone, 40 steps of one linear come out the same on average (7 % faster
// to 4 % slower).  Codes of a workgroup per unit with statistics are written through: at the end of a kernel the L2s write out what is dirty
// with the chip idle (20 steps of one linear 2.3 % on average, 0 ... 5; [1504 x 2080] 9.1 us -> 8.4, [4096 x 4096] 22.5 -> 20.8, a step 1504 x 2080 x 1568
// 59.9 -> 58.7, 2048 x 4096 x 4096 163.2 -> 160.1).  Without statistics and LDS it makes no difference.  Large tensors: qb_streams.
constexpr int kStream = 2, kThrough = 16;
constexpr int qb_threads(int nw, int stats) { return nw ? nw * (stats ? 64 : 128) : 256; }
template <int FMT_R, int FMT_C, int RULE, int STATS, int NW, int RBU, bool RAW_LDS, bool STREAM, bool APART>      // STATS: 0 none, 1 the chosen formats' errors, 2 both formats' errors
__global__ __launch_bounds__(qb_threads(NW, STATS), STATS ? 2 : 1) void quant_both_kernel(const uint16_t* __restrict__ x, int rows, int cols, int64_t ld,
                                                         uint8_t* __restrict__ codes_r, uint8_t* __restrict__ scales_r,
                                                         uint8_t* __restrict__ g4_r, int64_t kpitch_r,
                                                         uint8_t* __restrict__ codes_c, uint8_t* __restrict__ scales_c,
                                                         uint8_t* __restrict__ g4_c, int64_t kpitch_c,
                                                         double* __restrict__ partials, int eighth, int band_log2)
{
    constexpr bool COOP = NW != 0, SPLIT = STATS == 0;
    constexpr int STORE = STREAM ? kStream | kThrough : COOP && STATS ? kThrough : 0;
    static_assert(!STREAM || RAW_LDS || !COOP, "codes are streamed by the forms for large tensors");
    constexpr int WPB = qb_threads(NW, STATS) / 64, CW = APART ? NW : WPB;    // waves of a workgroup, those that store the columns
    static_assert(!APART || (SPLIT && !RAW_LDS), "waves of rows and of columns, each with its own loads");
    constexpr int kRowsMeet = 3;
    constexpr int ROWB = RBU * (FMT_C == kFP8 ? 32 : 16);
    constexpr int CPR = ROWB / 16;
    // RAW_LDS: the raw tiles first, and the column codes in the same place once every wave has its part of them
    constexpr int RAW = kBlock * kColsPerWave * 2;                            // bytes of a raw tile
    __shared__ __attribute__((aligned(16))) uint8_t stage[COOP ? 1 : kWavesPerBlock][RAW_LDS && NW * RAW > kColsPerWave * ROWB ? NW * RAW : kColsPerWave * ROWB];
    __shared__ __attribute__((aligned(4))) uint8_t scale_stage[COOP ? RBU * kColsPerWave : 4];   // COOP: scale byte of (tile, column)
    static_assert(!SPLIT || NW == RBU, "a wave of either kind has one tile");
    static_assert(SPLIT || !RAW_LDS, "with statistics a wave reads its tile itself");
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* const reg = stage[COOP ? 0 : wib];
    const int wave = __builtin_amdgcn_readfirstlane(blockIdx.x * WPB + wib);
    const int nwaves = gridDim.x * kWavesPerBlock;
    const int ncg = (cols + kColsPerWave - 1) / kColsPerWave;
    const int nrb = rows / kBlock;
    const int nru = (nrb + RBU - 1) / RBU;
    const int units = ncg * nru;
    const int nblk = cols / kBlock;                       // blocks per row of the row-direction output
    const int pitch_x = (int)ld * 2;
    const int pitch_r = FMT_R == kFP8 ? cols : cols / 2, pitch_c = FMT_C == kFP8 ? rows : rows / 2;      // bytes of a stored row
    float s0 = 0.f, se_c = 0.f, se_r = 0.f;
    float so_c = 0.f, so_r = 0.f;                         // STATS == 2: error sums of the format not chosen
    // COOP: the order of the units (qb_place and qb_eighths in picks.h; the grid is a multiple of 8 workgroups); else row unit by row unit
    const int bands = COOP ? qb_bands(nrb / RBU, nru, eighth, band_log2) : 0;
    const int v_end = !COOP ? units : eighth ? 8 * eighth : (units + 63) / 64 * 64;
    for (int v = COOP ? (int)blockIdx.x : wave; v < v_end; v += COOP ? (int)gridDim.x : nwaves) {
        const int u = COOP ? qb_unit(v, eighth) : v;
        if (COOP && u >= units) continue;
        const QbPlace place = qb_place(u, bands, band_log2, ncg);
        const int ru = place.ru, cg = place.cg;
        const int c0 = cg * kColsPerWave;
        const bool act = c0 + lane * 2 < cols;                        // column direction: this lane's 2 columns
        const bool ract = c0 + (lane & 15) * 8 < cols;                // row direction: this lane's 8 columns
        const int rb0 = ru * RBU;
        const int nb = min(nrb - rb0, RBU);
        const int swz_lo = lane & (CPR - 1);
        unsigned g4_lo = 0, g4_hi = 0;
        auto tile_x = [&](int k) { return tile_rsrc(x + (int64_t)(rb0 + k) * kBlock * ld + c0); };
        // Four row blocks done (the last group of a tensor may hold fewer: blocks 0 .. last): their scale bytes of a
        // column are one dword of the row-major array (when the row length allows it) and exactly one dword of the
        // grouped copy.
        auto store_col_scales = [&](int rbh, int last, unsigned lo, unsigned hi) {
            const rsrc_t ss = tile_rsrc(scales_c + (int64_t)c0 * nrb + rbh);
            const int voff = act ? 2 * lane * nrb : kPast;
            if ((nrb & 3) == 0) {
                __builtin_amdgcn_raw_buffer_store_b32(lo, ss, voff, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b32(hi, ss, voff, nrb, 0);
            } else if (!COOP) {
                for (int i = 0; i <= last; ++i) {
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(lo >> (8 * i)), ss, voff, i, 0);
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(hi >> (8 * i)), ss, voff, nrb + i, 0);
                }
            }
            if (g4_c)
                __builtin_amdgcn_raw_buffer_store_b64(v2u_t{lo, hi}, tile_rsrc(g4_c + ((int64_t)(rbh / kRowBlocksPerUnit) * kpitch_c + c0) * 4),
                                                      act ? lane * 8 : kPast, 0, 0);
        };
        auto fetch_col = [&](int k, unsigned (&cv)[32]) {
            const rsrc_t sx = tile_x(k);
            const int voff = act ? lane * 4 : kPast;
            int soff = 0;
#pragma unroll
            for (int i = 0; i < 32; ++i) { cv[i] = __builtin_amdgcn_raw_buffer_load_b32(sx, voff, soff, 0); step(soff, pitch_x); }
        };
        auto fetch_row = [&](int k, uint4 (&rv)[8]) {
            const rsrc_t sx = tile_x(k);
            const int voff = ract ? (lane >> 4) * pitch_x + (lane & 15) * 16 : kPast;
            int soff = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const v4u_t v = __builtin_amdgcn_raw_buffer_load_b128(sx, voff, soff, 0);
                rv[j] = make_uint4(v[0], v[1], v[2], v[3]);
                step(soff, 4 * pitch_x);
            }
        };
        auto work_col = [&](int k, unsigned (&cv)[32]) {
            unsigned y0, y1;
            if (STATS == 0) {
                ColBlock b;
                pair_col_block(cv, b);
                y0 = quant_one_column<FMT_C, RULE, false>(b.lo, b.am_lo, reg + (2 * lane) * ROWB, k, swz_lo, s0, se_c);
                y1 = quant_one_column<FMT_C, RULE, false>(b.hi, b.am_hi, reg + (2 * lane + 1) * ROWB, k, swz_lo, s0, se_c);
            } else {
                float xc[32];
#pragma unroll
                for (int i = 0; i < 32; ++i) { xc[i] = __uint_as_float(cv[i] << 16); acc_sq(cv[i], s0); }
                y0 = quant_column_stats<FMT_C, RULE, STATS>(xc, reg + (2 * lane) * ROWB, k, swz_lo, se_c, so_c);
                __builtin_amdgcn_sched_barrier(0);             // (both columns at once would not fit the registers)
#pragma unroll
                for (int i = 0; i < 32; ++i) xc[i] = __uint_as_float(cv[i] & 0xFFFF0000u);
                y1 = quant_column_stats<FMT_C, RULE, STATS>(xc, reg + (2 * lane + 1) * ROWB, k, swz_lo, se_c, so_c);
            }
            if (COOP) {
                // the four tiles of a dword belong to four waves: the bytes meet in LDS after the unit's barrier
                *reinterpret_cast<uint16_t*>(scale_stage + k * kColsPerWave + 2 * lane) = (uint16_t)(y0 | (y1 << 8));
            } else {
                g4_lo |= y0 << (8 * (k & 3));
                g4_hi |= y1 << (8 * (k & 3));
                if ((k & 3) == 3 || k == nb - 1) {
                    store_col_scales(rb0 + (k & ~3), k & 3, g4_lo, g4_hi);
                    g4_lo = 0; g4_hi = 0;
                }
            }
        };
        auto work_row = [&](int k, uint4 (&rv)[8]) {
            const int row0 = (rb0 + k) * kBlock;
            const rsrc_t sc_codes = tile_rsrc(codes_r + (int64_t)row0 * pitch_r + (FMT_R == kFP8 ? c0 : c0 / 2));
            const int voff = ract ? (lane >> 4) * pitch_r + (lane & 15) * (FMT_R == kFP8 ? 8 : 4) : kPast;
            int soff = 0;
            int d_lo = 0, d_hi = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (APART && j == kRowsMeet) __builtin_amdgcn_s_barrier();      // the one in front of the columns' stores
                const unsigned w[4] = {rv[j].x, rv[j].y, rv[j].z, rv[j].w};
                float x8[8];
                unsigned am;
                if (STATS == 0) {
                    am = quad_max(amax8(rv[j]));
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) unpack2(w[i], x8[2 * i], x8[2 * i + 1]);
                    am = quad_max(__float_as_uint(max_abs<8>(x8))) >> 16;
                }
                const unsigned byte = scale_byte<FMT_R, RULE>(am), other = scale_byte<1 - FMT_R, RULE>(am);
                const float sc = scale_operand(byte), sco = scale_operand(other);
                const bool bad = byte == 0xFFu;
                if (FMT_R == kFP8) {
                    unsigned e0 = STATS ? enc8x4<RULE>(x8, sc, byte) : enc8<RULE>(w[0], w[1], sc, byte);
                    unsigned e1 = STATS ? enc8x4<RULE>(x8 + 4, sc, byte) : enc8<RULE>(w[2], w[3], sc, byte);
                    if (bad) { e0 = 0; e1 = 0; }
                    __builtin_amdgcn_raw_buffer_store_b64(v2u_t{e0, e1}, sc_codes, voff, soff, STORE);
                    if (STATS) { err8x4(x8, e0, sc, se_r); err8x4(x8 + 4, e1, sc, se_r); }
                    if (STATS == 2) err4x8(x8, enc4x8(x8, sco), sco, so_r);
                } else {
                    unsigned e4 = STATS ? enc4x8(x8, sc) : enc4(w[0], w[1], w[2], w[3], sc);
                    if (bad) e4 = 0;
                    __builtin_amdgcn_raw_buffer_store_b32(e4, sc_codes, voff, soff, STORE);
                    if (STATS) err4x8(x8, e4, sc, se_r);
                    if (STATS == 2) {
                        err8x4(x8, enc8x4<RULE>(x8, sco, other), sco, so_r);
                        err8x4(x8 + 4, enc8x4<RULE>(x8 + 4, sco, other), sco, so_r);
                    }
                }
                step(soff, 4 * pitch_r);
                // the four block bytes of this row's 128 columns as a dword, in all 16 lanes of the row; quad j % 4 keeps it
                int d = (int)(byte << (8 * ((lane >> 2) & 3)));
                d |= __builtin_amdgcn_update_dpp(0, d, 0x124, 0xF, 0xF, true);                  // row_ror:4
                d |= __builtin_amdgcn_update_dpp(0, d, 0x128, 0xF, 0xF, true);                  // row_ror:8
                int& keep = j < 4 ? d_lo : d_hi;
                if ((j & 3) == 0) keep = __builtin_amdgcn_update_dpp(keep, d, 0xE4, 0xF, 1, false);
                if ((j & 3) == 1) keep = __builtin_amdgcn_update_dpp(keep, d, 0xE4, 0xF, 2, false);
                if ((j & 3) == 2) keep = __builtin_amdgcn_update_dpp(keep, d, 0xE4, 0xF, 4, false);
                if ((j & 3) == 3) keep = __builtin_amdgcn_update_dpp(keep, d, 0xE4, 0xF, 8, false);
            }
            // the tile's 32 dwords at once: one of the grouped copy and, when rows hold a whole number of groups, of the
            // row-major array per row
            const int row = 16 * (lane & 1) + 4 * ((lane >> 2) & 3) + (lane >> 4);
            const int d = lane & 1 ? d_hi : d_lo;
            const bool mine = (lane & 2) == 0;
            const rsrc_t ss = tile_rsrc(scales_r + (int64_t)row0 * nblk + cg * 4);
            const int soff_r = mine ? row * nblk : kPast;
            if ((nblk & 3) == 0) {
                __builtin_amdgcn_raw_buffer_store_b32(d, ss, soff_r, 0, 0);
            } else {
                // (four lanes to a row: all of a quad hold both dwords)
                int l = lane;
                asm volatile("" : "+v"(l));                    // (computed here, kept over the units it is registers that other waves need)
                const int b = l & 3, off = cg * 4 + b < nblk ? (4 * ((l >> 2) & 3) + (l >> 4)) * nblk + b : kPast;
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)((unsigned)d_lo >> (8 * b)), ss, off, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)((unsigned)d_hi >> (8 * b)), ss, off, 16 * nblk, 0);
            }
            if (g4_r) __builtin_amdgcn_raw_buffer_store_b32(d, tile_rsrc(g4_r + ((int64_t)cg * kpitch_r + row0) * 4), mine ? row * 4 : kPast, 0, 0);
        };
        if (RAW_LDS) {
            // 1 KB copies of four rows straight into LDS, dealt to all waves
#pragma unroll
            for (int i = 0; i < 8 * RBU / WPB; ++i) {
                const int q = i * WPB + wib;
                if (q < nb * 8)
                    copy_to_lds<kStream>(tile_x(q >> 3), reg + q * 1024, ract ? (lane >> 4) * pitch_x + (lane & 15) * 16 : kPast, (q & 7) * 4 * pitch_x);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0)
            __syncthreads();                                   // the raw tiles are there
            const int k = wib < NW ? wib : wib - NW;
            const uint8_t* raw = reg + k * RAW;
            // (behind the second barrier, the same one for both kinds, the tiles are in registers)
            if (wib < NW) {
                unsigned cv[32];
#pragma unroll
                for (int i = 0; i < 32; ++i) cv[i] = *reinterpret_cast<const unsigned*>(raw + i * 256 + lane * 4);
                __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0)
                __syncthreads();
                if (k < nb) work_col(k, cv);
            } else {
                uint4 rv[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) rv[j] = *reinterpret_cast<const uint4*>(raw + j * 1024 + lane * 16);
                __builtin_amdgcn_s_waitcnt(0xC07F);
                __syncthreads();
                if (k < nb) work_row(k, rv);
            }
        } else if (SPLIT) {
            const int k = wib < NW ? wib : wib - NW;
            if (wib < NW && k < nb) {
                unsigned cv[32];
                fetch_col(k, cv);
                work_col(k, cv);
            } else if (k < nb) {
                uint4 rv[8];
                fetch_row(k, rv);
                work_row(k, rv);
            } else if (APART && wib >= NW) {
                __builtin_amdgcn_s_barrier();
            }
        } else {
            for (int k = COOP ? wib : 0; k < nb; k += COOP ? NW : 1) {
                unsigned cv[32];
                uint4 rv[8];
                fetch_col(k, cv);
                fetch_row(k, rv);
                work_col(k, cv);
                work_row(k, rv);
            }
        }
        if (!APART || wib < NW) {                              // (the rows' waves have met this barrier on their way)
            if (COOP) {
                __syncthreads();                                   // all tiles of the unit are staged
                for (int g = wib; 4 * g < nb; g += CW) {
                    const int last = min(3, nb - 1 - 4 * g);
                    unsigned lo = 0, hi = 0;
                    for (int i = 0; i <= last; ++i) {
                        const unsigned v = *reinterpret_cast<const uint16_t*>(scale_stage + (4 * g + i) * kColsPerWave + 2 * lane);
                        lo |= (v & 0xFFu) << (8 * i);
                        hi |= (v >> 8) << (8 * i);
                    }
                    store_col_scales(rb0 + 4 * g, last, lo, hi);
                }
                // Rows of no whole number of dwords: bytes, four lanes to a column, the columns dealt to the waves (a lane for two whole
                // columns, in one wave, is four times the requests).
                if ((nrb & 3) != 0)
                    for (int p = wib; p < (nb + 3) / 4 * 8; p += CW) {
                        int l = lane;
                        asm volatile("" : "+v"(l));
                        const int blk = p / 8 * 4 + (l & 3), col = p % 8 * 16 + (l >> 2);
                        __builtin_amdgcn_raw_buffer_store_b8(scale_stage[blk * kColsPerWave + col], tile_rsrc(scales_c + (int64_t)c0 * nrb + rb0),
                                                             blk < nb && c0 + col < cols ? col * nrb + blk : kPast, 0, 0);
                    }
            }
            const rsrc_t sc_codes = tile_rsrc(codes_c + (int64_t)c0 * pitch_c + (int64_t)ru * ROWB);
            int l = lane;
            if (!COOP) asm volatile("" : "+v"(l));                 // (computed here: kept over the tiles, the addresses below spill registers)
            const int chunk = l % CPR, blk = FMT_C == kFP8 ? chunk >> 1 : chunk;
            const int lane_off = (l / CPR) * pitch_c + chunk * 16;
#pragma unroll
            for (int it = COOP ? wib : 0; it < kColsPerWave * CPR / 64; it += COOP ? CW : 1) {
                const int row = it * (64 / CPR) + l / CPR;
                const v4u_t q = *reinterpret_cast<const v4u_t*>(reg + row * ROWB + ((chunk ^ ((row >> 1) & (CPR - 1))) * 16));
                // (no scalar offset in a 16-byte store: see tile_rsrc)
                __builtin_amdgcn_raw_buffer_store_b128(q, sc_codes, c0 + row < cols && blk < nb ? lane_off + it * (64 / CPR) * pitch_c : kPast, 0, STORE);
            }
        }
        if (COOP) __syncthreads();                             // the staging areas go to the next unit
    }
    if (STATS) {
        s0 = wave_sum(s0);
        se_r = wave_sum(se_r);
        se_c = wave_sum(se_c);
        if (STATS == 2) { so_r = wave_sum(so_r); so_c = wave_sum(so_c); }
        const float sums[6] = {s0, FMT_R == kFP4 ? se_r : so_r, FMT_R == kFP8 ? se_r : so_r,
                               s0, FMT_C == kFP4 ? se_c : so_c, FMT_C == kFP8 ? se_c : so_c};
        store_wave_sums<WPB>(sums, wib, lane, partials);
    }
}

// Statistics only, both formats, column blocks.  Grid: blockIdx.y = row split; a wave owns a
// column group and the rows of its split, so per-column sums stay in the lane.
template <int RULE>
__global__ __launch_bounds__(256) void stats_col_kernel(const uint16_t* __restrict__ x, int rows,
                                                        int cols, int64_t ld, int nsplit,
                                                        float* __restrict__ partials,
                                                        float* __restrict__ line_partials)
{
    const int lane = threadIdx.x & 63;
    const int wave_x = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
    const int nwaves_x = gridDim.x * kWavesPerBlock;
    const int split = blockIdx.y;
    const int ncg = (cols + kColsPerWave - 1) / kColsPerWave;
    const int nrb = rows / kBlock;
    const int rb0 = (int)((int64_t)nrb * split / nsplit), rb1 = (int)((int64_t)nrb * (split + 1) / nsplit);
    float t0 = 0.f, t4 = 0.f, t8 = 0.f;
    for (int cg = wave_x; cg < ncg; cg += nwaves_x) {
        const int c = cg * kColsPerWave + lane * 2;
        const bool act = c < cols;
        float a0[2] = {0.f, 0.f}, a4[2] = {0.f, 0.f}, a8[2] = {0.f, 0.f};
        for (int rb = rb0; rb < rb1; ++rb) {
            unsigned v[32];
            const uint16_t* const p = x + (int64_t)rb * kBlock * ld + c;
#pragma unroll
            for (int i = 0; i < 32; ++i) v[i] = act ? ld4(p + (int64_t)i * ld) : 0u;     // (with load_col_tile: 192 registers, 10 % slower)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float xc[32], sq[4] = {0.f, 0.f, 0.f, 0.f};          // (a block's squares on their own: fewer roundings of the large sum)
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    xc[i] = __uint_as_float(h ? v[i] & 0xFFFF0000u : v[i] << 16);
                    sq[i & 3] = fmaf(xc[i], xc[i], sq[i & 3]);
                }
                a0[h] += (sq[0] + sq[1]) + (sq[2] + sq[3]);
                const unsigned am = magnitude_bits(max_abs<32>(xc));
                both_errors<32, RULE>(xc, am, a4[h], a8[h]);
                if (am >= 0x7F80u) { a4[h] = __builtin_nanf(""); a8[h] = __builtin_nanf(""); }
            }
        }
        if (line_partials && act) {
            float* lp = line_partials + ((int64_t)split * cols + c) * 3;
            lp[0] = a0[0]; lp[1] = a4[0]; lp[2] = a8[0];
            lp[3] = a0[1]; lp[4] = a4[1]; lp[5] = a8[1];
        }
        t0 += a0[0] + a0[1]; t4 += a4[0] + a4[1]; t8 += a8[0] + a8[1];
    }
    t0 = wave_sum(t0); t4 = wave_sum(t4); t8 = wave_sum(t8);
    if (lane == 0) {
        float* p = partials + ((int64_t)split * nwaves_x + wave_x) * 3;
        p[0] = t0; p[1] = t4; p[2] = t8;
    }
}

// Statistics for BOTH block directions from one read of the matrix (the complete Step-1 record of a tensor:
// its forward operands are blocked along rows, its backward ones down columns, Sec. 2.2).
// A wave takes 32 x 128 tiles w, w + waves, ... (row-major), so that the chip reads one band of rows at a time; a lane
// reads two adjacent columns of every row.  The column-direction errors come straight from those registers
// (a column's block never leaves the lane).  For the row direction the raw tile goes through the
// wave's 8 KB of LDS and comes back as eight 16-byte pieces per lane: two whole 32-element row blocks, so that
// the row direction, too, forms a block's maximum and scales inside one lane.  LDS operations of one wave execute in order,
// so no barrier is needed between the writes and the reads.
// Bound by vector arithmetic: 18 instructions per element, 4 of them conversions (two at half the rate).  Against waves that
// own a column group and a range of rows, a branch around every load (us per call): [16384 x 4096] 57.6 -> 45.5, [11008 x
// 4096] 43.8 -> 35.4, [16384 x 11008] 130 -> 118, [16384 x 96] 32 -> 7.7.  Loading the next tile during the row phase needs
// 142 registers and is slower (50.8, 37.5, 120).
// partials: [workgroups][6] = {sum x^2, row err4, row err8, sum x^2, col err4, col err8}.
template <int RULE>
__global__ __launch_bounds__(256) void stats_both_kernel(const uint16_t* __restrict__ x, int rows,
                                                         int cols, int64_t ld,
                                                         double* __restrict__ partials)
{
    __shared__ __attribute__((aligned(16))) unsigned tile[kWavesPerBlock][kBlock * 64];
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned* const raw = tile[wib];
    const int nwaves = gridDim.x * kWavesPerBlock;
    const int ncg = (cols + kColsPerWave - 1) / kColsPerWave;
    const int ntiles = rows / kBlock * ncg;
    float t0 = 0.f, r4 = 0.f, r8 = 0.f, c4 = 0.f, c8 = 0.f;
    bool bad = false;
    // LDS image of the raw tile: row i holds its sixteen 16-byte pieces at positions piece ^ (i % 4), so that the
    // 16 lanes served together by a 16-byte read (4 rows x 4 blocks) fall into 16 different bank groups.
    int wpos[4], rpos[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        wpos[t] = (((lane >> 2) ^ t) << 2) | (lane & 3);                                   // dword lane of a row with i % 4 == t
        rpos[t] = (lane >> 2) * 64 + ((((lane & 3) * 4 + t) ^ ((lane >> 2) & 3)) << 2);    // piece t of block lane % 4, row lane / 4
    }
    for (int t = blockIdx.x * kWavesPerBlock + wib; t < ntiles; t += nwaves) {
        const int rb = t / ncg, c0 = (t - rb * ncg) * kColsPerWave;
        unsigned v[32];
        load_col_tile(x + (int64_t)rb * kBlock * ld, c0, lane, cols, ld, v);
#pragma unroll
        for (int i = 0; i < 32; ++i) raw[i * 64 + wpos[i & 3]] = v[i];
        // ---- column direction ----
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float xc[32];
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                xc[i] = __uint_as_float(h ? v[i] & 0xFFFF0000u : v[i] << 16);
                if (h == 0) acc_sq(v[i], t0);
            }
            const unsigned am = magnitude_bits(max_abs<32>(xc));
            both_errors<32, RULE>(xc, am, c4, c8);
            bad |= am >= 0x7F80u;
        }
        // ---- row direction: the lane takes two whole blocks, block lane % 4 of tile rows lane / 4 and
        //      16 + lane / 4, as four 16-byte pieces each, so that a block's maximum and its two scales are
        //      formed once per 32 elements, inside the lane ----
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float xr[32];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint4 q = *reinterpret_cast<const uint4*>(raw + h * 16 * 64 + rpos[k]);
                unpack2(q.x, xr[8 * k + 0], xr[8 * k + 1]);
                unpack2(q.y, xr[8 * k + 2], xr[8 * k + 3]);
                unpack2(q.z, xr[8 * k + 4], xr[8 * k + 5]);
                unpack2(q.w, xr[8 * k + 6], xr[8 * k + 7]);
            }
            const unsigned am = magnitude_bits(max_abs<32>(xr));
            both_errors<32, RULE>(xr, am, r4, r8);
            bad |= am >= 0x7F80u;
        }
    }
    if (bad) { r4 = c4 = r8 = c8 = __builtin_nanf(""); }     // a non-finite element poisons every error sum of the wave
    t0 = wave_sum(t0); r4 = wave_sum(r4); r8 = wave_sum(r8); c4 = wave_sum(c4); c8 = wave_sum(c8);
    const float sums[6] = {t0, r4, r8, t0, c4, c8};
    store_wave_sums<kWavesPerBlock>(sums, wib, lane, partials);
}

// Second stages: one workgroup adds n partials in double, in a fixed order: thread t takes partials t, t + 512, ..., wave j
// then adds component j over the threads.
constexpr int kReduceThreads = 512;
template <int N>
__device__ __forceinline__ double reduce_workgroup(const double (&a)[N], double (*sh)[kReduceThreads])      // sh[N]; sum of component j in every lane of wave j
{
#pragma unroll
    for (int j = 0; j < N; ++j) sh[j][threadIdx.x] = a[j];
    __syncthreads();
    const int j = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double t = 0.0;
    if (j < N) {
#pragma unroll
        for (int k = 0; k < kReduceThreads / 64; ++k) t += sh[j][k * 64 + lane];
        t = wave_sum(t);
    }
    return t;
}

// Partials [n][6] of both block directions; out_row and out_col receive three doubles each.
__global__ __launch_bounds__(kReduceThreads) void reduce_both_kernel(const double* __restrict__ partials, int n,
                                                           double* __restrict__ out_row, double* __restrict__ out_col,
                                                           int mode_row, int mode_col)
{
    __shared__ double sh[6][kReduceThreads];
    double a[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += kReduceThreads) {
        const double2* p = reinterpret_cast<const double2*>(partials + (size_t)i * 6);
        const double2 v0 = p[0], v1 = p[1], v2 = p[2];
        a[0] += v0.x; a[1] += v0.y; a[2] += v1.x;
        a[3] += v1.y; a[4] += v2.x; a[5] += v2.y;
    }
    const double t = reduce_workgroup<6>(a, sh);
    // mode 0: all three sums; mode 1 (fused FP4): the FP8 field is NaN; mode 2 (fused FP8): the FP4 field is NaN
    const int j = threadIdx.x >> 6;
    if (j < 6 && (threadIdx.x & 63) == 0) {
        const int f = j % 3;
        const int mode = j < 3 ? mode_row : mode_col;
        double* out = j < 3 ? out_row : out_col;
        const bool absent = (mode == 1 && f == 2) || (mode == 2 && f == 1);
        if (out) out[f] = absent ? __builtin_nan("") : t;
    }
}

// Partials [n][3] of one block direction.
// mode 0: out = {p0, p1, p2}; mode 1 (fused FP4): out = {p0, p1, NaN}; mode 2 (fused FP8): {p0, NaN, p1}.
__global__ __launch_bounds__(kReduceThreads) void reduce_partials_kernel(const float* __restrict__ partials, int n,
                                                                         int mode, double* __restrict__ out)
{
    __shared__ double sh[3][kReduceThreads];
    double a[3] = {0.0, 0.0, 0.0};
#pragma unroll 8
    for (int i = threadIdx.x; i < n; i += kReduceThreads) {
        const float* p = partials + (size_t)i * 3;
        a[0] += (double)p[0]; a[1] += (double)p[1]; a[2] += (double)p[2];
    }
    const double t = reduce_workgroup<3>(a, sh);
    const int j = threadIdx.x >> 6;
    if (j < 3 && (threadIdx.x & 63) == 0) {
        // the fused statistics deliver two sums: p1 is the error of the format that was written
        if (mode == 0 || j == 0) out[j] = t;
        else if (j == 1) { out[mode] = t; out[3 - mode] = __builtin_nan(""); }
    }
}

// Per-column sums: add the row splits in order.
__global__ __launch_bounds__(256) void reduce_lines_kernel(const float* __restrict__ line_partials, int nsplit,
                                                           int64_t n3, float* __restrict__ per_line)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n3) return;
    double a = 0.0;
    for (int s = 0; s < nsplit; ++s) a += (double)line_partials[(int64_t)s * n3 + i];
    per_line[i] = (float)a;
}

int col_splits(int64_t rows, int64_t cols, int* gx)
{
    const int ncg = (int)((cols + kColsPerWave - 1) / kColsPerWave);
    int g = (ncg + kWavesPerBlock - 1) / kWavesPerBlock;
    if (g > kStreamBlocks) g = kStreamBlocks;
    const int nrb = (int)(rows / kBlock);
    int64_t want = kStreamWaves / ((int64_t)g * kWavesPerBlock);
    if (want < 1) want = 1;
    if (want > kMaxColSplits) want = kMaxColSplits;
    if (want > nrb) want = nrb > 0 ? nrb : 1;
    *gx = g;
    return (int)want;
}

}  // namespace

size_t workspace_bytes(int64_t rows, int64_t cols)
{
    (void)rows;
    return stream_workspace_bytes(cols);
}

// Workgroups for `units` equal work units that waves take in turn: as many waves as give every wave the
// same number of units (the last one possibly fewer), at most kStreamWaves.  11008 units on 8192 waves would
// leave three quarters of the device idle during the second turn; 5504 waves take two units each.
static int balanced_blocks(int64_t units)
{
    if (units <= 0) return 1;
    const int64_t per_wave = (units + kStreamWaves - 1) / kStreamWaves;
    const int64_t waves = (units + per_wave - 1) / per_wave;
    return (int)((waves + kWavesPerBlock - 1) / kWavesPerBlock);
}

// Returns the number of workgroups launched (= partial-sum slots used, times kWavesPerBlock).
template <int FMT, int RULE, bool STATS, bool SR = false>
static int launch_q(const QuantArgs& a, float* partials, hipStream_t s)
{
    const uint2 seed = make_uint2((unsigned)a.sr_seed, (unsigned)(a.sr_seed >> 32));
    int blocks;
    // pitch of the block-major scale copy = padded number of STORED rows
    if (a.axis == 0) {
        // without statistics (a partial-sum slot per wave) a wave per unit: the dispatcher hands them out more evenly than a
        // fixed grid takes them ([8192 x 8192] FP4 33.3 -> 30.9 us, [16384 x 11008] 87.9 -> 81.4, FP8 115.6 -> 105.8, [1920 x 9088] 13.3 -> 12.4)
        const int64_t units = ((a.rows + kUnroll - 1) / kUnroll) * ((a.cols + kSeg - 1) / kSeg), groups = (units + kWavesPerBlock - 1) / kWavesPerBlock;
        blocks = STATS ? balanced_blocks(units) : (int)(groups < kMostBlocks ? groups : kMostBlocks);
        hipLaunchKernelGGL((quant_row_kernel<FMT, RULE, STATS, SR>), dim3(blocks), dim3(256), 0, s,
                           a.x, (int)a.rows, (int)a.cols, a.ld, a.codes, a.scales, a.scales_g4,
                           g4_pitch(a.rows), partials, seed);
    } else {
        const int64_t nrb = a.rows / kBlock;
        const int rbu = (FMT == kFP8 || SR) ? kRowBlocksPerUnit : 2 * kRowBlocksPerUnit;       // as in quant_col_kernel
        const int64_t units = ((a.cols + kColsPerWave - 1) / kColsPerWave) * ((nrb + rbu - 1) / rbu);
        // a workgroup per unit (see quant_col_kernel); SNIP_QUANT_COL_UNIT=wave|workgroup, read at every call, fixes
        // the choice for tests and measurements
        bool coop = true;
        if (const char* e = getenv("SNIP_QUANT_COL_UNIT")) coop = !(e[0] == 'w' && e[1] == 'a');
        if (coop) {
            // Without statistics as many workgroups as units, except that units of eight row blocks (FP4 to nearest) keep the
            // fixed grid: us per call, fixed grid -> all units, [8192 x 8192] FP8 43 -> 39.3, stochastic 42 -> 38.2, [16384 x 11008]
            // 108.7 -> 105.2 and 109 -> 99.5, FP4 88.0 -> 89.9.
            const int64_t most = STATS || rbu > kRowBlocksPerUnit ? kStreamBlocks : kMostBlocks;
            blocks = (int)(units < most ? units : most);
            hipLaunchKernelGGL((quant_col_kernel<FMT, RULE, STATS, SR, true>), dim3(blocks), dim3(256), 0, s,
                               a.x, (int)a.rows, (int)a.cols, a.ld, a.codes, a.scales, a.scales_g4,
                               g4_pitch(a.cols), partials, seed);
        } else {
            blocks = balanced_blocks(units);
            hipLaunchKernelGGL((quant_col_kernel<FMT, RULE, STATS, SR, false>), dim3(blocks), dim3(256), 0, s,
                               a.x, (int)a.rows, (int)a.cols, a.ld, a.codes, a.scales, a.scales_g4,
                               g4_pitch(a.cols), partials, seed);
        }
    }
    return blocks;
}

hipError_t launch_quantize(const QuantArgs& a, hipStream_t s)
{
    if (a.rows == 0 || a.cols == 0) {
        if (a.stats) {
            hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(kReduceThreads), 0, s,
                               (const float*)a.workspace, 0, a.fmt == kFP4 ? 1 : 2, a.stats);
        }
        return hipGetLastError();
    }
    float* partials = (float*)a.workspace;
    const bool st = a.stats != nullptr;
    if (a.stochastic) {
        if (a.fmt != kFP4 || st) return hipErrorInvalidValue;
        if (a.rule == 0) launch_q<kFP4, 0, false, true>(a, partials, s);
        else             launch_q<kFP4, 1, false, true>(a, partials, s);
        return hipGetLastError();
    }
    const int key = (a.fmt << 2) | (a.rule << 1) | (st ? 1 : 0);
    int blocks = 0;
    switch (key) {
        case 0: blocks = launch_q<kFP8, 0, false>(a, partials, s); break;
        case 1: blocks = launch_q<kFP8, 0, true>(a, partials, s); break;
        case 2: blocks = launch_q<kFP8, 1, false>(a, partials, s); break;
        case 3: blocks = launch_q<kFP8, 1, true>(a, partials, s); break;
        case 4: blocks = launch_q<kFP4, 0, false>(a, partials, s); break;
        case 5: blocks = launch_q<kFP4, 0, true>(a, partials, s); break;
        case 6: blocks = launch_q<kFP4, 1, false>(a, partials, s); break;
        case 7: blocks = launch_q<kFP4, 1, true>(a, partials, s); break;
        default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (st) {
        hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(kReduceThreads), 0, s,
                           (const float*)partials, blocks * kWavesPerBlock, a.fmt == kFP4 ? 1 : 2, a.stats);
        e = hipGetLastError();
    }
    return e;
}

// Work distribution of quant_both_kernel: waves of a workgroup x tiles of the unit they share (Apart: APART, Lds: RAW_LDS), or a wave
// per unit.
enum class QbForm { k4x4, k4x4Apart, k4x4Lds, k4x8, kWave };

template <int FMT_R, int FMT_C, int RULE, int STATS, int NW, int RBU, bool RAW_LDS = false, bool STREAM = false, bool APART = false>
static int launch_qb_form(const QuantBothArgs& a, double* partials, hipStream_t s)
{
    const int64_t nrb = a.rows / kBlock;
    const int64_t units = ((a.cols + kColsPerWave - 1) / kColsPerWave) * ((nrb + RBU - 1) / RBU);
    // order of the units (picks.h)
    const int64_t column_bytes = FMT_C == kFP8 ? a.rows : a.rows / 2;
    const bool eighths = qb_eighths(a.rows, a.cols, a.ld, column_bytes, STATS != 0);
    const int band_log2 = eighths ? 1 : qb_band_log2(a.cols, column_bytes);
    const int64_t eighth = eighths ? (units + 7) / 8 : 0;
    // A workgroup per unit.  With statistics it also needs a partial-sum slot, and its waves' sums cost as much as a sixth
    // of a tile: at most kStreamBlocks workgroups with equal shares of the units then.
    const int64_t most = STATS ? kStreamBlocks / 8 : (int64_t)1 << 24, run = eighths ? eighth : (units + 63) / 64 * 8, share = (run + most - 1) / most;
    const int blocks = NW ? (int)(8 * ((run + share - 1) / share)) : balanced_blocks(units);
    hipLaunchKernelGGL((quant_both_kernel<FMT_R, FMT_C, RULE, STATS, NW, RBU, RAW_LDS, STREAM, APART>), dim3(blocks), dim3(qb_threads(NW, STATS)), 0, s,
                       a.x, (int)a.rows, (int)a.cols, a.ld, a.codes_r, a.scales_r, a.g4_r, g4_pitch(a.rows),
                       a.codes_c, a.scales_c, a.g4_c, g4_pitch(a.cols), partials, (int)eighth, band_log2);
    return blocks;
}

template <int FMT_R, int FMT_C, int RULE, int STATS>
static int launch_qb(const QuantBothArgs& a, double* partials, QbForm form, hipStream_t s)
{
    const bool stream = qb_streams(a.rows, a.cols, FMT_R == kFP8, FMT_C == kFP8, STATS != 0, (uintptr_t)a.codes_r, (uintptr_t)a.codes_c);
    if constexpr (STATS != 0)
        if (form == QbForm::kWave)
            return stream ? launch_qb_form<FMT_R, FMT_C, RULE, STATS, 0, FMT_C == kFP8 ? 4 : 8, false, true>(a, partials, s)
                          : launch_qb_form<FMT_R, FMT_C, RULE, STATS, 0, FMT_C == kFP8 ? 4 : 8>(a, partials, s);
    if constexpr (FMT_C == kFP4 && STATS != 0)
        if (form == QbForm::k4x8) return launch_qb_form<FMT_R, FMT_C, RULE, STATS, 4, 8>(a, partials, s);
    if constexpr (STATS == 0)
        if (form == QbForm::k4x4Lds)
            return stream ? launch_qb_form<FMT_R, FMT_C, RULE, STATS, 4, 4, true, true>(a, partials, s)
                          : launch_qb_form<FMT_R, FMT_C, RULE, STATS, 4, 4, true>(a, partials, s);
    if constexpr (STATS == 0)
        if (form == QbForm::k4x4Apart) return launch_qb_form<FMT_R, FMT_C, RULE, STATS, 4, 4, false, false, true>(a, partials, s);
    return launch_qb_form<FMT_R, FMT_C, RULE, STATS, 4, 4>(a, partials, s);
}

// Which distribution serves a call (measured, us per call back to back in a graph):
//   - four waves with a tile each (for either direction, without statistics) wherever nothing else is said: the loads of a
//     tile are a wave's whole chain.  Against four waves with two tiles each (FP4 codes of columns): [2048 x 2048] 9.0 -> 6.4,
//     [4096 x 4096] 15.5 -> 12.8, [8192 x 4096] 27.2 -> 21.9.
//   - without statistics the tiles go through LDS where qb_through_lds (picks.h) says so.
//   - the complete statistics fill the registers (two waves per SIMD in any form), and a workgroup's barrier and sums cost
//     8-20 %: a wave per unit as soon as that gives every SIMD work, from 28 M elements (48 M with FP4 codes of columns: eight
//     tiles per unit): [3072 x 8192] FP8 41.2 (wave) against 38.8 (4 x 4), [8192 x 4096] 41.9 against 47.2; FP4 between
//     12 M and 48 M elements four waves with two tiles each: [4096 x 4096] 26.0 against 28.6 (4 x 4) and 42.7 (wave).
//   - statistics of the written formats: a wave per unit from 56 M elements on ([16384 x 4096] FP4 62.9 (4 x 4) -> 61.7, FP8 71.2
//     -> 71.1, [16384 x 8192] 122 -> 109 and 141 -> 128; [12288 x 4096] 50.8 against 59.0 and 56.6 against 57.9), if at two
//     waves per SIMD the last round is not too empty ([24576 x 4096] FP4, 0.75 of whole rounds, 95.2 -> 88.8; [16384 x 5120],
//     0.62, 82.6 against 88.0) and, for FP4 columns, rows start on whole lines ([12320 x 8224] 118 against 116, 4 x 8 112).
//     FP4 columns that a wave per unit does not serve take four waves with two tiles each from 20 M on ([8192 x 4096] 37.7 (4 x 4) ->
//     34.6, beside FP8 rows 39.2 -> 36.1, [16384 x 5120] 81 -> 77; [4096 x 5120] 27.0 against 27.1, [4096 x 3072] 19.6 against 19.9).
constexpr int64_t kTwoWavesPerSimd = 2048;
static QbForm pick_qb_form(const QuantBothArgs& a, int stats)
{
    QbForm direct = QbForm::k4x4;
    bool through_lds = false;
    if (stats == 0) {
        const int64_t units = ((a.cols + kColsPerWave - 1) / kColsPerWave) * ((a.rows / kBlock + 3) / 4), ncu = gemm_compute_units();
        if (qb_rows_apart(units, ncu)) direct = QbForm::k4x4Apart;
        through_lds = qb_through_lds(a.cols, units, ncu);
    }
    // SNIP_QUANT_BOTH_UNIT=4x4|lds|4x8|wave in the environment, read at every call, fixes the form where it exists for the
    // call, =workgroup keeps to a workgroup per unit; for tests and measurements
    bool group = false;
    if (const char* e = getenv("SNIP_QUANT_BOTH_UNIT")) {
        const bool fp4 = a.fmt_c == kFP4;
        const struct { const char* name; QbForm form; bool exists; } kForms[] = {
            {"4x4", direct, true}, {"4x8", QbForm::k4x8, fp4 && stats != 0}, {"lds", QbForm::k4x4Lds, stats == 0}, {"wave", QbForm::kWave, stats != 0}};
        for (const auto& f : kForms)
            if (!strcmp(e, f.name) && f.exists) return f.form;
        group = !strcmp(e, "workgroup");
    }
    const int64_t elems = a.rows * a.cols;
    if (stats == 0) return through_lds ? QbForm::k4x4Lds : direct;
    if (stats == 1) {
        const int64_t tiles = a.fmt_c == kFP8 ? 4 : 8, waves = ((a.cols + kColsPerWave - 1) / kColsPerWave) * ((a.rows / kBlock + tiles - 1) / tiles);
        const int64_t rounds = (waves + kTwoWavesPerSimd - 1) / kTwoWavesPerSimd;
        const bool many = elems > ((int64_t)56 << 20), full = 100 * waves >= 65 * rounds * kTwoWavesPerSimd;
        if (many && full && (a.fmt_c == kFP8 || a.ld % 128 == 0) && !group) return QbForm::kWave;
        return a.fmt_c == kFP4 && elems > ((int64_t)20 << 20) ? QbForm::k4x8 : QbForm::k4x4;
    }
    if (elems > ((int64_t)(a.fmt_c == kFP8 ? 28 : 48) << 20) && !group) return QbForm::kWave;
    return a.fmt_c == kFP4 && elems > ((int64_t)12 << 20) ? QbForm::k4x8 : QbForm::k4x4;
}

// quant_both_kernel addresses a tile, and the column codes of a unit, with 32-bit offsets.
static bool qb_offsets_fit(const QuantBothArgs& a)
{
    const int64_t most = (int64_t)1 << 31;
    return a.ld * 2 * kBlock + 256 < most && a.cols * kBlock + 256 < most && a.rows * kColsPerWave + 256 < most;
}

// Rows longer than that (32 M elements of a source row, 16 M rows): one orientation at a time, and the complete record from
// the statistics kernel.  Codes and scales are the same bytes.
static hipError_t launch_quantize_each(const QuantBothArgs& a, hipStream_t s)
{
    for (int axis = 0; axis < 2; ++axis) {
        QuantArgs q;
        q.x = a.x; q.rows = a.rows; q.cols = a.cols; q.ld = a.ld;
        q.fmt = axis ? a.fmt_c : a.fmt_r; q.axis = axis; q.rule = a.rule;
        q.codes = axis ? a.codes_c : a.codes_r; q.scales = axis ? a.scales_c : a.scales_r; q.scales_g4 = axis ? a.g4_c : a.g4_r;
        q.stats = a.both_formats ? nullptr : axis ? a.stats_c : a.stats_r;
        q.workspace = a.workspace;
        const hipError_t e = launch_quantize(q, s);
        if (e != hipSuccess) return e;
    }
    if (!a.stats_r || !a.both_formats) return hipSuccess;
    StatsArgs t;
    t.x = a.x; t.rows = a.rows; t.cols = a.cols; t.ld = a.ld;
    t.axis = 0; t.rule = a.rule; t.stats = a.stats_r; t.per_line = nullptr; t.workspace = a.workspace;
    return launch_stats_both(t, a.stats_c, s);
}

hipError_t launch_quantize_both(const QuantBothArgs& a, hipStream_t s)
{
    if (a.rows > 0 && a.cols > 0 && !qb_offsets_fit(a)) return launch_quantize_each(a, s);
    double* partials = (double*)a.workspace;
    const bool st = a.stats_r != nullptr;
    // second stage: which field of each triple is "not computed" (NaN); none when both formats are wanted
    const int mode_r = a.both_formats ? 0 : (a.fmt_r == kFP4 ? 1 : 2), mode_c = a.both_formats ? 0 : (a.fmt_c == kFP4 ? 1 : 2);
    if (a.rows == 0 || a.cols == 0) {
        if (st) hipLaunchKernelGGL(reduce_both_kernel, dim3(1), dim3(kReduceThreads), 0, s, (const double*)partials, 0, a.stats_r, a.stats_c, mode_r, mode_c);
        return hipGetLastError();
    }
    const int mode = !st ? 0 : (a.both_formats ? 2 : 1);
    const QbForm form = pick_qb_form(a, mode);
    int blocks = 0;
    const int key = (a.fmt_r << 4) | (a.fmt_c << 3) | (a.rule << 2) | mode;
    switch (key) {
#define SNIP_QB_CASE(FR, FC, RU) \
        case ((FR) << 4) | ((FC) << 3) | ((RU) << 2) | 0: blocks = launch_qb<FR, FC, RU, 0>(a, partials, form, s); break; \
        case ((FR) << 4) | ((FC) << 3) | ((RU) << 2) | 1: blocks = launch_qb<FR, FC, RU, 1>(a, partials, form, s); break; \
        case ((FR) << 4) | ((FC) << 3) | ((RU) << 2) | 2: blocks = launch_qb<FR, FC, RU, 2>(a, partials, form, s); break;
        SNIP_QB_CASE(0, 0, 0) SNIP_QB_CASE(0, 0, 1) SNIP_QB_CASE(0, 1, 0) SNIP_QB_CASE(0, 1, 1)
        SNIP_QB_CASE(1, 0, 0) SNIP_QB_CASE(1, 0, 1) SNIP_QB_CASE(1, 1, 0) SNIP_QB_CASE(1, 1, 1)
#undef SNIP_QB_CASE
        default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (st) {
        hipLaunchKernelGGL(reduce_both_kernel, dim3(1), dim3(kReduceThreads), 0, s, (const double*)partials, blocks,
                           a.stats_r, a.stats_c, mode_r, mode_c);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_stats_both(const StatsArgs& a, double* out_col, hipStream_t s)
{
    double* partials = (double*)a.workspace;
    if (a.rows == 0 || a.cols == 0) {
        hipLaunchKernelGGL(reduce_both_kernel, dim3(1), dim3(kReduceThreads), 0, s, (const double*)partials, 0, a.stats, out_col, 0, 0);
        return hipGetLastError();
    }
    // every wave the same number of tiles or one less
    const int64_t tiles = (a.rows / kBlock) * ((a.cols + kColsPerWave - 1) / kColsPerWave), most = kStreamWaves;
    const int64_t share = (tiles + most - 1) / most, waves = (tiles + share - 1) / share;
    const int blocks = (int)((waves + kWavesPerBlock - 1) / kWavesPerBlock);
    if (a.rule == 0)
        hipLaunchKernelGGL((stats_both_kernel<0>), dim3(blocks), dim3(256), 0, s, a.x, (int)a.rows, (int)a.cols, a.ld, partials);
    else
        hipLaunchKernelGGL((stats_both_kernel<1>), dim3(blocks), dim3(256), 0, s, a.x, (int)a.rows, (int)a.cols, a.ld, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_both_kernel, dim3(1), dim3(kReduceThreads), 0, s, (const double*)partials, blocks,
                       a.stats, out_col, 0, 0);
    return hipGetLastError();
}

hipError_t launch_stats(const StatsArgs& a, hipStream_t s)
{
    float* partials = (float*)a.workspace;
    if (a.rows == 0 || a.cols == 0) {
        hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(kReduceThreads), 0, s, (const float*)partials, 0, 0, a.stats);
        return hipGetLastError();
    }
    int npart;
    if (a.axis == 0) {
        const int blocks = balanced_blocks(a.rows);             // a wave per row
        if (a.rule == 0)
            hipLaunchKernelGGL((stats_row_kernel<0>), dim3(blocks), dim3(256), 0, s,
                               a.x, (int)a.rows, (int)a.cols, a.ld, partials, a.per_line);
        else
            hipLaunchKernelGGL((stats_row_kernel<1>), dim3(blocks), dim3(256), 0, s,
                               a.x, (int)a.rows, (int)a.cols, a.ld, partials, a.per_line);
        npart = blocks * kWavesPerBlock;
    } else {
        int gx;
        const int nsplit = col_splits(a.rows, a.cols, &gx);
        float* lines = a.per_line ? (float*)((char*)a.workspace + kPartialBytes) : nullptr;
        if (a.rule == 0)
            hipLaunchKernelGGL((stats_col_kernel<0>), dim3(gx, nsplit), dim3(256), 0, s,
                               a.x, (int)a.rows, (int)a.cols, a.ld, nsplit, partials, lines);
        else
            hipLaunchKernelGGL((stats_col_kernel<1>), dim3(gx, nsplit), dim3(256), 0, s,
                               a.x, (int)a.rows, (int)a.cols, a.ld, nsplit, partials, lines);
        npart = gx * kWavesPerBlock * nsplit;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (a.per_line) {
            const int64_t n3 = a.cols * 3;
            hipLaunchKernelGGL(reduce_lines_kernel, dim3((unsigned)((n3 + 255) / 256)), dim3(256), 0, s,
                               (const float*)lines, nsplit, n3, a.per_line);
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(kReduceThreads), 0, s, (const float*)partials, npart, 0, a.stats);
    return hipGetLastError();
}

}  // namespace snip

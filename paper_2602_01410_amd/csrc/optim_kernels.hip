// AdamW factor of the weight-divergence estimate (SNIP Sec. 4.3.2 "Impact on Weight Divergence").
// With m = beta1 m' + (1 - beta1) g and v = beta2 v' + (1 - beta2) g^2, the update direction
// h(g) = m / (sqrt(v) + eps) has the element-wise derivative
//     (1 - beta1) / (sqrt(v) + eps)  -  (1 - beta2) m g / (sqrt(v) (sqrt(v) + eps)^2),
// and Step 1 of the method collects its Frobenius norm.  One streaming pass over m, v (fp32) and
// g (fp32 or bf16): 12 or 10 bytes per element read, nothing written but one partial per wave: bound by
// HBM.  fp32 arithmetic: square root and quotients come from the hardware's approximations and a Newton step each, the
// root and eps are rounded together: over 2^20 elements the sum is within 4e-9 of 64-bit arithmetic, where a correctly rounded
// root plus eps was up to 3e-8 off (eps is a constant number of units in the root's last place).  One element's squared first
// part is 0.9e-7 off (rms; correctly rounded 0.9-1.0e-7), its second part 1.9e-7 (1.9-2.5e-7); with one approximated root
// in the second part and no step for it it was 1.9-2.2e-7.  An element takes 29 vector instructions, not 46.  Sums per lane
// (four, added in double) and wave in fp32, across waves in double in a fixed order.
#include "snip_internal.h"

namespace snip {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

// Correctly rounded square root and divisions, for any argument.
__device__ __forceinline__ float sens_any(float m, float v, float g, float c1, float c2, float eps)
{
    const float root = __fsqrt_rn(v);
    const float d = root + eps;
    const float first = __fdiv_rn(c1, d);
    // v == 0: AdamW has m = g = 0 there and the second part is taken as zero (the expression is 0/0)
    const float second = v > 0.f ? __fdiv_rn(c2 * m * g, root * d * d) : 0.f;
    return first - second;
}

// The same where v is 0 or in [kLow, kHigh] and eps in [kLow, 1] (nothing under- or overflows on the way that the result does
// not); `w` is v, or 1 in place of 0.  A NaN in v reaches the term: it is told from 0 by ==, not by >.
constexpr float kLow = 0x1p-96f, kHigh = 0x1p96f;
__device__ __forceinline__ float sens_normal(float m, float v, float w, float g, float c1, float c2, float eps)
{
    const float y = __builtin_amdgcn_rsqf(w);
    const float s = w * y, h = 0.5f * y;
    // s plus the rest of the root and eps, rounded once (eps is a fixed number of units in the last place of the root)
    const float d = v == 0.f ? eps : s + fmaf(fmaf(-s, s, w), h, eps);
    const float r0 = __builtin_amdgcn_rcpf(d);
    const float r = fmaf(r0, fmaf(-d, r0, 1.f), r0);
    const float second = v == 0.f ? 0.f : c2 * m * g * r * r * fmaf(h, fmaf(-s, y, 1.f), y);      // (1 / root last: it may be 2^48)
    const float q = c1 * r, first = fmaf(fmaf(-q, d, c1), r, q);
    return first - second;
}

// Four elements; acc[i] += (term of element i)^2.
__device__ __forceinline__ void sens4(v4f m, v4f v, v4f g, float c1, float c2, float eps, bool eps_normal, v4f& acc)
{
    v4f w, t;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = v[i] == 0.f ? 1.f : v[i];
    const float lo = fminf(fminf(w[0], w[1]), fminf(w[2], w[3])), hi = fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3]));
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(lo >= kLow && hi <= kHigh && eps_normal)) == 0, 1)) {       // wave-uniform
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = sens_normal(m[i], v[i], w[i], g[i], c1, c2, eps);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = sens_any(m[i], v[i], g[i], c1, c2, eps);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = fmaf(t[i], t[i], acc[i]);
}

template <bool G_BF16>
__global__ __launch_bounds__(256) void adamw_sens_kernel(const float* __restrict__ m, const float* __restrict__ v,
                                                         const void* __restrict__ g, int64_t n, float c1, float c2,
                                                         float eps, float* __restrict__ partials)
{
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t nthreads = (int64_t)gridDim.x * 256;
    const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t n4 = n / 4;
    const bool eps_normal = eps >= kLow && eps <= 1.f;
    v4f acc4 = {0.f, 0.f, 0.f, 0.f};
    // streaming (non-temporal) loads: nothing is read twice and the three arrays exceed every cache
    auto load = [&](int64_t q, v4f& mm, v4f& vv, v4f& gg) {
        mm = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(m) + q);
        vv = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(v) + q);
        if (G_BF16) {
            const v2u w = __builtin_nontemporal_load(reinterpret_cast<const v2u*>(g) + q);
            gg = v4f{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u),
                     __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xFFFF0000u)};
        } else {
            gg = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(g) + q);
        }
    };
    for (int64_t q = tid; q < n4; q += nthreads) {
        v4f mm, vv, gg;
        load(q, mm, vv, gg);
        sens4(mm, vv, gg, c1, c2, eps, eps_normal, acc4);
    }
    float acc = (float)(((double)acc4[0] + acc4[1]) + ((double)acc4[2] + acc4[3]));
    // the last n % 4 elements
    const int64_t i = n4 * 4 + tid;
    if (i < n) {
        const float gi = G_BF16 ? __uint_as_float((unsigned)reinterpret_cast<const uint16_t*>(g)[i] << 16)
                                : reinterpret_cast<const float*>(g)[i];
        const float t = sens_any(m[i], v[i], gi, c1, c2, eps);
        acc = fmaf(t, t, acc);
    }
    acc = wave_sum(acc);
    if (lane == 0) partials[wave] = acc;
}

}  // namespace

hipError_t launch_adamw_sensitivity(const AdamwArgs& a, hipStream_t s)
{
    float* partials = (float*)a.workspace;
    // At most 1024 workgroups (four waves per SIMD): more waves in flight than that only spread the three
    // streams over more memory pages.  [11008 x 4096], bf16 gradient, us with 512 / 768 / 1024 / 1536 / 2048 workgroups: 83 / 75.5 /
    // 75 / 76 / 80 (correctly rounded divisions, 2048: 82); [4096 x 4096] 34 / 31 / 30 / 32 / 32 (34), fp32 gradient [28671 x 8191] 427 /
    // 413 / 431 / 461 / 502 (480).  Fewer of them with equal shares leave compute units with three beside others with four: 2.05 M
    // elements 9.7 -> 8.1, 2.5 M 10.2 -> 8.8, 4.5 M 13.3 -> 12.0.
    constexpr int64_t most = 1024;
    static_assert(most <= kStreamBlocks, "partials");
    const int64_t groups = (a.n + 4 * 256 - 1) / (4 * 256);
    const int blocks = (int)(groups < most ? groups : most);
    if (a.n > 0) {
        const float c1 = 1.0f - a.beta1, c2 = 1.0f - a.beta2;
        if (a.g_bf16)
            hipLaunchKernelGGL(adamw_sens_kernel<true>, dim3(blocks), dim3(256), 0, s, a.m, a.v, a.g, a.n, c1, c2, a.eps, partials);
        else
            hipLaunchKernelGGL(adamw_sens_kernel<false>, dim3(blocks), dim3(256), 0, s, a.m, a.v, a.g, a.n, c1, c2, a.eps, partials);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_sum_partials(partials, blocks * kWavesPerBlock, a.out, s);
}

}  // namespace snip

// Internal launcher interface between the C-ABI layer (api.hip) and the kernel files.
// Nothing here is exported.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "picks.h"

namespace snip {

constexpr int kFP8 = 0;   // E4M3
constexpr int kFP4 = 1;   // E2M1
constexpr int kBlock = 32;  // elements per scale

// Number of waves the streaming kernels are launched with; also the number of per-wave
// partial-sum slots at the start of the workspace.  Fixed (not device dependent) so that
// reductions run in the same order everywhere.
constexpr int kStreamBlocks = 2048;
constexpr int kWavesPerBlock = 4;
constexpr int kStreamWaves = kStreamBlocks * kWavesPerBlock;
constexpr int64_t kMostBlocks = (int64_t)1 << 22;    // workgroups of a launch that needs no slot per workgroup (threads are counted in 32 bits)
constexpr int kMaxColSplits = 64;    // row splits of the column-statistics kernel
// Workspace of the streaming kernels: partial sums, for one block direction [kStreamWaves][3] fp32 of waves, for both at most
// [kStreamBlocks][6] fp64 of workgroups; then [kMaxColSplits][cols][3] fp32 per-column partials for the per-line column
// statistics.
constexpr size_t kPartialBytes = (size_t)kStreamWaves * 6 * sizeof(float);
static_assert((size_t)kStreamBlocks * 6 * sizeof(double) <= kPartialBytes && (size_t)kStreamWaves * 3 * sizeof(float) <= kPartialBytes, "partial sums");
constexpr size_t stream_workspace_bytes(int64_t cols) { return kPartialBytes + (size_t)kMaxColSplits * (size_t)cols * 3 * sizeof(float); }
constexpr int kG4Align = 256;    // row pitch (in dwords) of the grouped scale copy is a multiple of this
__host__ __device__ inline int64_t g4_pitch(int64_t rows) { return (rows + kG4Align - 1) / kG4Align * kG4Align; }

// Sum over a wave (all lanes active), in every lane: a balanced tree of adds of neighbours, rows of 16 lanes and pairs of rows by
// DPP, a few cycles a step where a shuffle through LDS takes about 100.  A statistics kernel ends with three to five such sums, its
// second stage with one on doubles; both together, us per call: quantize with statistics [256 x 512] 7.9 -> 7.55, [1504 x 1568]
// 10.3 -> 9.8, [2048 x 2048] 11.5 -> 11.1.
template <int CTRL, int ROWS> __device__ __forceinline__ int dpp_or_zero(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false); }
template <int CTRL, int ROWS> __device__ __forceinline__ float dpp_add(float v) { return v + __int_as_float(dpp_or_zero<CTRL, ROWS>(__float_as_int(v))); }
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v)
{
    return v + __hiloint2double(dpp_or_zero<CTRL, ROWS>(__double2hiint(v)), dpp_or_zero<CTRL, ROWS>(__double2loint(v)));
}
template <class T> __device__ __forceinline__ T wave_tree(T v)      // in lane 63
{
    // DPP reads a register two wait states after a vector instruction wrote it; the compiler does not keep that distance to
    // inline assembly, which is where the sums of squares come from
    asm volatile("s_nop 4" : "+v"(v));
    v = dpp_add<0x111, 0xF>(v);                 // row_shr:1, 2, 4, 8: lane 15 of a row has the row's sum
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);                 // row_bcast:15 to rows 1 and 3
    return dpp_add<0x143, 0xC>(v);              // row_bcast:31 to rows 2 and 3
}
__device__ __forceinline__ float wave_sum(float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_tree(v)), 63)); }
__device__ __forceinline__ double wave_sum(double v)
{
    v = wave_tree(v);
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63), __builtin_amdgcn_readlane(__double2loint(v), 63));
}

struct QuantArgs {
    const uint16_t* x;
    int64_t rows, cols, ld;
    int fmt, axis, rule;
    uint8_t* codes;
    uint8_t* scales;
    uint8_t* scales_g4;       // [ceil(stored cols / 128)][g4_pitch(stored rows)][4] or nullptr
    double* stats;        // device snip_stats (3 doubles) or nullptr
    void* workspace;
    bool stochastic = false;  // FP4 only: stochastic rounding with the byte stream of sr_seed
    uint64_t sr_seed = 0;
};

// One source matrix quantized in both orientations by one pass (snip_quantize_both).
struct QuantBothArgs {
    const uint16_t* x;
    int64_t rows, cols, ld;
    int rule;
    int fmt_r, fmt_c;                        // row-direction output [rows][cols], column-direction output [cols][rows]
    uint8_t *codes_r, *scales_r, *g4_r;
    uint8_t *codes_c, *scales_c, *g4_c;
    double *stats_r, *stats_c;               // both or neither
    bool both_formats = false;               // statistics: also the error of the format not written
    void* workspace;
};

struct StatsArgs {
    const uint16_t* x;
    int64_t rows, cols, ld;
    int axis, rule;
    double* stats;        // device, 3 doubles
    float* per_line;      // device [L][3] or nullptr
    void* workspace;
};

struct GemmArgs {
    const uint8_t* a_codes; const uint8_t* a_scales; const uint8_t* a_scales_g4; int fmt_a;
    const uint8_t* b_codes; const uint8_t* b_scales; const uint8_t* b_scales_g4; int fmt_b;
    int64_t I, J, R;      // C[I][J] = sum_r A[I][r] B[J][r]
    void* c; int64_t ldc; int out_fp32;
    // optional: squared Frobenius norm of the stored output.  norm_partials has room for
    // gemm_norm_partials(I, J) floats (one per workgroup of the launch); norm_out is one double.
    float* norm_partials = nullptr;
    double* norm_out = nullptr;
};
inline double gemm_operand_bytes(const GemmArgs& a)
{
    return (double)a.I * a.R * (a.fmt_a == kFP8 ? 1.0 : 0.5) + (double)a.J * a.R * (a.fmt_b == kFP8 ? 1.0 : 0.5);
}
// Whether the result is stored streaming.
template <class Args> bool gemm_streams(const Args& a) { return streams_result((uintptr_t)a.c, a.ldc, a.out_fp32); }
constexpr double kColdBytes = 10e6;      // operands of more than that are taken to come from memory (the tables in gemm.hip say why)
// Upper bound of the number of partials either GEMM kernel writes for an I x J output (128 x 128 tiles).
inline int64_t gemm_norm_partials(int64_t I, int64_t J) { return ((I + 127) / 128) * ((J + 127) / 128); }

struct AdamwArgs {
    const float* m; const float* v; const void* g; int g_bf16;
    int64_t n;
    float beta1, beta2, eps;
    double* out;          // device, one double
    void* workspace;      // room for kStreamWaves floats
};

// The paper's own recipe (real-valued scale per 1x128 tile or 128x128 block): quantize (stats == nullptr)
// or statistics of both formats (stats != nullptr; codes / scales unused).
struct PaperArgs {
    const uint16_t* x;
    int64_t rows, cols, ld;
    int fmt, axis;
    bool blocks;           // false: 1x128 tiles, true: 128x128 blocks (stored orientation)
    uint8_t* codes;
    float* scales;
    double* stats;         // device, 3 doubles
    void* workspace;       // statistics only: paper_workspace_bytes(rows, cols)
};
struct GemmPaperArgs {
    const uint8_t* a_codes; const float* a_scales; int a_group; int fmt_a;     // group: 1 (tiles) or 128 (blocks)
    const uint8_t* b_codes; const float* b_scales; int b_group; int fmt_b;
    int64_t I, J, R;      // C[I][J] = sum_r (A[I][r] / sa) (B[J][r] / sb)
    void* c; int64_t ldc; int out_fp32;
};
// Every row's scales on 16 bytes: the 256 x 128 kernel then copies four slabs' at once.
inline bool gemm_paper_scales16(const GemmPaperArgs& a) { return a.R % 512 == 0 && (((uintptr_t)a.a_scales | (uintptr_t)a.b_scales) & 15) == 0; }
hipError_t launch_gemm_paper(const GemmPaperArgs& a, hipStream_t s);
bool gemm_paper_wide_eligible(const GemmPaperArgs& a);
hipError_t launch_gemm_paper_wide(const GemmPaperArgs& a, hipStream_t s);
size_t paper_workspace_bytes(int64_t rows, int64_t cols);
hipError_t launch_paper(const PaperArgs& a, hipStream_t s);

size_t workspace_bytes(int64_t rows, int64_t cols);
hipError_t launch_adamw_sensitivity(const AdamwArgs& a, hipStream_t s);
// out[i] = sum of partials[i * stride ... i * stride + n) in a fixed order, in double, for i < sums; n may be 0
hipError_t launch_sum_partials(const float* partials, int64_t n, double* out, hipStream_t s, int sums = 1, int64_t stride = 0);
hipError_t launch_quantize(const QuantArgs& a, hipStream_t s);
hipError_t launch_quantize_both(const QuantBothArgs& a, hipStream_t s);
hipError_t launch_stats(const StatsArgs& a, hipStream_t s);
// both block directions from one read: a.stats receives the row-direction record, out_col the column one
// (a.axis and a.per_line are ignored)
hipError_t launch_stats_both(const StatsArgs& a, double* out_col, hipStream_t s);
hipError_t launch_gemm(const GemmArgs& a, hipStream_t s);
// Workgroup tiles of the GEMM kernels: the persistent kernel's (gemm_fast.hip), those of one tile per workgroup
// (gemm_small.hip) and the general kernel's (gemm.hip).
enum class GemmTile { kBig, kWide, k128x128, k64x64, k64x32, k32x32, kGeneral };
bool gemm_fast_eligible(const GemmArgs& a);
bool gemm_small_eligible(const GemmArgs& a);
hipError_t launch_gemm_fast(const GemmArgs& a, GemmTile tile, hipStream_t s);
hipError_t launch_gemm_small(const GemmArgs& a, GemmTile tile, hipStream_t s);
int gemm_compute_units();   // of the current device, a multiple of 8

}  // namespace snip

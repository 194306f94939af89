// Source ranges of the GEMM kernels' copies through raw buffer descriptors, apart from the kernels so that they can be
// checked without a GPU.
//
// A copy's source byte is the descriptor's base + a wave-uniform offset + an offset per lane, and it is in range while the
// lane's offset lies below size - uniform offset.  That difference is unsigned: a uniform offset past the size need not
// give zeros, so every range below keeps it within the size.  What is not there is put out of range by the size or by the
// lane's offset.
#pragma once
#ifdef __HIPCC__
#define SNIP_HD __host__ __device__
#else
#define SNIP_HD
#endif

namespace snip {

struct CopyRange { unsigned size, uniform; };

// Sizes stay below 2^31, so that kNoSource (gemm_common.h) is past every one of them and a group past the last one still has
// a 32-bit offset.
constexpr bool descriptor_covers(long long bytes) { return bytes < 1ll << 31; }

// Codes of stage `st`: `bytes` of a tile's rows, `step` bytes of a row per stage.  Past the last stage nothing is in range.
SNIP_HD constexpr CopyRange code_range(int st, int nstage, unsigned bytes, unsigned step)
{
    return st < nstage ? CopyRange{bytes, (unsigned)st * step} : CopyRange{0u, 0u};
}

// Grouped scales of stage `st` (`ng` groups of 128 contraction elements) for the rows from byte `row0` of a group on: `ngrp`
// groups, `pitch` bytes apart.  A lane's offset is scale_lane(group inside the stage, row); for the group that an odd `ngrp`
// leaves out of a last stage it lies at or past size - uniform.
SNIP_HD constexpr unsigned scale_size(int ngrp, unsigned pitch, unsigned row0) { return (unsigned)ngrp * pitch - row0; }
SNIP_HD constexpr unsigned scale_uniform(int st, int ng, unsigned pitch) { return (unsigned)(st * ng) * pitch; }
SNIP_HD constexpr CopyRange scale_range(int st, int nstage, int ngrp, int ng, unsigned pitch, unsigned row0)
{
    return st < nstage ? CopyRange{scale_size(ngrp, pitch, row0), scale_uniform(st, ng, pitch)} : CopyRange{0u, 0u};
}
SNIP_HD constexpr unsigned scale_lane(int group, int row, unsigned pitch) { return (unsigned)group * pitch + (unsigned)row * 4u; }

}  // namespace snip

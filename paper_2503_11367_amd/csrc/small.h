// Which shares run in the single-launch kernels of small.hip, and their entry points.
#pragma once
#include "common.h"

namespace mm {

// most 32-token units of the sequence, and of the share, which is no longer; most blocks of it (of at
// least 16 tokens): what the kernels' lists in LDS hold
constexpr int kSmallUnits = 128, kSmallBlocks = 2 * kSmallUnits;

inline bool small_fits(const AttnArgs& a) { return a.S <= 32 * kSmallUnits; }
inline int64_t small_row_units(const AttnArgs& a) { return ((int64_t)a.n_blocks * a.block + 31) / 32; }
inline int64_t small_fwd_wgs(const AttnArgs& a) { return small_row_units(a) * (a.Hq / a.Hkv) * a.kv_count; }

// Forward: as long as the general path's launches cost more than it gains by sharing K/V tiles
// between rows and heads.  Few workgroups may have at most 2048 keys each (from there on the
// general path's slices, which spread over the chip, are ahead: 4096 tokens, 256 rows, 2 / 1 heads,
// 16 workgroups 22.9 us here, 21.7 there), many of them at most 2^21 / workgroups (32 / 8 heads:
// 2048 tokens, 1024 rows 45 us here, 53 there at head_dim 128, 30 and 32 at 64; 2048 rows, 128 and 70).
inline bool small_fwd_wanted(const AttnArgs& a) {
    const int64_t wgs = small_fwd_wgs(a);
    return small_fits(a) && wgs <= 1024 && wgs * a.S <= (1 << 21) && (a.S <= 2048 || wgs * 64 >= a.S);
}
// Workgroups of four wavefronts, of which two or three share a CU, where the chip has no room for
// all of eight at once (2048 tokens, 1024 rows, 16 / 4 heads, 512 workgroups: 19.6 us with four, 27 with
// eight), and where there is hardly a unit for each of eight (256 tokens 7.0 / 7.5 us).
inline bool small_fwd_four(const AttnArgs& a) { return small_fwd_wgs(a) > 256 || a.S <= 256; }

// Backward (workgroups: 32 keys of a KV head for dK, as many for dV, 32 rows of a head for dQ): up to
// about three rounds of one workgroup per CU, and no dK / dV workgroup with more than 24 units per
// wavefront.  Beyond either the general path, whose tiles are shared by 128 keys, is level or ahead (2048
// tokens, 1024 rows, 32 / 8 heads: 157 us both at head_dim 128, 100 here and 92 there at 64; 2048 rows,
// 8 / 1 heads, sinks and a window, 64 units per wavefront: 161 and 107 us).
inline bool small_bwd_wanted(const AttnArgs& a) {
    const int64_t rows = small_row_units(a), wgs = 2 * (a.S / 32) * a.Hkv + rows * a.Hq;
    return small_fits(a) && wgs <= 768 && rows * (a.Hq / a.Hkv) <= 192;
}

// `err`: the call's status word and its spare words (kFlagInts)
int launch_fwd_small(const AttnArgs& a, void* o, float* lse, int32_t* err, hipStream_t st);
int launch_bwd_small(const AttnArgs& a, const void* o, const float* lse, const void* d_o, void* dq, void* dk, void* dv,
                     int32_t* err, hipStream_t st);

}  // namespace mm

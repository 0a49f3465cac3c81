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
// 16 workgroups 22.9 us here, 21.7 there), many of them at most 3 * 2^20 / workgroups, and 2^22 at head_dim 64,
// where three share a CU.  Here / there, us, head_dim 128: 2560 tokens, 12 / 4 heads (960) 56 / 66; 3584 tokens, 8 / 8
// heads, window (896) 39 / 56; 4096 tokens, 6 / 2 heads (768) 61 / 68; beyond, 3072 tokens, 12 / 4 heads (1152)
// 79 / 77, 1280 tokens, 64 / 8 heads (2560) 70 / 68.  Head_dim 64: 2560 tokens, 16 / 16 heads (1280) 41 / 57, 1024
// tokens, 64 / 16 heads (2048) 36 / 41; beyond, 1536 tokens, 48 / 16 heads (2304) 35 / 29.
inline bool small_fwd_wanted(const AttnArgs& a) {
    const int64_t wgs = small_fwd_wgs(a);
    const int64_t most = a.D == 128 ? 1024 : 2048, most_keys = a.D == 128 ? (int64_t)3 << 20 : (int64_t)1 << 22;
    return small_fits(a) && wgs <= most && wgs * a.S <= most_keys && (a.S <= 2048 || wgs * 64 >= a.S);
}
// Workgroups of four wavefronts, of which two or three share a CU, where the chip has no room for
// all of eight at once (2048 tokens, 1024 rows, 16 / 4 heads, 512 workgroups: 19.6 us with four, 27 with
// eight), and where there is hardly a unit for each of eight (256 tokens 7.0 / 7.5 us).
inline bool small_fwd_four(const AttnArgs& a) { return small_fwd_wgs(a) > 256 || a.S <= 256; }

// Backward (workgroups: 32 keys of a KV head for dK, as many for dV, 32 rows of a head for dQ): up to
// six rounds of one workgroup per CU, beyond 1536 tokens, where walks are longer and a causal mask has
// the two paths level sooner, three, or five at head_dim 64; and no dK / dV workgroup with more than 28 units per
// wavefront.  Beyond, the general path, whose tiles are shared by 128 keys, is level or ahead.  Here / there, us,
// up to 1536 tokens: 1280 tokens, 12 / 4 heads (800 workgroups) 49 / 90, 768 tokens, 32 / 8 heads (1152) 53 / 74, 1024
// tokens, 32 / 8 heads (1536) 85 / 115; head_dim 64, 512 tokens, 64 / 16 heads (1536) 60 / 66; beyond, 1280 tokens,
// 16 / 16 heads (1920) 90 / 84, 1024 tokens, 64 / 16 heads of 64 (3072) 137 / 117.  Longer: 3584 tokens, 2 / 1
// heads of 64 (448, 28 units) 36 / 61, 3072 tokens, 1536 rows, 4 / 4 heads of 64 (960) 42 / 62; beyond, 2048 tokens, 512 rows, 32 / 8 heads (1536) 98 / 98, 4096 tokens, 6 / 2
// heads (1280, 48 units) 202 / 198.
inline bool small_bwd_wanted(const AttnArgs& a) {
    const int64_t rows = small_row_units(a), wgs = 2 * (a.S / 32) * a.Hkv + rows * a.Hq;
    return small_fits(a) && wgs <= (a.S <= 1536 ? 1536 : a.D == 64 ? 1280 : 768) && rows * (a.Hq / a.Hkv) <= 224;
}

// `err`: the call's status word and its spare words (kFlagInts)
int launch_fwd_small(const AttnArgs& a, void* o, float* lse, int32_t* err, hipStream_t st);
int launch_bwd_small(const AttnArgs& a, const void* o, const float* lse, const void* d_o, void* dq, void* dk, void* dv,
                     int32_t* err, hipStream_t st);

}  // namespace mm

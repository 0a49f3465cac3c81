// Device bodies of the tile map (paper section 3.2.1) and of the block-list check, shared
// by the public tile-map kernel and by the first launch of the attention passes, where
// they run side by side with that pass's other independent preparation work.
#pragma once
#include <algorithm>
#include <type_traits>
#include "common.h"

namespace mm {

constexpr int kTmThreads = 256;
constexpr int kTmWaves = kTmThreads / kWave;
constexpr int kTmGroup = 32;       // most q-tiles and most k-tiles of a workgroup
constexpr int64_t kTmNarrow = (int64_t)1 << 30;      // up to this length positions are 32-bit
constexpr int kTmSplit = 3;        // more runs than this in a q-tile are shared out over the idle threads
constexpr int kTmAhead = 4;        // tiles whose words a wavefront requests together

// One launch serves up to two maps of the same rows (the second map's workgroups follow
// the first's in the one-dimensional grid).  A workgroup takes gq q-tiles x gk k-tiles (powers
// of two, at most kTmGroup each).
struct TileMapJob {
    int32_t tq, tk, nq, nk, gq, gk;
    int32_t kpw;                         // > 0: row by row, four wavefronts of kpw k-tiles each
    uint32_t gx, gy;                     // workgroups this map needs
    uint8_t* cls;
    uint32_t* cnt;
};
struct TileMapJobs { TileMapJob j[2]; };

// What a kernel's copy of the code below is for: maps counted row by row with up to 64, 128, any
// number of rows per tile, the same at positions beyond 32 bits, maps whose tiles are cut into
// runs.  A kernel for all of them needs 21 KiB more LDS and twice the code where neither is used:
// small maps took 0.2 to 0.5 us longer (64 x 64 tiles of 64 x 64: 6.3 against 6.0 us).  kTmBeside:
// other workgroups of the launch stream through memory, so that the map may not take much LDS.
// kTmWhole: the rows are the whole sequence, no list of blocks to look positions up in.
enum : int { kTmRows1 = 1, kTmRows2 = 2, kTmRows4 = 4, kTmWide = 8, kTmByRuns = 16, kTmBeside = 32, kTmWhole = 64 };

// A run: consecutive tokens of a tile that carry the same fields (x: the attend word of query
// rows, the modality of keys) at consecutive positions.  A list of runs ends with an entry
// whose `at` is the tile's length.  (One form for both: with shorter entries for keys the cutting
// took 6 % longer on large maps.  That whole multiples of 64 bytes lie between lists does not matter: padded by 16, the same times.)
struct TmRun { uint32_t ss, x, pos, at; };

// the value held by the next lower lane; lane 0 gets `first`
__device__ __forceinline__ uint32_t lane_below(uint32_t v, uint32_t first) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}

// Pairs (row, key) with key position <= row position for n rows and m keys at consecutive
// positions, summed row by row from prefix(x) = sum of min(t, m) over t = 1..x: the first row
// looks at d = row position - first key position + 1 keys.  Modulo 2^32 throughout (a tile
// has at most 2^31 pairs).
__device__ __forceinline__ uint32_t prefix_pairs(int32_t x, uint32_t m) {
    if (x <= 0) return 0u;
    const uint32_t y = min((uint32_t)x, m);
    const uint32_t tri = (y & 1u) ? ((y + 1u) >> 1) * y : (y >> 1) * (y + 1u);
    return tri + ((uint32_t)x - y) * m;
}
__device__ __forceinline__ uint32_t pairs_upto(int32_t d, int32_t n, uint32_t m) {
    return prefix_pairs(d + n - 1, m) - prefix_pairs(d - 1, m);
}

// A pair's count and class
__device__ __forceinline__ void tile_map_put(const TileMapJob& J, int64_t rows, int64_t i, int64_t j, uint32_t total) {
    const uint32_t full = (uint32_t)rows * (uint32_t)J.tk;
    if (J.cnt) J.cnt[i * J.nk + j] = total;
    if (J.cls)
        J.cls[i * J.nk + j] = total == 0 ? MMATTN_TILE_EMPTY
                              : (total == full ? MMATTN_TILE_FULL : MMATTN_TILE_PARTIAL);
}

// The rows that a map covers: all of the sequence, or those of a list of blocks.  The list may be
// a caller's unchecked one: an entry outside [0, n_seq_blocks) counts as block 0, exactly as
// validate_blocks_body rewrites it.
struct TmRows {
    const uint64_t* __restrict__ bits;
    const int32_t* __restrict__ blocks;
    int32_t block;
    int64_t n_seq_blocks, n_rows;
    // rows of q-tile i (the last one may be ragged)
    __device__ __forceinline__ int64_t of_tile(int32_t tq, int32_t i) const {
        return min((int64_t)tq, n_rows - (int64_t)i * tq);
    }
    __device__ __forceinline__ int64_t pos(int64_t r) const {
        if (!blocks) return r;
        const uint32_t b = (uint32_t)r / (uint32_t)block;    // a share has fewer than 2^31 rows
        int64_t g = blocks[b];
        if (g < 0 || g >= n_seq_blocks) g = 0;
        return g * block + ((uint32_t)r - b * (uint32_t)block);
    }
};

// The pairs first + bit of `left` of a group of tiles (from i0, j0 on; 1 << log_gk k-tiles wide),
// one after the other by a whole wavefront, row by row: up to 64 kRows rows in registers, kept
// while the q-tile stays the same, their words in flight together; a lane counts its rows
// against each run of keys.  The next 64 keys' words are requested ahead
// of their use, also those of the next pair.  kTiles == 2 (q-tiles of at most 32 rows): the
// tile below goes along on the other half of the lanes when it is in `left` too.  T holds a
// position.  Bound by the instructions per (64 kRows rows, run of keys).
template <int kRows, int kTiles, int kAtOnce, class T>
__device__ __forceinline__ void tile_map_by_rows(const TileMapJob& J, const TmRows& in, int32_t i0, int32_t j0,
                                                 int log_gk, uint64_t left, int first) {
    constexpr int kLanes = kWave / kTiles;
    const int lane = threadIdx.x & (kWave - 1), below = lane / kLanes;       // below: second tile
    const int gk = 1 << log_gk;
    const int32_t tq = J.tq, tk = J.tk;
    const uint64_t* __restrict__ bits = in.bits;
    T q[kRows];
    uint32_t ss_q[kRows], att[kRows];
    bool spans[kRows], windows = false;
    auto first_keys = [&](uint64_t of) -> uint64_t {         // of the first pair in `of`
        if (!of || lane >= tk) return 0;
        const int p = first + __ffsll((unsigned long long)of) - 1;
        return bits[(int64_t)(j0 + (p & (gk - 1))) * tk + lane];
    };
    uint64_t wk_first = first_keys(left);
    int64_t have = -1;                                       // the q-tile(s) whose rows are in registers
    while (left) {
        const int bit = __ffsll((unsigned long long)left) - 1, p = first + bit;
        const bool both = kTiles == 2 && bit + gk < 64 && (left >> (bit + gk) & 1u);
        left &= left - 1;
        if (both) left &= ~(1ull << (bit + gk));
        const uint64_t wk_mine = wk_first;
        wk_first = first_keys(left);
        const int32_t i = i0 + (p >> log_gk), j = j0 + (p & (gk - 1));
        const int64_t k0 = (int64_t)j * tk;
        const int32_t rows = kTiles == 2 && below && !both ? 0 : (int32_t)in.of_tile(tq, i + below);
        uint32_t part = 0;
        for (int32_t r0 = 0; kTiles == 2 ? r0 == 0 : r0 < rows; r0 += kRows * kWave) {
            const int n_r = kTiles == 2 ? 1 : min(kRows, (rows - r0 + kWave - 1) / kWave);
            uint64_t wk_next = r0 == 0 ? wk_mine : lane < tk ? bits[k0 + lane] : 0;
            if (have != 2 * (int64_t)i + both || (kTiles == 1 && rows > kRows * kWave)) {      // wave-uniform
                have = 2 * (int64_t)i + both;
                uint64_t w[kRows];
#pragma unroll
                for (int u = 0; u < kRows; ++u) {
                    q[u] = 0;
                    w[u] = 0;                                // (a word of zeros sees nothing)
                    const int32_t r = r0 + u * kWave + lane % kLanes;
                    if (u < n_r && r < rows) {
                        const int64_t pos = in.pos((int64_t)(i + below) * tq + r);
                        q[u] = (T)pos;
                        w[u] = bits[pos];
                    }
                }
                bool any = false;
#pragma unroll
                for (int u = 0; u < kRows; ++u) {
                    ss_q[u] = word_ss(w[u]);
                    att[u] = word_att(w[u]);
                    spans[u] = (ss_q[u] & 0xFFFFu) != 0u;
                    any = any || att_window(att[u]) != 0u;
                }
                windows = __any(any);
            }
            for (int kc = 0; kc < tk; kc += kWave) {
                // run starts among these keys: a key whose fields differ from its predecessor's
                const int n_keys = min(kWave, tk - kc);
                const uint64_t wk = wk_next;
                if (kc + kWave < tk) wk_next = kc + kWave + lane < tk ? bits[k0 + kc + kWave + lane] : 0;
                const uint32_t ss_k = word_ss(wk), mod_k = word_mod(wk);
                const uint32_t b_ss = lane_below(ss_k, 0u), b_mod = lane_below(mod_k, 0u);
                const bool starts = lane < n_keys && (lane == 0 || ss_k != b_ss || mod_k != b_mod);
                uint64_t m = __ballot(starts);
                while (m) {
                    // run v is keys at[v] .. at[v + 1] - 1 (past the last run: none)
                    int at[kAtOnce + 1];
                    at[0] = __ffsll((unsigned long long)m) - 1;
#pragma unroll
                    for (int v = 0; v < kAtOnce; ++v) {
                        m &= m - 1;
                        at[v + 1] = m ? __ffsll((unsigned long long)m) - 1 : n_keys;
                    }
#pragma unroll
                    for (int v = 0; v < kAtOnce; ++v) {
                        const int a = v == 0 ? at[0] : at[v] & (kWave - 1);
                        const uint32_t ss_r = (uint32_t)__builtin_amdgcn_readlane((int)ss_k, a);
                        const uint32_t mod_r = (uint32_t)__builtin_amdgcn_readlane((int)mod_k, a);
                        const T before = (T)(k0 + kc + at[v] - 1), len = (T)(at[v + 1] - at[v]);
#pragma unroll
                        for (int u = 0; u < kRows; ++u) {
                            if (kRows > 1 && u >= n_r) continue;     // wave-uniform
                            const bool same_span = spans[u] && ss_q[u] == ss_r;
                            const bool back = (ss_q[u] >> 16) == (ss_r >> 16) && ((att[u] >> mod_r) & 1u);
                            // keys of the run at or before the row's position, minus those a look-back
                            // window over the row's own modality cuts off
                            T seen = max(T(0), min((T)(q[u] - before), len));
                            if (windows) {                   // wave-uniform
                                const T win = (T)att_window(att[u]);
                                const T cut = max(T(0), min((T)(q[u] - win - before), len));
                                if (win != 0 && mod_r == att_modality(att[u])) seen -= cut;
                            }
                            part += (uint32_t)(same_span ? len : (back ? seen : T(0)));
                        }
                    }
                }
            }
        }
        for (int off = kLanes / 2; off > 0; off >>= 1) part += __shfl_xor(part, off);
        if (lane % kLanes == 0 && (below == 0 || both)) tile_map_put(J, rows, i + below, j, part);
    }
}

// kMany: for tiles of many runs, two of which at once keep a wavefront busier (tiles of 64 x 64
// over 32768 tokens in spans of 1 to 3: 555 -> 538 us) and where short tiles go two together
// (32 x 32: 1290 -> 725 us, with both 610).  Tiles of one run would pay for a second that is not there.
template <int CODE, bool kMany>
__device__ __forceinline__ void tile_map_by_rows_any(const TileMapJob& J, const TmRows& in, int32_t i0, int32_t j0,
                                                     int log_gk, uint64_t left, int first) {
    constexpr int kAtOnce = kMany ? 2 : 1;
    if constexpr (kMany && (CODE & kTmRows1))
        if (J.tq <= kWave / 2) return tile_map_by_rows<1, 2, kAtOnce, int32_t>(J, in, i0, j0, log_gk, left, first);
    if constexpr ((CODE & kTmRows1) != 0)
        if (J.tq <= kWave) return tile_map_by_rows<1, 1, kAtOnce, int32_t>(J, in, i0, j0, log_gk, left, first);
    if constexpr ((CODE & kTmRows2) != 0)
        if (J.tq <= 2 * kWave) return tile_map_by_rows<2, 1, kAtOnce, int32_t>(J, in, i0, j0, log_gk, left, first);
    if constexpr ((CODE & kTmRows4) != 0) tile_map_by_rows<4, 1, kAtOnce, int32_t>(J, in, i0, j0, log_gk, left, first);
    if constexpr ((CODE & kTmWide) != 0) tile_map_by_rows<4, 1, kAtOnce, int64_t>(J, in, i0, j0, log_gk, left, first);
}

// A layout is a handful of runs, so a tile is one to three of them, and the pairs of a run of
// rows and a run of keys have a closed form: all of them inside one span, a (clamped) triangle
// where the rows look back at the keys, minus a second triangle for a look-back window.  The
// workgroup's wavefronts cut its q-tiles and k-tiles into runs once (every word of the group is
// requested before the first is used), then each thread counts one tile pair.  Bound by the
// latency of the words and the integer work per run pair; the group's shape trades words read
// per pair, (gq + gk) / (gq gk) tiles, against workgroups in flight.  Measured per launch:
// 1024 x 1024 tiles of 128 x 128 302 -> 21 us, 512 x 512 88 -> 12 us against counting every
// row of a tile against every run of keys (back to back 19 and 10; 25 and 13 without a way out for tiles of one run, and
// with a branch and a look at the block list around every word; tiles of 512 x 512, one 64-word step
// in flight instead of eight, 256 x 256 of them 19 -> 12 us).  Where a group has fewer pairs than threads, tiles of
// more than kTmSplit runs have theirs shared out over several (256 x 256 tiles of 16 x 16 in
// spans of 1 to 3 tokens 61 -> 24 us; tiles of few runs would pay 0.9 us for nothing).
// Counted by rows all the same: tiles of more than kTmRuns runs, and q-tiles of more than most_q
// of them, where a lane's serial loop over run pairs (about 45 instructions each) takes longer
// than the wavefront's over runs of keys (14 and 14 scalar ones, up to 64 rows at a time, two tiles
// of 32).  Medium runs (spans of 4 to 12 tokens), 32768 tokens: 64 x 64 tiles 182 -> 87 us, 64 x 128
// 180 -> 83 us; spans of 1 to 3: 16 x 16 tiles 2238 -> 668 us, 32 x 32 1044 -> 610, 64 x 64 524 -> 539,
// 128 x 128 489 -> 355 (before: by rows of a q-tile in LDS).
// kTmRuns: 27 leave room for five workgroups per CU, 15 for nine (spans of 4 to 12 tokens, 64 x 128
// tiles over 32768 tokens: 15 201 us, 27 83; but the forward of 32768 tokens at head_dim 64, whose
// key norms run beside its map, 593.4 us with 27 and 590.4 with 15).
template <int CODE>
__device__ __forceinline__ void tile_map_runs(const TileMapJob& J, const TmRows& in, uint32_t wg, int lane, int wave) {
    const int32_t tq = J.tq, tk = J.tk, nq = J.nq, nk = J.nk;
    const uint64_t* __restrict__ bits = in.bits;
    constexpr int kTmRuns = CODE & kTmBeside ? 15 : 27;      // runs of a tile that are kept in LDS
    const int gq = J.gq, gk = J.gk, log_gk = __ffs(gk) - 1;      // gk is a power of two
    const int32_t i0 = (int32_t)(wg / J.gx) * gq, j0 = (int32_t)(wg % J.gx) * gk;
    __shared__ TmRun runs[2 * kTmGroup][kTmRuns + 1];        // q-tiles, then k-tiles
    __shared__ int32_t n_runs[2 * kTmGroup];
    __shared__ uint64_t left_s[kTmGroup * kTmGroup / kWave];     // pairs that the runs do not serve

    // tile `slot` of the group (q-tiles first): its length (0: past the end of the map) and first row or key
    auto length_of = [&](int slot) -> int32_t {
        if (slot < gq) return i0 + slot < nq ? (int32_t)in.of_tile(tq, i0 + slot) : 0;
        return slot < gq + gk && j0 + slot - gq < nk ? tk : 0;
    };
    auto start_of = [&](int slot) -> uint32_t {
        return slot < gq ? (uint32_t)(i0 + slot) * (uint32_t)tq : (uint32_t)(j0 + slot - gq) * (uint32_t)tk;
    };
    // position of element e of a tile (of its first one past the end, so that no load hangs on a branch).
    // Called for all elements of a batch before the first word is requested: the block indices of a
    // share are a load of their own.
    auto position = [&](int slot, uint32_t start, int32_t len, int32_t e) -> uint32_t {
        const uint32_t r = (len > 0 ? start : 0u) + (uint32_t)(e < len ? e : 0);
        return (CODE & kTmWhole) || slot >= gq ? r : (uint32_t)in.pos((int64_t)r);
    };
    // 64 elements at0 .. of a tile (n of them valid) appended to its list of runs; (p_ss, p_x,
    // p_pos): the last element of the 64 before
    auto append = [&](int slot, int32_t at0, int32_t n, uint64_t w, uint32_t pos, int32_t& count, uint32_t& p_ss,
                      uint32_t& p_x, uint32_t& p_pos) {
        const uint32_t ss = word_ss(w), x = slot < gq ? word_att(w) : word_mod(w);
        // (all lanes exchange before any lane decides)
        const uint32_t b_ss = lane_below(ss, p_ss), b_x = lane_below(x, p_x), b_pos = lane_below(pos, p_pos);
        const bool same = ss == b_ss && x == b_x && pos == b_pos + 1u;
        const bool starts = lane < n && (!same || (lane == 0 && at0 == 0));
        const uint64_t m = __ballot(starts);
        const int32_t idx = count + __popcll(m & ((1ull << lane) - 1));
        if (starts && idx < kTmRuns) runs[slot][idx] = TmRun{ss, x, pos, (uint32_t)(at0 + lane)};
        count += __popcll(m);
        p_ss = (uint32_t)__builtin_amdgcn_readlane((int)ss, 63);
        p_x = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
        p_pos = (uint32_t)__builtin_amdgcn_readlane((int)pos, 63);
    };
    auto finish = [&](int slot, int32_t len, int32_t count) {
        if (lane == 0) {
            n_runs[slot] = count;
            if (count <= kTmRuns) runs[slot][count].at = (uint32_t)len;
        }
    };
    // A tile, or some hundred tokens of a larger one, is usually one run: then no word differs from the first (equal
    // words have equal fields) and positions are consecutive, one comparison per word, and all that
    // is left is to see whether the run goes on.
    auto one_run = [&](int slot, int32_t at0, int32_t n, uint64_t w0, uint32_t pos0, int32_t& count, uint32_t& p_ss,
                       uint32_t& p_x, uint32_t& p_pos) {
        const uint32_t ss = word_ss(w0), x = slot < gq ? word_att(w0) : word_mod(w0);
        if (at0 == 0 || ss != p_ss || x != p_x || pos0 != p_pos + 1u) {
            if (lane == 0 && count < kTmRuns) runs[slot][count] = TmRun{ss, x, pos0, (uint32_t)at0};
            ++count;
        }
        p_ss = ss;
        p_x = x;
        p_pos = pos0 + (uint32_t)n - 1u;
    };
    auto first_word = [&](uint64_t w) -> uint64_t {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(w >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)w);
    };
    if (max(tq, tk) <= 2 * kWave) {
        // tiles of one or two words per lane, the words of kTmAhead tiles in flight together
        for (int s0 = wave; s0 < gq + gk; s0 += kTmWaves * kTmAhead) {
            uint64_t w[kTmAhead][2];
            uint32_t pos[kTmAhead][2];
#pragma unroll
            for (int s = 0; s < kTmAhead; ++s) {
                const int slot = s0 + kTmWaves * s;
                const int32_t len = length_of(slot);
                const uint32_t start = start_of(slot);
#pragma unroll
                for (int c = 0; c < 2; ++c) pos[s][c] = position(slot, start, len, c * kWave + lane);
            }
#pragma unroll
            for (int s = 0; s < kTmAhead; ++s)
#pragma unroll
                for (int c = 0; c < 2; ++c) w[s][c] = bits[pos[s][c]];
#pragma unroll
            for (int s = 0; s < kTmAhead; ++s) {
                const int slot = s0 + kTmWaves * s;
                const int32_t len = length_of(slot);
                if (len == 0) continue;                      // wave-uniform
                int32_t count = 0;
                uint32_t p_ss = 0u, p_x = 0u, p_pos = 0u;
                const uint64_t w0 = first_word(w[s][0]);
                const uint32_t pos0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos[s][0]);
                bool same = (lane >= len || w[s][0] == w0) && (kWave + lane >= len || w[s][1] == w0);
                if (!(CODE & kTmWhole))
                    same = same && (lane >= len || pos[s][0] == pos0 + lane) &&
                           (kWave + lane >= len || pos[s][1] == pos0 + kWave + lane);
                if (__all(same)) {                           // wave-uniform
                    one_run(slot, 0, len, w0, pos0, count, p_ss, p_x, p_pos);
                } else {
                    append(slot, 0, len, w[s][0], pos[s][0], count, p_ss, p_x, p_pos);
                    if (len > kWave) append(slot, kWave, len - kWave, w[s][1], pos[s][1], count, p_ss, p_x, p_pos);
                }
                finish(slot, len, count);
            }
        }
    } else {
        auto larger = [&](auto CH_) __attribute__((always_inline)) {
            constexpr int CH = decltype(CH_)::value;         // times 64 words of a tile in flight together
            for (int slot = wave; slot < gq + gk; slot += kTmWaves) {
                const int32_t len = length_of(slot);
                if (len == 0) continue;
                const uint32_t start = start_of(slot);
                int32_t count = 0;
                uint32_t p_ss = 0u, p_x = 0u, p_pos = 0u;
                for (int32_t at = 0; at < len; at += CH * kWave) {
                    uint64_t w[CH];
                    uint32_t pos[CH];
#pragma unroll
                    for (int c = 0; c < CH; ++c) pos[c] = position(slot, start, len, at + c * kWave + lane);
#pragma unroll
                    for (int c = 0; c < CH; ++c) w[c] = bits[pos[c]];
                    const uint64_t w0 = first_word(w[0]);
                    const uint32_t pos0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos[0]);
                    bool same = true;
#pragma unroll
                    for (int c = 0; c < CH; ++c)
                        same = same && (at + c * kWave + lane >= len ||
                                        (w[c] == w0 && ((CODE & kTmWhole) || pos[c] == pos0 + c * kWave + lane)));
                    if (__all(same)) {                           // wave-uniform
                        one_run(slot, at, min(len - at, CH * kWave), w0, pos0, count, p_ss, p_x, p_pos);
                    } else {
#pragma unroll
                        for (int c = 0; c < CH; ++c)
                            if (at + c * kWave < len)
                                append(slot, at + c * kWave, len - at - c * kWave, w[c], pos[c], count, p_ss, p_x, p_pos);
                    }
                }
                finish(slot, len, count);
            }
        };
        if (max(tq, tk) <= 4 * kWave) larger(std::integral_constant<int, 4>{});
        else larger(std::integral_constant<int, 8>{});
    }
    __syncthreads();

    const int most_q = min(kTmRuns, tq <= kWave / 4 ? 16 : tq <= kWave / 2 ? 10 : tq <= kWave ? 20 : kTmRuns);
    auto put = [&](int32_t i, int32_t j, uint32_t total) { tile_map_put(J, in.of_tile(tq, i), i, j, total); };
    // the pair of q-tile qi and k-tile ki, counted for every f-th run of rows from `sub` on
    auto closed = [&](int qi, int ki, int sub, int f) -> uint32_t {
        const TmRun* qr = runs[qi];
        const int nqr = n_runs[qi], nkr = n_runs[gq + ki];
        uint32_t total = 0;
        for (int a = sub; a < nqr; a += f) {
            const TmRun A = qr[a];
            const int32_t n = (int32_t)(qr[a + 1].at - A.at);
            const int32_t win = (int32_t)att_window(A.x);
            const uint32_t mod = att_modality(A.x);
            const TmRun* kr = runs[gq + ki];
            TmRun B = kr[0];
            for (int b = 0; b < nkr; ++b) {
                const TmRun next = kr[b + 1];
                const uint32_t m = next.at - B.at;
                if ((A.ss & 0xFFFFu) != 0u && A.ss == B.ss) {
                    total += (uint32_t)n * m;
                } else if ((A.ss >> 16) == (B.ss >> 16) && ((A.x >> B.x) & 1u)) {
                    const int32_t d = (int32_t)(A.pos - B.pos) + 1;
                    total += pairs_upto(d, n, m);
                    if (win != 0 && B.x == mod) total -= pairs_upto(d - win, n, m);
                }
                B = next;
            }
        }
        return total;
    };
    bool any_left = false;
    if (gq * gk < kTmThreads && __any(lane < gq && i0 + lane < nq && n_runs[lane] > kTmSplit)) {      // workgroup-uniform
        // fewer pairs than threads and more than a few runs: several threads per pair
        const int log_f = __ffs(kTmThreads / (gq * gk)) - 1, f = 1 << log_f;
        const int pair = (int)threadIdx.x >> log_f, sub = threadIdx.x & (f - 1);
        const int qi = pair >> log_gk, ki = pair & (gk - 1);
        const bool mine = i0 + qi < nq && j0 + ki < nk;
        const bool few = mine && n_runs[qi] <= most_q && n_runs[gq + ki] <= kTmRuns;
        uint32_t total = few ? closed(qi, ki, sub, f) : 0u;
        for (int off = 1; off < f; off <<= 1) total += __shfl_xor(total, off);
        if (few && sub == 0) put(i0 + qi, j0 + ki, total);
        if (threadIdx.x < kTmThreads / kWave) left_s[threadIdx.x] = 0;
        __syncthreads();
        if (mine && !few) {                                  // the other pairs
            any_left = true;
            if (sub == 0) atomicOr((unsigned long long*)&left_s[pair / kWave], 1ull << (pair % kWave));
        }
    } else {
        for (int p0 = 0; p0 < gq * gk; p0 += kTmThreads) {
            const int pair = p0 + threadIdx.x;
            const int qi = pair >> log_gk, ki = pair & (gk - 1);
            const bool mine = pair < gq * gk && i0 + qi < nq && j0 + ki < nk;
            const bool few = mine && n_runs[qi] <= most_q && n_runs[gq + ki] <= kTmRuns;
            if (few) put(i0 + qi, j0 + ki, closed(qi, ki, 0, 1));
            const uint64_t left = __ballot(mine && !few);    // the other pairs
            if (lane == 0) left_s[p0 / kWave + wave] = left;
            any_left = any_left || left != 0;
        }
    }
    // by whole wavefronts, every fourth pair to each
    if (!__syncthreads_or(any_left)) return;                 // the usual case
    for (int m = 0; m * kWave < gq * gk; ++m) {
        const uint64_t all = left_s[m] & (0x1111111111111111ull << wave);
        const uint64_t left = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(all >> 32)) << 32) |
                              (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)all);
        tile_map_by_rows_any<CODE, true>(J, in, i0, j0, log_gk, left, m * kWave);
    }
}

// Workgroup `wg_index` (of tile_map_workgroups(jobs)) of the map(s); kTmThreads threads.
// `blocks` may be a caller's unchecked list (see TmRows).
template <int CODE>
__device__ __forceinline__ void
tile_map_body(uint32_t wg_index, const uint64_t* __restrict__ bits,
              const int32_t* __restrict__ blocks, int32_t block, int64_t n_seq_blocks, int64_t n_rows,
              const TileMapJobs& jobs) {
    const uint32_t n_first = jobs.j[0].gx * jobs.j[0].gy;
    const bool second = wg_index >= n_first;                 // workgroup-uniform
    const TileMapJob& J = jobs.j[second ? 1 : 0];
    const uint32_t wg = wg_index - (second ? n_first : 0u);
    const TmRows in{bits, blocks, block, n_seq_blocks, n_rows};
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (!(CODE & kTmByRuns) || J.kpw > 0) {                  // workgroup-uniform
        const int32_t i = (int32_t)(wg / J.gx), j0 = ((int32_t)(wg % J.gx) * kTmWaves + wave) * J.kpw;
        const int32_t n = min(J.kpw, J.nk - j0);
        for (int32_t c = 0; c < n; c += kWave)
            tile_map_by_rows_any<CODE, false>(J, in, i, j0 + c, 6, n - c < kWave ? (1ull << (n - c)) - 1 : ~0ull, 0);
        return;
    }
    if constexpr ((CODE & kTmByRuns) != 0) tile_map_runs<CODE>(J, in, wg, threadIdx.x & (kWave - 1), wave);
}

// ---- block list ------------------------------------------------------------
// One workgroup of 256 threads: clears the error flag block (kFlagInts int32 words), then
// copies the block list, replacing out-of-range entries by 0 and raising the flag.
constexpr int kFlagInts = 4;
__device__ __forceinline__ void
validate_blocks_body(const int32_t* __restrict__ blocks, int32_t n_blocks, int64_t n_seq_blocks,
                     int32_t* __restrict__ clean, int32_t* __restrict__ err) {
    int bad = 0;
    for (int i = threadIdx.x; i < n_blocks; i += 256) {
        int32_t b = blocks[i];
        if (b < 0 || b >= n_seq_blocks) {
            bad = 1;
            b = 0;
        }
        clean[i] = b;
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x < kFlagInts) err[threadIdx.x] = threadIdx.x == 0 ? bad : 0;
}

inline TileMapJob tile_map_job(int64_t S, int64_t n_rows, int32_t tq, int32_t tk, uint8_t* d_cls,
                               uint32_t* d_cnt) {
    const int64_t nq = (n_rows + tq - 1) / tq;
    const int32_t nk = (int32_t)(S / tk);
    // Row by row, J.kpw pairs per wavefront, as long as that is as fast: up to 4096 pairs (one each:
    // cutting tiles into runs first costs 1 to 3 us more), up to 16384 if the tiles are small (64
    // rows x 64 keys each: 128 x 128 tiles of 64 x 64 8.6 us, 9.2 by runs; 128 x 64 tiles of 128 x 64
    // 7.5 / 9.1; but 64 x 128 of 512 x 64 15 / 10.6); and at positions beyond kTmNarrow.
    const int64_t steps = nq * nk * ((tq + kWave - 1) / kWave) * ((tk + kWave - 1) / kWave);
    if (nq * nk <= 4096 || steps <= 16384 || (int64_t)nk * tk > kTmNarrow) {
        // (workgroups: a thousand or more, at most about 2^23)
        const int64_t pairs = nq * nk;
        const int32_t kpw = (int32_t)std::max<int64_t>({1, std::min<int64_t>(8, pairs / (kTmWaves * 1024)), pairs >> 25});
        const int32_t per_wg = kTmWaves * kpw;
        return TileMapJob{tq, tk, (int32_t)nq, nk, 1, per_wg, kpw, (uint32_t)((nk + per_wg - 1) / per_wg), (uint32_t)nq,
                          d_cls, d_cnt};
    }
    // by runs: as many pairs per workgroup as leave about a thousand workgroups
    int32_t gq = 1, gk = kTmWaves;
    auto groups = [&]() { return ((nq + gq - 1) / gq) * (((int64_t)nk + gk - 1) / gk); };
    while (groups() > 1024 && gq * gk < kTmGroup * kTmGroup) {
        int32_t& g = (gq <= gk && gq < nq) || gk == kTmGroup ? gq : gk;
        g *= 2;
    }
    return TileMapJob{tq, tk, (int32_t)nq, nk, gq, gk, 0, (uint32_t)((nk + gk - 1) / gk),
                      (uint32_t)((nq + gq - 1) / gq), d_cls, d_cnt};
}

// whether a launch needs the code that cuts tiles into runs
inline bool tile_map_by_runs(const TileMapJobs& jobs) { return jobs.j[0].kpw == 0 || jobs.j[1].kpw == 0; }

inline uint32_t tile_map_workgroups(const TileMapJobs& jobs, int n_maps) {
    uint32_t n = jobs.j[0].gx * jobs.j[0].gy;
    if (n_maps > 1) n += jobs.j[1].gx * jobs.j[1].gy;
    return n;
}

}  // namespace mm

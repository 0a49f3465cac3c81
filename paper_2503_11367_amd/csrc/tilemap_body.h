// Device bodies of the tile map (paper section 3.2.1) and of the block-list check, shared
// by the public tile-map kernel and by the first launch of the attention passes, where
// they run side by side with that pass's other independent preparation work.
#pragma once
#include <algorithm>
#include "common.h"

namespace mm {

constexpr int kTmThreads = 256;
constexpr int kTmWaves = kTmThreads / kWave;
constexpr int kTmGroup = 32;       // most q-tiles and most k-tiles of a workgroup
constexpr int kTmRuns = 15;        // runs of a tile that are kept in LDS
constexpr int kTmAhead = 4;        // tiles whose words a wavefront requests together

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// One launch serves up to two maps of the same rows (the second map's workgroups follow
// the first's in the one-dimensional grid).  A workgroup takes gq q-tiles x gk k-tiles (powers
// of two, at most kTmGroup each).
struct TileMapJob {
    int32_t tq, tk, nq, nk, gq, gk;
    uint32_t gx, gy;                     // workgroups this map needs
    uint8_t* cls;
    uint32_t* cnt;
};
struct TileMapJobs { TileMapJob j[2]; };

// A run: consecutive tokens of a tile that carry the same fields (x: the attend word of query
// rows, the modality of keys) at consecutive positions.  A list of runs ends with an entry
// whose `at` is the tile's length.
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

// Workgroup `wg_index` (of tile_map_workgroups(jobs)) of the map(s); kTmThreads threads.
// `blocks` may be a caller's unchecked list: an entry outside [0, n_seq_blocks) counts
// as block 0, exactly as validate_blocks_body rewrites it.
//
// A layout is a handful of runs, so a tile is one to three of them, and the pairs of a run of
// rows and a run of keys have a closed form: all of them inside one span, a (clamped) triangle
// where the rows look back at the keys, minus a second triangle for a look-back window.  The
// workgroup's wavefronts cut its q-tiles and k-tiles into runs once (every word of the group is
// requested before the first is used), then each lane counts one tile pair.  Bound by the
// latency of the words and the integer work per run pair; the group's shape trades words read
// per pair, (gq + gk) / (gq gk) tiles, against workgroups in flight.  Measured per launch:
// 1024 x 1024 tiles of 128 x 128 302 -> 25 us, 512 x 512 88 -> 13 us against counting every
// row of a tile against every run of keys.
// Counted that way still, one wavefront per pair and a row per lane: tiles of more than kTmRuns
// runs (spans of a few tokens), sequences whose positions do not fit 30 bits, and maps of up to
// 4096 pairs (a pair per wavefront; cutting tiles into runs first made these 1.2 us slower).
__device__ __forceinline__ void
tile_map_body(uint32_t wg_index, const uint64_t* __restrict__ bits,
              const int32_t* __restrict__ blocks, int32_t block, int64_t n_seq_blocks, int64_t n_rows,
              const TileMapJobs& jobs) {
    const uint32_t n_first = jobs.j[0].gx * jobs.j[0].gy;
    const bool second = wg_index >= n_first;                 // workgroup-uniform
    const TileMapJob& J = jobs.j[second ? 1 : 0];
    const uint32_t wg = wg_index - (second ? n_first : 0u);
    const int32_t tq = J.tq, tk = J.tk, nq = J.nq, nk = J.nk;
    const int gq = J.gq, gk = J.gk, log_gk = __ffs(gk) - 1;      // gk is a power of two
    const int32_t i0 = (int32_t)(wg / J.gx) * gq, j0 = (int32_t)(wg % J.gx) * gk;
    __shared__ TmRun runs[2 * kTmGroup][kTmRuns + 1];        // q-tiles, then k-tiles
    __shared__ int32_t n_runs[2 * kTmGroup];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const bool small = gq * gk == kTmWaves;                  // workgroup-uniform
    const bool narrow = (int64_t)nk * tk <= ((int64_t)1 << 30);      // positions fit 30 bits
    const bool by_runs = !small && narrow;

    // rows of q-tile i (the last one may be ragged)
    auto rows_of = [&](int32_t i) -> int64_t { return min((int64_t)tq, n_rows - (int64_t)i * tq); };
    auto pos_of = [&](int64_t r) -> int64_t {
        if (!blocks) return r;
        const uint32_t b = (uint32_t)r / (uint32_t)block;    // a share has fewer than 2^31 rows
        int64_t g = blocks[b];
        if (g < 0 || g >= n_seq_blocks) g = 0;
        return g * block + ((uint32_t)r - b * (uint32_t)block);
    };
    // tile `slot` of the group (q-tiles first): its length (0: past the end of the map), and the
    // position of its element e
    auto length_of = [&](int slot) -> int32_t {
        if (slot < gq) return i0 + slot < nq ? (int32_t)rows_of(i0 + slot) : 0;
        return slot < gq + gk && j0 + slot - gq < nk ? tk : 0;
    };
    auto element = [&](int slot, int32_t e) -> uint32_t {
        return slot < gq ? (uint32_t)pos_of((int64_t)(i0 + slot) * tq + e)
                         : (uint32_t)(j0 + slot - gq) * (uint32_t)tk + (uint32_t)e;
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
    if (by_runs && max(tq, tk) <= 2 * kWave) {
        // tiles of one or two words per lane, the words of kTmAhead tiles in flight together
        for (int s0 = wave; s0 < gq + gk; s0 += kTmWaves * kTmAhead) {
            uint64_t w[kTmAhead][2];
            uint32_t pos[kTmAhead][2];
#pragma unroll
            for (int s = 0; s < kTmAhead; ++s) {
                const int slot = s0 + kTmWaves * s;
                const int32_t len = length_of(slot);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    pos[s][c] = 0u;
                    w[s][c] = 0u;
                    if (c * kWave + lane < len) {
                        pos[s][c] = element(slot, c * kWave + lane);
                        w[s][c] = bits[pos[s][c]];
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < kTmAhead; ++s) {
                const int slot = s0 + kTmWaves * s;
                const int32_t len = length_of(slot);
                if (len == 0) continue;                      // wave-uniform
                int32_t count = 0;
                uint32_t p_ss = 0u, p_x = 0u, p_pos = 0u;
                append(slot, 0, len, w[s][0], pos[s][0], count, p_ss, p_x, p_pos);
                if (len > kWave) append(slot, kWave, len - kWave, w[s][1], pos[s][1], count, p_ss, p_x, p_pos);
                finish(slot, len, count);
            }
        }
    } else if (by_runs) {
        for (int slot = wave; slot < gq + gk; slot += kTmWaves) {
            const int32_t len = length_of(slot);
            if (len == 0) continue;
            int32_t count = 0;
            uint32_t p_ss = 0u, p_x = 0u, p_pos = 0u;
            for (int32_t at = 0; at < len; at += kWave) {
                const uint32_t pos = at + lane < len ? element(slot, at + lane) : 0u;
                append(slot, at, len - at, at + lane < len ? bits[pos] : 0u, pos, count, p_ss, p_x, p_pos);
            }
            finish(slot, len, count);
        }
    }
    if (by_runs) __syncthreads();

    // the pair's count and class
    auto put = [&](int32_t i, int32_t j, uint32_t total) {
        const uint32_t full = (uint32_t)rows_of(i) * (uint32_t)tk;
        if (J.cnt) J.cnt[(int64_t)i * nk + j] = total;
        if (J.cls)
            J.cls[(int64_t)i * nk + j] = total == 0 ? MMATTN_TILE_EMPTY
                                         : (total == full ? MMATTN_TILE_FULL : MMATTN_TILE_PARTIAL);
    };
    // The pairs first + bit of `left`, one after the other by the whole wavefront, row by row: up
    // to 256 rows in registers, kept while the q-tile stays the same, their words in flight
    // together; the next 64 keys' words are requested ahead of their use.  T holds a
    // position.  Bound by the instructions per (64 rows, run of keys): positions in 32 bits where they
    // fit, the window's only where a row has one.  Measured on spans of 1 to 3 tokens, 32768 of
    // them in all, against a wavefront per pair with its rows in LDS: tiles of 128 x 128 476 -> 367
    // us, 256 x 256 528 -> 284, 16 x 16 2185 -> 774 (these by runs), 64 x 64 515 -> 586.
    auto by_rows = [&](auto zero, uint64_t left, int first) {
        typedef decltype(zero) T;
        constexpr int kRows = 4;
        T q[kRows];
        uint32_t ss_q[kRows], att[kRows];
        bool spans[kRows], windows = false;
        int32_t have = -1;                                   // the q-tile whose rows are in registers
        while (left) {
            const int p = first + __ffsll((unsigned long long)left) - 1;
            left &= left - 1;
            const int32_t i = i0 + (p >> log_gk), j = j0 + (p & (gk - 1));
            const int64_t rows = rows_of(i), k0 = (int64_t)j * tk;
            uint32_t part = 0;
            for (int64_t r0 = 0; r0 < rows; r0 += kRows * kWave) {
                const int n_r = (int)min((int64_t)kRows, (rows - r0 + kWave - 1) / kWave);
                uint64_t wk_next = lane < tk ? bits[k0 + lane] : 0;
                if (have != i || rows > kRows * kWave) {     // wave-uniform
                    have = i;
                    uint64_t w[kRows];
#pragma unroll
                    for (int u = 0; u < kRows; ++u) {
                        q[u] = 0;
                        w[u] = 0;                            // (a word of zeros sees nothing)
                        const int64_t r = r0 + u * kWave + lane;
                        if (u < n_r && r < rows) {
                            const int64_t pos = pos_of((int64_t)i * tq + r);
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
                        const int a = __ffsll((unsigned long long)m) - 1;
                        m &= m - 1;
                        const int b = m ? __ffsll((unsigned long long)m) - 1 : n_keys;   // the run is keys a..b-1
                        const uint32_t ss_r = (uint32_t)__builtin_amdgcn_readlane((int)ss_k, a);
                        const uint32_t mod_r = (uint32_t)__builtin_amdgcn_readlane((int)mod_k, a);
                        const T before = (T)(k0 + kc + a - 1), len = (T)(b - a);
#pragma unroll
                        for (int u = 0; u < kRows; ++u) {
                            if (u >= n_r) continue;          // wave-uniform
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
            const uint32_t total = wave_sum(part);
            if (lane == 0) put(i, j, total);
        }
    };
    __shared__ uint64_t left_s[kTmGroup * kTmGroup / kWave];     // pairs that the runs do not serve
    uint64_t any_left = 0;
    for (int p0 = 0; !small && p0 < gq * gk; p0 += kTmThreads) {
        const int pair = p0 + threadIdx.x;
        const int qi = pair >> log_gk, ki = pair & (gk - 1);
        const bool mine = pair < gq * gk && i0 + qi < nq && j0 + ki < nk;
        const bool few = mine && by_runs && n_runs[qi] <= kTmRuns && n_runs[gq + ki] <= kTmRuns;
        if (few) {
            const TmRun* qr = runs[qi];
            const int nqr = n_runs[qi], nkr = n_runs[gq + ki];
            uint32_t total = 0;
            for (int a = 0; a < nqr; ++a) {
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
            put(i0 + qi, j0 + ki, total);
        }

        // the other pairs
        const uint64_t left = __ballot(mine && !few);
        if (lane == 0) left_s[p0 / kWave + wave] = left;
        any_left |= left;
    }
    // by whole wavefronts, every fourth pair to each
    auto count_rows = [&](uint64_t left, int first) {
        if (narrow) by_rows(int32_t(0), left, first);
        else by_rows(int64_t(0), left, first);
    };
    if (small) {
        count_rows(j0 + wave < nk ? 1u : 0u, wave);
        return;
    }
    if (!__syncthreads_or(any_left != 0)) return;            // the usual case
    for (int m = 0; m * kWave < gq * gk; ++m) count_rows(left_s[m] & (0x1111111111111111ull << wave), m * kWave);
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
    // one q-tile x four k-tiles (a pair per wavefront, should the runs not serve) while the map
    // has few pairs, more pairs per workgroup once about a thousand workgroups remain
    int32_t gq = 1, gk = kTmWaves;
    auto groups = [&]() { return ((nq + gq - 1) / gq) * (((int64_t)nk + gk - 1) / gk); };
    while (groups() > 1024 && gq * gk < kTmGroup * kTmGroup) {
        int32_t& g = (gq <= gk && gq < nq) || gk == kTmGroup ? gq : gk;
        g *= 2;
    }
    return TileMapJob{tq, tk, (int32_t)nq, nk, gq, gk, (uint32_t)((nk + gk - 1) / gk),
                      (uint32_t)((nq + gq - 1) / gq), d_cls, d_cnt};
}

inline uint32_t tile_map_workgroups(const TileMapJobs& jobs, int n_maps) {
    uint32_t n = jobs.j[0].gx * jobs.j[0].gy;
    if (n_maps > 1) n += jobs.j[1].gx * jobs.j[1].gy;
    return n;
}

}  // namespace mm

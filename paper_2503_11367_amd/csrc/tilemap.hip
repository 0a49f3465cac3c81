// Tile map (paper section 3.2.1): for every (q-tile, k-tile) the number of
// unmasked (query,key) pairs and the class EMPTY / FULL / PARTIAL; a tile whose
// mask block is all zeros is the one the attention kernels skip.  Row sums give
// the per-block workloads W_b that Alg. 1 balances.
//
// A k-tile is a handful of "runs" (maximal stretches of keys with the same
// sample/span/modality fields: a text run, a modality span), a q-tile likewise, and
// the visible pairs of two runs have a closed form; on small maps, and for tiles of
// many short runs, a lane takes a query row and counts it against each run of keys
// (the whole run if it is the row's own span, the keys up to the row's position and
// inside its look-back window if the row looks back at that modality in its sample,
// else none).  Exact for any layout.
//
// The same device code serves the attention kernels' private maps: there the q rows
// are a rank's local rows (positions looked up through its block list) and the
// last q-tile may be ragged.
#include "tilemap_body.h"

namespace mm {

template <int CODE>
__global__ void __launch_bounds__(kTmThreads)
tile_map_kernel(const uint64_t* __restrict__ bits, const int32_t* __restrict__ blocks, int32_t block,
                int64_t n_seq_blocks, int64_t n_rows, const TileMapJobs jobs) {
    tile_map_body<CODE>(blockIdx.x, bits, blocks, block, n_seq_blocks, n_rows, jobs);
}

// A row per wavefront, 1024 counts of it in flight
constexpr int kRowWaves = 4, kRowAhead = 16;
__global__ void __launch_bounds__(kRowWaves * kWave)
row_pairs_kernel(const uint32_t* __restrict__ cnt, int32_t nq, int32_t nk, uint64_t* __restrict__ rowpairs) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t i = (int64_t)blockIdx.x * kRowWaves + threadIdx.x / kWave;
    if (i >= nq) return;
    uint64_t s = 0;
    for (int j0 = 0; j0 < nk; j0 += kRowAhead * kWave) {
        uint32_t c[kRowAhead];
#pragma unroll
        for (int u = 0; u < kRowAhead; ++u) {
            const int j = j0 + u * kWave + lane;
            c[u] = 0u;
            if (j0 + u * kWave < nk && j < nk) c[u] = cnt[i * nk + j];
        }
#pragma unroll
        for (int u = 0; u < kRowAhead; ++u) s += c[u];
    }
    for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) rowpairs[i] = s;
}

int launch_tile_map(const uint64_t* d_bits, int64_t S, const int32_t* d_blocks, int32_t block,
                    int64_t n_rows, int32_t tq, int32_t tk, uint8_t* d_cls, uint32_t* d_cnt,
                    uint64_t* d_rowpairs, hipStream_t st) {
    if (n_rows <= 0) return MMATTN_OK;
    TileMapJobs jobs;
    jobs.j[0] = jobs.j[1] = tile_map_job(S, n_rows, tq, tk, d_cls, d_cnt);
    const bool runs = tile_map_by_runs(jobs);
    // (kTmWhole: not with a list of blocks)
    auto for_rows = [&](auto ROWS_) {
        constexpr int ROWS = decltype(ROWS_)::value;
        return !runs      ? tile_map_kernel<ROWS>
               : d_blocks ? tile_map_kernel<kTmByRuns | ROWS>
                          : tile_map_kernel<kTmByRuns | kTmWhole | ROWS>;
    };
    const auto kernel = S > kTmNarrow     ? tile_map_kernel<kTmWide>
                        : tq <= kWave     ? for_rows(std::integral_constant<int, kTmRows1>{})
                        : tq <= 2 * kWave ? for_rows(std::integral_constant<int, kTmRows2>{})
                                          : for_rows(std::integral_constant<int, kTmRows4>{});
    hipLaunchKernelGGL(kernel, dim3(jobs.j[0].gx * jobs.j[0].gy), dim3(kTmThreads), 0, st, d_bits, d_blocks, block,
                       d_blocks ? S / block : (int64_t)0, n_rows, jobs);
    MM_LAUNCH_CHECK();
    if (d_rowpairs) {
        hipLaunchKernelGGL(row_pairs_kernel, dim3((unsigned)((jobs.j[0].nq + kRowWaves - 1) / kRowWaves)),
                           dim3(kRowWaves * kWave), 0, st, d_cnt, jobs.j[0].nq, jobs.j[0].nk, d_rowpairs);
        MM_LAUNCH_CHECK();
    }
    return MMATTN_OK;
}

}  // namespace mm

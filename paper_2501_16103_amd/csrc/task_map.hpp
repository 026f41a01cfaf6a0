// Task-map construction and decode for the statically batched MoE GEMM (gfx950).
//
// Builds, on the device, what Sec. 4.1 asks for after the token route: the
// per-expert counts, the list sigma of non-empty experts, the inclusive
// TilePrefix over the non-empty experts (Alg. 1), and the per-expert token
// index arrays of Sec. 4.3 (here a stable counting sort of the flat row ids,
// so the result does not depend on atomic ordering).  `mapping()` is Alg. 2
// for a 64-lane wavefront; `decode_block()` adds the sigma stage of Alg. 4.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/moe_sb.h"

namespace moe {

constexpr int kChunkRows = 1024;  // routed rows handled by one scatter workgroup
constexpr int kMapThreads = 1024; // = kChunkRows: one row per thread, 16 wavefronts
constexpr int kMaxE = 1024;
constexpr int kWaves = kMapThreads / 64;

struct MapLayout {
    int E64;
    size_t off_counts, off_offsets, off_sigma, off_prefix, off_records, off_rows;
};

__host__ __device__ inline MapLayout map_layout(int E) {
    MapLayout L;
    L.E64 = (E + 63) / 64 * 64;
    L.off_counts = MOE_MAP_HDR_WORDS;
    L.off_offsets = L.off_counts + L.E64;
    L.off_sigma = L.off_offsets + L.E64 + 64;
    L.off_prefix = L.off_sigma + L.E64;
    L.off_records = L.off_prefix + L.E64;
    L.off_rows = L.off_records + 4 * (size_t)L.E64;
    return L;
}

__host__ __device__ inline size_t round_up64(size_t v) { return (v + 63) / 64 * 64; }
// per-chunk histogram row: E64 expert columns + 64 spare (column E64 counts bad ids)
__host__ __device__ inline int hist_stride(int E64) { return E64 + 64; }

// Inclusive scan over the lanes of a wavefront, all of them active.  In the lanes' own registers (DPP: shifts by 1, 2, 4 and 8
// inside each row of 16, then the last lane of a row to the rows behind it): the same with __shfl_up is six round trips through
// the LDS crossbar, one after the other, and a small build has two to four such scans in its chain.
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return v;
}

// ---------------------------------------------------------------- decode

// Alg. 2 on one wavefront: lane t tests p = (B >= TilePrefix[t]); the ballot is the
// warp vote, its population count is the task index h.  Pads are INT32_MAX and never vote.
// The prefix comes from the packed task records {TilePrefix, expert, count, row offset}, so the record of
// task h is already in a register of lane h when the vote is over: rec = that record, l = tile index in the task.
// More than 64 tasks (Sec. 3.1, two-level TilePrefix): the last entry of every group of 64 tasks is the
// first level; one vote over it (read in place, up to 64 groups) finds the group, a second vote the task in it.
// `first` is records[lane] (the caller loads it early, next to the header); B must be below the total tile count.
__device__ __forceinline__ void mapping(const int4* __restrict__ records, int E64, int B, int4 first, int& h, int& l, int4& rec) {
    const int lane = __lane_id();
    int4 r = first;
    int base = 0, kprev = 0;
    if (E64 > 64) {
        const int groups = E64 >> 6;  // <= 16 for E <= 1024
        const int top = lane < groups ? records[64 * lane + 63].x : 0x7fffffff;
        const int grp = __popcll(__ballot(B >= top));  // groups that end at or before B
        if (grp > 0) {
            base = grp << 6;
            kprev = __builtin_amdgcn_readlane(top, grp - 1);
            r = records[base + lane];
        }
    }
    const int votes = __popcll(__ballot(B >= r.x));  // < 64: the group's last entry is above B
    h = base + votes;
    rec.x = __builtin_amdgcn_readlane(r.x, votes);
    rec.y = __builtin_amdgcn_readlane(r.y, votes);
    rec.z = __builtin_amdgcn_readlane(r.z, votes);
    rec.w = __builtin_amdgcn_readlane(r.w, votes);
    if (votes > 0) kprev = __builtin_amdgcn_readlane(r.x, votes - 1);
    l = B - kprev;
}

struct TileCoord {
    int e, m_tile, n_tile, rows, row_base;  // row_base: index into sorted_rows of the tile's first row
    int small;                              // task type (Alg. 3): 1 = the expert uses the small tiling strategy
    int m_tiles;                            // m-tiles of the expert: 1 = no other tile reads this tile's weight panel
    int streams = 0;                        // tiles of the launch, as it runs them, times the workgroups that share one (halves, parts along K)
};

// Tiling strategy of an expert with cnt rows: tile_m_small when cnt <= small_max_rows (0 = one strategy).
__host__ __device__ __forceinline__ int expert_tile_m(int cnt, int tile_m, int tile_m_small, int small_max_rows) {
    return (small_max_rows > 0 && cnt <= small_max_rows) ? tile_m_small : tile_m;
}
// m-tiles of an expert with cnt rows.  With slack > 0 the last tile of a big-strategy expert may hold up to
// tile_m + slack rows, so a remainder of at most `slack` rows does not open a tile of its own.
__host__ __device__ __forceinline__ int expert_m_tiles(int cnt, const moe_tiling& g) {
    if (cnt <= 0) return 0;
    if (g.small_max_rows > 0 && cnt <= g.small_max_rows) return (cnt + g.tile_m_small - 1) / g.tile_m_small;
    const int mt = (cnt - g.tile_m_slack + g.tile_m - 1) / g.tile_m;
    return mt < 1 ? 1 : mt;
}

// Alg. 2 + Alg. 4 for workgroup B, then the tile index split m-fastest (the task function's own convention).
__device__ __forceinline__ TileCoord decode_block(const int32_t* __restrict__ map, const MapLayout& L, const moe_tiling& g, int B,
                                                  int4 first_record) {
    int h, l;
    int4 rec;
    mapping(reinterpret_cast<const int4*>(map + L.off_records), L.E64, B, first_record, h, l, rec);
    TileCoord c;
    c.e = rec.y;
    const int cnt = rec.z;
    c.small = g.small_max_rows > 0 && cnt <= g.small_max_rows;
    const int tile_m = c.small ? g.tile_m_small : g.tile_m;
    const int mt = expert_m_tiles(cnt, g);
    c.m_tiles = mt;
    c.n_tile = l / mt;
    c.m_tile = l - c.n_tile * mt;
    const int left = cnt - c.m_tile * tile_m;
    c.rows = c.m_tile + 1 < mt ? tile_m : left;
    c.row_base = rec.w + c.m_tile * tile_m;
    return c;
}

// ---------------------------------------------------------------- build

// Among the lanes of a wavefront holding the same key: my rank (lanes below me with
// my key), the group size and the lanes themselves.  Invalid lanes take no part.
__device__ __forceinline__ unsigned long long wave_match(int key, bool valid, int nbits, int& rank, int& size) {
    unsigned long long peers = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
        const int bit = (key >> b) & 1;
        const unsigned long long m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    const unsigned long long below = (1ull << __lane_id()) - 1ull;
    rank = __popcll(peers & below);
    size = __popcll(peers);
    return peers;
}

// Inclusive scan across the threads of the block (at most kMapThreads; s_tmp: >= kWaves ints of LDS).
__device__ __forceinline__ int block_incl_scan(int v, int* s_tmp) {
    const int w = threadIdx.x >> 6, lane = __lane_id();
    const int incl = wave_incl_scan(v);
    __syncthreads();
    if (lane == 63) s_tmp[w] = incl;
    __syncthreads();
    int base = 0;
    for (int i = 0; i < w; ++i) base += s_tmp[i];
    return incl + base;
}

__device__ __forceinline__ int bit_reverse(int r, int nbits) { return nbits ? (int)(__brev((unsigned)r) >> (32 - nbits)) : 0; }

// Ints of LDS finish_map needs: three totals per wavefront, then the heavy-tile sum of order 2.
constexpr int kTmpInts = 3 * kWaves + 8;

// From the per-expert count held by thread e (< E64; 0 beyond E): write counts, offsets, sigma, tile_prefix, the task
// records and the header.  Executed by all threads of one block of at least E64 threads.
// The build is a few microseconds of latency, so what counts is the chain of barriers and memory round trips:
//   - order 0: sigma is ascending, so the TilePrefix of a non-empty expert is the plain inclusive scan of the tile counts
//     in expert order (empty experts add nothing), and its position the scan of the non-empty flags: the three scans
//     (rows, non-empty, tiles) run together, with one barrier, or none at E <= 64, where they are one wavefront's;
//   - every word is written once, by the thread that knows it: an empty expert's thread writes one of the pads.
// order 1 (spread, our reading of the interval-halving placement of Sec. 4.2): non-empty experts ranked by tile count
// (largest first, ties by lower index), rank r keyed by bitrev(r) over ceil(log2 M) bits, sigma by increasing key.
// order 2: heavy experts (more than a quarter of an m-tile) by falling tile count, ties by lower index, then the light ones
// by rising index; the tiles of the heavy part are summed for the header.
// s_tmp: kTmpInts ints, s_work: >= 2*E64 ints of LDS (orders 1 and 2 only).  Returns this thread's exclusive row offset
// (valid for tid < E).  `write` is false for the workgroups that only need that (every scatter workgroup repeats this
// function; the first one stores its results).
__device__ __forceinline__ int finish_map(int32_t* __restrict__ map, const MapLayout& L, int cnt, int bad, int T, int k,
                                          int E, int N, const moe_tiling& g, int* s_tmp, int* s_work, bool write = true) {
    const int tid = threadIdx.x, w = tid >> 6;
    const int R = T * k;
    const int nt = (N + g.tile_n - 1) / g.tile_n;
    const bool nonempty = cnt > 0;
    const int tiles = expert_m_tiles(cnt, g) * nt;
    const int order = g.order;
    int rows_incl = wave_incl_scan(cnt);
    int ne_incl = __popcll(__ballot(nonempty) & (~0ull >> (63 - __lane_id())));
    int tile_incl = wave_incl_scan(tiles);
    int M, total;
    if (L.E64 > 64 || order != 0) {
        if (__lane_id() == 63) {
            s_tmp[3 * w] = rows_incl;
            s_tmp[3 * w + 1] = ne_incl;
            s_tmp[3 * w + 2] = tile_incl;
        }
        if (tid == 0) s_tmp[3 * kWaves] = 0;
        __syncthreads();
        M = 0;
        total = 0;
        for (int i = 0; i < (L.E64 >> 6); ++i) {
            const int r = s_tmp[3 * i], n = s_tmp[3 * i + 1], t = s_tmp[3 * i + 2];
            if (i < w) { rows_incl += r; ne_incl += n; tile_incl += t; }
            M += n;
            total += t;
        }
    } else {   // (only the first wavefront holds experts, and only it uses these)
        M = __builtin_amdgcn_readlane(ne_incl, 63);
        total = __builtin_amdgcn_readlane(tile_incl, 63);
    }
    const int off = rows_incl - cnt;
    int heavy_tiles = 0;
    if (order == 0) {
        if (write && tid < L.E64) {
            // position in sigma; empty experts take the pads behind the M tasks, in order
            const int pos = nonempty ? ne_incl - 1 : M + tid - ne_incl;
            const int prefix = nonempty ? tile_incl : 0x7fffffff, ex = nonempty ? tid : -1;
            map[L.off_sigma + pos] = ex;
            map[L.off_prefix + pos] = prefix;
            reinterpret_cast<int4*>(map + L.off_records)[pos] = make_int4(prefix, ex, cnt, nonempty ? off : 0);
        }
    } else {
        int pos = 0;
        if (order == 1) {
            if (tid < L.E64) s_work[tid] = nonempty ? tiles : -1;
            __syncthreads();
            int rank = 0;
            if (nonempty)
                for (int j = 0; j < L.E64; ++j) {
                    const int tj = s_work[j];
                    rank += (tj > tiles) || (tj == tiles && j < tid);
                }
            int nbits = 0;
            while ((1 << nbits) < M) ++nbits;
            const int key = bit_reverse(rank, nbits);
            if (tid < L.E64) s_work[L.E64 + tid] = nonempty ? key : 0x7fffffff;
            __syncthreads();
            if (nonempty)
                for (int j = 0; j < L.E64; ++j) pos += s_work[L.E64 + j] < key;
        } else {
            const bool light = 4 * cnt <= g.tile_m;
            const int heavy_key = light ? 0 : tiles;   // every heavy expert has at least one tile
            if (tid < L.E64) s_work[tid] = nonempty ? heavy_key : -1;
            __syncthreads();
            if (nonempty) {
                for (int j = 0; j < L.E64; ++j) {
                    const int tj = s_work[j];
                    pos += (tj > heavy_key) || (tj == heavy_key && j < tid);
                }
                if (!light) atomicAdd(&s_tmp[3 * kWaves], tiles);   // integer sum: the order of the adds does not matter
            }
        }
        __syncthreads();
        heavy_tiles = s_tmp[3 * kWaves];
        if (!nonempty) pos = M + tid - ne_incl;
        if (tid < L.E64) {
            s_work[pos] = nonempty ? tiles : 0;
            if (write) {
                map[L.off_sigma + pos] = nonempty ? tid : -1;
                map[L.off_records + 4 * pos + 1] = nonempty ? tid : -1;
                map[L.off_records + 4 * pos + 2] = cnt;
                map[L.off_records + 4 * pos + 3] = nonempty ? off : 0;
            }
        }
        __syncthreads();
        // Alg. 1 over the non-empty experts in sigma order
        const int prefix = block_incl_scan(tid < M ? s_work[tid] : 0, s_tmp);
        if (write && tid < L.E64) {
            map[L.off_prefix + tid] = tid < M ? prefix : 0x7fffffff;
            map[L.off_records + 4 * tid] = tid < M ? prefix : 0x7fffffff;
        }
    }
    if (!write) return off;
    if (tid < L.E64) {
        map[L.off_counts + tid] = cnt;
        map[L.off_offsets + tid] = tid < E ? off : (tid == E ? R - bad : R);
    }
    if (tid < 64) map[L.off_offsets + L.E64 + tid] = L.E64 + tid == E ? R - bad : R;
    if (tid < MOE_MAP_HDR_WORDS) {
        int v = 0;
        switch (tid) {
            case MOE_HDR_MAGIC: v = MOE_MAP_MAGIC; break;
            case MOE_HDR_T: v = T; break;
            case MOE_HDR_K_TOP: v = k; break;
            case MOE_HDR_E: v = E; break;
            case MOE_HDR_N: v = N; break;
            case MOE_HDR_TILE_M: v = g.tile_m; break;
            case MOE_HDR_TILE_N: v = g.tile_n; break;
            case MOE_HDR_NT: v = nt; break;
            case MOE_HDR_M: v = M; break;
            case MOE_HDR_TOTAL_TILES: v = bad ? 0 : total; break;
            case MOE_HDR_ORDER: v = 0; break;
            case MOE_HDR_STATUS: v = bad; break;
            case MOE_HDR_R: v = R; break;
            case MOE_HDR_E64: v = L.E64; break;
            case MOE_HDR_SIGMA_ORDER: v = order; break;
            case MOE_HDR_TILE_M_SMALL: v = g.tile_m_small; break;
            case MOE_HDR_SMALL_MAX_ROWS: v = g.small_max_rows; break;
            case MOE_HDR_TILE_M_SLACK: v = g.tile_m_slack; break;
            case MOE_HDR_HEAVY_TILES: v = (order == 2 && !bad) ? heavy_tiles : 0; break;
            default: v = 0;
        }
        map[tid] = v;
    }
    return off;
}

__device__ __forceinline__ int key_bits(int E) {
    int nb = 1;
    while ((1 << nb) < E) ++nb;
    return nb;
}

// Exclusive scan of the per-wavefront counts of expert `e` in row order, in place; returns their sum.
__device__ __forceinline__ int scan_waves(int* s_wave, int E64, int nwaves, int e) {
    int run = 0;
    for (int i = 0; i < nwaves; ++i) {
        const int c = s_wave[i * E64 + e];
        s_wave[i * E64 + e] = run;
        run += c;
    }
    return run;
}

// A second map from the same routing, flattened: T * k tokens with one expert each (the second product of a layer).  Rows,
// counts and offsets are those of the first map; only its tiling and N differ.  map == nullptr: none.
struct TwinMap {
    int32_t* map;
    int N;
    moe_tiling g;
};

// One-workgroup build for R <= kChunkRows: histogram, scans and stable scatter fused.  As many wavefronts as rows or
// experts need: a decode step's few rows are one wavefront's work, and a barrier of one wavefront costs nothing
// (R = 6, E = 64: 6.2 -> 3.1 us against a workgroup of 16).
// Dynamic LDS: (wavefronts + 1) * E64 ints (per-wavefront counts, offsets) + kTmpInts + 1 + 2 * E64 (ordering).
__host__ __device__ inline int small_build_threads(int64_t R, int E64) { return (int)(R > E64 ? (R + 63) / 64 * 64 : E64); }
__host__ __device__ inline size_t small_build_lds(int threads, int E64) {
    return ((size_t)(threads / 64 + 3) * E64 + kTmpInts + 1) * sizeof(int);
}
__device__ __forceinline__ void build_small(const int32_t* __restrict__ ids, int32_t* __restrict__ map, int T, int k, int E, int N,
                                            const moe_tiling& g, const TwinMap& twin, int* s_mem) {
    const MapLayout L = map_layout(E);
    const int nwaves = blockDim.x >> 6;
    int* s_wave = s_mem;                   // [nwaves][E64]
    int* s_off = s_mem + nwaves * L.E64;   // [E64]
    int* s_work = s_off + L.E64;           // [2*E64]
    int* s_tmp = s_work + 2 * L.E64;       // [kTmpInts], then the count of bad ids
    const int tid = threadIdx.x, w = tid >> 6;
    const int R = T * k;
    const bool in_range = tid < R;
    const int e = in_range ? ids[tid] : 0;
    for (int i = tid; i < nwaves * L.E64; i += blockDim.x) s_wave[i] = 0;
    if (tid == 0) s_tmp[kTmpInts] = 0;
    __syncthreads();
    const bool valid = in_range && e >= 0 && e < E;
    int rank, size;
    wave_match(e, valid, key_bits(E), rank, size);
    if (valid && rank == 0) s_wave[w * L.E64 + e] = size;
    const int nbad = __popcll(__ballot(in_range && !valid));
    if (nbad && __lane_id() == 0) atomicAdd(&s_tmp[kTmpInts], nbad);
    __syncthreads();
    const int bad = s_tmp[kTmpInts];
    const int cnt = tid < L.E64 ? scan_waves(s_wave, L.E64, nwaves, tid) : 0;
    const int off = finish_map(map, L, cnt, bad, T, k, E, N, g, s_tmp, s_work);
    if (twin.map) {
        __syncthreads();   // (the two share the scratch)
        finish_map(twin.map, L, cnt, bad, R, 1, E, twin.N, twin.g, s_tmp, s_work);
    }
    if (tid < L.E64) s_off[tid] = off;
    __syncthreads();
    if (valid) {
        const size_t at = L.off_rows + s_off[e] + s_wave[w * L.E64 + e] + rank;
        map[at] = tid;
        if (twin.map) twin.map[at] = tid;
    }
}

__global__ __launch_bounds__(kMapThreads) void map_build_small(const int32_t* __restrict__ ids, int32_t* __restrict__ map,
                                                                int T, int k, int E, int N, moe_tiling g, TwinMap twin) {
    extern __shared__ int s_mem[];
    build_small(ids, map, T, k, E, N, g, twin, s_mem);
}

// Larger builds: one workgroup per chunk of kChunkRows rows.  Every workgroup needs the counts of all experts over all
// rows and over the rows before its own chunk; it then repeats the scans (the first one writes counts / offsets / sigma /
// TilePrefix / task records / header) and scatters its chunk of rows, stably, into the token index arrays.
// Up to kFusedChunks chunks every workgroup counts all ids itself (R * 4 bytes out of L2, one LDS add per id), which
// costs less than a second launch; beyond that a first launch leaves one histogram per chunk.  Measured, one launch
// against two, back to back: 5 chunks, E = 64: 5.1 / 6.6 us; 16 chunks, E = 256: 7.3 / 8.3; 24 chunks, E = 64: 7.5 / 7.2;
// 64 chunks, E = 256: 13.6 / 9.5.  (One row after another summed the chunk histograms before, and every scan had its own
// pair of barriers: 13, 18, 17 and 35 us.)
constexpr int kFusedChunks = 16;

// Per-chunk histogram (integer LDS atomics: order-free).
__global__ __launch_bounds__(kMapThreads) void map_hist(const int32_t* __restrict__ ids, int R, int E, int E64,
                                                         int32_t* __restrict__ chunk_hist) {
    extern __shared__ int s_mem[];
    const int hs = hist_stride(E64);
    const int r = blockIdx.x * kChunkRows + threadIdx.x;
    const int e = r < R ? ids[r] : 0;
    for (int i = threadIdx.x; i < hs; i += kMapThreads) s_mem[i] = 0;
    __syncthreads();
    if (r < R) atomicAdd(&s_mem[(e >= 0 && e < E) ? e : E64], 1);
    __syncthreads();
    for (int i = threadIdx.x; i < hs; i += kMapThreads) chunk_hist[(size_t)blockIdx.x * hs + i] = s_mem[i];
}

// chunk_hist == nullptr: count the ids here.  Dynamic LDS: kWaves * E64 ints (per-wavefront counts) + E64 ints (this
// chunk's destination per expert) + 2 * hist_stride(E64) ints (counts of the rows before this chunk, of the others).
__global__ __launch_bounds__(kMapThreads) void map_scan_scatter(const int32_t* __restrict__ ids, int32_t* __restrict__ map,
                                                                const int32_t* __restrict__ chunk_hist, int nchunks,
                                                                int T, int k, int E, int N, moe_tiling g, TwinMap twin) {
    extern __shared__ int s_mem[];
    __shared__ int s_tmp[kTmpInts];
    __shared__ int s_bad[kWaves];
    const MapLayout L = map_layout(E);
    const int hs = hist_stride(L.E64);
    int* s_wave = s_mem;                  // [kWaves][E64]
    int* s_off = s_mem + kWaves * L.E64;  // [E64]
    int* s_hist = s_off + L.E64;          // [2][hs]: before this chunk, not before it; column E64 counts bad ids
    const int tid = threadIdx.x, w = tid >> 6;
    const int R = T * k;
    const int chunk = blockIdx.x;
    const int r = chunk * kChunkRows + tid;
    const bool in_range = r < R;
    const int e = in_range ? ids[r] : 0;
    for (int i = tid; i < kWaves * L.E64; i += kMapThreads) s_wave[i] = 0;
    for (int i = tid; i < 2 * hs; i += kMapThreads) s_hist[i] = 0;
    __syncthreads();
    const bool valid = in_range && e >= 0 && e < E;
    int rank, size;
    wave_match(e, valid, key_bits(E), rank, size);
    if (valid && rank == 0) s_wave[w * L.E64 + e] = size;
    const int wave_bad = __popcll(__ballot(in_range && !valid));
    if (__lane_id() == 0) s_bad[w] = wave_bad;
    if (chunk_hist) {
        // thread (column, part): the parts share out the chunks
        const int cols = L.E64 + 1, parts = kMapThreads / L.E64;
        const int col = tid % L.E64, part = tid / L.E64;
        if (part < parts) {
            int before = 0, rest = 0;
#pragma unroll 4
            for (int c = part; c < nchunks; c += parts) {
                const int v = chunk_hist[(size_t)c * hs + col];
                if (c < chunk) before += v; else rest += v;
            }
            if (before) atomicAdd(&s_hist[col], before);
            if (rest) atomicAdd(&s_hist[hs + col], rest);
        }
        int b = 0;
        for (int c = tid; c < nchunks; c += kMapThreads) b += chunk_hist[(size_t)c * hs + cols - 1];
        if (b) atomicAdd(&s_hist[L.E64], b);
    } else {
        const int batch = 4;
        for (int c0 = 0; c0 < nchunks; c0 += batch) {
            int v[batch];
#pragma unroll
            for (int j = 0; j < batch; ++j) {
                const int rr = (c0 + j) * kChunkRows + tid;
                v[j] = c0 + j < nchunks && rr < R ? ids[rr] : -2;
            }
#pragma unroll
            for (int j = 0; j < batch; ++j) {
                const int rr = (c0 + j) * kChunkRows + tid;
                if (c0 + j < nchunks && rr < R)
                    atomicAdd(&s_hist[(c0 + j < chunk ? 0 : hs) + ((v[j] >= 0 && v[j] < E) ? v[j] : L.E64)], 1);
            }
        }
    }
    __syncthreads();
    const int bad = s_hist[L.E64] + s_hist[hs + L.E64];
    const int before = tid < L.E64 ? s_hist[tid] : 0;
    const int cnt = tid < L.E64 ? before + s_hist[hs + tid] : 0;
    const int own = tid < L.E64 ? scan_waves(s_wave, L.E64, kWaves, tid) : 0;
    __syncthreads();   // (the ordering work below reuses s_hist)
    const int off = finish_map(map, L, cnt, bad, T, k, E, N, g, s_tmp, s_hist, chunk == 0);
    if (twin.map && chunk == 0) {
        __syncthreads();   // (the two share the scratch)
        finish_map(twin.map, L, cnt, bad, R, 1, E, twin.N, twin.g, s_tmp, s_hist);
    }
    if (tid < L.E64) s_off[tid] = off + before;
    __syncthreads();
    if (valid) {
        const size_t at = L.off_rows + s_off[e] + s_wave[w * L.E64 + e] + rank;
        map[at] = r;
        if (twin.map) twin.map[at] = r;
    }
    // The scratch parts hold the histogram of every chunk either way.
    const size_t hist_at = L.off_rows + round_up64((size_t)R) + (size_t)chunk * hs;
    if (!chunk_hist || twin.map) {
        for (int i = tid; i < hs; i += kMapThreads) {
            int v = i < L.E64 ? own : 0;   // (i == tid there)
            if (i == L.E64)
                for (int j = 0; j < kWaves; ++j) v += s_bad[j];
            if (!chunk_hist) map[hist_at + i] = v;
            if (twin.map) twin.map[hist_at + i] = v;
        }
    }
}

// Full per-block table from the compressed map, one wavefront per block index.
__global__ __launch_bounds__(256) void map_expand(const int32_t* __restrict__ map, int E, int32_t* __restrict__ table,
                                                   long long grid) {
    const MapLayout L = map_layout(E);
    const int total = map[MOE_HDR_TOTAL_TILES];
    moe_tiling g;
    g.tile_m = map[MOE_HDR_TILE_M]; g.tile_n = map[MOE_HDR_TILE_N]; g.order = map[MOE_HDR_SIGMA_ORDER];
    g.tile_m_small = map[MOE_HDR_TILE_M_SMALL]; g.small_max_rows = map[MOE_HDR_SMALL_MAX_ROWS];
    g.tile_m_slack = map[MOE_HDR_TILE_M_SLACK];
    const long long wave = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long nwaves = (long long)gridDim.x * 4;
    for (long long B = wave; B < grid; B += nwaves) {
        int4 out = make_int4(-1, -1, -1, -1);
        if (B < total) {
            const TileCoord c = decode_block(map, L, g, (int)B, reinterpret_cast<const int4*>(map + L.off_records)[__lane_id()]);
            out = make_int4(c.e, c.m_tile, c.n_tile, c.rows);
        }
        if (__lane_id() == 0) reinterpret_cast<int4*>(table)[B] = out;
    }
}

}  // namespace moe

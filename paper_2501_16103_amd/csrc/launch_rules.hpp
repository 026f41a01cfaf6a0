// Which form of launch a call takes, where that is decided by sizes alone: host rules, no kernels and no HIP calls.
// Times quoted in comments are those of one product, HIP events around launches back to back on one set of weights.
#pragma once
#include <math.h>
#include <stdint.h>

#include "../../include/moe_sb.h"

namespace moe {

constexpr int kXcdCus = 32;   // CUs of each of the 8 XCDs
constexpr int kCus = 8 * kXcdCus;
constexpr int kStreamExperts = 256;   // experts whose task records the streaming launch holds in registers
constexpr int kStreamScales = 2048;   // scales (T + E) that the fp8 one holds in LDS
constexpr int kSpareSlots = 16;   // workgroups a launch's grid holds beyond the bound on its tiles (see grouped_gemm_impl)

// The work items of a launch are counted in 32 bits: with more, workgroups are left out and no error is reported.
constexpr bool work_items_fit(int64_t workgroups, int threads) { return workgroups * threads <= 0xffffffffll; }
static_assert(work_items_fit((1 << 23) - 1, 512) && !work_items_fit(1 << 23, 512) && work_items_fit(1 << 23, 256), "2^32 - 1");

// Tiles of 16 rows that a uniform routing gives: one for each expert it hits; from half a tile of rows per expert on, rows
// fill a tile half on average.
inline double expected_tiles16(int64_t R, int E, int64_t nt) {
    const double hit = E * (1.0 - pow(1.0 - 1.0 / E, (double)R)), filled = R / 16.0 + E / 2.0;
    return (R >= 8 * (int64_t)E && filled > hit ? filled : hit) * (double)nt;
}

// Whether the streaming launch runs the rows of several 16-row tiles as one tile (see moe_gemm_stream_kernel): nt n-tiles as it runs
// them.  From 8 to 32 rows per expert on average and from 16 k-tiles on.  At 8 to 10 rows an even routing gives nearly every expert
// one tile, and the larger task function costs 1 to 2 % (bf16, 256 experts, 2048 -> 2048, 6 %: 317 -> 339 us), but skewed ones gain ten
// times that (the same 332 -> 281; 64 experts, 2048 -> 2816, 122 -> 110); below 8 rows the cost stays (fp8, 32 tokens, 1 to 3 %).  Beyond 32, few
// experts are left with too few workgroups (8 experts, K = 256, 75 rows each: 7.4 -> 11.5 us), and such maps are not the default; with a
// short K the rows of a full tile take longer than its panel (64 experts, 1024 -> 2048, fp8, a skewed routing of 200 tokens 28.6 -> 35.0).
// Tiles that all start at once gain nothing from being fewer, the longest of them only gets longer: below two tiles per CU, it takes
// a round less under a uniform routing (tiles expected one by one / merged; fp8, us: 8 experts, 2048 -> 2816, 20 rows, 154 / 88, 17.2
// -> 18.1 and, skewed, 16.7 -> 20.9; 32 experts, 10 rows, 396 / 352, 35.3 -> 36.4, skewed 36.2 -> 40.4, but 16 rows, 528 / 352, 41.5 -> 37.6;
// 16 experts, 4096 -> 4096, 16 rows, 384 / 256, 61.5 -> 47.3).  A launch of a given number of workgroups merges by rows and K alone.
constexpr bool merges16(int64_t R, int E, int64_t nt, int k_tiles, int mode) {
    if (R < 8 * (int64_t)E || R > 32 * (int64_t)E || k_tiles < 16) return false;
    const int64_t merged = E * nt, single = R * nt / 16 + merged / 2;
    return mode >= MOE_LAUNCH_RESIDENT || merged >= 2 * kCus || (single + kCus - 1) / kCus > (merged + kCus - 1) / kCus;
}
static_assert(merges16(64 * 8, 64, 11, 16, MOE_LAUNCH_AUTO) && !merges16(64 * 8 - 1, 64, 11, 16, MOE_LAUNCH_AUTO), "many tiles");
static_assert(!merges16(8 * 20, 8, 11, 16, MOE_LAUNCH_AUTO) && !merges16(32 * 10, 32, 11, 16, MOE_LAUNCH_AUTO), "few tiles, no round less");
static_assert(merges16(32 * 16, 32, 11, 16, MOE_LAUNCH_AUTO) && merges16(16 * 16, 16, 16, 32, MOE_LAUNCH_AUTO), "a round less");

// The 16-row tiles over [E][K][N] weights, 256 or 128 columns wide, as the launches run them: threads of a workgroup and stages of its ring
// (the same for both types).
struct Rows16Form { int threads, stages; };
struct Rows16Forms {
    Rows16Form deep;      // a CU by itself
    Rows16Form shallow;   // two workgroups per CU
    Rows16Form small;     // the same with two wavefronts
    Rows16Form pairs;     // two n-tiles of 128 columns as one, a CU by itself
};
constexpr Rows16Forms rows16_forms(int tile_n) {
    return tile_n == 256 ? Rows16Forms{{512, 3}, {512, 2}, {128, 2}, {0, 0}} : Rows16Forms{{256, 6}, {256, 4}, {128, 4}, {512, 3}};
}

// Form of the launch for a map of 16-row tiles (MOE_ROWS16_*); `grid`: bound on its tiles with the spare slots.
//
// One workgroup per tile.  Two workgroups per CU, so that one's start and store do not leave the CU idle.  128-wide tiles always run so (64 experts,
// 2048 -> 2816, a CU each / two per CU, us: fp8, 127 tiles expected 10.9 / 10.3, 243 17.8 / 15.8, 559 32.2 / 27.9; bf16 243 29.4 / 28.0,
// 559 55.1 / 51.4).  256-wide ones up to one per CU take a CU each, which keeps more of a stream in flight (bf16 121 tiles 29.2 / 42.3,
// 179 33.4 / 45.2), and beyond two per CU with at least 32 k-tiles (384 experts, 2048 -> 2816, bf16, 4213 tiles 678 / 701); else two per CU
// (280 tiles 57.6 / 53.6, 450 67.9 / 67.3).  Two wavefronts each for launches of more work items than their count holds in the other forms.
//
// Resident workgroups (not in MOE_LAUNCH_PER_TILE), as many as stay resident at once.  256-wide tiles: from two
// tiles per workgroup on, counted by the bound.  128-wide ones: once more are expected than the CUs hold in the two-workgroup form,
// for up to there no tile waits for a second round (64 experts, 2048 -> 1408, fp8: 363 tiles 19.7 us per tile,
// 22.2 streaming; 572 tiles 32.4 / 28.6); where N holds a whole number of 256-wide ones, the map's n-tiles are
// run in pairs once more of them are expected than CUs (fp8, 64 experts,
// 2048 -> 2816: 3 tokens, 330 tiles, 22.5 -> 18.0 us, 20.5 with two workgroups per CU; 32 tokens 56 -> 52).  A K too short for the deep ring
// streams in a form of two workgroups per CU.  bf16: from two tiles per workgroup on (per tile / streaming, us: 256 experts, K = 128, 2 rows each,
// N = 2048 24.4 / 22.3, N = 1024 14.2 / 13.2; skewed 16.7 / 17.5, 10.6 / 12.6).  fp8: the scales behind the rings leave room for two workgroups
// of two wavefronts only (kStreamScales), which one workgroup per tile, of four, overtakes: 64 experts, 512 -> 1408, 100 tokens, top-6, even 12.4 /
// 16.3, skewed 13.5 / 16.8; 128 experts, 512 -> 1920, 256 tokens, top-8, 36.1 / 40.7 and 38.1 / 45.6; 256 experts, 512 -> 3968, 600 tokens 158
// / 162 and 153 / 167.  They lead where tiles are sixteen per CU and nearly empty: 128 experts, 512 -> 8064, 40 tokens 90.9 / 85.6 and
// 67.3 / 66.6, 150 tokens 114 / 110 and 117 / 120; 256 experts, 512 -> 3968, 150 tokens 98 / 95 and 85 / 88, 256 tokens 108 / 103 and 108 / 111.
// (Between one and two 256-wide tiles per CU the deep form is kept: where a uniform routing is expected to give 280 tiles, it takes 57 us
// against 54 with two workgroups per CU, but a skewed one of the same size, with less than one per CU, 34 against 45.)
inline int rows16_form(bool fp8, int tile_n, int T, int64_t R, int E, int K, int N, int64_t grid, int mode) {
    const Rows16Forms f = rows16_forms(tile_n);
    const bool wide = tile_n == 256, asked = mode >= MOE_LAUNCH_RESIDENT;
    const int k_tiles = K / (fp8 ? 128 : 64);
    const double expected = expected_tiles16(R, E, N / tile_n);
    if (mode != MOE_LAUNCH_PER_TILE && E <= kStreamExperts && (!fp8 || T + E <= kStreamScales)) {
        if (!wide && N % 256 == 0 && k_tiles >= f.pairs.stages && (asked || expected > kCus))
            return merges16(R, E, N / 256, k_tiles, mode) ? MOE_ROWS16_PAIRS_MERGED : MOE_ROWS16_PAIRS;
        if (k_tiles >= f.deep.stages) {
            if (asked || (wide ? grid >= 2 * kCus : expected > 2 * kCus))
                return merges16(R, E, N / tile_n, k_tiles, mode) ? MOE_ROWS16_STREAM_MERGED : MOE_ROWS16_STREAM;
            if (wide) return MOE_ROWS16_PER_TILE_DEEP;
        } else if (k_tiles >= f.shallow.stages) {
            const bool many = fp8 ? expected >= 16 * kCus && R < 12 * (int64_t)E : grid >= 4 * kCus;
            if (asked || many) return MOE_ROWS16_STREAM_SHORT_K;
        }
    }
    const bool deep = wide && (expected <= kCus || (expected > 2 * kCus && k_tiles >= 32));
    if (deep && work_items_fit(grid, f.deep.threads)) return MOE_ROWS16_PER_TILE_DEEP;
    if (work_items_fit(grid, f.shallow.threads)) return MOE_ROWS16_PER_TILE;
    if (work_items_fit(grid, f.small.threads)) return MOE_ROWS16_PER_TILE_SMALL;
    return MOE_ERR_UNSUPPORTED;
}

// Form of the one launch that builds the maps of a layer's step as well (bf16, see moe_gemm_with_map_kernel), that of moe_grouped_gemm for the same
// tiles; 0: two launches.  Up to 64 rows and experts (a wavefront's lanes), each tile of the map by itself.
inline int with_map_form(int tile_n, int T, int64_t R, int E, int K, int N, int64_t grid) {
    const int k_tiles = K / 64;
    if (R < 1 || R > 64 || E > 64 || k_tiles < 3 || merges16(R, E, N / 256, k_tiles, MOE_LAUNCH_AUTO) || merges16(R, E, N / 128, k_tiles, MOE_LAUNCH_AUTO))
        return 0;
    const int form = rows16_form(false, tile_n, T, R, E, K, N, grid, MOE_LAUNCH_AUTO);
    if (tile_n == 256) return form == MOE_ROWS16_STREAM || form == MOE_ROWS16_PER_TILE_DEEP ? form : 0;
    const bool per_tile = form == MOE_ROWS16_PER_TILE && expected_tiles16(R, E, N / tile_n) <= kCus;
    return form == MOE_ROWS16_PAIRS || per_tile ? form : 0;
}

}  // namespace moe

// The plan of a fused step launch: tile height, z chunk and store hint as functions of
// the lattice and the device alone (host code, no HIP).
#pragma once

#include <algorithm>
#include <cstddef>

namespace tslb {

// What a plan depends on.
struct PlanShape {
    int nx, ny, nz;
    bool phase;  // two components
    bool wide;   // 20-row tiles serve the lattice (two components, equal densities)
    bool half;   // 16-bit moments (all of them, or the stress)
    int cus;     // compute units of the device
};

// Tile height (16 or 20 rows) and z chunk.
struct FusedPlan {
    int rows = 16;
    int lz = 1;
};

constexpr int kTileX = 32;  // columns of a tile of either height

inline long long fused_tiles(const PlanShape &s, int rows) {
    return (((long long)s.nx + kTileX - 1) / kTileX) * (((long long)s.ny + rows - 1) / rows);
}

// Chunks of lz planes over nz planes, and the length under the bound L that makes as
// many chunks of near-equal length.
inline long long chunk_count(int nz, int lz) { return ((long long)nz + lz - 1) / lz; }
inline int chunk_under_bound(int nz, int L) {
    const long long k = chunk_count(nz, L);
    return (int)((nz + k - 1) / k);
}

// Tile height and z planes per workgroup.  A workgroup on a chunk of lz planes
// walks lz planes and the fill of its pipeline, and the W work items of a launch
// give each CU ceil(W / CUs) of them, so the cost of a plan is
// ceil(W / CUs) (lz + fill) c, with c the time of one pipeline plane of a
// workgroup: 1 for 16 rows and kWideCost for 20 rows.
// fill: one round of workgroups takes 1.97 (lz + 6.2 to 6.6) us with two components
// and 1.57 (lz + 4.4 to 4.9) with one (32^3 to 64^3 lattices, lz 1 to 12, launch
// included), of which 3 are planes of the loop and, with two, the geometry's prologue;
// 6.5 and 4.5 are taken.  So the shortest chunks pay as long as they fill idle CUs: 32^3
// droplet 20.2 us a step at 4 planes, 14.4 at 1; 48^3 20.9 at 4, 16.8 at 2; 40^3 vortex
// 13.7 at 4, 9.0 at 1.
// Cost of 20 rows, from jets timed at both heights: about 1.25 in one round of
// workgroups, 1.15 to 1.30 in several, where the last round is not full and neighbours
// share less.  Of 32 jets in binary32 1.22 takes the faster height or one within 4.7 %
// (512 x 512 x 2048: 20 rows 1.5 % faster in one process and 1.5 % slower in another;
// 320 x 240 x 640 16 rows, 1116 and 1081 us; 157 x 229 x 103 20 rows, 110 and 115), 0.45 %
// on average.  With 16-bit moments their geometry, four waves' work there, is the
// longer chain of phase A: 1.23 to 1.32, of 31 jets in each type 1.26 takes the faster or
// one within 3.5 %, 0.06 % on average (at 1.35 0.7 %, up to 6.9 %: 200 x 200 x 400 FP16Q
// 465 us on 16 rows, 438 on 20; 103 x 97 x 514 175 and 164; at 1.18 1.8 %).
// Long chunks recompute less halo, short ones keep every unit busy; ties go to the
// shorter chunk, then to 16 rows.  Chunks are capped at kMaxChunk planes:
// workgroups that share halo columns run side by side, but over a long chunk
// they drift apart in z and their shared halo planes leave L2 before the
// neighbour reads them (HBM reads 1.48x the state at 2048 planes on a
// 512 x 512 x 2048 lattice, against 1.06x at 64 on 128 x 128 x 512).  On that
// lattice 16 rows take 11.65 and 11.38 ms at 64 and 128 planes, 20 rows 11.80 and 11.58.
// 20 rows serve the two-component step with equal densities; the one-component
// and the variable-density step take 16.  A height or chunk length fixed with
// tslb_set_tile / tslb_set_kernel is taken as given.
constexpr int kMaxChunk = 128;
constexpr double kWideCost = 1.22, kWideCostHalf = 1.26;

// Planes a workgroup on a chunk of lz planes walks, doubled.
inline long long fused_walk2(const PlanShape &s, int lz) { return 2ll * lz + (s.phase ? 13 : 9); }

// Cheapest chunk length for `rows` (chunk_z > 0 fixes it) and its cost, in 16-row plane
// times.
inline double best_chunk(const PlanShape &s, int rows, int chunk_z, int *lz_out) {
    const long long tiles = fused_tiles(s, rows), cus = std::max(1, s.cus);
    const double f = rows == 16 ? 1.0 : s.half ? kWideCostHalf : kWideCost;
    auto cost_of = [&](int lz) {
        const long long w = tiles * chunk_count(s.nz, lz);
        return (double)((w + cus - 1) / cus) * (0.5 * (double)fused_walk2(s, lz)) * f;
    };
    if (chunk_z > 0) {
        *lz_out = std::min(chunk_z, s.nz);
        return cost_of(*lz_out);
    }
    double best = -1.0;
    int last = 0;
    for (int L = std::min(s.nz, kMaxChunk); L >= 1; --L) {
        const int lz = chunk_under_bound(s.nz, L);
        if (lz == last) continue;
        last = lz;
        const double cost = cost_of(lz);
        if (best < 0 || cost <= best) {
            best = cost;
            *lz_out = lz;
        }
    }
    return best;
}

// The plan of a lattice; chunk_z and tile_rows as set by the caller (0: open).
inline FusedPlan plan_fused(const PlanShape &s, int chunk_z, int tile_rows) {
    FusedPlan pl;
    int lz20 = 0;
    const double c16 = best_chunk(s, 16, chunk_z, &pl.lz);
    if (!s.wide || tile_rows == 16) return pl;
    const double c20 = best_chunk(s, 20, chunk_z, &lz20);
    if (tile_rows == 20 || c20 < c16) {
        pl.rows = 20;
        pl.lz = lz20;
    }
    return pl;
}

// Whether the step's stores carry the non-temporal hint, where a launch writes
// launch_bytes in all (a launch over several lattices takes what most of its bytes
// call for).  A line stored with it goes out at once; without it the line
// stays in L2 until it is complete and then in the 256 MB cache behind.
//  - A lattice up to kTinyState bytes: hint.  Its launch is a few planes long and
//    would end with the lines still to be written back (61 x 45 x 83 box 18.6 us a step
//    with, 19.5 without; 64^3 vortex 10.6, 11.0; 66^3 droplet, 12.7 MB, 22.6 both).
//  - Rows that do not begin at 128-byte lines: none.  The two tiles that share a
//    line write it at different times, and the halves go to memory as partial writes
//    (250 x 256 x 400 jet: 26.4 M write requests against 18.0 M at 256 wide; 250 x 250 x
//    400 jet 832 us with, 618 without; 300 x 300 x 600 jet 1919 and 1418; 200 x 200 x 400
//    FP16Q 506 and 487).
//  - Whole lines, state and new state within the cache: none, the next step reads from
//    it (128^3 droplet 55.4 and 48.6, 128^3 vortex 42.1 and 34.4).
//  - Whole lines, larger: hint, since lines written without it take L2 from the halo
//    lines that neighbouring workgroups read again (512 x 512 x 2048 jet 12.3 ms and
//    12.6, 512 x 512 x 1024 5.46 and 5.79, 256^3 vortex 263 us and 274, 160^3 droplet
//    101.5 and 102).
//  - 16-bit rows of a tile are half a line, so that two tiles share it at any width; on
//    widths of whole lines the hint makes little difference: 512 x 512 x 2048 jet FP16
//    11.03 ms with, 11.12 without, BF16 11.43 and 11.42, FP16Q 11.72 and 11.78; 256 x 256 x
//    512 674 us and 666, 697 and 694, 678 and 679; one component 256^3 FP16 265 and 263,
//    384^3 FP16Q 1037 and 1009.  They follow the rule of binary32.
constexpr size_t kTinyState = 13u << 20, kFarCache = 256u << 20;
inline bool stream_stores(const PlanShape &s, size_t launch_bytes) {
    if (launch_bytes <= kTinyState) return true;
    if (s.nx % (s.half ? 64 : 32)) return false;  // words of a 128-byte line
    return 2 * launch_bytes > kFarCache;
}

// Workgroups of one launch when `items` are left: a launch takes at most 2^32 - 1
// threads, 4194303 workgroups of 1024.  Chunks of 128 planes stay far below that on
// every lattice that is wide enough to fill its tiles; a lattice of one column and more
// than 5e8 planes, or one whose chunk the caller sets to a plane, does not.
inline long long launch_blocks(long long items, int threads) { return std::min(items, 0xFFFFFFFFll / threads); }

}  // namespace tslb

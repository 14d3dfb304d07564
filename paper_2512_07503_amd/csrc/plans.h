// Which projection kernels a forward of M rows runs through: row groups (kernels_skinny.hip.h), LDS tiles
// (kernels_lds.hip.h) or tile kernels (kernels_tile.hip.h), chosen by their expected times.  Plain host code, without
// HIP: the choice can be computed and tested on a machine without a GPU.
#pragma once
#include <stddef.h>

#include <algorithm>

#include "../../include/sjd.h"

inline int plan_div(int a, int b) { return (a + b - 1) / b; }   // rounded up

// What the choice depends on beside the rows.
struct ProjShape {
    int d_model, n_heads, n_kv_heads, d_ff, n_sampled, n_cus, kernel_flags;
    int q_dim() const { return d_model; }                                                          // n_heads * head dimension
    int qkv_groups() const { return (n_heads + 2 * n_kv_heads) * (d_model / n_heads / 64); }        // groups of two column blocks
    int gate_up_groups() const { return d_ff / 32; }
    int head_groups() const { return plan_div(plan_div(n_sampled, 32), 2); }
};

constexpr int TILE_M = 256;   // rows of the larger tile of kernels_tile.hip.h

// ---- LDS tiles.  Tile shapes (TMT, TNB, WM, WN, S) of kernels_lds.hip.h.  Shape 4 is the head's where a wavefront has to hold a
// conditional and an unconditional row tile.  Shape 5 (QKV and gate/up) moves the fewest bytes per MFMA but leaves a CU to one
// workgroup and its epilogue uncovered: it is for launches of one workgroup per CU at most.  Kernel times in repeated prompt
// forwards, without -> with it: 2040 x 6144 x 4096 117 -> 101 us (128-row tiles), 900 x 12288 x 4096 110 -> 104 and 1008 x 12288
// 113 -> 106 (the same), 1280 x 12288 136 -> 113 (192 x 128), 2040 x 6912 x 1280 50 -> 42 (192 x 128); with several per CU it
// gains nothing (2048 x 28672 x 4096 434 us against 430).
#define SJD_LDS_TILES(X) X(0, 2, 2, 2, 1, 6) X(1, 4, 2, 4, 1, 6) X(2, 4, 4, 4, 2, 5) X(3, 6, 4, 2, 2, 4) X(4, 4, 4, 2, 2, 4) X(5, 8, 8, 2, 4, 4)
constexpr int kLdsTiles = 4, kLdsTileHeadZ = 4, kLdsTileBig = 5;
struct LdsTile { int tmt, tnb, cb; double t1, t2, tn; };
// t1, t2, tn: microseconds per pipeline stage of a CU with one workgroup, with two, and per workgroup of more.  Measured on
// models 768 to 4096 wide at 118 to 2040 rows, weights from HBM, before the kernels had their first arguments in registers: launches
// of up to 500 rows now take 5 to 30 % less than this says (row groups of 126 rows of 1280: 40 %), larger ones are within 13 %
// (2040 x 3840 x 1280: 15 % more).
inline LdsTile lds_tile(int cfg) {
    static const LdsTile t[6] = {{2, 2, 2, 0.22, 0.33, 0.14}, {4, 2, 2, 0.27, 0.45, 0.19}, {4, 4, 2, 0.38, 0.56, 0.30}, {6, 4, 2, 0.42, 0.72, 0.37},
                                 {4, 4, 2, 0.40, 0.62, 0.33}, {8, 8, 2, 0.80, 1e3, 1e3}};
    return t[cfg];
}

// Time of an LDS-tile launch: stages x the busiest CU's workgroups (the column tiles of an XCD run on its CUs only).
inline double lds_us(int cfg, int M, int n_blocks, int KB, int ks, int n_cus) {
    const LdsTile t = lds_tile(cfg);
    const int wgs_xcd = plan_div(plan_div(n_blocks, t.tnb), 8) * plan_div(M, 32 * t.tmt) * ks;
    const int n = plan_div(wgs_xcd, std::max(1, n_cus / 8));
    return (cfg == kLdsTileBig ? 8.0 : 4.0) + (double)plan_div(KB, 2 * ks) * (n == 1 ? t.t1 : n == 2 ? t.t2 : n * t.tn);
}
// ... of a row-group launch (kernels_skinny.hip.h): a CU moves 52 GB/s of weights and activations
inline double skinny_us(int wgs, double wg_bytes, bool norm, int n_cus) {
    return 5.0 + plan_div(wgs, n_cus) * wg_bytes / 52e3 + (norm ? 2.5 : 0.0);
}
// ... and of the kernel that adds ks partial sums of M rows of d columns
inline double reduce_us(int M, int d, int ks) { return std::max(6.7, 3.0 + (ks + 2.0) * M * d * 4.0 / 5e6); }

// ---- tile kernels
// Rows per workgroup tile for n_blocks column blocks over M rows.  256 rows (two 32-row tiles per wavefront) need
// the fewest operand bytes per MFMA: 0.75 KiB against 1.25 KiB for 128 rows, whose weight fragments alone would
// take the whole LDS bandwidth at full MFMA rate.  128 rows are chosen where they spread the work better: when
// 256-row tiles would not even fill the CUs, or when the most loaded CU (a launch takes as long as that one)
// gets less work - ceil(workgroups / CUs) tiles of 256 rows against as many half-size ones.
inline int tile_rows_for(int M, int n_blocks, int ksplit, int n_cus) {
    const int col_tiles = (n_blocks + 3) / 4;
    const long wg2 = (long)col_tiles * ((M + 255) / 256) * ksplit, wg1 = (long)col_tiles * ((M + 127) / 128) * ksplit;
    if (wg2 < n_cus) return 128;
    const long cost2 = 2 * ((wg2 + n_cus - 1) / n_cus), cost1 = (wg1 + n_cus - 1) / n_cus;
    return cost1 < cost2 ? 128 : 256;
}

// Time of a launch: 32-wide K stages x the busiest CU's tiles (the column tiles of an XCD run on its CUs only): 0.27 us a
// 128-row tile (0.40 alone on its CU), 0.45 a 256-row tile, 0.27 per 128 x 128 in a launch of both heights.  Measured on
// models 1280 to 4096 wide at 260 to 2040 rows.
inline bool tile_two_heights(int M, int n_blocks, int ksplit, int n_cus) {
    const int col_tiles = (n_blocks + 3) / 4, rt2 = (M + 255) / 256, rt1 = (M + 127) / 128;
    return ksplit == 1 && rt1 > rt2 && col_tiles * rt2 > n_cus && col_tiles * rt2 < 2 * n_cus && n_cus / rt2 >= 8 && (col_tiles * rt1) % n_cus != 0;
}
inline double tile_us(int M, int n_blocks, int KB, int ksplit, int n_cus) {
    const int col_tiles = (n_blocks + 3) / 4, rows = tile_rows_for(M, n_blocks, ksplit, n_cus);
    const double stages = KB / (2.0 * ksplit);
    if (tile_two_heights(M, n_blocks, ksplit, n_cus)) {
        const int rt2 = (M + 255) / 256, ct_split = n_cus / rt2 / 8 * 8;
        return 12.0 + stages * 0.27 * (2.0 * ct_split * rt2 + (double)(col_tiles - ct_split) * ((M + 127) / 128)) / n_cus;
    }
    const int per_xcd = (col_tiles + 7) / 8 * ((M + rows - 1) / rows) * ksplit, cus = n_cus >= 8 ? n_cus / 8 : 1, n = (per_xcd + cus - 1) / cus;
    return 12.0 + stages * (rows == 256 ? 0.45 * n : n == 1 ? 0.40 : 0.27 * n);
}

// ---- the choice
inline int resid_nbw(int d) { return plan_div(d, 32) >= 128 ? 2 : 1; }   // column blocks per workgroup of an output / down projection
// More than 32 rows and so few column groups that a workgroup per group and 32-row tile still finds a CU of its own
inline bool rows_of_32(const ProjShape &s, int M, int groups) {
    return M > 32 && 2 * plan_div(M, 64) * 8 * plan_div(groups, 8) <= s.n_cus && !(s.kernel_flags & SJD_NO_ROW_SPLIT);
}

// How a projection runs: row groups (lds < 0) or LDS tiles of shape `lds`; ks: splits of K (output / down projections, whose
// partial sums resid_reduce_kernel adds); us: its expected time, on which the choice rests.
struct ProjPlan { int lds, ks; double us; };
inline ProjPlan with_lds(const ProjShape &s, int M, int n_blocks, int KB, int max_ks, ProjPlan p, double extra_us) {
    if (M <= 64 || (s.kernel_flags & SJD_KERNELS_ROWGROUPS)) return p;
    for (int cfg = 0; cfg < kLdsTiles; ++cfg)
        for (int ks = 1; ks <= max_ks; ks *= 2) {
            if (ks > 1 && KB / ks < 32) continue;
            const double t = extra_us + lds_us(cfg, M, n_blocks, KB, ks, s.n_cus) + (ks > 1 ? reduce_us(M, s.d_model, ks) : 0.0);
            if (t < p.us) p = {cfg, ks, t};
        }
    return p;
}
// Shape 5 in the place of p where it is expected to be faster (QKV and gate/up only).
inline ProjPlan with_big(const ProjShape &s, int M, int n_blocks, ProjPlan p) {
    if (M < TILE_M || (s.kernel_flags & (SJD_KERNELS_ROWGROUPS | SJD_KERNELS_TILES))) return p;
    const double t = lds_us(kLdsTileBig, M, n_blocks, s.d_model / 16, 1, s.n_cus);
    return t < p.us ? ProjPlan{kLdsTileBig, 1, t} : p;
}
// QKV, gate/up and head: groups of two column blocks, whole K.  (2 us: the sums of squares that the row-group kernel takes
// from its operands come from the writer of the rows with LDS tiles.)
inline ProjPlan norm_plan(const ProjShape &s, int M, int groups) {
    const int d = s.d_model, mt = M <= 32 || rows_of_32(s, M, groups) ? 1 : 2;
    const ProjPlan p = {-1, 1, skinny_us(plan_div(M, 32 * mt) * groups, (double)(64 + 32 * mt) * d * 2.0, true, s.n_cus)};
    return with_lds(s, M, groups * 2, d / 16, 1, p, 2.0);
}
inline ProjPlan resid_plan(const ProjShape &s, int M, int K) {
    const int d = s.d_model, KB = K / 16, nbw = resid_nbw(d), groups = plan_div(plan_div(d, 32), nbw);
    const int mt = M <= 32 || rows_of_32(s, M, groups) ? 1 : 2;
    const double wg_bytes = (double)(nbw * 32 + mt * 32) * K * 2.0;
    int ks = 1;
    if (wg_bytes > 512e3) {   // one workgroup's share is too much for its CU
        ks = std::min(8, std::max(1, s.n_cus / (groups * plan_div(M, 64))));
        while (ks > 1 && KB / ks < 32) --ks;
        ks = plan_div(KB, plan_div(KB, ks));
    }
    const ProjPlan p = {-1, ks, skinny_us(plan_div(M, 32 * mt) * groups * ks, wg_bytes / ks, false, s.n_cus) + (ks > 1 ? reduce_us(M, d, ks) : 0.0)};
    return with_lds(s, M, plan_div(d, 32), KB, 4, p, 0.0);
}

// The tile kernels (kernels_tile.hip.h): K splits of an output / down projection, and the same estimate for a layer.
inline int tile_splits(const ProjShape &s, int M, int KB) {
    int ks = std::min(8, std::max(1, s.n_cus / (plan_div(plan_div(s.d_model, 64) * 2, 4) * plan_div(M, TILE_M))));
    while (ks > 1 && KB / ks < 32) --ks;
    return plan_div(KB, plan_div(KB, ks));
}
inline double tile_layer_us(const ProjShape &s, int M) {
    const int d = s.d_model;
    auto resid = [&](int K) {
        const int ks = tile_splits(s, M, K / 16);
        return tile_us(M, plan_div(d, 64) * 2, K / 16, ks, s.n_cus) + (ks > 1 ? reduce_us(M, d, ks) : 0.0);
    };
    return tile_us(M, s.qkv_groups() * 2, d / 16, 1, s.n_cus) + tile_us(M, s.d_ff / 32 * 2, d / 16, 1, s.n_cus) +
           resid(s.q_dim()) + resid(s.d_ff);
}
// From 256 rows on: the tile kernels where their heights fit the rows and the CUs, else the mix of LDS tiles and row groups (shape 5
// apart: it takes its place in either afterwards).
// Measured, prompts through 6 layers of the 4096-wide shape, ms: 260 rows 1.38 (tile kernels) against 1.19; 700 2.39 / 2.05;
// 1000 2.62 / 2.87; 1400 4.22 / 3.97; 2040 5.28 / 5.47; 1280-wide, 16 layers: 1000 rows 2.01 / 1.69, 2040 3.18 / 2.71.
inline bool tile_forward(const ProjShape &s, int M) {
    if (M < TILE_M || (s.kernel_flags & SJD_KERNELS_ROWGROUPS)) return false;
    if (s.kernel_flags & SJD_KERNELS_TILES) return true;
    return tile_layer_us(s, M) < norm_plan(s, M, s.qkv_groups()).us + norm_plan(s, M, s.d_ff / 32).us +
                                     resid_plan(s, M, s.q_dim()).us + resid_plan(s, M, s.d_ff).us;
}

struct ForwardPlan {
    bool tile;                             // every projection through the tile kernels, but QKV or gate/up of LDS tile shape 5
    ProjPlan qkv, o, gate_up, down, head;  // else each its own
};
// windows32: windows of 32 whose guidance branches the head combines, which needs both row tiles of a sequence in one wavefront
inline ForwardPlan forward_plan(const ProjShape &s, int M, bool windows32) {
    ForwardPlan f = {tile_forward(s, M), norm_plan(s, M, s.qkv_groups()), resid_plan(s, M, s.q_dim()), norm_plan(s, M, s.gate_up_groups()),
                     resid_plan(s, M, s.d_ff), norm_plan(s, M, s.head_groups())};
    if (f.tile) {
        f.qkv = {-1, 1, tile_us(M, s.qkv_groups() * 2, s.d_model / 16, 1, s.n_cus)};
        f.gate_up = {-1, 1, tile_us(M, s.gate_up_groups() * 2, s.d_model / 16, 1, s.n_cus)};
    }
    f.qkv = with_big(s, M, s.qkv_groups() * 2, f.qkv);
    f.gate_up = with_big(s, M, s.gate_up_groups() * 2, f.gate_up);
    if (f.head.lds >= 0 && windows32) f.head.lds = kLdsTileHeadZ;
    return f;
}

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
// gains nothing (2048 x 28672 x 4096 434 us against 430).  Shape 6 (QKV, whole-K output and down), eight wavefronts on 256 x 128 and a
// workgroup per CU as well, is for launches of one a CU that are long: 512 x 12288 x 4096 84 -> 66 us (128 x 64 tiles), 2048 x 4096 x
// 4096 86 -> 74 (128 x 128), x 14336 249 -> 220 (tile kernels, whose four wavefronts wait for LDS in turn).  Prompts of 512 to 2048 rows,
// 2048 to 5120 wide, 42 of them: 1.019 times in the geometric mean, 1.068 to 0.99.
#define SJD_LDS_TILES(X) X(0, 2, 2, 2, 1, 6) X(1, 4, 2, 4, 1, 6) X(2, 4, 4, 4, 2, 5) X(3, 6, 4, 2, 2, 4) X(4, 4, 4, 2, 2, 4) X(5, 8, 8, 2, 4, 4) X(6, 8, 4, 4, 2, 6)
constexpr int kLdsTiles = 4, kLdsTileHeadZ = 4, kLdsTileBig = 5, kLdsTileWide = 6;
// What a projection's epilogue is, as far as its time goes.
enum PlanEpi { PLAN_QKV = 0, PLAN_SWIGLU = 1, PLAN_RESID = 2, PLAN_PARTIAL = 3 };   // (the head: as SWIGLU)

// The expected times below are fits to launches one after the other over weights from HBM, models of 768, 1280, 2048, 3072 and 4096
// (grouped heads and not) at 66 to 2040 rows, 4 860 of them; the standard deviation of expected against measured is 5 to 9 % for
// the row groups and the LDS tiles, 11 % for the tile kernels.  Set by hand within that, so that near ties fall as whole forwards
// measured: t1, t2 and tn of shapes 2, 4 and 5, and the rates in tile_us().  Over those models and rows the four projections chosen take 1.018
// of the fastest launches' time in the geometric mean; with the rates measured before the kernels had their first arguments in
// registers, and one family of kernels for a whole layer, it was 1.047.
struct LdsTile { int tmt, tnb, cb; double t1, t2, tn, fixed[4], hbm, tflops; };
// t1, t2, tn: microseconds per pipeline stage of a CU with one workgroup, with two, and per workgroup of more; fixed: launch,
// first operands and epilogue; hbm: MB of weights per microsecond that a launch is held to; tflops: what it sustains at most (long
// launches run into the power limit; short ones, at higher clocks, do not)
inline LdsTile lds_tile(int cfg) {
    static const LdsTile t[7] = {{2, 2, 2, 0.142, 0.228, 0.109, {4.1, 3.5, 4.4, 4.6}, 3.83, 480}, {4, 2, 2, 0.166, 0.316, 0.167, {4.5, 3.5, 5.9, 5.1}, 4.28, 780},
                                 {4, 4, 2, 0.240, 0.511, 0.2634, {5.6, 3.9, 6.5, 5.7}, 4.75, 950}, {6, 4, 2, 0.305, 0.608, 0.328, {11.2, 7.8, 13.9, 6.2}, 4.38, 1090},
                                 {4, 4, 2, 0.240, 0.511, 0.2634, {5.6, 3.9, 6.5, 5.7}, 4.75, 950}, {8, 8, 2, 0.697, 1e3, 1e3, {11.5, 9.6, 0.0, 0.0}, 5.91, 1110},
                                 {8, 4, 2, 0.43, 1e3, 1e3, {13.5, 0.0, 16.3, 0.0}, 5.91, 1170}};
    return t[cfg];
}

// Time of an LDS-tile launch: stages x the busiest CU's workgroups (the column tiles of an XCD run on its CUs only).
inline double lds_us(int cfg, PlanEpi epi, int M, int n_blocks, int KB, int ks, int n_cus) {
    const LdsTile t = lds_tile(cfg);
    const int wgs_xcd = plan_div(plan_div(n_blocks, t.tnb), 8) * plan_div(M, 32 * t.tmt) * ks;
    const int n = plan_div(wgs_xcd, std::max(1, n_cus / 8));
    const double us = t.fixed[epi] + (double)plan_div(KB, 2 * ks) * (n == 1 ? t.t1 : n == 2 ? t.t2 : n * t.tn);
    // Launches of shape 3 from 0.3 TFLOP on sustain its rate over whole row tiles, and at no lower clocks as they grow: gate/up of 4096 and 5120 wide, 24
    // launches of 0.35 to 0.75 TFLOP, 1042 to 1100 TFLOP/s (1500 rows of 28672 x 4096 338 us, 1950 and 2048, 11 tiles of 192 both, 470 and 471; 1900 of
    // 35840 x 5120 659).  Shorter ones of all shapes were fitted with the rows that are asked for, and the choice among them holds
    // better with those: counted in whole tiles 61 prompts that would change took 1.017 times as long.
    const double flops = 1024.0 * M * n_blocks * KB, done = cfg == 3 && flops > 3e11 ? flops * plan_div(M, 192) * 192 / M : flops;
    return std::max({us, 4.0 + n_blocks * (KB * 1024.0) / (t.hbm * 1e6), t.fixed[epi] + done / (t.tflops * 1e6)});
}
// ... of a row-group launch (kernels_skinny.hip.h) over row groups of 32 mt rows and column groups of nbw blocks: a CU moves 65 GB/s
// of weights and activations, its workgroups but the first cost `more` each on top, and all CUs move 6 TB/s of weights
inline int skinny_per_cu(int M, int mt, int groups, int ks, int n_cus) {
    return plan_div(plan_div(groups, 8) * plan_div(M, 32 * mt) * ks, std::max(1, n_cus / 8));
}
inline double skinny_us(PlanEpi epi, int M, int mt, int groups, int nbw, int KB, int ks, int n_cus) {
    static const double fixed[4][2][2] = {{{4.6, 4.6}, {6.9, 6.9}}, {{4.1, 4.1}, {5.6, 5.6}}, {{2.8, 3.9}, {3.5, 5.7}}, {{5.1, 5.1}, {4.7, 6.0}}};   // [epilogue][mt - 1][nbw - 1]
    static const double more[2][2] = {{0.0, 1.0}, {1.5, 2.4}};
    const int n = skinny_per_cu(M, mt, groups, ks, n_cus);
    const double us = fixed[epi][mt - 1][nbw - 1] + (n - 1) * more[mt - 1][nbw - 1] + n * (double)(nbw + mt) * KB / ks * 1024.0 / 65e3;
    return std::max(us, 4.0 + (double)groups * nbw * KB * 1024.0 / 6e6);
}
// ... and what the kernel that adds ks partial sums of M rows of d columns adds to the launch before it (on its own it takes 2 us more, but with
// those in here the 33 forwards in which a K split then went were 2.7 % slower)
inline double reduce_us(int M, int d, int ks) { return 0.3 + (ks + 2.0) * M * d * 4.0 / 3.28e6; }

// ---- fp32
// Whether an fp32 projection that starts with a norm has it, and what follows, inside (gemm_f32_kernel) or as kernels of their own.  Inside
// saves two launches (QKV: norm and rotation, gate/up: norm and SwiGLU) or one (the head's norm), and costs every wavefront the norm of its
// rows and one multiplication more per four, so what it costs grows with the results, M x N.  The lines lie where neither way gains;
// steps and prompts of 2 layers, us, inside / apart: QKV of 240 rows of 256 91 / 98, 180 of 512 122 / 126 and 240 143 / 140, 60 of 2048
// 354 / 357 and 118 602 / 583; gate/up of 240 rows of 256 91 / 93 and 512 138 / 134, 180 of 512 122 / 120, 32 of 2048 215 / 225 and 118
// 602 / 599; head of 4096 ids, 512 wide, 32 rows 159 / 156 and 512 477 / 456, of 16384 ids, 512 rows of 64 307 / 234.
enum { F32_QKV_INSIDE = 320000, F32_GATE_UP_INSIDE = 480000, F32_HEAD_INSIDE = 160000 };
inline bool f32_inside(int M, int N, long results) { return (long)M * N <= results; }

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

// Time of a launch: 32-wide K stages x the busiest CU's tiles (the column tiles of an XCD run on its CUs only): 0.25 us a
// 128-row tile (0.33 alone on its CU), 0.47 a 256-row tile, 0.25 per 128 x 128 in a launch of both heights.  QKV projections, whose
// epilogue is the longest, take more (medians of 20 launches of 3072 to 5120 wide, all heads their own): 256-row tiles 0.60 (1700 and 1964
// rows of 4096 250 and 268 us, 1300 and 1900 of 5120 310 and 352), 128-row tiles 0.27 (1300 rows of 4096 185, 1700 of 5120 314), both heights 0.34 (1300 and
// 1600 rows of 3072 126 and 137).  With the rates of the others, which expected 195 us of 268, 4096 wide prompts took 7 to 8 % longer
// than with 128 x 128 LDS tiles (1964 rows, 226 us) or 192 x 128 (1300 rows, 153).
inline bool tile_two_heights(int M, int n_blocks, int ksplit, int n_cus) {
    const int col_tiles = (n_blocks + 3) / 4, rt2 = (M + 255) / 256, rt1 = (M + 127) / 128;
    return ksplit == 1 && rt1 > rt2 && col_tiles * rt2 > n_cus && col_tiles * rt2 < 2 * n_cus && n_cus / rt2 >= 8 && (col_tiles * rt1) % n_cus != 0;
}
inline double tile_us(PlanEpi epi, int M, int n_blocks, int KB, int ksplit, int n_cus) {
    static const double fixed[4] = {16.8, 7.2, 22.1, 5.4};
    const int col_tiles = (n_blocks + 3) / 4, rows = tile_rows_for(M, n_blocks, ksplit, n_cus);
    const double stages = KB / (2.0 * ksplit);
    if (tile_two_heights(M, n_blocks, ksplit, n_cus)) {
        const int rt2 = (M + 255) / 256, ct_split = n_cus / rt2 / 8 * 8;
        return fixed[epi] + stages * (epi == PLAN_QKV ? 0.34 : 0.25) * (2.0 * ct_split * rt2 + (double)(col_tiles - ct_split) * ((M + 127) / 128)) / n_cus;
    }
    const int per_xcd = (col_tiles + 7) / 8 * ((M + rows - 1) / rows) * ksplit, cus = n_cus >= 8 ? n_cus / 8 : 1, n = (per_xcd + cus - 1) / cus;
    return fixed[epi] + stages * (rows == 256 ? (epi == PLAN_QKV ? 0.60 : 0.465) * n : n == 1 ? 0.328 : (epi == PLAN_QKV ? 0.27 : 0.25) * n);
}

// ---- the choice
inline int resid_nbw(int d) { return plan_div(d, 32) >= 128 ? 2 : 1; }   // column blocks per workgroup of an output / down projection
// More than 32 rows and so few column groups that a workgroup per group and 32-row tile still finds a CU of its own
inline bool rows_of_32(const ProjShape &s, int M, int groups) {
    return M > 32 && 2 * plan_div(M, 64) * 8 * plan_div(groups, 8) <= s.n_cus && !(s.kernel_flags & SJD_NO_ROW_SPLIT);
}

// ---- few rows (kernels_few.hip.h): 16-row tiles of a workgroup, 0 where the row-group kernels run.  Wherever two workgroups per column
// group and 16 or 32 rows still find a CU each; 64 rows of 1280 x 6912 (gate/up), 432 workgroups, took 2 % of a step more than 216
// of whole groups.  (SJD_NO_ROW_SPLIT: all rows in one workgroup; the same sums together with SJD_NO_K_ROTATION, since a workgroup's number
// says where its k starts.)
inline int few_wgs(int M, int groups, int rt) { return 16 * plan_div(groups, 8) * plan_div(M, 16 * rt); }
inline int few_rows(const ProjShape &s, int M, int groups) {
    if (M > 64) return 0;
    const int rt = few_wgs(M, groups, 1) <= s.n_cus ? 1 : few_wgs(M, groups, 2) <= s.n_cus ? 2 : 0;
    return rt && (s.kernel_flags & SJD_NO_ROW_SPLIT) ? (M <= 16 ? 1 : M <= 32 ? 2 : 4) : rt;
}
// How a projection runs: row groups (lds < 0, not tile), LDS tiles of shape `lds`, or the tile kernels; ks: splits of
// K (output / down projections, whose partial sums resid_reduce_kernel adds); us: its expected time, on which the choice rests.
struct ProjPlan { int lds, ks; double us; bool tile = false; };
inline int tile_splits(const ProjShape &s, int M, int KB) {   // K splits of an output / down projection through the tile kernels
    int ks = std::min(8, std::max(1, s.n_cus / (plan_div(plan_div(s.d_model, 64) * 2, 4) * plan_div(M, TILE_M))));
    while (ks > 1 && KB / ks < 32) --ks;
    return plan_div(KB, plan_div(KB, ks));
}
// The better of p and the kernels for more rows than a row group's
inline ProjPlan with_tiles(const ProjShape &s, PlanEpi epi, int M, int n_blocks, int KB, ProjPlan p, bool tile_kernels) {
    if (M <= 64 || (s.kernel_flags & SJD_KERNELS_ROWGROUPS)) return p;
    const bool resid = epi == PLAN_RESID;
    auto reduced = [&](int ks) { return ks > 1 ? reduce_us(M, s.d_model, ks) : 0.0; };
    auto kind = [&](int ks) { return ks > 1 ? PLAN_PARTIAL : epi; };
    for (int cfg = 0; cfg < kLdsTiles; ++cfg)
        for (int ks = 1; ks <= (resid ? 4 : 1); ks *= 2) {
            if (ks > 1 && KB / ks < 32) continue;
            const double t = lds_us(cfg, kind(ks), M, n_blocks, KB, ks, s.n_cus) + reduced(ks);
            if (t < p.us) p = {cfg, ks, t};
        }
    if (M < TILE_M) return p;
    const int ks = resid ? tile_splits(s, M, KB) : 1;
    const double t = tile_us(kind(ks), M, n_blocks, KB, ks, s.n_cus) + reduced(ks);
    if (tile_kernels && (t < p.us || (s.kernel_flags & SJD_KERNELS_TILES))) p = {-1, ks, t, true};
    if (!resid && !(s.kernel_flags & SJD_KERNELS_TILES)) {
        const double big = lds_us(kLdsTileBig, epi, M, n_blocks, KB, 1, s.n_cus);
        if (big < p.us) p = {kLdsTileBig, 1, big};
    }
    // Shape 6 in place of the tile kernels' output and down projections: 2000 rows of 4096, K = 14336 249 -> 220 us; prompts of 4096 wide with
    // MLPs of 5728 to 8032, 1926 to 2042 rows, 13 of them: 0.970 to 0.985 of the time.  (A line at K = 2 d kept these in the tile kernels, and at
    // 1.75 d to 2 d the whole layer left them for it: MLP 8032, 1980 rows 3478 us, without the line 3376.)  Such projections have been compared from
    // 1154 rows on: 12 prompts of 5120 wide, 1164 to 1278 rows, were 1.02 to 1.06 times faster with it.
    if ((epi == PLAN_QKV || (resid && M > 1024)) && !(s.kernel_flags & SJD_KERNELS_TILES)) {
        const double t = lds_us(kLdsTileWide, epi, M, n_blocks, KB, 1, s.n_cus);
        if (t < p.us) p = {kLdsTileWide, 1, t};
    }
    return p;
}
inline int skinny_mt(const ProjShape &s, int M, int groups) { return M <= 32 || rows_of_32(s, M, groups) ? 1 : 2; }   // 32-row tiles per row group
// Whether launch p of an output / down projection has CUs to spare for touching the next projection's weights (32 at least; no more
// weights than the L2s hold)
inline bool warms(const ProjShape &s, int M, const ProjPlan &p, size_t next_bytes) {
    if (p.lds >= 0 || p.tile || p.ks > 1 || (s.kernel_flags & SJD_NO_L2_WARM)) return false;
    const int groups = plan_div(plan_div(s.d_model, 32), resid_nbw(s.d_model));
    return s.n_cus - 8 * plan_div(groups, 8) * plan_div(M, 32 * skinny_mt(s, M, groups)) >= 32 && next_bytes <= (size_t)24 << 20;
}
// Row groups as a choice.  Beyond 512 rows and one workgroup per CU their many short workgroups take far longer than the bytes
// they move say (1434 rows of 512, output projection in row groups of 32: 11.3 us, expected 5.8): not there, except where the flag asks.
// With a workgroup per CU at most they are the better kernels of narrow models at any number of rows (prompts through 12 layers with LDS
// tiles in their place: 743 rows of 256 361 -> 422 us, 558 of 512 430 -> 457, 637 of 384 397 -> 412).
inline ProjPlan row_groups(const ProjShape &s, PlanEpi epi, int M, int mt, int groups, int nbw, int KB, int ks) {
    if (M > 512 && skinny_per_cu(M, mt, groups, ks, s.n_cus) > 1 && !(s.kernel_flags & SJD_KERNELS_ROWGROUPS)) return {-1, ks, 1e9};
    return {-1, ks, skinny_us(epi, M, mt, groups, nbw, KB, ks, s.n_cus) + (ks > 1 ? reduce_us(M, s.d_model, ks) : 0.0)};
}
// QKV, gate/up: groups of two column blocks, whole K.  Row groups of a CU each whose weights the launch before has touched take
// about 0.82 of the time (LDS tiles gain a tenth or nothing): 1024 wide, MLP of 3584, 71 and 128 prompt rows, gate/up in row groups 415
// and 419 us, in LDS tiles 440 and 435.
inline ProjPlan norm_plan(const ProjShape &s, PlanEpi epi, int M, int groups, bool tile_kernels, const ProjPlan &before) {
    const int KB = s.d_model / 16, mt = skinny_mt(s, M, groups);
    ProjPlan p = row_groups(s, epi, M, mt, groups, 2, KB, 1);
    if (skinny_per_cu(M, mt, groups, 1, s.n_cus) == 1 && warms(s, M, before, (size_t)groups * 64 * s.d_model * 2)) p.us *= 0.82;
    return with_tiles(s, epi, M, groups * 2, KB, p, tile_kernels);
}
inline ProjPlan resid_row_groups(const ProjShape &s, int M, int K) {
    const int d = s.d_model, KB = K / 16, nbw = resid_nbw(d), groups = plan_div(plan_div(d, 32), nbw);
    int mt = skinny_mt(s, M, groups), ks = 1;
    if ((double)(nbw + mt) * KB * 1024.0 > 512e3 && (M <= 64 || nbw > 1)) {   // one workgroup's share is too much for its CU
        mt = M <= 32 ? 1 : 2;
        ks = std::min(8, std::max(1, s.n_cus / (groups * plan_div(M, 64))));
        while (ks > 1 && KB / ks < 32) --ks;
        ks = plan_div(KB, plan_div(KB, ks));
    }
    return row_groups(s, ks > 1 ? PLAN_PARTIAL : PLAN_RESID, M, mt, groups, nbw, KB, ks);
}
inline ProjPlan resid_plan(const ProjShape &s, int M, int K, bool tile_kernels) {
    return with_tiles(s, PLAN_RESID, M, plan_div(s.d_model, 32), K / 16, resid_row_groups(s, M, K), tile_kernels);
}

// K splits of an output / down projection at most, whatever is chosen
inline int max_splits(const ProjShape &s, int M, int K) {
    const int KB = K / 16, groups = plan_div(plan_div(s.d_model, 32), resid_nbw(s.d_model));
    int ks = KB >= 32 ? std::min(std::min(8, KB / 32), std::max(1, s.n_cus / (groups * plan_div(M, 64)))) : 1;
    if (M > 64) ks = std::max(ks, KB >= 128 ? 4 : KB >= 64 ? 2 : 1);
    return M >= TILE_M ? std::max(ks, tile_splits(s, M, KB)) : ks;
}

struct ForwardPlan {
    bool tile;                             // some projection runs through the tile kernels, and so does the head
    ProjPlan qkv, o, gate_up, down, head;
};
// windows32: windows of 32 whose guidance branches the head combines, which needs both row tiles of a sequence in one wavefront
inline ForwardPlan layer_plan(const ProjShape &s, int M, bool tile_kernels) {
    ForwardPlan f{};
    // An output / down projection in row groups touches the weights of the projection behind it, which gains by that: row groups where the
    // two together are expected to take 3 % less.  70 prompt rows of 1280: down 9.6 us against 9.4 in LDS tiles, QKV then 6.9 against 8.4;
    // 12 layers 469 -> 418 us, 86 rows of 640 396 -> 363.  (Below 3 % the other side was faster: 88 rows of 2048 193 against 204 us.)
    auto pair = [&](int K, ProjPlan &first, PlanEpi epi, int groups, ProjPlan &next) {
        first = resid_plan(s, M, K, tile_kernels);
        next = norm_plan(s, epi, M, groups, tile_kernels, first);
        if (s.kernel_flags & SJD_KERNELS_TILES) return;
        const ProjPlan rg = resid_row_groups(s, M, K), after_rg = norm_plan(s, epi, M, groups, tile_kernels, rg);
        if (rg.us + after_rg.us < 0.97 * (first.us + next.us)) { first = rg; next = after_rg; }
    };
    pair(s.q_dim(), f.o, PLAN_SWIGLU, s.gate_up_groups(), f.gate_up);
    pair(s.d_ff, f.down, PLAN_QKV, s.qkv_groups(), f.qkv);
    f.tile = f.qkv.tile || f.o.tile || f.gate_up.tile || f.down.tile;
    return f;
}
inline double layer_us(const ForwardPlan &f) { return f.qkv.us + f.o.us + f.gate_up.us + f.down.us; }
inline ForwardPlan forward_plan(const ProjShape &s, int M, bool windows32) {
    // The tile kernels are a third set of kernels for the same rows: only where a layer is expected to gain 2 % by them, which is
    // where the fits tell the sets apart (2000 rows of 1280: expected 0.4 % less, 8 % more as whole prompts; 34 prompts of 2560 to 5120 wide, 396 to 2044 rows,
    // that were expected to gain 1.5 to 2 %: 28 of them slower through the tile kernels, all in the mean by 1.3 %, 5.8 % at most), and 8 % in narrow models
    // whose gate/up takes less than 85 us: the fits have launches one by one, and so short ones lose more beside their neighbours than
    // that (84 forwards of 256 to 2040 rows that were expected to gain 2 to 10 %: below 3072 wide and 85 us 42 of 49 were slower, by 2.3 %
    // in the mean; the other 35 were 1.4 % faster).
    ForwardPlan f = layer_plan(s, M, (s.kernel_flags & SJD_KERNELS_TILES) != 0);
    if (M >= TILE_M && !(s.kernel_flags & (SJD_KERNELS_ROWGROUPS | SJD_KERNELS_TILES))) {
        const ForwardPlan g = layer_plan(s, M, true);
        if (layer_us(g) < (s.d_model >= 3072 || g.gate_up.us >= 85.0 ? 0.98 : 0.92) * layer_us(f)) f = g;
    }
    const int groups = s.head_groups(), mt = skinny_mt(s, M, groups);
    f.head = {-1, 1, skinny_us(PLAN_SWIGLU, M, mt, groups, 2, s.d_model / 16, 1, s.n_cus)};
    // (by its own time in such forwards, and with weights touched ahead in them: 0.1 % over 60, 2 % at best)
    if (f.tile) f.head = {-1, 1, tile_us(PLAN_SWIGLU, M, groups * 2, s.d_model / 16, 1, s.n_cus), true};
    if (!f.tile && M > 64 && !(s.kernel_flags & SJD_KERNELS_ROWGROUPS))
        for (int cfg = 0; cfg < kLdsTiles; ++cfg) {
            const double t = lds_us(cfg, PLAN_SWIGLU, M, groups * 2, s.d_model / 16, 1, s.n_cus);
            if (t < f.head.us) f.head = {cfg, 1, t};
        }
    if (f.head.lds >= 0 && windows32) f.head.lds = kLdsTileHeadZ;
    return f;
}

// ---- touching weights ahead
// Launches of row groups and LDS tiles carry workgroups that touch the weights of the projection behind them, so that those are in the
// L2 of the XCD that will read them (the launches are short and latency-bound, and the chip is mostly idle).
// Computing workgroups of a launch: LDS tiles over n_blocks column blocks, row groups over `groups` column groups
inline int lds_wgs(int cfg, int M, int n_blocks) {
    const LdsTile t = lds_tile(cfg);
    return 8 * plan_div(plan_div(n_blocks, t.tnb), 8) * plan_div(M, 32 * t.tmt);
}
inline int row_group_wgs(int M, int groups, bool rows32) {
    const int m_groups = plan_div(M, 64);
    if (rows32) return 2 * m_groups * 8 * plan_div(groups, 8);
    return m_groups > 1 ? m_groups * 8 * plan_div(groups, 8) : groups;
}
// What the launch before needs to know about a projection: n slabs (its column tiles) of nbw column blocks x KB k-blocks
struct Slabs { int n, nbw, KB; bool whole, lds; };
inline Slabs slabs_of(const ProjPlan &p, int n_blocks, int KB, int nbw) {
    if (p.lds < 0) return {plan_div(n_blocks, nbw), nbw, KB, p.ks == 1, false};
    const int tnb = lds_tile(p.lds).tnb;
    return {n_blocks / tnb, tnb, KB, p.ks == 1, true};   // whole tiles only: a ragged last one ends with the matrix
}
// Workgroups that a launch of cur_wgs, expected to take cur_us, carries, and how many of the next launch's slabs they touch.
// LDS tiles gain about 1 us where their weights are touched ahead, which a launch of less than 12 us loses and more (500
// rows of 1280: output projection 11.5 -> 14.8 us, gate/up 15.3 -> 14.0; 948 rows: 18.7 -> 18.2 and 25.0 -> 23.2).
struct Touch { int wgs, slabs; };
inline Touch touch(const ProjShape &s, int M, int cur_wgs, double cur_us, const Slabs &next) {
    if (!next.whole || (next.lds && cur_us < 12.0)) return {0, 0};
    const size_t slab = (size_t)next.nbw * next.KB * 1024;
    int fit = (int)std::min<size_t>(next.n, ((size_t)24 << 20) / slab);   // what the L2s hold beside the current weights
    int wgs = (int)((fit * slab / (96 << 10) + 7) / 8 * 8);
    wgs = std::min(wgs, (s.n_cus - cur_wgs) / 8 * 8);
    if (wgs < 8 || (M > 64 && wgs < 32)) return {0, 0};   // long-window launches: a handful of CUs only delays them
    // few CUs left: touch no more than they get through while the launch computes (a CU streams ~45 GB/s from
    // HBM, the launches take 7-10 us: 320 KB each), the first slabs
    fit = (int)std::min<size_t>(fit, (size_t)wgs * (320 << 10) / slab);
    return fit < 1 ? Touch{0, 0} : Touch{wgs, fit};
}

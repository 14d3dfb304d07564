// Projections of at most 64 rows whose column groups number so few that a workgroup per group leaves most CUs idle: the
// row-group kernels (kernels_skinny.hip.h) with a column group split over two workgroups, 16 columns of each of its blocks, and
// the rows over groups of 16 or 32, on v_mfma_f32_16x16x32_bf16.  8 wavefronts take the steps of 32 k round-robin and meet in LDS.
//
// What bounds it: a CU's share of the operands.  A CU has some 36 KB of reads under way at most, 38 - 45 GB/s of weights that come from
// HBM; its wavefronts' first operands arrive 1.1 - 1.5 us after the start.  So the bytes of a workgroup are what counts, not those
// of the launch: 32 rows of the 1280-wide model (MLP 3456) in 240, 160, 216 and 160 workgroups of 123, 82, 164 and 221 KB (QKV,
// output, gate/up, down) take 4.5, 2.6, 5.5 and 5.5 us from the first workgroup's start to the last one's end, without workgroups that touch
// the next launch's weights.  In 120, 80, 108 and 80 workgroups beside such (the row-group kernels) they took 4.3, 3.4, 4.5 and
// 5.0 and 0.4 us more between two launches, and the launch in front of each was longer by the touching.
// Steps of that model, 36 layers: window 16 1.137 -> 1.091 ms, window 1 behind a 120-token prompt 1.14 -> 1.06; 66 steps of models of 512
// to 4096, 2 to 64 rows: 1.07 times in the geometric mean, none slower (2048 wide, 2 rows 308 -> 272 us; 3072 wide, 64 rows 518 -> 515).
// Touching weights ahead beside these kernels costs what it gains or more: over 48 divisions of the idle CUs' time between the five launches
// of a layer the 32-row step took 1.081 to 1.170 ms, 1.083 to 1.099 without.  (With all layers' weights in the memory-side cache
// touching would pay, 1.053 -> 0.985 ms.)  Keys and values are touched by the launch ahead of the attention as before.
// That holds where the launch behind is one of row groups that finds its weights cold, too (gate/up of 33 to 64 rows: 7.4 us where the output projection's
// launch touched them, now 9.1).  Steps with 48 to 200 KB of them touched by each CU that the output projection leaves idle: 1280 wide, 64 rows 1183 -> 1208 to
// 1227 us, 40 rows 1188 -> 1196 to 1295; 1536 wide, 64 rows 992 -> 999 to 1072; 1024 wide (MLP 5632), 16 rows 758 -> 811 to 822; 2048 wide, 16 rows 991 ->
// 1031 to 1060, 64 rows 1302 to 1322 -> 1295 to 1338; 1024 wide (MLP 2816), 64 rows 708 -> 703 to 709.
// Error of the logits against float64 (tests/test_gpu_few_rows.py, 9 models, 22 sequences and branches): 0.9995 of the row-group kernels' in the
// geometric mean, 0.977 to 1.008.
// Five steps of loads are under way per wavefront: 2, 3 and 4 take 1 - 2 % longer, 7, 10 and 14 (down) 1 - 2 % as well.
#pragma once
#include "kernels_skinny.hip.h"

typedef float acc16_t __attribute__((ext_vector_type(4)));

// RT: 16-row tiles of a workgroup; NBW: column blocks of a group, of each of which the workgroup takes 16 columns.  Epilogues, norm
// (gains in the weights or, ROWS, in the rows) and the order of k as in the row-group kernels.
template <int RT, int NBW, int EPI, bool ROWS>
__global__ __launch_bounds__(512) void gemm_few_kernel(SJD_HOT_PARAMS, SkinnyArgs a) {
    SJD_HOT_TAKE(a);
    constexpr int NW = 8, DEPTH = 5;
    constexpr bool kNorm = EPI != EPI_RESID;
    constexpr bool kSsqLoop = kNorm && !ROWS;
    static_assert(EPI == EPI_RESID || ((EPI == EPI_QKV || EPI == EPI_SWIGLU) && NBW == 2), "epilogues of whole-K projections");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // id = 8 j + x is entry j of XCD x's list: group g = x + 8 (j / (2 m_groups)), of which all column halves and row groups
    // follow each other
    const int per = 2 * a.m_groups, n_compute = 8 * ((a.groups + 7) / 8) * per;
    if ((int)blockIdx.x >= n_compute) {
        l2_warm_kv(a, blockIdx.x, n_compute, tid, NW * 64);
        return;
    }
    const int j = blockIdx.x >> 3, g = (blockIdx.x & 7) + 8 * (j / per), sub = j % per, ch = sub & 1, mg = sub >> 1;
    if (g >= a.groups) return;
    const int KB = a.KB, m_base = mg * RT * 16, blk0 = g * NBW;
    // operands of the MFMA, 16 rows (columns of the product) x 32 k, out of two 32-row fragments: lane l holds row l % 16, k from
    // 8 (l / 16) on; every 16 lanes read 256 contiguous bytes
    const int off = ((lane >> 5) * 64) + ((lane >> 4) & 1) * 32 + (lane & 15);
    const u32x4 *Wp = reinterpret_cast<const u32x4 *>(a.W) + (size_t)blk0 * KB * 64 + ch * 16 + off;
    const u32x4 *Ap[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) Ap[r] = reinterpret_cast<const u32x4 *>(a.A) + (size_t)((m_base + 16 * r) >> 5) * KB * 64 + (((m_base + 16 * r) >> 4) & 1) * 16 + off;
    const int n_k = KB >> 1;   // steps of 32 k; wavefront w takes w, w + NW, ...
    const int n_it = wave < n_k ? (n_k - wave + NW - 1) / NW : 0;
    const int rot = n_it > 0 ? (int)(((blockIdx.x >> 3) * (unsigned)a.k_rot) % (unsigned)n_it) : 0;
    auto k_of = [&](int it) {
        const int r = it + rot;
        return (size_t)(wave + (r >= n_it ? r - n_it : r) * NW) * 128;
    };

    // What a thread stores: accumulator register v = u % 4 of row tile u / 4, u = wave, wave + NW, ...: row 4 (l / 16) + v of the
    // tile, column l % 16 of each block's half
    constexpr int NU = 4 * RT, EPT = (NU + NW - 1) / NW;
    const int col = ch * 16 + (lane & 15);
    auto row_of = [&](int i) { const int u = wave + NW * i; return 16 * (u >> 2) + 4 * (lane >> 4) + (u & 3); };
    [[maybe_unused]] float xpre[EPT][NBW];
    float gpre[NBW];
    [[maybe_unused]] QkvRow qrow[EPT];
    [[maybe_unused]] float rot_c[EPT], rot_s[EPT];
    auto request_epilogue = [&]() {
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            gpre[i] = 1.0f;
            if constexpr (EPI == EPI_RESID && ROWS)
                if (const int n = (blk0 + i) * 32 + col; n < a.N) gpre[i] = a.gain[n];
        }
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int m = m_base + row_of(e);
            const bool mine = wave + NW * e < NU && m < a.M;
            if constexpr (EPI == EPI_RESID) {
#pragma unroll
                for (int i = 0; i < NBW; ++i) {
                    const int n = (blk0 + i) * 32 + col;
                    xpre[e][i] = mine && n < a.N ? a.x[(size_t)m * a.N + n] : 0.0f;
                }
            } else if constexpr (EPI == EPI_QKV) {
                qrow[e].pos = -1;
                rot_c[e] = 1.0f;
                rot_s[e] = 0.0f;
                if (mine) {
                    qrow[e] = qkv_row(a, m);
                    qkv_rotation(a, m, g, col, rot_c[e], rot_s[e]);
                }
            }
        }
    };

    acc16_t acc[RT][NBW];
    float ssq[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        ssq[r] = 0.0f;
#pragma unroll
        for (int i = 0; i < NBW; ++i) acc[r][i] = acc16_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
    if (n_it > 0) {
        u32x4 bq[DEPTH][NBW], aq[DEPTH][RT];
        auto load = [&](int s, int it) {
            const size_t k = k_of(it);
#pragma unroll
            for (int i = 0; i < NBW; ++i) bq[s][i] = __builtin_nontemporal_load(Wp + (size_t)i * KB * 64 + k);
#pragma unroll
            for (int r = 0; r < RT; ++r) aq[s][r] = Ap[r][k];
        };
        auto consume = [&](int s) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const bf16x8 av = __builtin_bit_cast(bf16x8, aq[s][r]);
                if (kSsqLoop) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t pr = aq[s][r][e];
                        const float lo = __builtin_bit_cast(float, pr << 16), hi = __builtin_bit_cast(float, pr & 0xFFFF0000u);
                        ssq[r] = fmaf(lo, lo, ssq[r]);
                        ssq[r] = fmaf(hi, hi, ssq[r]);
                    }
                }
#pragma unroll
                for (int i = 0; i < NBW; ++i) acc[r][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bq[s][i]), acc[r][i], 0, 0, 0);
            }
        };
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) load(s, s < n_it ? s : n_it - 1);
        __builtin_amdgcn_sched_barrier(0);
        request_epilogue();
        __builtin_amdgcn_sched_barrier(0);
        int it0 = 0;
        for (; it0 + 2 * DEPTH <= n_it; it0 += DEPTH) {
#pragma unroll
            for (int s = 0; s < DEPTH; ++s) {
                consume(s);
                load(s, it0 + s + DEPTH);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            if (it0 + s < n_it) {
                consume(s);
                if (it0 + s + DEPTH < n_it) load(s, it0 + s + DEPTH);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int s = 0; s < DEPTH; ++s)
            if (it0 + DEPTH + s < n_it) consume(s);
    } else {
        request_epilogue();
    }

    // the wavefronts' partial tiles, a register of 64 lanes at a time (no bank conflicts)
    __shared__ float red[NW][RT * NBW][4][64];
    __shared__ float ssq_lds[NW][RT * 16];
    if (kNorm) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            float t;
            if constexpr (kSsqLoop) {
                t = ssq[r] + __shfl_xor(ssq[r], 16, 64);
                t += __shfl_xor(t, 32, 64);
            } else {
                const int m = m_base + 16 * r + (lane & 15);
                t = m < a.M ? row_ssq_sum(a, m, wave, NW) : 0.0f;
            }
            if (lane < 16) ssq_lds[wave][16 * r + lane] = t;
        }
    }
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int i = 0; i < NBW; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][r * NBW + i][v][lane] = acc[r][i][v];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int u = wave + NW * e;
        if (u >= NU) continue;
        const int row = row_of(e), m = m_base + row;
        float vals[NBW], inv = 1.0f;
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            float t = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) t += red[w][(u >> 2) * NBW + i][u & 3][lane];
            vals[i] = t;
        }
        if (kNorm) {
            float t = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) t += ssq_lds[w][row];
            inv = 1.0f / sqrtf(t / (float)(KB * 16) + a.eps);
        }
        if (m >= a.M) continue;
        if constexpr (EPI == EPI_QKV) {
            qkv_store<true>(a, qrow[e], g, col, vals[0] * inv, vals[NBW - 1] * inv, rot_c[e], rot_s[e]);
        } else {
            float xin[NBW];
#pragma unroll
            for (int i = 0; i < NBW; ++i) xin[i] = EPI == EPI_RESID ? xpre[e][i] : 0.0f;
            skinny_epilogue<EPI, NBW>(a, 0, m, blk0, col, vals, inv, xin, gpre);
            if constexpr (EPI == EPI_RESID) {
                if (a.ssq_out) {   // the row's columns of this half group lie in a quarter wavefront
                    float sq = 0.0f;
#pragma unroll
                    for (int i = 0; i < NBW; ++i) {
                        const float f = (blk0 + i) * 32 + col < a.N ? ssq_value<ROWS>(xin[i] + vals[i]) : 0.0f;
                        sq = fmaf(f, f, sq);
                    }
#pragma unroll
                    for (int o = 8; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
                    if ((lane & 15) == 0) a.ssq_out[(size_t)(2 * g + ch) * a.M + m] = sq;
                }
            }
        }
    }
}

template <int RT, int EPI, bool ROWS>
inline hipError_t launch_few_rt(hipStream_t st, const SkinnyArgs &a, int grid) {
    constexpr int NBW = EPI == EPI_RESID ? 1 : 2;
    gemm_few_kernel<RT, NBW, EPI, ROWS><<<grid, 512, 0, st>>>(SJD_HOT_PASS(a), a);
    return hipGetLastError();
}
// rt: 16-row tiles of a workgroup (1, 2 or 4); groups: column groups of one block (RESID) or two
template <int EPI>
inline hipError_t launch_few(hipStream_t st, const SkinnyArgs &a_in, int rt, int groups) {
    SkinnyArgs a = a_in;
    if (a.M <= 0 || a.M > 64 || groups <= 0 || (a.KB & 1) || a.ksplit != 1) return hipErrorInvalidValue;
    a.groups = groups;
    a.m_groups = ceil_div(a.M, 16 * rt);
    const int grid = 8 * ceil_div(groups, 8) * 2 * a.m_groups + a.kv_wgs;
    const bool rows = EPI == EPI_RESID ? a.gain != nullptr : a.row_ssq_part != nullptr;
    switch (rt) {
    case 1: return rows ? launch_few_rt<1, EPI, true>(st, a, grid) : launch_few_rt<1, EPI, false>(st, a, grid);
    case 2: return rows ? launch_few_rt<2, EPI, true>(st, a, grid) : launch_few_rt<2, EPI, false>(st, a, grid);
    case 4: return rows ? launch_few_rt<4, EPI, true>(st, a, grid) : launch_few_rt<4, EPI, false>(st, a, grid);
    }
    return hipErrorInvalidValue;
}

// Projections of the fp32 forward with the element-wise steps around them inside: RMSNorm of the rows ahead of the product,
// rotation and cache write, SwiGLU or the residual sum behind it.
//
// Same sums as the kernels they stand for (gemm_reference_kernel, addnorm_kernel, rope_kv_kernel, swiglu_kernel), bit for bit:
// every product in gemm_reference_kernel's order of k and lanes, a row's sum of squares in addnorm_kernel's (256 strided
// threads, lanes 32, 16, ..., 1 apart, then the four wavefronts), every element rounded where they round it.
//
// Bound: a step of the fp32 model is a chain of short dependent launches (2 layers of 256: 4 us each whatever they do), so what
// counts is their number, nine a layer before and five now (where results are many, the norm and what follows are on their own again:
// f32_inside, plans.h).  The four wavefronts of a workgroup share the sums of squares of their
// eight rows, two rows each: 10 exchanges and a barrier.
#pragma once
#include "kernels_attention.hip.h"
#include "kernels_gemm.hip.h"

enum { F32_QKV = 0, F32_RESID = 1, F32_SWIGLU = 2, F32_LOGITS = 3 };

struct F32Args {
    int M, N, K;            // N: columns of W
    const float *gain;      // RMSNorm of the rows of A (QKV, SWIGLU, LOGITS)
    float eps;
    float *out;             // RESID: the stream, added to; SWIGLU: [M][N / 2]; LOGITS: [M][N]
    // QKV
    RowMap rm;
    const float *rope_cos, *rope_sin;
    float *q_out;
    KvPool pool;
    int L, H, Hkv, hd;
};

// One wavefront per (8 rows, NC columns), as gemm_reference_kernel.  QKV and SWIGLU work on pairs of columns (a rotary pair of a
// head, a gate and its up): a wavefront has NC / 2 pairs, first members in the lower half of its columns, so that a pair ends up
// in lanes 32 apart.
template <int NC, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ A, const float *__restrict__ W, F32Args a) {
    constexpr bool kNorm = EPI != F32_RESID, kPair = EPI == F32_QKV || EPI == F32_SWIGLU;
    static_assert(!kPair || NC % 2 == 0, "pairs of columns");
    constexpr int U = 4, NV = 8 * NC, NP = NC / 2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int M = a.M, N = a.N, K = a.K;
    const int unit = blockIdx.x * (blockDim.x >> 6) + wave;   // of NC columns
    const int m0 = blockIdx.y * 8;
    const int half = a.hd >> 1, n_pairs = N >> 1;
    // column c of this wavefront (past the end: the last one, never stored)
    auto column = [&](int c) -> int {
        if constexpr (!kPair) return min(unit * NC + c, N - 1);
        const int p = min(unit * NP + c % NP, n_pairs - 1);
        if constexpr (EPI == F32_SWIGLU) return p + (c >= NP ? n_pairs : 0);
        return p / half * a.hd + p % half + (c >= NP ? half : 0);
    };
    const float *wrow[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) wrow[c] = W + (size_t)column(c) * K;
    auto load = [&](int k, float (&av)[8], float (&wv)[NC], float &g) {
#pragma unroll
        for (int c = 0; c < NC; ++c) wv[c] = wrow[c][k];
        if constexpr (kNorm) g = a.gain[k];
#pragma unroll
        for (int j = 0; j < 8; ++j) av[j] = A[(size_t)min(m0 + j, M - 1) * K + k];
    };
    float acc[NV];   // [column][row]
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0f;
    float inv[8];
    auto add = [&](const float (&av)[8], const float (&wv)[NC], float g) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x[j] = av[j];
            if constexpr (kNorm) x[j] = av[j] * inv[j] * g;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[c * 8 + j] = fmaf(x[j], wv[c], acc[c * 8 + j]);
    };
    // the first four rounds are in flight while the sums of squares are taken
    float av[U][8], wv[U][NC], g[U];
    int k = lane;
    const bool full = 64 * U <= K;
    if (full) {
#pragma unroll
        for (int u = 0; u < U; ++u) load(k + 64 * u, av[u], wv[u], g[u]);
    }
    if constexpr (kNorm) {
        __shared__ float row_inv[8];
        float s[8];   // [thread group of 64 of 256][row 2 wave, 2 wave + 1]
#pragma unroll
        for (int v = 0; v < 8; ++v) s[v] = 0.0f;
        for (int k0 = 0; k0 < K; k0 += 256) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = A[(size_t)min(m0 + 2 * wave + (i & 1), M - 1) * K + min(k0 + 64 * (i >> 1) + lane, K - 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (k0 + 64 * (i >> 1) + lane < K) s[i] = fmaf(v[i], v[i], s[i]);
        }
        (void)add_lanes<32, 8>(s, lane, 0);   // lane l: thread group l / 16, row (l / 8) % 2
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) t += __shfl(s[0], w * 16 + (lane & 8), 64);
        if ((lane & ~8) == 0) row_inv[2 * wave + (lane >> 3)] = 1.0f / sqrtf(t / (float)K + a.eps);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; ++j) inv[j] = row_inv[j];
    }
    if (full) {
#pragma unroll
        for (int u = 0; u < U; ++u) add(av[u], wv[u], g[u]);
        k += 64 * U;
    }
    for (; k - lane + 64 * U <= K; k += 64 * U) {
#pragma unroll
        for (int u = 0; u < U; ++u) load(k + 64 * u, av[u], wv[u], g[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) add(av[u], wv[u], g[u]);
    }
    for (; k < K; k += 64) {
        load(k, av[0], wv[0], g[0]);
        add(av[0], wv[0], g[0]);
    }
    const int idx = add_lanes<32, NV>(acc, lane, 0);
    const int m = m0 + (idx & 7), c = idx >> 3;
    float v = 0.0f + acc[0];   // (a sum of one partial product, as the element-wise kernels take it: no -0)
    if constexpr (EPI == F32_RESID || EPI == F32_LOGITS) {
        const int n = unit * NC + c;
        if ((lane & (64 / NV - 1)) != 0 || m >= M || n >= N) return;
        if constexpr (EPI == F32_RESID) a.out[(size_t)m * N + n] += acc[0];
        else a.out[(size_t)m * N + n] = acc[0];
    } else {
        const float other = __shfl_xor(v, 32, 64);   // the other member of the pair, of the same row
        const int p = unit * NP + c % NP;
        const bool first = c < NP;
        if ((lane & (64 / NV - 1)) != 0 || m >= M || p >= n_pairs) return;
        if constexpr (EPI == F32_SWIGLU) {
            if (first) a.out[(size_t)m * n_pairs + p] = v / (1.0f + expf(-v)) * other;
        } else {
            if (a.rm.row_tok[m] < 0) return;
            int seg, i_win, q_tile0;
            row_place(a.rm, a.L, m, seg, i_win, q_tile0);
            const int pos = a.rm.row_pos[m], h = p / half, i = p % half, j = first ? i : i + half;
            typedef Layout<float> Lay;
            if (h < a.H + a.Hkv) {
                float r0 = first ? v : other, r1 = first ? other : v;
                rotate_pair(r0, r1, a.rope_cos[(size_t)pos * half + i], a.rope_sin[(size_t)pos * half + i]);
                v = first ? r0 : r1;
            }
            const int page = a.pool.page_table[seg * a.pool.pages_per_seg + pos / a.pool.page_tokens], t = pos % a.pool.page_tokens;
            const size_t blk = (size_t)a.pool.page_tokens * a.hd;
            if (h < a.H) a.q_out[((size_t)(q_tile0 + (i_win >> 5)) * a.H + h) * 32 * a.hd + Lay::q_index(i_win & 31, j, a.hd)] = v;
            else if (h < a.H + a.Hkv) ((float *)a.pool.k)[((size_t)page * a.Hkv + (h - a.H)) * blk + Lay::k_index(t, j, a.hd)] = v;
            else ((float *)a.pool.v)[((size_t)page * a.Hkv + (h - a.H - a.Hkv)) * blk + Lay::v_index(t, j, a.hd)] = v;
        }
    }
}

// Columns per wavefront: as launch_gemm_reference, a pair at least where columns come in pairs
template <int EPI>
inline hipError_t launch_gemm_f32(hipStream_t st, const float *A, const float *W, const F32Args &a) {
    const int rows = (a.M + 7) / 8;
    constexpr int few = EPI == F32_QKV || EPI == F32_SWIGLU ? 2 : 1;
    if ((long)a.N * rows >= 6144) gemm_f32_kernel<4, EPI><<<dim3((a.N + 15) / 16, rows), 256, 0, st>>>(A, W, a);
    else gemm_f32_kernel<few, EPI><<<dim3((a.N + 4 * few - 1) / (4 * few), rows), 256, 0, st>>>(A, W, a);
    return hipGetLastError();
}

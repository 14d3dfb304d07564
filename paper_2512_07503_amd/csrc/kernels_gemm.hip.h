// Projection GEMMs  C[m][n] = sum_k A[m][k] W[n][k]  (QKV, output, gate/up, down and the vocabulary
// head: the dense contractions of the forward, Sec. 4.1 Step 2).
//
// M = 2 * sequences * window is small (32 ... 512) while the weights are large, so below M ~ 300 the
// kernels are bound by streaming W from HBM exactly once.  bf16 operands are stored fragment-major
// (see Layout<bf16_t>): a wavefront reads a 32 x 16 operand fragment with one coalesced 1 KiB load and
// feeds it straight into v_mfma_f32_32x32x16_bf16; W never passes through LDS.  K is split across
// workgroups to fill the 256 CUs; the partial sums [splits][M][N] are reduced, in a fixed order, by the
// element-wise kernel that consumes them.
#pragma once
#include "common.hip.h"

// ------------------------------------------------------------------------------------ reference
// Adds v[0 .. N) over the lanes in pairs OFF, OFF / 2, ..., 1 apart: while there are several values, a lane bit picks the half
// a lane goes on with, so the exchanges halve as well.  Returns the index of the value this lane ends up with in v[0].
template <int OFF, int N, int NV>
SJD_D int add_lanes(float (&v)[NV], int lane, int idx) {
    if constexpr (OFF == 0) {
        return idx;
    } else if constexpr (N > 1) {
        const bool up = (lane & OFF) != 0;
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const float keep = up ? v[i + N / 2] : v[i], send = up ? v[i] : v[i + N / 2];
            v[i] = keep + __shfl_xor(send, OFF, 64);
        }
        return add_lanes<OFF / 2, N / 2>(v, lane, 2 * idx + (up ? 1 : 0));
    } else {
        v[0] += __shfl_xor(v[0], OFF, 64);
        return add_lanes<OFF / 2, 1>(v, lane, idx);
    }
}

// One wavefront per (NC output columns, block of 8 rows): lane l sums k = l, l + 64, ... in order, then the lanes are added in
// pairs 32, 16, ..., 1 apart.  The fp32 forward runs on this kernel, so its sums keep that order whatever NC and the
// unrolling are.  Works for both dtypes through the layout functions; fp32 accumulation with fused multiply-adds.
// Bound: at the fp32 model's sizes the latency of a wavefront's loads (K / 64 rounds of them), so four rounds are requested
// together, without conditions (rows past M re-read the last one and are not stored); with enough columns to fill the chip
// four per wavefront share its activation loads.  The 8 x NC sums are reduced together, each exchange halving the values
// a lane holds, 32 exchanges for 32 sums instead of 192.  fp32, launches back to back: 32 x 256 x 1024 17.5 -> 4.0 us,
// 32 x 2048 x 256 10.2 -> 3.9, 32 x 4096 x 256 17.2 -> 4.8, 62 x 768 x 256 9.1 -> 4.0.
template <typename T, int NC>
__global__ __launch_bounds__(256) void gemm_reference_kernel(const T *__restrict__ A, const T *__restrict__ W, float *__restrict__ C, int M, int N,
                                                             int K) {
    constexpr int U = 4, NV = 8 * NC;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n0 = (blockIdx.x * (blockDim.x >> 6) + wave) * NC;
    const int m0 = blockIdx.y * 8;
    if (n0 >= N) return;
    float acc[NV];   // [column][row]
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0f;
    auto round = [&](int k, float (&av)[8], float (&wv)[NC]) {
#pragma unroll
        for (int c = 0; c < NC; ++c) wv[c] = to_float<T>(W[Layout<T>::w_index(min(n0 + c, N - 1), k, K)]);
#pragma unroll
        for (int j = 0; j < 8; ++j) av[j] = to_float<T>(A[Layout<T>::a_index(min(m0 + j, M - 1), k, K)]);
    };
    auto add = [&](const float (&av)[8], const float (&wv)[NC]) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[c * 8 + j] = fmaf(av[j], wv[c], acc[c * 8 + j]);
    };
    int k = lane;
    for (; k - lane + 64 * U <= K; k += 64 * U) {
        float av[U][8], wv[U][NC];
#pragma unroll
        for (int u = 0; u < U; ++u) round(k + 64 * u, av[u], wv[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) add(av[u], wv[u]);
    }
    for (; k < K; k += 64) {
        float av[8], wv[NC];
        round(k, av, wv);
        add(av, wv);
    }
    const int idx = add_lanes<32, NV>(acc, lane, 0);
    const int m = m0 + (idx & 7), n = n0 + (idx >> 3);
    if ((lane & (64 / NV - 1)) == 0 && m < M && n < N) C[(size_t)m * N + n] = acc[0];
}

// ------------------------------------------------------------------------------------ MFMA, bf16
// Workgroup = 4 wavefronts; wavefront w owns NBW column blocks of 32 and MT row tiles of 32 over the
// k-blocks [split * kb_per_split, ...).  grid = (ceil(NB / (4 NBW)), splits, ceil(MTILES / MT)).
template <int MT, int NBW>
__global__ __launch_bounds__(256) void gemm_bf16_mfma_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W,
                                                             float *__restrict__ C, int M, int N, int KB, int kb_per_split) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int NB = (N + 31) >> 5, MTILES = (M + 31) >> 5;
    const int nb0 = (blockIdx.x * 4 + wave) * NBW;
    if (nb0 >= NB) return;
    const int mt0 = blockIdx.z * MT;
    const int kb_begin = blockIdx.y * kb_per_split;
    const int kb_end = kb_begin + kb_per_split < KB ? kb_begin + kb_per_split : KB;

    const u32x4 *Ap = reinterpret_cast<const u32x4 *>(A);
    const u32x4 *Wp = reinterpret_cast<const u32x4 *>(W);
    // fragment (tile, kb) starts at 16-byte index (tile * KB + kb) * 64; out-of-range tiles are clamped
    // (their results are never stored)
    size_t a_off[MT], w_off[NBW];
#pragma unroll
    for (int j = 0; j < MT; ++j) a_off[j] = (size_t)(mt0 + j < MTILES ? mt0 + j : MTILES - 1) * KB * 64 + lane;
#pragma unroll
    for (int i = 0; i < NBW; ++i) w_off[i] = (size_t)(nb0 + i < NB ? nb0 + i : NB - 1) * KB * 64 + lane;

    f32x16 acc[MT][NBW];
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int i = 0; i < NBW; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;

    for (int kb = kb_begin; kb < kb_end; ++kb) {
        u32x4 b[NBW], a[MT];
#pragma unroll
        for (int i = 0; i < NBW; ++i) b[i] = __builtin_nontemporal_load(Wp + w_off[i] + (size_t)kb * 64);
#pragma unroll
        for (int j = 0; j < MT; ++j) a[j] = Ap[a_off[j] + (size_t)kb * 64];
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int i = 0; i < NBW; ++i)
                acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[j]),
                                                                    __builtin_bit_cast(bf16x8, b[i]), acc[j][i], 0, 0, 0);
    }

    // accumulator element v of lane l is C[row = 8 (v / 4) + 4 (l / 32) + v % 4][col = l % 32] of the tile
    float *Cs = C + (size_t)blockIdx.y * M * N;
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        if (mt0 + j >= MTILES) continue;
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            const int col = (nb0 + i) * 32 + (lane & 31);
            if (nb0 + i >= NB || col >= N) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = (mt0 + j) * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (row < M) Cs[(size_t)row * N + col] = acc[j][i][v];
            }
        }
    }
}

struct GemmPlan {
    int mt, nbw, splits, kb_per_split;
    dim3 grid;
};

// Split-K factor and tile shape for an M x N x K bf16 GEMM: aim at >= ~4 wavefronts per SIMD worth of
// independent weight streams while keeping at least 8 k-blocks (128 k) per split.
inline GemmPlan plan_gemm_bf16(int M, int N, int K, int force_splits) {
    GemmPlan p;
    const int NB = (N + 31) / 32, KB = K / 16, MTILES = (M + 31) / 32;
    p.mt = MTILES >= 2 ? 2 : 1;
    p.nbw = NB >= 512 ? 2 : 1;
    const int mz = (MTILES + p.mt - 1) / p.mt;
    const int waves = ((NB + p.nbw - 1) / p.nbw) * mz;
    int splits = force_splits > 0 ? force_splits : (2048 + waves - 1) / waves;
    int max_splits = KB / 8 > 0 ? KB / 8 : 1;
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    p.kb_per_split = (KB + splits - 1) / splits;
    p.splits = (KB + p.kb_per_split - 1) / p.kb_per_split;
    p.grid = dim3((NB + 4 * p.nbw - 1) / (4 * p.nbw), p.splits, mz);
    return p;
}

inline hipError_t launch_gemm_bf16(hipStream_t st, const GemmPlan &p, const bf16_t *A, const bf16_t *W, float *C, int M, int N,
                                   int K) {
    const int KB = K / 16;
    if (p.mt == 1 && p.nbw == 1) gemm_bf16_mfma_kernel<1, 1><<<p.grid, 256, 0, st>>>(A, W, C, M, N, KB, p.kb_per_split);
    else if (p.mt == 1 && p.nbw == 2) gemm_bf16_mfma_kernel<1, 2><<<p.grid, 256, 0, st>>>(A, W, C, M, N, KB, p.kb_per_split);
    else if (p.mt == 2 && p.nbw == 1) gemm_bf16_mfma_kernel<2, 1><<<p.grid, 256, 0, st>>>(A, W, C, M, N, KB, p.kb_per_split);
    else gemm_bf16_mfma_kernel<2, 2><<<p.grid, 256, 0, st>>>(A, W, C, M, N, KB, p.kb_per_split);
    return hipGetLastError();
}

template <typename T>
inline hipError_t launch_gemm_reference(hipStream_t st, const T *A, const T *W, float *C, int M, int N, int K) {
    const int rows = (M + 7) / 8;
    // one column per wavefront / four: 32 x 768 x 256 3.2 / 3.5 us, 62 x 768 x 256 4.0 / 3.8, 32 x 2048 x 256 4.7 / 3.9
    if ((long)N * rows >= 6144) gemm_reference_kernel<T, 4><<<dim3((N + 15) / 16, rows), 256, 0, st>>>(A, W, C, M, N, K);
    else gemm_reference_kernel<T, 1><<<dim3((N + 3) / 4, rows), 256, 0, st>>>(A, W, C, M, N, K);
    return hipGetLastError();
}

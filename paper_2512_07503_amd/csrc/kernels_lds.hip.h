// Projection GEMMs for more than 64 rows (windows and batches of a few hundred rows, prompts): a dense contraction whose
// operands pass through LDS once per workgroup.
//
// Workgroup = WM x WN wavefronts on a tile of TMT x TNB MFMA tiles (32 rows x 32 columns each) over a K range; a wavefront
// owns (TMT / WM) x (TNB / WN) of them.  Both operands are stored fragment-major, so a fragment (1 KiB) goes from global
// memory straight into LDS with one load per lane that never touches a register, lands in the order in which ds_read_b128
// hands it to the matrix core (no bank conflict, no swizzle), and is read by every wavefront that needs it.
// A pipeline stage is two k-steps of 16; S stages of LDS, all but the one being read in flight.  Per stage one barrier; a stage's
// MFMAs run on registers while the next stage's fragments come out of LDS into a second set.  With one set, read a k-step ahead,
// every k-step ended in the latency of its last read: six prompts of 948 rows through 36 layers of 1280 and a step of 192
// 5194 -> 5122 us a pass, the others of these kernels' cases 0 - 1 %.
// What the epilogue reads (partial sums of squares, destinations of rows, residual values) is asked for ahead of the k-loop, as far
// as registers go: left to the epilogue it took two or three round trips there, 2.0 of 10.3 us of 238 x 6912 x 1280, now 1.1
// (a pass as above 5300 -> 5194, a 120-token prompt and a step 3043 -> 3015, 2793 -> 2755).
//
// The product is taken transposed (weights as the A operand of the MFMA): a lane then holds 4 consecutive output columns of
// one row per accumulator quad, which is 8 bytes of the next GEMM's operand layout, 16 bytes of the residual stream or of the
// logits: the epilogues store whole quads instead of single elements.
//
// What bounds it: the operand bytes of a CU.  192 x 4096 x 11008 whole K in 128 x 128 tiles, 64 workgroups: 80 us; with the loads
// alone 80, from L2 55 (70 and 102 GB/s, with 64 or with 128 KB in flight alike).  A K split over two or four groups of
// wavefronts in the workgroup, which brings MFMAs and LDS reads down to 53 us together, is therefore no faster (83 us), and
// slower on short K.  Hence small tiles while a launch has fewer workgroups than CUs, larger ones
// (fewer bytes per MFMA) as rows are added; lds_us() (plans.h) holds the measured rates.
// Against the row-group kernels, which split K over the wavefronts of a 64-row workgroup: 4096-wide, 192 rows: QKV
// 68.6 -> 43.3 us, gate/up 97.8 -> 60.3, down 65 -> 41 with its reduction, head (65 536 ids) 263 -> 135; 1280-wide, 500 rows:
// gate/up 35.9 -> 18.1, QKV 24.2 -> 15.6, down 27.2 -> 24.2.
#pragma once
#include <type_traits>

#include "kernels_skinny.hip.h"
#include "plans.h"

typedef __attribute__((address_space(3))) void lds_ptr_t;
typedef const __attribute__((address_space(1))) void glb_ptr_t;

SJD_D uint2 pack_bf16x4(float a, float b, float c, float d) {
    uint2 r;
    r.x = (uint32_t)float_to_bf16(a) | ((uint32_t)float_to_bf16(b) << 16);
    r.y = (uint32_t)float_to_bf16(c) | ((uint32_t)float_to_bf16(d) << 16);
    return r;
}

// waits until at most `stages` stages of NL loads are in flight (a constant after unrolling)
template <int NL> SJD_D void wait_stages(int stages) {
    switch (stages * NL) {
#define SJD_WAIT(n) case n: asm volatile("s_waitcnt vmcnt(" #n ")" ::: "memory"); break;
#define SJD_WAIT8(a, b, c, d, e, f, g, h) SJD_WAIT(a) SJD_WAIT(b) SJD_WAIT(c) SJD_WAIT(d) SJD_WAIT(e) SJD_WAIT(f) SJD_WAIT(g) SJD_WAIT(h)
        SJD_WAIT8(1, 2, 3, 4, 5, 6, 7, 8) SJD_WAIT8(9, 10, 11, 12, 13, 14, 15, 16) SJD_WAIT8(17, 18, 19, 20, 21, 22, 23, 24)
        SJD_WAIT8(25, 26, 27, 28, 29, 30, 31, 32) SJD_WAIT8(33, 34, 35, 36, 37, 38, 39, 40) SJD_WAIT8(41, 42, 43, 44, 45, 46, 47, 48)
        SJD_WAIT8(49, 50, 51, 52, 53, 54, 55, 56) SJD_WAIT(57) SJD_WAIT(58) SJD_WAIT(59) SJD_WAIT(60) SJD_WAIT(61) SJD_WAIT(62) SJD_WAIT(63)
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
}

// (two wavefronts per SIMD at least: two workgroups of the four-wavefront shapes share a CU if LDS and registers admit them, and
// the 256 x 256 shape, whose 128 KiB of LDS admit one workgroup, has eight wavefronts)
template <int TMT, int TNB, int WM, int WN, int S, int EPI>
__global__ __launch_bounds__(WM * WN * 64, 2) void gemm_lds_kernel(SJD_TILE_PARAMS, int col_tiles, int row_tiles, SkinnyArgs a) {
    SJD_TILE_TAKE(a);
    constexpr int NW = WM * WN, RT = TMT / WM, CB = TNB / WN;   // wavefronts; MFMA tiles of a wavefront: RT x CB
    constexpr int FR = 2 * (TMT + TNB);                         // fragments of a stage
    constexpr int NL = FR / NW;                                 // ... that a wavefront fetches
    static_assert((S - 1) * NL <= 63 && TMT % WM == 0 && TNB % WN == 0 && FR % NW == 0, "tile does not divide");
    constexpr bool kNorm = EPI != EPI_RESID && EPI != EPI_PARTIAL;
    constexpr bool kPair = EPI == EPI_QKV || EPI == EPI_SWIGLU;
    static_assert(!kPair || CB % 2 == 0, "rotary and gate/up pairs of column blocks stay in one wavefront");
    __shared__ u32x4 smem[S * FR * 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup id -> tile: all row tiles of a column tile on one XCD (ids go to the 8 XCDs round-robin), whose L2 then
    // fetches the column tile's weights once; the grid is padded to a multiple of 8 column tiles
    const int ct = (blockIdx.x & 7) + 8 * ((int)(blockIdx.x >> 3) / row_tiles), rt = (int)(blockIdx.x >> 3) % row_tiles;
    if (ct >= col_tiles) {
        // past the padded grid: a workgroup that only touches what the next launch reads (l2_warm_next)
        const int n_compute = 8 * ((col_tiles + 7) >> 3) * row_tiles;
        if ((int)blockIdx.x >= n_compute) l2_warm_next(a, blockIdx.x, n_compute, tid, NW * 64);
        return;
    }
    const int KB = a.KB, ks = blockIdx.y;
    const int kb_lo = ks * a.kb_per_split;
    const int kb_hi = kb_lo + a.kb_per_split < KB ? kb_lo + a.kb_per_split : KB;
    const int n_st = (kb_hi - kb_lo) >> 1;   // K is a multiple of 32 and so is a split's range
    const int row_tiles32 = (a.M + 31) >> 5;

    // this wavefront's fragments of a stage: f = wave + NW i = (operand tile f / 2, k-step f % 2); tiles past the end are
    // clamped (their products are never stored)
    const char *src[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int f = wave + NW * i, t = f >> 1;
        const size_t tile = t < TMT ? (size_t)min(rt * TMT + t, row_tiles32 - 1) : (size_t)min(ct * TNB + t - TMT, n_blocks - 1);
        src[i] = (const char *)(t < TMT ? a.A : a.W) + (tile * KB + kb_lo + (f & 1)) * 1024;
    }
    const int lane16 = lane * 16;
    auto fetch1 = [&](int i, int st, int buf) {
        __builtin_amdgcn_global_load_lds((glb_ptr_t *)(src[i] + (size_t)st * 2048 + lane16), (lds_ptr_t *)&smem[(buf * FR + wave + NW * i) * 64], 16, 0, 0);
    };
    auto fetch = [&](int st, int buf) {
#pragma unroll
        for (int i = 0; i < NL; ++i) fetch1(i, st, buf);
    };
    const int wm = wave / WN, wn = wave % WN;
    struct Frags { bf16x8 act[2][RT], wgt[2][CB]; };   // of a stage: both k-steps
    constexpr int NR = 2 * (RT + CB);
    auto read1 = [&](Frags &f, int o, int buf) {   // operand o of the wavefront: k-step by k-step, its row tiles, then its column blocks
        const int kk = o / (RT + CB), u = o % (RT + CB);
        if (u < RT) f.act[kk][u < RT ? u : 0] = __builtin_bit_cast(bf16x8, smem[(buf * FR + (wm * RT + u) * 2 + kk) * 64 + lane]);
        else f.wgt[kk][u >= RT ? u - RT : 0] = __builtin_bit_cast(bf16x8, smem[(buf * FR + (TMT + wn * CB + u - RT) * 2 + kk) * 64 + lane]);
    };
    f32x16 acc[RT][CB];
#pragma unroll
    for (int j = 0; j < RT; ++j)
#pragma unroll
        for (int i = 0; i < CB; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;
    // One stage's MFMAs on `f`, with the reads of the next stage's operands into `nxt` (n_read of them) and the loads of a stage
    // (n_load) spread between them: issued in a block they would hold the MFMAs behind them back while the load unit takes
    // them one by one.
    auto stage_step = [&](const Frags &f, Frags &nxt, auto n_read, int rbuf, auto n_load, int st, int lbuf) {
        constexpr int NM = 2 * RT * CB, NRD = decltype(n_read)::value, NO = NRD + decltype(n_load)::value;
#pragma unroll
        for (int u = 0; u < NM; ++u) {
            const int kk = u / (RT * CB), v = u % (RT * CB);
            acc[v / CB][v % CB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.wgt[kk][v % CB], f.act[kk][v / CB], acc[v / CB][v % CB], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int o = u * NO / NM; o < (u + 1) * NO / NM; ++o) {
                if (o < NRD) read1(nxt, o, rbuf);
                else fetch1(o >= NRD ? o - NRD : 0, st, lbuf);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr std::integral_constant<int, NR> kReads{};
    constexpr std::integral_constant<int, NL> kLoads{};
    constexpr std::integral_constant<int, 0> kNone{};
    auto barrier = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wavefront is done reading the buffer that is refilled next
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // What the epilogue needs from memory and one lane can hold is requested ahead of the operands (older loads: the waits below, which
    // count what is outstanding, cover them): partial sums of squares, even ones in the lower half wavefront, odd ones in the upper;
    // destinations of the rows; residual values.
    const int h4 = 4 * (lane >> 5), blk0 = ct * TNB + wn * CB;
    constexpr int kSsq = !kNorm ? 0 : RT == 1 ? (NW == 8 ? 10 : 20) : RT == 2 ? 10 : RT == 3 ? 8 : 0;
    constexpr bool kEarlyRow = EPI == EPI_QKV && RT <= 2 && NW < 8, kEarlyX = EPI == EPI_RESID && RT == 1;
    [[maybe_unused]] float ssq[RT][kSsq + 1];
    [[maybe_unused]] QkvRow qrow[RT];
    [[maybe_unused]] float4 xin[CB][4];
    auto row_m = [&](int j) { return min((rt * TMT + wm * RT + j) * 32 + (lane & 31), a.M - 1); };   // past the end: the last row
    auto load_x = [&](int m) {
#pragma unroll
        for (int i = 0; i < CB; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)   // N is a multiple of 32: a block is inside or past the end as a whole
                xin[i][q] = *reinterpret_cast<const float4 *>(a.x + (size_t)m * a.N + min(blk0 + i, n_blocks - 1) * 32 + 8 * q + h4);
    };
    if constexpr (kNorm) {
#pragma unroll
        for (int j = 0; j < RT; ++j)
#pragma unroll
            for (int u = 0; u < kSsq; ++u) ssq[j][u] = a.row_ssq_part[(size_t)min((lane >> 5) + 2 * u, a.row_ssq_n - 1) * a.M + row_m(j)];
    }
    if constexpr (kEarlyRow) {
#pragma unroll
        for (int j = 0; j < RT; ++j) qrow[j] = qkv_row(a, row_m(j));
    }
    if constexpr (kEarlyX) load_x(row_m(0));
    __builtin_amdgcn_sched_barrier(0);

#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s < n_st) fetch(s, s);
    // stage 0 has landed once at most the younger stages' loads are outstanding
    wait_stages<NL>(n_st >= S ? S - 1 : 0);
    barrier();
    Frags f, g;
    if (n_st > 0)
#pragma unroll
        for (int o = 0; o < NR; ++o) read1(f, o, 0);
    int it = 0, buf = 0;
    auto next_of = [](int b) { return b + 1 == S ? 0 : b + 1; };
    // stage `it` from cur, while nxt takes stage it + 1 out of LDS and stage it + S takes its buffer, which every wavefront has read
    auto steady = [&](const Frags &cur, Frags &nxt) {
        wait_stages<NL>(S - 2);   // stage it + 1
        barrier();
        stage_step(cur, nxt, kReads, next_of(buf), kLoads, it + S, buf);
        buf = next_of(buf);
        ++it;
    };
    while (it + S + 1 < n_st) {
        steady(f, g);
        steady(g, f);
    }
    if (it + S < n_st) {
        steady(f, g);
        f = g;
    }
    // the last S stages: nothing left to fetch (t stages to go, conditions are uniform); operands of stage S are in f, of S - 1 in g, ...
    if (((n_st - it) ^ S) & 1) g = f;
#pragma unroll
    for (int t = S; t >= 1; --t) {
        if (n_st - it != t) continue;
        Frags &cur = (t ^ S) & 1 ? g : f, &nxt = (t ^ S) & 1 ? f : g;
        if (t > 1) {
            wait_stages<NL>(t - 2);
            barrier();
            stage_step(cur, nxt, kReads, next_of(buf), kNone, 0, 0);
            buf = next_of(buf);
        } else {
            stage_step(cur, nxt, kNone, 0, kNone, 0, 0);
        }
        ++it;
    }

    // ---- epilogue: accumulator register v = 4 q + e of lane l is row l % 32 of the row tile, column 8 q + 4 (l / 32) + e of
    //      the column block
    float inv[RT];
#pragma unroll
    for (int j = 0; j < RT; ++j) {
        inv[j] = 1.0f;
        if constexpr (kNorm) {
            // 1 / rms: those requested ahead of the k-loop, then the rest
            float t = 0.0f;
#pragma unroll
            for (int u = 0; u < kSsq; ++u) t += (lane >> 5) + 2 * u < a.row_ssq_n ? ssq[j][u] : 0.0f;
            if (2 * kSsq < a.row_ssq_n) t += row_ssq_sum(a, row_m(j), (lane >> 5) + 2 * kSsq, 2);
            t += __shfl_xor(t, 32, 64);
            inv[j] = 1.0f / sqrtf(t / (float)(KB * 16) + a.eps);
        }
    }
    if constexpr (EPI == EPI_HEAD && RT % 2 == 0) {
        if (a.z_mode == 1) {   // row tiles (2 s, 2 s + 1): conditional and unconditional rows of sequence s's window of 32
#pragma unroll
            for (int j = 0; j < RT; j += 2) {
                const int mc = (rt * TMT + wm * RT + j) * 32 + (lane & 31), mu = mc + 32;
                if (mu >= a.M) continue;
                float *zrow = a.z_out + ((size_t)(mc >> 6) * 32 + (lane & 31)) * a.N;
#pragma unroll
                for (int i = 0; i < CB; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int n = (ct * TNB + wn * CB + i) * 32 + 8 * q + h4;
                        float4 z, lc, lu;
                        float *zp = &z.x, *cp = &lc.x, *up = &lu.x;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            zp[e] = guided_z(acc[j][i][4 * q + e], inv[j], acc[j + 1][i][4 * q + e], inv[j + 1], a.cfg_scale, a.inv_t);
                            cp[e] = acc[j][i][4 * q + e] * inv[j];
                            up[e] = acc[j + 1][i][4 * q + e] * inv[j + 1];
                        }
                        if ((a.N & 3) == 0 && n + 3 < a.N) {
                            *reinterpret_cast<float4 *>(zrow + n) = z;
                            if (a.logits) {
                                *reinterpret_cast<float4 *>(a.logits + (size_t)mc * a.N + n) = lc;
                                *reinterpret_cast<float4 *>(a.logits + (size_t)mu * a.N + n) = lu;
                            }
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (n + e < a.N) {
                                    zrow[n + e] = zp[e];
                                    if (a.logits) {
                                        a.logits[(size_t)mc * a.N + n + e] = cp[e];
                                        a.logits[(size_t)mu * a.N + n + e] = up[e];
                                    }
                                }
                        }
                    }
            }
            return;
        }
    }
#pragma unroll
    for (int j = 0; j < RT; ++j) {
        const int m = (rt * TMT + wm * RT + j) * 32 + (lane & 31);
        [[maybe_unused]] float sq = 0.0f;
        if (m < a.M) {
            if constexpr (EPI == EPI_QKV) {
                const QkvRow r = kEarlyRow ? qrow[j] : qkv_row(a, m);
                const int pairs = a.hd >> 6, half = a.hd >> 1;
#pragma unroll
                for (int i = 0; i < CB; i += 2) {
                    const int g = (blk0 + i) >> 1, head = g / pairs, j0 = (g % pairs) * 32 + h4;
                    if (blk0 + i >= n_blocks || r.pos < 0) continue;
                    const float4 *rot = reinterpret_cast<const float4 *>(a.row_rot + (size_t)m * half + j0);
                    const bool is_q = head < a.H, is_v = head >= a.H + a.Hkv;
                    const size_t blk = (size_t)a.pool.page_tokens * a.hd;
                    bf16_t *dst = is_q ? a.q_out + (size_t)head * 32 * a.hd + r.q_off
                                : is_v ? (bf16_t *)a.pool.v + ((size_t)r.page * a.Hkv + (head - a.H - a.Hkv)) * blk + r.v_off
                                       : (bf16_t *)a.pool.k + ((size_t)r.page * a.Hkv + (head - a.H)) * blk + r.k_off;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float v0[4], v1[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            v0[e] = acc[j][i][4 * q + e] * inv[j];
                            v1[e] = acc[j][i + 1][4 * q + e] * inv[j];
                        }
                        if (is_v) {   // a token's value dimensions are 16 bytes apart in the operand layout
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                dst[Layout<bf16_t>::v_index(0, j0 + 8 * q + e, a.hd)] = float_to_bf16(v0[e]);
                                dst[Layout<bf16_t>::v_index(0, j0 + 8 * q + e + half, a.hd)] = float_to_bf16(v1[e]);
                            }
                            continue;
                        }
                        const float4 r0 = rot[4 * q], r1 = rot[4 * q + 1];   // (cos, sin) of 4 consecutive dimensions
                        const float c[4] = {r0.x, r0.z, r1.x, r1.z}, s[4] = {r0.y, r0.w, r1.y, r1.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) rotate_pair(v0[e], v1[e], c[e], s[e]);
                        // queries and keys share the form of their row operand: 4 dimensions are 8 contiguous bytes
                        *reinterpret_cast<uint2 *>(dst + Layout<bf16_t>::q_index(0, j0 + 8 * q, a.hd)) = pack_bf16x4(v0[0], v0[1], v0[2], v0[3]);
                        *reinterpret_cast<uint2 *>(dst + Layout<bf16_t>::q_index(0, j0 + 8 * q + half, a.hd)) = pack_bf16x4(v1[0], v1[1], v1[2], v1[3]);
                    }
                }
            } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
                for (int i = 0; i < CB; i += 2) {
                    if (blk0 + i >= n_blocks) continue;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float s[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float gt = acc[j][i][4 * q + e] * inv[j], up = acc[j][i + 1][4 * q + e] * inv[j];
                            s[e] = silu(gt) * up;
                        }
                        *reinterpret_cast<uint2 *>(a.h + Layout<bf16_t>::a_index(m, ((blk0 + i) >> 1) * 32 + 8 * q + h4, a.F)) = pack_bf16x4(s[0], s[1], s[2], s[3]);
                    }
                }
            } else if constexpr (EPI == EPI_RESID) {
                if constexpr (!kEarlyX) load_x(m);
#pragma unroll
                for (int i = 0; i < CB; ++i) {
                    float4 gn[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) gn[q] = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
                    if (a.gain && (blk0 + i) * 32 < a.N) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) gn[q] = *reinterpret_cast<const float4 *>(a.gain + (blk0 + i) * 32 + 8 * q + h4);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int n = (blk0 + i) * 32 + 8 * q + h4;
                        if (n >= a.N) continue;
                        float4 v = xin[i][q];
                        v.x += acc[j][i][4 * q]; v.y += acc[j][i][4 * q + 1]; v.z += acc[j][i][4 * q + 2]; v.w += acc[j][i][4 * q + 3];
                        *reinterpret_cast<float4 *>(a.x + (size_t)m * a.N + n) = v;
                        const float4 g = gn[q];
                        const uint2 b = pack_bf16x4(v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w);
                        *reinterpret_cast<uint2 *>(a.xb + Layout<bf16_t>::a_index(m, n, a.N)) = b;
                        if (!a.gain) {   // the squares of what the copy holds
                            v.x = __builtin_bit_cast(float, b.x << 16); v.y = __builtin_bit_cast(float, b.x & 0xFFFF0000u);
                            v.z = __builtin_bit_cast(float, b.y << 16); v.w = __builtin_bit_cast(float, b.y & 0xFFFF0000u);
                        }
                        sq += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
                    }
                }
            } else {   // EPI_PARTIAL, EPI_HEAD: fp32 rows of N
                float *row = EPI == EPI_PARTIAL ? a.part + ((size_t)ks * a.M + m) * a.N : a.logits + (size_t)m * a.N;
#pragma unroll
                for (int i = 0; i < CB; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int n = (blk0 + i) * 32 + 8 * q + h4;
                        if ((a.N & 3) == 0 && n + 3 < a.N) {
                            *reinterpret_cast<float4 *>(row + n) =
                                make_float4(acc[j][i][4 * q] * inv[j], acc[j][i][4 * q + 1] * inv[j], acc[j][i][4 * q + 2] * inv[j], acc[j][i][4 * q + 3] * inv[j]);
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (n + e < a.N) row[n + e] = acc[j][i][4 * q + e] * inv[j];
                        }
                    }
            }
        }
        if constexpr (EPI == EPI_RESID) {
            // sum of squares of this wavefront's columns of the row, for the next projection's norm
            sq += __shfl_xor(sq, 32, 64);
            if (a.ssq_out && lane < 32 && m < a.M && blk0 * 32 < a.N) a.ssq_out[(size_t)(blk0 / CB) * a.M + m] = sq;
        }
    }
}

// a.ksplit K ranges of a.kb_per_split (even) k-blocks.
template <int EPI>
inline hipError_t launch_lds(hipStream_t st, const SkinnyArgs &a, int n_blocks, int cfg) {
    if (a.M <= 0 || n_blocks <= 0 || (a.KB & 1) || (a.kb_per_split & 1) || a.ksplit < 1 || (size_t)a.kb_per_split * a.ksplit < (size_t)a.KB ||
        (EPI != EPI_PARTIAL && a.ksplit != 1))
        return hipErrorInvalidValue;
#define SJD_LDS_ONE(I, TMT, TNB, WM, WN, S)                                                                                    \
    if constexpr (I < kLdsTiles || (I == kLdsTileHeadZ ? EPI == EPI_HEAD : I == kLdsTileBig ? EPI == EPI_QKV || EPI == EPI_SWIGLU : EPI == EPI_QKV || EPI == EPI_RESID)) \
        if (cfg == I) {                                                                                                        \
            const int col_tiles = ceil_div(n_blocks, TNB), row_tiles = ceil_div(a.M, 32 * TMT);                                \
            const dim3 grid(8 * ceil_div(col_tiles, 8) * row_tiles + (a.ksplit == 1 ? a.pf_wgs : 0), a.ksplit);                \
            gemm_lds_kernel<TMT, TNB, WM, WN, S, EPI><<<grid, WM * WN * 64, 0, st>>>(SJD_TILE_PASS(a), col_tiles, row_tiles, a);       \
            return hipGetLastError();                                                                                          \
        }
    SJD_LDS_TILES(SJD_LDS_ONE)
#undef SJD_LDS_ONE
    return hipErrorInvalidValue;
}

// "NT" GEMM  C[M,N] = sum_k A[M,k] * Bt[N,k]  for products of few output tiles, which the 128-wide kernels leave to a few CUs,
// each a chain of K steps with a memory round trip and two barriers per step.
//
// A workgroup of eight wavefronts owns one tile of T32 x T32 MFMA tiles; wavefront w takes the 128-byte K steps w, w + 8, ... and
// loads its fragments straight from memory (a step's loads cover whole 128-byte lines of its rows; LDS would only pass
// them on: no two wavefronts read the same), the next step's under this one's MFMAs, no barrier.  The eight sums meet
// in LDS, in a fixed order.  Bound by the loads' latency where a wavefront has a step or two, by the L2 traffic of small tiles
// where there are many.  Measurement of one head, n = 1600, m = 392, d = 64 in float: 73.8 -> 21.0 us; 256 x 64 x 256:
// 19.6 -> 12.5; four heads of n = 8192, m = 1024: 349 -> 152 (calls, with their transposes).  Against float64 a third of the
// error: eight chains of an eighth of the length.
//
// SPLIT (float): the products of csat_gemm_f32.h, the operands split in registers.  Synthesis of 1600 x 64 over 1600:
// 65 -> 19 us; 77 x 64 over 4096, eight heads 157 -> 39; error against float64 0.74 to 1.0 of the 128 x 64 kernel's, on dense
// rows and on rows of a few coefficients (1.5 to 1.8 with the two sets of products added before the wavefronts' sums meet).  A tile with a suspect sum (there) is formed again on the float MFMA, as the chain it always was.
#pragma once
#include "csat_gemm_f32.h"

namespace csat {

constexpr int kDeepWaves = 8;

template <typename T, int T32, bool SPLIT, typename Epi>
__global__ __launch_bounds__(512, T32 == 2 || SPLIT ? 2 : 4) void gemm_nt_deep_kernel(GemmArgs g, Epi epi) {
    constexpr int EPC = Elem<T>::per_chunk, NT = T32 * T32, SLOTS = kDeepWaves / 2, SETS = SPLIT ? 2 : 1;
    __shared__ f32x4 part[SLOTS][SETS * NT * 4][64];
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int z = blockIdx.z;
    const long long row0 = (long long)blockIdx.x * (32 * T32), col0 = (long long)blockIdx.y * (32 * T32);
    const int kchunks = (g.K + EPC - 1) / EPC, ksteps = (kchunks + kRowChunks - 1) / kRowChunks;
    // rows beyond the last: the last one's, not used
    const T* pa[T32];
    const T* pb[T32];
#pragma unroll
    for (int i = 0; i < T32; ++i) {
        const long long ra = row0 + 32 * i + li, rb = col0 + 32 * i + li;
        pa[i] = (const T*)g.A + (long long)z * g.strideA + (ra < g.M ? ra : g.M - 1) * g.lda;
        pb[i] = (const T*)g.Bt + (long long)z * g.strideB + (rb < g.N ? rb : g.N - 1) * g.ldb;
    }
    uint4 fa[2][4][T32], fb[2][4][T32];
    auto load = [&](int ks, auto bc) {
        constexpr int b = decltype(bc)::value;
#pragma unroll
        for (int gk = 0; gk < 4; ++gk) {
            const int kc = ks * kRowChunks + 2 * gk + lh, kb = kc < kchunks ? kc : 0;
            const int ka = g.a_kwrap > 0 ? kb % g.a_kwrap : kb;
#pragma unroll
            for (int i = 0; i < T32; ++i) {
                fa[b][gk][i] = *(const uint4*)(pa[i] + (long long)ka * EPC);
                fb[b][gk][i] = *(const uint4*)(pb[i] + (long long)kb * EPC);
            }
        }
    };
    f32x16 acc[T32][T32], corr[T32][T32];          // corr: SPLIT only, the five smaller products
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < T32; ++i)
#pragma unroll
            for (int j = 0; j < T32; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = corr[i][j][v] = 0.f;
    };
    auto multiply = [&](int ks, auto bc, auto plain) {
        constexpr int b = decltype(bc)::value;
        if ((ks + 1) * kRowChunks > kchunks) {         // the last step: chunks beyond K are zero
#pragma unroll
            for (int gk = 0; gk < 4; ++gk)
#pragma unroll
                for (int i = 0; i < T32; ++i) {
                    const bool in = ks * kRowChunks + 2 * gk + lh < kchunks;
                    fa[b][gk][i] = in ? fa[b][gk][i] : make_uint4(0, 0, 0, 0);
                    fb[b][gk][i] = in ? fb[b][gk][i] : make_uint4(0, 0, 0, 0);
                }
        }
        if constexpr (SPLIT && !decltype(plain)::value) {
#pragma unroll
            for (int gk = 0; gk < 4; gk += 2) {        // a lane's eight floats of two groups: one K slab of the bf16 product
                bf16x8 qa[T32][3], qb[T32][3];
                auto split = [](const uint4& x, const uint4& y, bf16x8 (&q)[3]) {
                    const f32x4 u = __builtin_bit_cast(f32x4, x), v = __builtin_bit_cast(f32x4, y);
                    u32x4 h, m, l;
                    uint32_t a[4], b2[4], c[4];
                    split3(u[0], u[1], a[0], b2[0], c[0]);
                    split3(u[2], u[3], a[1], b2[1], c[1]);
                    split3(v[0], v[1], a[2], b2[2], c[2]);
                    split3(v[2], v[3], a[3], b2[3], c[3]);
                    h = u32x4{a[0], a[1], a[2], a[3]}; m = u32x4{b2[0], b2[1], b2[2], b2[3]}; l = u32x4{c[0], c[1], c[2], c[3]};
                    q[0] = __builtin_bit_cast(bf16x8, h); q[1] = __builtin_bit_cast(bf16x8, m); q[2] = __builtin_bit_cast(bf16x8, l);
                };
#pragma unroll
                for (int i = 0; i < T32; ++i) {
                    split(fa[b][gk][i], fa[b][gk + 1][i], qa[i]);
                    split(fb[b][gk][i], fb[b][gk + 1][i], qb[i]);
                }
                constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
                for (int p = 0; p < 6; ++p)
#pragma unroll
                    for (int i = 0; i < T32; ++i)
#pragma unroll
                        for (int j = 0; j < T32; ++j) {
                            if (p < 5) corr[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa[i][PA[p % 5]], qb[j][PB[p % 5]], corr[i][j], 0, 0, 0);
                            else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa[i][0], qb[j][0], acc[i][j], 0, 0, 0);
                        }
            }
        } else {
#pragma unroll
            for (int gk = 0; gk < 4; ++gk)
#pragma unroll
                for (int i = 0; i < T32; ++i)
#pragma unroll
                    for (int j = 0; j < T32; ++j) mfma_group<T>(fa[b][gk][i], fb[b][gk][j], acc[i][j]);
        }
    };
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    clear();
    int ks = wave;
    if (ks < ksteps) load(ks, B0{});
    for (; ks < ksteps; ks += 2 * kDeepWaves) {
        if (ks + kDeepWaves < ksteps) load(ks + kDeepWaves, B1{});
        multiply(ks, B0{}, std::false_type{});
        if (ks + 2 * kDeepWaves < ksteps) load(ks + 2 * kDeepWaves, B0{});
        if (ks + kDeepWaves < ksteps) multiply(ks + kDeepWaves, B1{}, std::false_type{});
    }

    // the wavefronts' sums, in a fixed order: 4 .. 7 into 0 .. 3, then those.  SPLIT: the first products' and the smaller ones' apart up
    // to the end, as in one chain.  A few first products sum exactly, so that a row of few coefficients is rounded once.
    auto set = [&](int i) -> f32x16& { return i < NT * 4 ? acc[i / 4 / T32][i / 4 % T32] : corr[i / 4 % NT / T32][i / 4 % T32]; };
    auto put = [&](int s) {
#pragma unroll
        for (int i = 0; i < SETS * NT * 4; ++i) {
            const f32x16& a = set(i);
            part[s][i][lane] = f32x4{a[4 * (i & 3)], a[4 * (i & 3) + 1], a[4 * (i & 3) + 2], a[4 * (i & 3) + 3]};
        }
    };
    if (wave >= SLOTS) put(wave - SLOTS);
    __syncthreads();
    if (wave < SLOTS) {
#pragma unroll
        for (int i = 0; i < SETS * NT * 4; ++i) {
            const f32x4 v = part[wave][i][lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) set(i)[4 * (i & 3) + e] += v[e];
        }
        put(wave);
    }
    __syncthreads();
    constexpr int NI = (NT * 4 + kDeepWaves - 1) / kDeepWaves;
    f32x4 sum[NI];
    SplitSuspect suspect;
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        const int i = wave + n * kDeepWaves;
        if (i >= NT * 4) continue;
        sum[n] = part[0][i][lane];
#pragma unroll
        for (int s = 1; s < SLOTS; ++s) sum[n] += part[s][i][lane];
        if constexpr (SPLIT) {
            f32x4 small = part[0][NT * 4 + i][lane];
#pragma unroll
            for (int s = 1; s < SLOTS; ++s) small += part[s][NT * 4 + i][lane];
            sum[n] += small;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) suspect.add(sum[n][e]);
    }
    auto out = [&](int i, const f32x4& v) {
        const long long r = row0 + i / 4 / T32 * 32 + 8 * (i & 3) + 4 * lh, c = col0 + i / 4 % T32 * 32 + li;
#pragma unroll
        for (int e = 0; e < 4; ++e) epi(z, r + e, c, v[e]);
    };
    if (SPLIT && __syncthreads_or(suspect.any())) {    // the tile again on the float MFMA, as one chain
        if (wave != 0) return;
        clear();
        for (ks = 0; ks < ksteps; ++ks) {
            load(ks, B0{});
            multiply(ks, B0{}, std::true_type{});
        }
#pragma unroll
        for (int i = 0; i < NT * 4; ++i) {
            const f32x16& a = acc[i / 4 / T32][i / 4 % T32];
            out(i, f32x4{a[4 * (i & 3)], a[4 * (i & 3) + 1], a[4 * (i & 3) + 2], a[4 * (i & 3) + 3]});
        }
        return;
    }
#pragma unroll
    for (int n = 0; n < NI; ++n)
        if (wave + n * kDeepWaves < NT * 4) out(wave + n * kDeepWaves, sum[n]);
}

}  // namespace csat

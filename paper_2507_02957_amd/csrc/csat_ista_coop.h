// Fused ISTA decoder (bf16, m <= 416) for launches with few rows: the eight wavefronts of a workgroup share one 32-row
// tile.  The arithmetic is ista_fused_kernel's, product by product, in the same order (same bits) where one workgroup has the
// tile; what is shared out:
//   wavefronts 0, 1   GEMM-U and the threshold of the even and the odd chunks (a chunk's U is one accumulator chain, so
//                     it stays with one wavefront and takes two steps; consecutive chunks overlap by one)
//   wavefronts 2, 3   GEMM-R of every chunk, each for its half of the tiles of m (independent accumulators)
//   wavefronts 4 - 7  stage the packed chunks, global -> LDS (a wavefront is held while its requests drain)
// A step is one chunk: U's first part of chunk c, U's second part and threshold of chunk c - 1, R of chunk c - 2, while
// chunk c + 2 is being requested; five ring slots.  The iterate goes from the U to the R wavefronts as bf16 operands
// through LDS (2 KB per chunk), the next residual back once per iteration through a ring slot that is free then.
//
// Why: on the one-tile form of ista_fused_kernel a single wavefront did all the products, 52 MFMAs per chunk at
// m = 392 (1664 cycles; with the threshold and the waits 1.08 us a chunk), on one of the CU's four matrix pipes.  Here
// a chunk takes 0.13 + 0.035 us per tile of m: what grows with m is the 2 KB per tile that the CU pulls from L2 (about
// 32 bytes a clock) and the 6 KB it moves in LDS; the rest is the step's barrier, the ramp of the fragment reads and
// the threshold.  Column-wise short_video (96 tiles, m = 392, 20 iterations): 1106 -> 600 us a launch;
// 3330 rows of n = 1571, m = 197: 800 -> 520 us a call.  (U's first part as a half or five sixths: equal, 4 % slower.)
//
// Where there are fewer tiles than CUs, several workgroups (members) share a tile, each with its share of the columns, through
// all iterations; at the end of each they exchange their parts of the residual (fp32), and each sums all of them in the members'
// order: the same residual, bit for bit, in every member, but not the other decoders' order of summation.  The
// staging and the chain of chunks, which bound a workgroup, get shorter by their number; an exchange takes 4 to 7 us for
// two members (52 KB out and as much in per CU at m = 392: the volume through the memory-side cache once the chip is full, the latency
// of a store, a flag and a load before).  The 96 tiles above: 612 -> 417 us with two members, 8 tiles 592 -> 267 with five, 8 tiles of
// n = 16 384, m = 64 2835 -> 305 with sixteen.  Tried and dropped: all eight wavefronts summing the parts, the own one read back of two
// too (8 tiles equal, 96 tiles 489 against 422: half as much volume again); parts waited for one by one (30 tiles, four members 332
// against 310); the own part kept in registers beside the sum from three members on (30 tiles 327 against 299, 10 tiles of m = 224 253
// against 200: fewer loads on the way).
// Members need not all be resident at once: they take their numbers as they start, so a started member waits only for
// members of its own tile, of which the last started tile alone can lack some, and those start as soon as any CU is free.
#pragma once
#include "csat_ista_fused.h"

namespace csat {

constexpr int kCoopSlots = 5;
constexpr int kCoopMaxMT = 13;
constexpr size_t ista_coop_lds_bytes(int MT) { return (size_t)kCoopSlots * ista_fused_set_frags(MT) * 1024 + 4096; }

template <int MT>
__global__ __launch_bounds__(512, 1) void ista_coop_kernel(IstaFusedArgs a) {
    extern __shared__ uint4 lds[];
    constexpr int NF = 2 * MT, SETF = ista_fused_set_frags(MT), FW = SETF / 4, SLOT = SETF * 1024;
    constexpr int G = 2, D = 2;                        // fragments per LDS wait, groups of them on the way (3, 4: up to 5 % slower)
    constexpr int OFF_X = kCoopSlots * SLOT;           // two buffers of x operands, 2 KB each
    constexpr int RT = (MT + 1) / 2;                   // tiles of m per R wavefront (tile 2 j + its index)
    // fragments of U's first part: about as long as the rest with the threshold behind it
    constexpr int H = MT <= 3 ? NF : (NF * 2 / 3 + 1) / 2 * 2;
    const int lane = threadIdx.x & 63, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int iters = a.iters, G2 = a.tile_split;
    // G2 members to a tile, numbered in the order in which they start
    __shared__ int s_unit;
    int unit = blockIdx.x;
    if (G2 > 1) {
        if (threadIdx.x == 0) s_unit = atomicAdd(a.sync, 1);
        __syncthreads();
        unit = __builtin_amdgcn_readfirstlane(s_unit);
    }
    const int member = unit % G2;
    const int c0 = (int)((long long)a.nct * member / G2), nct = (int)((long long)a.nct * (member + 1) / G2) - c0;
    const long long rt = unit / G2, row = rt * 32 + (lane & 31);
    const bool row_ok = row < a.rows;
    const float* yrow = a.Y + (row_ok ? row : a.rows - 1) * a.ldy + 4 * lh;
    const uint32_t lds0 = (uint32_t)(size_t)(lds_ptr_t)lds;
    auto barrier = [&]() {       // LDS writes of this wavefront done; loads from memory stay in flight
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto next = [](int s, int by) { s += by; return s >= kCoopSlots ? s - kCoopSlots : s; };
    auto operands_at = [&](int k) { return lds + (next(next(k, nct % kCoopSlots), 3) * SLOT) / 16 + lane; };
    // Every wavefront walks the same steps: iterations 0 .. iters - 2 have nct + 2 of them, the last one nct + 1.
    // k: ring slot of the iteration's chunk 0.

    if (wave >= 4) {             // ---- staging ----
        auto issue = [&](int c, int slot) {
            const uint4* src = a.PhiPack + ((long long)(c0 + c) * SETF + (wave - 4) * FW) * 64 + lane;
            char* dst = (char*)lds + slot * SLOT + (wave - 4) * FW * 1024;
#pragma unroll
            for (int i = 0; i < FW; ++i) __builtin_amdgcn_global_load_lds((glb_ptr_t)(src + i * 64), (lds_ptr_t)(dst + i * 1024), 16, 0, 0);
        };
        issue(0, 0);
        issue(1, 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FW) : "memory");
        barrier();
        int k = 0;
        for (int t = 0; t < iters; ++t) {
            const bool last = t + 1 == iters;
            int s = next(k, 2);                                   // slot of chunk c + 2
            for (int c = 0; c < nct + 1; ++c) {
                const int cn = c + 2 < nct ? c + 2 : c + 2 - nct; // (beyond the end: the next iteration's first two)
                const bool want = c + 2 < nct || (!last && c < nct);
                if (want) issue(cn, s);
                s = next(s, 1);
                if (want) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FW) : "memory");     // chunk c + 1 has landed
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                barrier();
            }
            if (!last) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                barrier();
            }
            k = (k + nct) % kCoopSlots;
        }
        return;
    }

    if (wave >= 2) {             // ---- GEMM-R ----
        const int rw = wave - 2;
        const uint32_t nat16 = lds0 + rw * 1024 + frag_slot(lane & 31, lh) * 16;
        f32x16 racc[RT];
        // A shared tile's residual, at the end of an iteration: this wavefront's tiles of the member's part go out, the others'
        // come in and are summed.  Parts and flags go past the L2s (agent scope), so no cache is written back
        // or invalidated; a part is complete (vmcnt) before its flag is set.  A slot is written again two iterations
        // later: its readers have set their own next flags since, which this wavefront has waited for.
        bool gave_up = false;
        auto exchange = [&](int t) {
            constexpr int kAgent = 16;                            // sc1
            constexpr int GB = RT <= 2 ? 4 : RT <= 4 ? 2 : 1, JB = RT <= 5 ? RT : (RT + 1) / 2;     // members and tiles per batch of loads
            auto slot = [&](int g) {
                return __builtin_amdgcn_make_buffer_rsrc((void*)(a.xchg + (((rt * G2 + g) * 2 + (t & 1)) * MT + rw) * 256), 0, (MT - rw) * 4096, kBufferFlags);
            };
            int* flags = a.sync + 2 + 2 * rt * G2 + rw;
            const auto mine = slot(member);
#pragma unroll
            for (int j = 0; j < RT; ++j)                          // (an odd count's missing tile: out of the descriptor's range)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{racc[j][4 * g], racc[j][4 * g + 1], racc[j][4 * g + 2], racc[j][4 * g + 3]}),
                                                           mine, j * 8192 + g * 1024 + lane * 16, 0, kAgent);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) __hip_atomic_store(flags + 2 * member, t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (long long n = 0; !gave_up; ++n) {
                const bool there = lane >= G2 || __hip_atomic_load(flags + 2 * lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > t;
                if (__all(there)) break;
                if (n >= a.spin_limit) {
                    if (lane == 0) __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    gave_up = true;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            asm volatile("" ::: "memory");
            // Every member sums in the members' order, so that all hold the same residual: from three on the own part is read back too
            // (of two, own + other is the same sum; the zeros out of their way: 548 -> 544 us a column-wise short_video).
            const int parts = G2 == 2 ? 1 : G2;
            if (__builtin_expect(G2 > 2, 0)) {
#pragma unroll
                for (int j = 0; j < RT; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) racc[j][e] = 0.f;
            }
            for (int i = 0; i < parts; i += GB) {
#pragma unroll
                for (int j0 = 0; j0 < RT; j0 += JB) {
                    u32x4 v[GB][JB][4];
#pragma unroll
                    for (int b = 0; b < GB; ++b)
                        if (i + b < parts) {
                            const auto part = slot(G2 == 2 ? 1 - member : i + b);
#pragma unroll
                            for (int j = 0; j < JB; ++j)
#pragma unroll
                                for (int g = 0; g < 4; ++g) v[b][j][g] = __builtin_amdgcn_raw_buffer_load_b128(part, (j0 + j) * 8192 + g * 1024 + lane * 16, 0, kAgent);
                        }
#pragma unroll
                    for (int b = 0; b < GB; ++b)
                        if (i + b < parts) {
#pragma unroll
                            for (int j = 0; j < JB; ++j)
                                if (j0 + j < RT) {
#pragma unroll
                                    for (int g = 0; g < 4; ++g)
#pragma unroll
                                        for (int e = 0; e < 4; ++e) racc[j0 + j][4 * g + e] += __builtin_bit_cast(f32x4, v[b][j][g])[e];
                                }
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        barrier();
        int k = 0;
        for (int t = 0; t + 1 < iters; ++t) {
#pragma unroll
            for (int j = 0; j < RT; ++j) {
                const int mt = 2 * j + rw < MT ? 2 * j + rw : 0;  // (an odd count's missing tile: computed on, never used)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 y4 = member == 0 ? *(const f32x4*)(yrow + 32 * mt + 8 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 0; e < 4; ++e) racc[j][4 * g + e] = y4[e];
                }
            }
            barrier();
            barrier();
            int s = k;
            for (int c = 0; c < nct; ++c) {                       // step c + 2
                const uint32_t base = nat16 + s * SLOT, xa = lds0 + OFF_X + (c & 1) * 2048 + lane * 16;
                u32x4 x0, x1, fr[D][G];
                lds_read16<0>(x0, xa);
                lds_read16<1024>(x1, xa);
                constexpr int NR = 2 * RT, NG = NR / G;
                auto fetch_group = [&](auto kc) {
                    constexpr int q = decltype(kc)::value, f = q * G;
                    if constexpr (f < NR) {
                        lds_read16<((f / RT) * MT + 2 * (f % RT)) * 1024>(fr[q % D][0], base);
                        lds_read16<(((f + 1) / RT) * MT + 2 * ((f + 1) % RT)) * 1024>(fr[q % D][1], base);
                    }
                };
                auto run = [&](auto self, auto kc) {
                    constexpr int q = decltype(kc)::value;
                    if constexpr (q < NG) {
                        fetch_group(std::integral_constant<int, q + D - 1>{});
                        lds_wait_n<G * (NG - 1 - q < D - 1 ? NG - 1 - q : D - 1)>();
                        if constexpr (q == 0) { lds_pin(x0); lds_pin(x1); }
#pragma unroll
                        for (int i = 0; i < G; ++i) lds_pin(fr[q % D][i]);
#pragma unroll
                        for (int i = 0; i < G; ++i) {
                            const int f = q * G + i;
                            racc[f % RT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fr[q % D][i]),
                                                                                   __builtin_bit_cast(bf16x8, f < RT ? x0 : x1), racc[f % RT], 0, 0, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        self(self, std::integral_constant<int, q + 1>{});
                    }
                };
                fetch_group(std::integral_constant<int, 0>{});
                run(run, std::integral_constant<int, 0>{});
                s = next(s, 1);
                if (c + 1 < nct) barrier();
            }
            if (G2 > 1) exchange(t);
            uint4* op = operands_at(k);                           // the residual's operands, for the U wavefronts
#pragma unroll
            for (int j = 0; j < RT; ++j)
                if (2 * j + rw < MT) {
                    op[(2 * (2 * j + rw)) * 64] = __builtin_bit_cast(uint4, cvt8<0>(racc[j], 1.f));
                    op[(2 * (2 * j + rw) + 1) * 64] = __builtin_bit_cast(uint4, cvt8<8>(racc[j], 1.f));
                }
            barrier();
            k = (k + nct) % kCoopSlots;
        }
        for (int c = 0; c < nct + 1; ++c) barrier();              // last iteration: no residual
        return;
    }

    // ---- GEMM-U and threshold ----
    const uint32_t tr8 = lds0 + ((lane >> 4) & 1) * (MT * 1024) + frag_slot(4 * lh + ((lane & 15) >> 2), lane & 1) * 16 +
                         ((lane >> 1) & 1) * 8;
    f32x4* st = (f32x4*)a.state + (rt * a.nct + c0) * 256 + lane;
    bf16x8 rb[NF];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {                             // x = 0: r = y
        f32x16 r;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 y4 = *(const f32x4*)(yrow + 32 * mt + 8 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) r[4 * g + e] = y4[e];
        }
        rb[2 * mt] = cvt8<0>(r, 1.f);
        rb[2 * mt + 1] = cvt8<8>(r, 1.f);
    }
    barrier();
    f32x16 u;
    f32x4 old[4];
    // fragments [F0, F1) of the chunk in `slot` into u
    auto part = [&](auto f0c, auto f1c, int slot) {
        constexpr int F0 = decltype(f0c)::value, F1 = decltype(f1c)::value, NG = (F1 - F0 + G - 1) / G;
        const uint32_t base = tr8 + slot * SLOT;
        u32x2 ft[D][G][2];
        auto fetch_group = [&](auto kc) {
            constexpr int q = decltype(kc)::value, f = F0 + q * G;
            if constexpr (f < F1) {
                lds_read8_tr<(f >> 1) * 1024 + (f & 1) * 256>(ft[q % D][0][0], base);
                lds_read8_tr<(f >> 1) * 1024 + (f & 1) * 256 + 128>(ft[q % D][0][1], base);
                lds_read8_tr<((f + 1) >> 1) * 1024 + ((f + 1) & 1) * 256>(ft[q % D][1][0], base);
                lds_read8_tr<((f + 1) >> 1) * 1024 + ((f + 1) & 1) * 256 + 128>(ft[q % D][1][1], base);
            }
        };
        auto run = [&](auto self, auto kc) {
            constexpr int q = decltype(kc)::value;
            if constexpr (q < NG) {
                fetch_group(std::integral_constant<int, q + D - 1>{});
                lds_wait_n<2 * G * (NG - 1 - q < D - 1 ? NG - 1 - q : D - 1)>();
                lds_pin(ft[q % D][0][0], ft[q % D][0][1]);
                lds_pin(ft[q % D][1][0], ft[q % D][1][1]);
#pragma unroll
                for (int i = 0; i < G; ++i) {
                    const u32x4 fa = __builtin_shufflevector(ft[q % D][i][0], ft[q % D][i][1], 0, 1, 2, 3);
                    u = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa), rb[F0 + q * G + i], u, 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                self(self, std::integral_constant<int, q + 1>{});
            }
        };
        static_assert((F1 - F0) % G == 0, "whole groups");
        if constexpr (NG > 0) {
            fetch_group(std::integral_constant<int, 0>{});
            run(run, std::integral_constant<int, 0>{});
        }
    };
    auto first_part = [&](int c, int slot, bool first) {
        if (!first) {
#pragma unroll
            for (int g = 0; g < 4; ++g) old[g] = st[(long long)(c * 4 + g) * 64];
        } else {
#pragma unroll
            for (int g = 0; g < 4; ++g) old[g] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) u[v] = 0.f;
        part(std::integral_constant<int, 0>{}, std::integral_constant<int, H>{}, slot);
    };
    auto second_part = [&](int c, int slot, bool last) {
        part(std::integral_constant<int, H>{}, std::integral_constant<int, NF>{}, slot);
        f32x16 x;
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = soft_threshold(old[v >> 2][v & 3] + a.mu * u[v], a.theta);
        if (!last) {
            uint4* xo = lds + (OFF_X + (c & 1) * 2048) / 16 + lane;
            xo[0] = __builtin_bit_cast(uint4, cvt8<0>(x, -1.f));
            xo[64] = __builtin_bit_cast(uint4, cvt8<8>(x, -1.f));
#pragma unroll
            for (int g = 0; g < 4; ++g) st[(long long)(c * 4 + g) * 64] = f32x4{x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
        } else if (row_ok) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = 32 * (c0 + c) + 8 * g + 4 * lh;
                if (a.Xb && col < a.ldxb)
                    *(uint2*)(a.Xb + row * a.ldxb + col) = uint2{f2bf_pk(x[4 * g], x[4 * g + 1]), f2bf_pk(x[4 * g + 2], x[4 * g + 3])};
                if (a.Xout) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < a.n) a.Xout[row * (long long)a.n + col + e] = x[4 * g + e];
                }
            }
        }
    };
    int k = 0;
    for (int t = 0; t < iters; ++t) {
        const bool last = t + 1 == iters;
        int s = k;
        for (int c = 0; c < nct + 1; ++c) {
            if ((c & 1) == wave) {
                if (c < nct) first_part(c, s, t == 0);
            } else if (c > 0 && c <= nct) {
                second_part(c - 1, next(s, kCoopSlots - 1), last);
            }
            s = next(s, 1);
            barrier();
        }
        if (!last) {
            uint4* op = operands_at(k);
            barrier();
#pragma unroll
            for (int f = 0; f < NF; ++f) rb[f] = __builtin_bit_cast(bf16x8, op[f * 64]);
        }
        k = (k + nct) % kCoopSlots;
    }
}

}  // namespace csat

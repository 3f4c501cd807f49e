// Compressed attention when only its output is wanted:  Z = softmax(Q K~^T / sqrt(d_k)) V~  (section 3), bf16, d a
// multiple of 32 up to 128, any m.  No row of A~ is ever stored: the stage call without A, the block with zero
// iterations and the column-wise reading take this kernel.
//
// What bounds it: 8 vector-instruction slots per score (maximum, scaled difference, exp2 at a quarter of the rate,
// sum, half a conversion) against d / 8 MFMA cycles, so the vector units, behind which the products run; and memory for Q and
// Z, once each.  So the scores of two tiles of m at a time go through one softmax step with a running maximum and
// sum per row, which keeps a wavefront at 128 registers (d <= 64): four wavefronts per SIMD fill each other's waits,
// where the kernel that also delivers A~ has to hold all of a row's scores until its maximum is known.  The running
// maximum is only moved (and the output rescaled) when a row's scores grow by more than 2^8 over it, and after the
// first step that almost never happens.  The weights are 2^(s - ref - shift) with 2^shift >= 256 m: their sum is at most
// 1, so the unnormalised output cannot overflow where the normalised one does not.
//
// Layout as in csat_attention.h: everything transposed, S^T = K~ Q^T puts a query row into one lane pair, and the
// scores' accumulator layout is the B operand of Z^T = V~^T P^T.  The fragments of K~ and V~ of a head sit in LDS:
// all of them where they fit (RESIDENT; a workgroup then takes several rounds of one row tile per wavefront), else
// two tiles of m at a time, the next two in flight.
//
// Measured, stage call without A~ (rocprofv3): 48 heads x 8192 queries, m = 256, d = 64: 42 us plus 5 us of packing, where
// the kernel that keeps whole rows plus a product GEMM took 197 + 78 + 10 us (it wrote A~ and its bf16 copy, 0.6 GB, and
// read the copy back); floor: 100 MB of Q and Z = 21 us, 1.6e6 wavefront scores x 30 cycles of vector issue = 22 us.
// 48 heads x 1600 queries, m = 392, K~ as a pair, Z^T wanted (two tiles at a time): 29 us against 86 + 44.
#pragma once
#include <cfloat>

#include "csat_ista_fused.h"      // slab_slot
#include "csat_kernels.h"

namespace csat {

struct AttentionZArgs {
    const bf16_t* Q;               // [heads][n_q][d]
    const uint4* Kf;               // [heads][MT][PARTS * d / 16][64]: K~ (or its (hi | lo) pair) as A fragments
    const uint4* Vf;               // [heads][MT][d / 32][2][64]: V~ as A fragments of the output product
    bf16_t* Z;                     // [heads][n_q][d], or null
    bf16_t* ZT;                    // optional Z^T per head as a (hi | lo) pair: hi at [dd][row], lo at [dd][ldT / 2 + row]
    long long ldT, strideT;
    int n_q, m, MT;
    int tiles_per_head, rounds, wg_per_head;
    float scale_log2e;
    float shift;                   // 8 + log2(m), rounded up
};

// K~ rows [heads][m][PARTS * d] and V~ rows [heads][m][d] -> the fragments above, zero beyond m; either source may be
// null (its fragments exist already).  One thread per 16-byte piece; nk + nv pieces.
static __global__ void pack_kv_fragments_kernel(const bf16_t* K, const bf16_t* V, int m, int d, int parts, int MT,
                                                uint4* Kf, uint4* Vf, long long nk, long long nv) {
    long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = (int)(idx & 63), i = lane & 31, h = lane >> 5;
    if (idx < nk) {
        const int ns = parts * d / 16;
        const int s = (int)((idx >> 6) % ns);
        const long long t = (idx >> 6) / ns;                 // head * MT + mt
        const int mt = (int)(t % MT);
        const long long z = t / MT;
        const int r = 32 * mt + i;
        Kf[idx] = r < m ? *(const uint4*)(K + (z * m + r) * (long long)(parts * d) + 16 * s + 8 * h) : uint4{0u, 0u, 0u, 0u};
        return;
    }
    idx -= nk;
    if (idx >= nv) return;
    const int nz = d / 32;
    const int sl = (int)((idx >> 6) & 1);
    const int dt = (int)((idx >> 7) % nz);
    const long long t = (idx >> 7) / nz;
    const int mt = (int)(t % MT);
    const long long z = t / MT;
    const bf16_t* v = V + z * (long long)m * d + 32 * dt + i;
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 8; q += 2) {
        const int k0 = 32 * mt + 16 * sl + slab_slot(h, q), k1 = 32 * mt + 16 * sl + slab_slot(h, q + 1);
        const uint32_t lo = k0 < m ? v[(long long)k0 * d] : 0, hi = k1 < m ? v[(long long)k1 * d] : 0;
        w[q / 2] = lo | (hi << 16);
    }
    Vf[idx] = uint4{w[0], w[1], w[2], w[3]};
}

// LDS: PT tiles of m per slot, the tiles' K~ fragments, then V~'s
constexpr int kAttnZTiles = 2;
constexpr int attention_z_slot_bytes(int d, int parts) { return kAttnZTiles * (parts + 1) * (d / 16) * 1024; }
constexpr int kAttnZWaves = 8;

template <int NZ, int PARTS, bool RESIDENT>
__global__ __launch_bounds__(64 * kAttnZWaves, NZ <= 2 ? 4 : 2) void attention_z_kernel(AttentionZArgs a) {
    constexpr int NG = 2 * NZ, NS = PARTS * NG, D = 32 * NZ, NW = kAttnZWaves;
    constexpr int PT = kAttnZTiles, SLOTF = PT * (NS + NG);         // tiles, fragments per slot
    extern __shared__ uint4 lds[];
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int z = blockIdx.x / a.wg_per_head, chunk = blockIdx.x % a.wg_per_head;
    const int steps = (a.MT + PT - 1) / PT;
    const uint4* kf = a.Kf + (long long)z * a.MT * NS * 64;
    const uint4* vf = a.Vf + (long long)z * a.MT * NG * 64;

    // tiles PT p .. of m into slot `slot`; a tile beyond the last one as zeros (its scores are masked)
    auto stage = [&](int p, int slot) {
        const int nt = a.MT - PT * p < PT ? a.MT - PT * p : PT;
        for (int f = wave; f < SLOTF; f += NW) {
            const bool isk = f < PT * NS;
            const int g = isk ? f : f - PT * NS, per = isk ? NS : NG;
            const uint4* src = (isk ? kf : vf) + ((long long)PT * p * per + g) * 64 + lane;
            if (g < nt * per) __builtin_amdgcn_global_load_lds((glb_ptr_t)src, (lds_ptr_t)((char*)lds + (slot * SLOTF + f) * 1024), 16, 0, 0);
            else lds[(slot * SLOTF + f) * 64 + lane] = uint4{0u, 0u, 0u, 0u};
        }
    };
    if constexpr (RESIDENT) {
        for (int p = 0; p < steps; ++p) stage(p, p);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
    const float sl = a.scale_log2e;
    for (int r = 0; r < a.rounds; ++r) {
        const int rt = (chunk * a.rounds + r) * NW + wave;
        const bool active = rt < a.tiles_per_head;           // wavefront-uniform
        if (RESIDENT && !active) break;                      // (no barriers after the staging)
        const int row = rt * 32 + li;
        const bool row_ok = active && row < a.n_q;
        const long long grow = (long long)z * a.n_q + (row_ok ? row : a.n_q - 1);
        uint4 qf[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) qf[g] = *(const uint4*)(a.Q + grow * D + (2 * g + lh) * 8);
        f32x16 zacc[NZ];
#pragma unroll
        for (int dt = 0; dt < NZ; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) zacc[dt][v] = 0.f;
        // the row's reference score, what a weight's exponent takes off for it (scores of -inf have weight 0, also before the
        // row's first finite one) and this lane's share of the row's sum
        float ref = -INFINITY, off = __builtin_fmaf(FLT_MAX, sl, -a.shift), sum = 0.f;
        auto step = [&](int p, const uint4* slot) {
            f32x16 s[PT];
#pragma unroll
            for (int t = 0; t < PT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) s[t][v] = 0.f;
#pragma unroll
            for (int q = 0; q < NS; ++q) {
#pragma unroll
                for (int t = 0; t < PT; ++t) mfma_group<bf16_t>(slot[(t * NS + q) * 64 + lane], qf[q % NG], s[t]);
                if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);      // fragments of two groups in flight, not of all: registers
            }
            if (32 * PT * (p + 1) > a.m) {                   // uniform: only the last step overhangs m
#pragma unroll
                for (int t = 0; t < PT; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (32 * (PT * p + t) + 8 * (v >> 2) + 4 * lh + (v & 3) >= a.m) s[t][v] = -INFINITY;
            }
            float mx = s[0][0];
#pragma unroll
            for (int t = 0; t < PT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[t][v]);
            {   // the partner lane holds the row's other scores of these tiles
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
            }
            if (__builtin_amdgcn_ballot_w64((mx - ref) * sl > 8.f) != 0) {      // (both lanes of a pair agree)
                const float nm = fmaxf(mx, ref), base = fmaxf(nm, -FLT_MAX), alpha = __builtin_amdgcn_exp2f((ref - base) * sl);     // first step: 2^(-inf) = 0
                ref = nm;
                off = __builtin_fmaf(-base, sl, -a.shift);
                sum *= alpha;
#pragma unroll
                for (int dt = 0; dt < NZ; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) zacc[dt][v] *= alpha;
            }
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                float e[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    e[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][v], sl, off));
                    sum += e[v];
                }
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
                    const uint4 pf = uint4{f2bf_pk(e[8 * h2], e[8 * h2 + 1]), f2bf_pk(e[8 * h2 + 2], e[8 * h2 + 3]),
                                           f2bf_pk(e[8 * h2 + 4], e[8 * h2 + 5]), f2bf_pk(e[8 * h2 + 6], e[8 * h2 + 7])};
#pragma unroll
                    for (int dt = 0; dt < NZ; ++dt) mfma_group<bf16_t>(slot[(PT * NS + t * NG + dt * 2 + h2) * 64 + lane], pf, zacc[dt]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if constexpr (RESIDENT) {
            for (int p = 0; p < steps; ++p) step(p, lds + p * SLOTF * 64);
        } else {
            stage(0, 0);
            for (int p = 0; p < steps; ++p) {
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();                             // step p's tiles are there, and step p - 1's have been read
                if (p + 1 < steps) stage(p + 1, (p + 1) & 1);
                step(p, lds + (p & 1) * SLOTF * 64);
            }
            __syncthreads();
        }
        {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
            sum = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
        const float inv = 1.f / sum;
#pragma unroll
        for (int dt = 0; dt < NZ; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) zacc[dt][v] *= inv;
        if (a.Z) {
            // lane (i, h) holds columns 8 g + 4 h .. + 3 of its row: the pair exchanges so that each lane stores 16 bytes
            // (h = 0 the columns of an even g, h = 1 those of the next)
            bf16_t* zr = a.Z + ((long long)z * a.n_q + row) * D;
#pragma unroll
            for (int dt = 0; dt < NZ; ++dt)
#pragma unroll
                for (int g = 0; g < 4; g += 2) {
                    const uint32_t a0 = f2bf_pk(zacc[dt][4 * g], zacc[dt][4 * g + 1]), a1 = f2bf_pk(zacc[dt][4 * g + 2], zacc[dt][4 * g + 3]);
                    const uint32_t b0 = f2bf_pk(zacc[dt][4 * g + 4], zacc[dt][4 * g + 5]), b1 = f2bf_pk(zacc[dt][4 * g + 6], zacc[dt][4 * g + 7]);
                    const auto s0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
                    if (row_ok) *(uint4*)(zr + 32 * dt + 8 * (g + lh)) = uint4{s0[0], s1[0], s0[1], s1[1]};
                }
        }
        if (a.ZT && row_ok) {
            long long ld = a.ldT;
            asm volatile("" : "+s"(ld));       // (addresses formed here, not kept in registers across the rounds)
            bf16_t* t = a.ZT + (long long)z * a.strideT + row + 4 * lh * ld;
#pragma unroll
            for (int dt = 0; dt < NZ; ++dt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float x = zacc[dt][v];
                    const bf16_t hi = f2bf(x);
                    t[0] = hi;
                    t[ld / 2] = f2bf(x - bf2f(hi));
                    t += (v & 3) == 3 ? 5 * ld : ld;       // rows 8 (v / 4) + 4 h + v % 4 of the tile
                    asm volatile("" : "+v"(t));
                }
        }
    }
}

}  // namespace csat

// float "NT" GEMM  C[M,N] = sum_k A[M,k] * Bt[N,k]  on the bf16 matrix cores, without giving up float precision.
//
// The float MFMA (32x32x2) tops out at 157 TFLOP/s, a sixteenth of the bf16 one.  A float of at least 2^-109 is the exact
// sum of three bf16 values (hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid: 8 bits each, round to nearest), so the product of
// two floats is nine bf16 products, each exact in the MFMA's float accumulation.  The three smallest (mid lo, lo mid,
// lo lo) are left out: together at most 2^-24 of the product (mid is up to 2^-8 of its operand, lo up to 2^-17), the size of one
// float accumulation step's rounding, and usually far less.  Six bf16 MFMAs in place of eight float ones that each take
// twice as long: 6/16 of the time.
//
// Workgroup: 4 wavefronts (2 x 2), tile 128 x 64, 32 floats of K per step.  The operands are split on the way from the
// prefetch registers into LDS (5.5 vector instructions per element, under the other workgroups' MFMAs: three workgroups
// per CU), three planes of 64-byte rows whose four 16-byte chunks are XOR-swizzled with row / 2 (conflict-free
// fragment reads).  What bounds it is each workgroup's chain of load, split, barrier and MFMAs, so occupancy counts for
// more than operand re-use.  19200 x 1600 x 392 (ISTA update, with its epilogue): 193 us = 125 TFLOP/s of float
// arithmetic, three workgroups per CU; 200 us with 128 x 128 tiles and two; the residual product, 19200 x 392 x 1600:
// 176 us, 214 with two workgroups per CU.  The forward of that shape (20 of one, 19 of the other) went from 12.7 ms on
// the float MFMA to 7.3 ms.
// Error against float64 over the shapes measured (K = 30 to 4096): 0.3 to 1.0 of the float MFMA's; with one accumulator
// for all six products it was up to 1.4 of it, where the operand is sparse.
//
// Infinities and NaN: inf - inf in the split, or inf times a zero mid part, makes an accumulator NaN that the float
// product would have as inf.  Operands below 2^-109 lose the bits that their parts would hold below bf16's smallest number
// (at 10^-37 all but ten); where that matters, in rows without larger ones, the sums are as small.  A workgroup that
// finds an accumulator that is not finite, or not zero but below 2^-90, therefore computes its tile again with the float MFMA.
#pragma once
#include "csat_kernels.h"

namespace csat {

// x0, x1 -> the packed bf16 pairs of their three parts
__device__ __forceinline__ void split3(float x0, float x1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    hi = f2bf_pk(x0, x1);
    const float r0 = x0 - __uint_as_float(hi << 16), r1 = x1 - __uint_as_float(hi & 0xffff0000u);
    mid = f2bf_pk(r0, r1);
    lo = f2bf_pk(r0 - __uint_as_float(mid << 16), r1 - __uint_as_float(mid & 0xffff0000u));
}

// Whether results of split operands may not be what float arithmetic gives (see above)
struct SplitSuspect {
    uint32_t low = 0xffffffffu, high = 0u;      // smallest non-zero and largest magnitude, as bits shifted left
    __device__ __forceinline__ void add(float v) {
        const uint32_t u = __float_as_uint(v) << 1;
        low = low < u - 1 ? low : u - 1;        // (zero: 2^32 - 1)
        high = high > u ? high : u;
    }
    __device__ __forceinline__ bool any() const { return low < 2 * __float_as_uint(0x1p-90f) - 1 || high >= 0xff000000u; }
};

constexpr int kF32TileM = 128, kF32TileN = 64;

template <typename Epi>
__global__ __launch_bounds__(256, 3) void gemm_nt_f32_split_kernel(GemmArgs g, Epi epi) {
    constexpr int BM = kF32TileM, BN = kF32TileN, WM = 2, WN = 2, TM = BM / (WM * 32), TN = BN / (WN * 32);
    constexpr int RA = BM / 32, RB = BN / 32;               // float4 per thread and step
    constexpr int PLANE_A = BM * 4, PLANE_B = BN * 4;       // 16-byte chunks per plane
    constexpr int kSplit = 3 * (PLANE_A + PLANE_B), kPlain = (BM + BN) * kLdsRowChunks;
    __shared__ uint4 lds[kSplit > kPlain ? kSplit : kPlain];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN, li = lane & 31, lh = lane >> 5;
    const int z = blockIdx.z;
    // All column tiles of a row tile on one XCD (workgroups go round-robin over the eight): its rows of A are fetched
    // into one L2.  g.raster: column tiles; the grid is padded to whole groups of eight row tiles.
    const int slot = blockIdx.x >> 3;
    const long long row0 = ((long long)(slot / g.raster) * 8 + (blockIdx.x & 7)) * BM, col0 = (long long)(slot % g.raster) * BN;
    if (!has_late_rule<Epi>::value && row0 >= g.M) return;      // (what may run in the product's place shares out the rows itself)
    if constexpr (has_rule<Epi>::value) {
        if (epi.rule.sparse()) return;
    }
    uint2 words{0u, 0u};
    if constexpr (has_late_rule<Epi>::value) words = epi.rule.words();
    u32x4 packed{1u, 0u, 0u, 0u};
    if constexpr (has_screen<Epi>::value)
        packed = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc((void*)g.screen, 0, g.screen ? 16 : 0, kBufferFlags), 0, 0, 0);
    const float* A = (const float*)g.A + (long long)z * g.strideA;
    const float* Bt = (const float*)g.Bt + (long long)z * g.strideB;
    const int kchunks = (g.K + 3) / 4, ksteps = (kchunks + 7) / 8;

    // thread: chunk tid % 8 of rows tid / 8 + 32 i
    const int lrow = tid >> 3, lchunk = tid & 7;
    f32x4 ra[RA], rb[RB];
    auto load_global = [&](int ks) {
        const int kc = ks * 8 + lchunk;
#pragma unroll
        for (int i = 0; i < RA; ++i) {
            const long long r = row0 + lrow + 32 * i;
            ra[i] = r < g.M && kc < kchunks ? *(const f32x4*)(A + r * g.lda + (long long)kc * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const long long r = col0 + lrow + 32 * i;
            rb[i] = r < g.N && kc < kchunks ? *(const f32x4*)(Bt + r * g.ldb + (long long)kc * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // half `lchunk & 1` of 16-byte chunk lchunk / 2 of row r
    auto store_row = [&](const f32x4& v, uint4* plane0, int plane, int r) {
        uint32_t p[3][2];
        split3(v[0], v[1], p[0][0], p[1][0], p[2][0]);
        split3(v[2], v[3], p[0][1], p[1][1], p[2][1]);
        const int c = (lchunk >> 1) ^ ((r >> 1) & 3);
#pragma unroll
        for (int q = 0; q < 3; ++q)
            *(uint2*)((char*)(plane0 + q * plane + r * 4 + c) + (lchunk & 1) * 8) = uint2{p[q][0], p[q][1]};
    };
    uint4* sA = lds;
    uint4* sB = lds + 3 * PLANE_A;

    // hi hi apart from the five smaller products: the large sum is then rounded once per 16 K steps
    f32x16 acc[TM][TN], corr[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = corr[i][j][v] = 0.f;
    };
    clear();
    load_global(0);
    if constexpr (has_late_rule<Epi>::value) {
        static_assert(Epi::kLds <= sizeof(lds), "LDS");
        if (epi.rule.sparse(words)) {
            epi.instead(lds);
            return;
        }
        if (row0 >= g.M) return;
    }
    if constexpr (has_screen<Epi>::value) {
        if (g.screen && __builtin_amdgcn_readfirstlane(packed[0]) == 0) {
            if (row0 >= (long long)(uint32_t)__builtin_amdgcn_readfirstlane(packed[2])) return;
            epi.packed();
        }
    }
    for (int ks = 0; ks < ksteps; ++ks) {
#pragma unroll
        for (int i = 0; i < RA; ++i) store_row(ra[i], sA, PLANE_A, lrow + 32 * i);
#pragma unroll
        for (int i = 0; i < RB; ++i) store_row(rb[i], sB, PLANE_B, lrow + 32 * i);
        __syncthreads();
        if (ks + 1 < ksteps) load_global(ks + 1);
#pragma unroll
        for (int gk = 0; gk < 2; ++gk) {
            bf16x8 fa[3][TM], fb[3][TN];
            const int c = (2 * gk + lh) ^ ((li >> 1) & 3);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    fa[q][i] = __builtin_bit_cast(bf16x8, sA[q * PLANE_A + ((wm * TM + i) * 32 + li) * 4 + c]);
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    fb[q][j] = __builtin_bit_cast(bf16x8, sB[q * PLANE_B + ((wn * TN + j) * 32 + li) * 4 + c]);
            }
            constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        if (p < 5) corr[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[PA[p % 5]][i], fb[PB[p % 5]][j], corr[i][j], 0, 0, 0);
                        else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][i], fb[0][j], acc[i][j], 0, 0, 0);
                    }
        }
        __syncthreads();
    }

    SplitSuspect suspect;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[i][j][v] += corr[i][j][v];
                suspect.add(acc[i][j][v]);
            }
    if (__syncthreads_or(suspect.any())) {      // the tile again on the float MFMA, one K step at a time
        clear();
        for (int ks = 0; ks < ksteps; ++ks) {
            load_global(ks);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < RA; ++i) lds[(lrow + 32 * i) * kLdsRowChunks + lchunk] = __builtin_bit_cast(uint4, ra[i]);
#pragma unroll
            for (int i = 0; i < RB; ++i) lds[(BM + lrow + 32 * i) * kLdsRowChunks + lchunk] = __builtin_bit_cast(uint4, rb[i]);
            __syncthreads();
            for (int gk = 0; gk < kRowChunks / 2; ++gk) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        mfma_group<float>(lds[((wm * TM + i) * 32 + li) * kLdsRowChunks + 2 * gk + lh],
                                          lds[(BM + (wn * TN + j) * 32 + li) * kLdsRowChunks + 2 * gk + lh], acc[i][j]);
            }
        }
    }

#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const long long c = col0 + (wn * TN + j) * 32 + li, r0 = row0 + (wm * TM + i) * 32 + 4 * lh;
            if constexpr (has_rows_epilogue<Epi>::value) {
                epi.rows(r0, c, acc[i][j]);
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) epi(z, r0 + 8 * (v / 4) + (v % 4), c, acc[i][j][v]);
            }
        }
}

}  // namespace csat

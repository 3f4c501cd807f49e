// Decoders over the support of a sparse iterate: products with the iterate that cost what its non-zero coefficients cost.
//
// A thresholded iterate of the decoders here is mostly zeros (short_video: 4 to 8 of a row's 1600 coefficients), and which
// rows are is known only on the device, after the first threshold.  So the first iteration runs as always, a kernel
// counts what it left (support_count_kernel), and behind it both ways are launched, of which one returns at once: the
// products over all columns, or the kernels here.  Every workgroup reads the same count, so a call takes one way as a whole
// and repeats its bits.
#pragma once
#include "csat_kernels.h"

namespace csat {

// Adds the non-zero float4 that the mask bytes name to ctl[0].
static __global__ __launch_bounds__(256) void support_count_kernel(const uint4* mask, long long chunks, uint32_t* ctl) {
    uint32_t n = 0;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < chunks; i += (long long)gridDim.x * 256) {
        const uint4 v = mask[i];
        n += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(ctl, part[0] + part[1] + part[2] + part[3]);
}

// DT[j][i] = D[i][j], both [n, ld] with zero pads, 64 x 64 tiles through LDS.
static __global__ __launch_bounds__(256) void support_transpose_kernel(SupportRule rule, const bf16_t* D, bf16_t* DT, int n, int ld) {
    if (!rule.sparse()) return;
    __shared__ bf16_t tile[64][66];
    const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64, tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int i = ty; i < 64; i += 4) tile[i][tx] = r0 + i < n && c0 + tx < n ? D[(long long)(r0 + i) * ld + c0 + tx] : (bf16_t)0;
    __syncthreads();
    for (int i = ty; i < 64; i += 4)
        if (c0 + i < n && r0 + tx < ld) DT[(long long)(c0 + i) * ld + r0 + tx] = tile[tx][i];
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// The unrolled decoder over the support: all layers of a row in one wavefront, alpha <- eta(W + alpha + D alpha) with W = B y in
// registers and D's columns (rows of DT) gathered for the non-zero alpha only.  Lane l holds eight columns of every 512, 8l to
// 8l + 7, and the R % 8 columns of a last, narrower piece.  The coefficients go into the products rounded to bf16, as in
// the layers over all columns; two columns' elements are paired for the two-product MAC.  The final product C = alpha V
// runs over the same list.
//
// What bounds it: the gather of 2 n bytes per coefficient and layer out of L2 (D of n = 1600 is 5 MB), 37 GB in 1.8 ms of the
// 2.2 that short_video's 19 layers take (2 to 11 coefficients a row, most rows none and one in a thousand 240; 19 layers over
// all columns 8.4 ms); the rest is the thresholds, four instructions per 64 columns, and reading W.  Wavefronts in flight
// count: 128 registers (four a SIMD) 2.2 ms, 168 (three) 2.6.
constexpr int kSupportMaxLayers = 256;
struct ListaSupportArgs {
    SupportRule rule;
    const f32x4* W; long long tiles_n;      // accumulator order (EpiListaFirstTiled)
    const bf16_t* DT; int ld;
    float* X;
    const bf16_t* V; bf16_t* C;
    long long rows;
    int n_q, n, d, iters;
    float theta[kSupportMaxLayers];
};

template <int R>
__global__ __launch_bounds__(256, R <= 32 ? 4 : 2) void lista_support_kernel(ListaSupportArgs a) {
    constexpr int FULL = R / 8, TAIL = R % 8;
    static_assert(TAIL == 0 || TAIL == 2 || TAIL == 4, "a lane's share of the last piece is one load");
    if (!a.rule.sparse()) return;
    extern __shared__ uint4 lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ncol = (int)a.tiles_n * 32;
    const long long row0 = (long long)blockIdx.x * 4, row = row0 + wave;
    // column of register k
    auto column = [&](int k) { return k < 8 * FULL ? 512 * (k / 8) + 8 * lane + k % 8 : 512 * FULL + TAIL * lane + (k - 8 * FULL); };

    // W of the workgroup's four rows: they are one float4 per column
    float w[R], acc[R];
    {
        float* stage = (float*)lds;
        const long long rt = row0 >> 5;
        const int piece = (int)((row0 & 31) >> 2);      // rows 8 (piece / 2) + 4 (piece % 2) .. + 3 of the tile
        const f32x4* src = a.W + rt * a.tiles_n * 256 + (piece >> 1) * 64 + (piece & 1) * 32;
        for (int c = threadIdx.x; c < ncol; c += 256) {
            const f32x4 v = __builtin_nontemporal_load(src + (long long)(c >> 5) * 256 + (c & 31));
#pragma unroll
            for (int e = 0; e < 4; ++e) stage[e * ncol + c] = v[e];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int c = column(k);
            w[k] = acc[k] = c < a.n ? stage[wave * ncol + c] : 0.f;
        }
        __syncthreads();
    }
    if (row >= a.rows) return;
    uint32_t* list = (uint32_t*)lds + wave * ncol;      // (column << 16 | coefficient) of this row

    // eta: x in place of u; the list of its non-zeros; NEXT: u of the next layer starts at W + x
    auto threshold = [&](float theta, auto next) -> int {
        int cnt = 0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const float u = acc[k], x = u - __builtin_amdgcn_fmed3f(u, -theta, theta);
            const bool nz = x != 0.f;
            const uint64_t some = __builtin_amdgcn_ballot_w64(nz);
            if (some) {
                if (nz) list[cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u))] =
                    (uint32_t)column(k) << 16 | f2bf(x);
                cnt += __popcll(some);
            }
            acc[k] = decltype(next)::value ? w[k] + x : x;
        }
        __builtin_amdgcn_wave_barrier();
        return cnt;
    };
    struct Col { u32x4 f[FULL ? FULL : 1]; uint32_t t[2]; };
    auto load = [&](uint32_t entry) {
        Col c;
        __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.DT + (long long)(entry >> 16) * a.ld), 0, a.ld * 2, kBufferFlags);
#pragma unroll
        for (int k = 0; k < FULL; ++k) c.f[k] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, k * 1024, 0);
        if constexpr (TAIL == 4) {
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, lane * 8, FULL * 1024, 0);
            c.t[0] = t[0]; c.t[1] = t[1];
        }
        if constexpr (TAIL == 2) c.t[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, FULL * 1024, 0);
        return c;
    };
    auto add = [&](const Col& p, const Col& q, uint32_t e0, uint32_t e1) {
        const bf16x2 x = __builtin_bit_cast(bf16x2, (e0 & 0xffffu) | e1 << 16);
        auto two = [&](uint32_t dp, uint32_t dq, float& lo, float& hi) {
            lo = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(dq, dp, 0x05040100u)), x, lo, false);
            hi = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(dq, dp, 0x07060302u)), x, hi, false);
        };
#pragma unroll
        for (int k = 0; k < FULL; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) two(p.f[k][e], q.f[k][e], acc[8 * k + 2 * e], acc[8 * k + 2 * e + 1]);
#pragma unroll
        for (int e = 0; e < TAIL / 2; ++e) two(p.t[e], q.t[e], acc[8 * FULL + 2 * e], acc[8 * FULL + 2 * e + 1]);
    };

    for (int t = 0; t + 1 < a.iters; ++t) {
        const int cnt = threshold(a.theta[t], std::true_type{});
        for (int base = 0; base < cnt; base += 64) {
            const uint32_t mine = base + lane < cnt ? list[base + lane] : 0u;       // (0: column 0 with coefficient 0)
            const int c = cnt - base < 64 ? cnt - base : 64;
            for (int e = 0; e < c; e += 4) {
                const uint32_t e0 = __builtin_amdgcn_readlane(mine, e), e1 = __builtin_amdgcn_readlane(mine, e + 1);
                const Col p = load(e0), q = load(e1);
                if (e + 2 < c) {
                    const uint32_t e2 = __builtin_amdgcn_readlane(mine, e + 2), e3 = __builtin_amdgcn_readlane(mine, e + 3);
                    const Col p2 = load(e2), q2 = load(e3);
                    add(p, q, e0, e1);
                    add(p2, q2, e2, e3);
                } else {
                    add(p, q, e0, e1);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        // an infinite coefficient makes NaN of the pads
#pragma unroll
        for (int k = 0; k <= FULL; ++k)
            if (512 * (k + 1) > a.n || k == FULL) {
#pragma unroll
                for (int e = 8 * k; e < 8 * k + 8 && e < R; ++e) acc[e] = column(e) < a.n ? acc[e] : 0.f;
            }
    }
    const int cnt = threshold(a.theta[a.iters - 1], std::false_type{});
    if (a.X) {
        float* X = a.X + row * a.n;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int c = column(k);
            if (c < a.n) X[c] = acc[k];
        }
    }
    if (a.C) {
        const bf16_t* V = a.V + row / a.n_q * a.n * (long long)a.d;
        for (int c = lane; c < a.d; c += 64) {
            float s = 0.f;
            int e = 0;
            for (; e + 4 <= cnt; e += 4) {
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = bf2f(V[(long long)(list[e + j] >> 16) * a.d + c]);
#pragma unroll
                for (int j = 0; j < 4; ++j) s = fmaf(bf2f((bf16_t)list[e + j]), v[j], s);
            }
            for (; e < cnt; ++e) s = fmaf(bf2f((bf16_t)list[e]), bf2f(V[(long long)(list[e] >> 16) * a.d + c]), s);
            a.C[row * a.d + c] = f2bf(s);
        }
    }
}

}  // namespace csat

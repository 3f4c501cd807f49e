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

// n more in ctl[0]; a sum that a word does not hold sets ctl[1] (a dense iterate, whose sum would read as next to nothing).
__device__ __forceinline__ void support_add(uint32_t* ctl, float n) {
    const uint32_t more = n < 4294967040.f ? (uint32_t)n : 0xffffffffu, before = atomicAdd(ctl, more);
    if (before + more < before) ctl[1] = 1u;
}
// Adds the non-zero float4 that the mask bytes name to ctl[0].
// (packed rows, csat_screen.h: of their 32-row tiles, the number scaled to all rows, which the limit is for, and by `packed`, the limit's ratio to theirs)
// v (optional): ctl[1] is set where one of its pieces (bf16) holds an infinity or NaN.
static __global__ __launch_bounds__(256) void support_count_kernel(const uint4* mask, long long chunks, uint32_t* ctl, const uint32_t* screen, float packed, long long rows, const uint4* v,
                                                                   long long v_pieces) {
    if (holds_unbounded<bf16_t>(v, v_pieces, (long long)blockIdx.x * 256 + threadIdx.x, (long long)gridDim.x * 256)) ctl[1] = 1u;
    uint32_t n = 0;
    float scale = 1.f;
    if (screen && screen[0] == 0) {
        const long long left = screen[2];
        chunks = chunks / ((rows + 31) / 32) * ((left + 31) / 32);
        scale = left > 0 ? packed * rows / left : 0.f;
    }
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < chunks; i += (long long)gridDim.x * 256) {
        const uint4 v = mask[i];
        n += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) support_add(ctl, (part[0] + part[1] + part[2] + part[3]) * scale);
}

// DT[j][i] = D[i][j], both [n, ld] with zero pads, 64 x 64 tiles through LDS.
static __global__ __launch_bounds__(256) void support_transpose_kernel(SupportRule rule, const bf16_t* D, bf16_t* DT, int n, int ld) {
    if (!rule.sparse()) return;
    rule.note();
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

// r = y - Phi x over the support of the large-tile decoder's iterate (accumulator order with its masks, EpiIstaUpdateTiled), for
// the next iteration's operand R.  A wavefront takes four rows, those of one float4 of the iterate (a quad): it collects the columns
// whose float4 is not zero from the mask bytes, 64 at a time, and adds their multiples of Phi's columns (rows of PhiT, lane l
// elements 8l to 8l + 7 of every 512 and MR % 8 of a last piece) to the four sums.  Coefficients are rounded to bf16 as in the
// product over all columns.  The numbers of coefficients differ widely between rows, so the four wavefronts of a workgroup
// share out the columns of a quad with more than kSupportOwn of them (13 104 rows, n = 11 744, 100 pieces a quad on average: a forward
// 9.9 ms over all columns, 7.4 so).  A quad without any has r = y: nothing is written where R holds that already.
//
// What bounds it: with hardly any coefficient the masks, 16 us for 28 544 rows, n = 1824 (41 with every row of R written again, the
// product over all columns 118); else the gather, 2 m bytes a column: 38 976 rows, n = 9744, m = 1024, 5 coefficients a row 142 us (790).
// Wavefronts in flight count: with eight a CU, in the product's place, 19 and 189.
struct ResidualSupportArgs {
    const uint8_t* Mask; const f32x4* Xs; long long tiles_n;
    const bf16_t* PhiT; int ldm;
    const float* Y; long long ldY;
    bf16_t* R;
    uint8_t* Same;      // [quads] 1: R holds the quad's y (read from the second launch on: before it, it holds every row's)
    long long rows;
    int m, first;
    const uint32_t* screen = nullptr; const float* Yp = nullptr; long long ldYp = 0;      // packed rows (csat_screen.h) and their y
};
constexpr int kSupportOwn = 64, kSupportList = 1024 + 128;
template <int MR, int WAVES>
struct ResidualSupportLds {
    uint16_t lists[WAVES][kSupportList];
    float part[WAVES][64 * MR];
    int heavy[3];        // bit w: wavefront w's quad is shared; a word each for three rounds in turn
};

// Workgroup `block` of `blocks`, of WAVES wavefronts.
template <int MR, int kSupportWaves>
__device__ __forceinline__ void residual_support(ResidualSupportArgs a, ResidualSupportLds<MR, kSupportWaves>& l, long long block, long long blocks) {
    constexpr int FULL = MR / 8, TAIL = MR % 8;
    static_assert(TAIL == 0 || TAIL == 2 || TAIL == 4, "a lane's share of the last piece is one load");
    auto& lists = l.lists;
    auto& part = l.part;
    auto& heavy = l.heavy;
    if (a.screen && a.screen[0] == 0) {
        a.rows = a.screen[2];
        a.Y = a.Yp;
        a.ldY = a.ldYp;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint16_t* list = lists[wave];
    const long long quads = (a.rows + 3) / 4, step = blocks * kSupportWaves;
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    auto column = [&](int k) { return k < 8 * FULL ? 512 * (k / 8) + 8 * lane + k % 8 : 512 * FULL + TAIL * lane + (k - 8 * FULL); };
    // bit i: column 32 ct + 16 (lane & 1) + i of the quad, ct = ct0 + lane / 2
    auto scan = [&](long long quad, long long ct0, long long ct1) {
        const long long ct = ct0 + (lane >> 1);
        if (ct >= ct1) return 0u;
        const uint4 v = *(const uint4*)(a.Mask + ((quad >> 3) * a.tiles_n + ct) * 64 + (quad & 1) * 32 + (lane & 1) * 16);
        const int g = (int)(quad & 7) >> 1;
        auto four = [&](uint32_t w) { w = (w >> g) & 0x01010101u; return (w | w >> 7 | w >> 14 | w >> 21) & 15u; };
        return four(v.x) | four(v.y) << 4 | four(v.z) << 8 | four(v.w) << 12;
    };

    if (threadIdx.x < 3) heavy[threadIdx.x] = 0;
    __syncthreads();
    int round = 0;
    for (long long quad0 = block * kSupportWaves; quad0 < quads; quad0 += step, round = round == 2 ? 0 : round + 1) {
        const long long own = quad0 + wave;
        int pieces = 0;
        if (own < quads) {
            for (long long ct0 = 0; ct0 < a.tiles_n; ct0 += 32) pieces += __popc(scan(own, ct0, a.tiles_n));
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) pieces += __shfl_xor(pieces, o, 64);
            pieces = __builtin_amdgcn_readfirstlane(pieces);
            if (pieces > kSupportOwn && lane == 0) atomicOr(&heavy[round], 1 << wave);
        }
        // (the next round's word: its readers of two rounds ago passed the barrier of the last, and nobody sets it before this one)
        if (threadIdx.x == 0) heavy[round == 2 ? 0 : round + 1] = 0;
        __syncthreads();
        const int shared = __builtin_amdgcn_readfirstlane(heavy[round]);

        // job -1: this wavefront's own quad; then the shared ones, a share of the columns each
        for (int job = -1; job < kSupportWaves; ++job) {
            const bool alone = job < 0;
            if (alone ? own >= quads || pieces > kSupportOwn : !(shared >> job & 1)) continue;
            const long long quad = alone ? own : quad0 + job;
            if (alone) {
                const bool same = a.first || a.Same[quad] != 0;
                if (lane == 0) a.Same[quad] = pieces == 0;
                if (pieces == 0 && same) continue;
            } else if (wave == job && lane == 0) a.Same[quad] = 0;
            const long long share = (a.tiles_n + kSupportWaves - 1) / kSupportWaves;
            const long long ct_lo = alone ? 0 : wave * share, ct_hi = alone ? a.tiles_n : ct_lo + share < a.tiles_n ? ct_lo + share : a.tiles_n;
            const long long tile0 = (quad >> 3) * a.tiles_n;
            const int g = (int)(quad & 7) >> 1, lh = (int)quad & 1;      // rows 8 g + 4 lh .. + 3 of the 32-row tile
            float acc[4][MR];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int k = 0; k < MR; ++k) acc[r][k] = 0.f;

            auto add = [&](int head, int c) {      // c <= 64 columns of the list
                int col = 0;
                u32x2 x = {0u, 0u};      // rows 0 | 1, 2 | 3
                if (lane < c) {
                    col = list[head + lane];
                    const f32x4 v = a.Xs[(tile0 + (col >> 5)) * 256 + g * 64 + lh * 32 + (col & 31)];
                    x = u32x2{f2bf_pk(v[0], v[1]), f2bf_pk(v[2], v[3])};
                }
                struct Col { u32x4 f[FULL]; uint32_t t[2]; };
                auto load = [&](int e) {
                    Col q;
                    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                        (void*)(a.PhiT + (long long)__builtin_amdgcn_readlane(col, e) * a.ldm), 0, a.ldm * 2, kBufferFlags);
#pragma unroll
                    for (int k = 0; k < FULL; ++k) q.f[k] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, k * 1024, 0);
                    if constexpr (TAIL == 4) {
                        const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, lane * 8, FULL * 1024, 0);
                        q.t[0] = t[0]; q.t[1] = t[1];
                    }
                    if constexpr (TAIL == 2) q.t[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, FULL * 1024, 0);
                    return q;
                };
                auto pair = [&](const Col& p, const Col& q, int e) {
                    uint32_t d[MR];      // element k of both columns
                    auto two = [&](uint32_t dp, uint32_t dq, uint32_t& lo, uint32_t& hi) {
                        lo = __builtin_amdgcn_perm(dq, dp, 0x05040100u);
                        hi = __builtin_amdgcn_perm(dq, dp, 0x07060302u);
                    };
#pragma unroll
                    for (int k = 0; k < FULL; ++k)
#pragma unroll
                        for (int i = 0; i < 4; ++i) two(p.f[k][i], q.f[k][i], d[8 * k + 2 * i], d[8 * k + 2 * i + 1]);
#pragma unroll
                    for (int i = 0; i < TAIL / 2; ++i) two(p.t[i], q.t[i], d[8 * FULL + 2 * i], d[8 * FULL + 2 * i + 1]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const uint32_t x0 = __builtin_amdgcn_readlane(x[r >> 1], e), x1 = __builtin_amdgcn_readlane(x[r >> 1], e + 1);
                        const uint32_t xp = (r & 1) ? (x0 >> 16) | (x1 & 0xffff0000u) : (x0 & 0xffffu) | (x1 << 16);
                        if ((xp & 0x7fff7fffu) == 0) continue;
#pragma unroll
                        for (int k = 0; k < MR; ++k)
                            acc[r][k] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, d[k]), __builtin_bit_cast(bf16x2, xp), acc[r][k], false);
                    }
                };
                for (int e = 0; e < c; e += 4) {
                    const Col p = load(e), q = load(e + 1);
                    if (e + 2 < c) {
                        const Col p2 = load(e + 2), q2 = load(e + 3);
                        pair(p, q, e);
                        pair(p2, q2, e + 2);
                    } else {
                        pair(p, q, e);
                    }
                }
            };

            int cnt = 0;
            for (long long ct0 = ct_lo; ct0 < ct_hi && (!alone || pieces); ct0 += 32) {
                uint32_t bits = scan(quad, ct0, ct_hi);
                const int c0 = (int)(ct0 + (lane >> 1)) * 32 + (lane & 1) * 16;
                for (uint64_t some; (some = __builtin_amdgcn_ballot_w64(bits != 0)) != 0;) {
                    if (bits) {
                        list[cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u))] =
                            (uint16_t)(c0 + __builtin_ctz(bits));
                        bits &= bits - 1;
                    }
                    cnt += __popcll(some);
                }
                __builtin_amdgcn_wave_barrier();
                const bool last = ct0 + 32 >= ct_hi;
                int head = 0;
                for (; cnt - head >= 64 || (last && head < cnt); head += 64) add(head, cnt - head < 64 ? cnt - head : 64);
                if (head && head < cnt) {      // (fewer than 64 are left)
                    const uint16_t v = list[head + lane];
                    __builtin_amdgcn_wave_barrier();
                    list[lane] = v;
                    __builtin_amdgcn_wave_barrier();
                }
                cnt = head < cnt ? cnt - head : 0;
            }

#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const long long row = quad * 4 + r < a.rows ? quad * 4 + r : a.rows - 1;
                const bool live = quad * 4 + r < a.rows;
                const float* y = a.Y + row * a.ldY;
                bf16_t* out = a.R + row * a.ldm;
                if (alone) {
                    auto store = [&](int k0, auto width) {      // elements k0 .. k0 + width - 1 of this lane
                        constexpr int N = decltype(width)::value;
                        const int c = column(k0);
                        if (c >= a.ldm || !live) return;
#pragma unroll
                        for (int i = 0; i < N; i += 2)
                            *(uint32_t*)(out + c + i) = f2bf_pk(c + i < a.m ? y[c + i] - acc[r][k0 + i] : 0.f, c + i + 1 < a.m ? y[c + i + 1] - acc[r][k0 + i + 1] : 0.f);
                    };
#pragma unroll
                    for (int k = 0; k < FULL; ++k) store(8 * k, std::integral_constant<int, 8>{});
                    if constexpr (TAIL > 0) store(8 * FULL, std::integral_constant<int, TAIL>{});
                    continue;
                }
                __syncthreads();        // (uniform: every wavefront of the workgroup takes every shared job)
#pragma unroll
                for (int k = 0; k < MR; ++k) part[wave][column(k)] = acc[r][k];
                __syncthreads();
                for (int c = threadIdx.x * 2; live && c < a.ldm; c += 128 * kSupportWaves) {
                    float s[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        float sum = part[0][c + e];
#pragma unroll
                        for (int v = 1; v < kSupportWaves; ++v) sum += part[v][c + e];
                        s[e] = c + e < a.m ? y[c + e] - sum : 0.f;
                    }
                    *(uint32_t*)(out + c) = f2bf_pk(s[0], s[1]);
                }
            }
        }
    }
}

// As a launch of its own, beside the product over all columns.
template <int MR>
__global__ __launch_bounds__(256, MR > 12 ? 3 : 4) void residual_support_kernel(SupportRule rule, ResidualSupportArgs a) {
    if (!rule.sparse()) return;
    if (a.first) rule.note();
    __shared__ ResidualSupportLds<MR, 4> l;
    residual_support<MR, 4>(a, l, blockIdx.x, gridDim.x);
}

// The residual product over all columns on large tiles (Epi: EpiResidualTiled, or EpiStorePart for its parts along K), or in its place the
// one above (MR = 0: in another launch): a launch that returned at once beside it would cost a small iteration 3 %.  One workgroup per
// CU either way.
struct EpiStorePart : EpiStore<float> {
    __device__ __forceinline__ void packed() {}
};
template <typename Epi, int MR>
struct EpiResidualEither : Epi {
    static constexpr bool kLate = true;       // (the rule's words come with the first stage)
    static constexpr int kWaves = 8;
    SupportRule rule;
    ResidualSupportArgs s;
    __device__ __forceinline__ void instead(void* lds, uint32_t block, uint32_t all) const {
        if constexpr (MR > 0) {
            const uint32_t blocks = all < 256 ? all : 256;
            if (s.first) rule.note();
            if (block < blocks) residual_support<MR, kWaves>(s, *(ResidualSupportLds<MR, kWaves>*)lds, block, blocks);
        }
    }
};

// Non-zero elements of every `stride`-th row of a float iterate [rows, ld], times stride, to ctl[0] (packed rows as support_count_kernel);
// ctl[1] where the operand holds an infinity or NaN: its coefficient may be zero here (float's threshold gives zero for NaN), and
// zero times it is not.
static __global__ __launch_bounds__(256) void support_count_f32_kernel(const float* X, long long ld, long long rows, int n, int stride, uint32_t* ctl, const uint32_t* screen,
                                                                       const float* operand, long long elements) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < elements; i += (long long)gridDim.x * 256)
        if (!(fabsf(operand[i]) < INFINITY)) ctl[1] = 1u;
    const long long all = rows;
    if (screen && screen[0] == 0) rows = screen[2];
    uint32_t c = 0;
    for (long long r = (long long)blockIdx.x * stride; r < rows; r += (long long)gridDim.x * stride)
        for (int i = threadIdx.x; i < n; i += 256) c += X[r * ld + i] != 0.f;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) support_add(ctl, (part[0] + part[1] + part[2] + part[3]) * (float)stride * ((float)all / (rows > 0 ? rows : 1)));
}

// r = y - Phi x over the support of a float iterate, in float: a wavefront per row, which collects the row's non-zero coefficients as it reads
// it and adds their multiples of Phi's columns (rows of PhiT, lane l elements 4l to 4l + 3 of every 256); the four wavefronts of a workgroup share
// out the columns of a row with more than kSupportOwn coefficients.  Exact products, one rounding a term: fewer terms than the
// product over all columns sums, none of them split.  4300 packed rows of 37 coefficients, n = 1600, m = 392: 77 us over all columns (238 tiles
// of a long contraction), 50 so, most of it the latency of reading a row and then its columns.
struct ResidualSupportF32Args {
    const float* X; long long ldx;
    const float* PhiT; int ldm;
    const float* Y; long long ldY;
    float* R;
    long long rows;
    int n, m;
    const uint32_t* screen; const float* Yp; long long ldYp;
};
template <int MR>
struct ResidualSupportF32Lds {
    uint32_t cols[4][512];
    float vals[4][512];
    float part[4][256 * MR];
    int heavy[3];        // as ResidualSupportLds
};
template <int MR>
__device__ __forceinline__ void residual_support_f32(ResidualSupportF32Args a, ResidualSupportF32Lds<MR>& l, long long block, long long blocks) {
    if (a.screen && a.screen[0] == 0) {
        a.rows = a.screen[2];
        a.Y = a.Yp;
        a.ldY = a.ldYp;
    }
    constexpr int UN = MR <= 2 ? 8 : 4;      // columns on the way
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x < 3) l.heavy[threadIdx.x] = 0;
    __syncthreads();
    int round = 0;
    const int share = ((a.n + 3) / 4 + 255) / 256 * 256;      // columns of a wavefront's part of a shared row
    for (long long row0 = block * 4; row0 < a.rows; row0 += blocks * 4, round = round == 2 ? 0 : round + 1) {
        const long long own = row0 + wave;
        int count = 0;
        if (own < a.rows) {
            const float* x = a.X + own * a.ldx;
            for (int c = 4 * lane; c < a.n; c += 256) {      // (rows are padded to whole float4 with zeros)
                const f32x4 v = *(const f32x4*)(x + c);
                count += (v[0] != 0.f) + (v[1] != 0.f) + (v[2] != 0.f) + (v[3] != 0.f);
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) count += __shfl_xor(count, o, 64);
            count = __builtin_amdgcn_readfirstlane(count);
            if (count > kSupportOwn && lane == 0) atomicOr(&l.heavy[round], 1 << wave);
        }
        if (threadIdx.x == 0) l.heavy[round == 2 ? 0 : round + 1] = 0;
        __syncthreads();
        const int shared = __builtin_amdgcn_readfirstlane(l.heavy[round]);
        for (int job = -1; job < 4; ++job) {
            const bool alone = job < 0;
            if (alone ? own >= a.rows || count > kSupportOwn : !(shared >> job & 1)) continue;
            const long long row = alone ? own : row0 + job;
            const float* x = a.X + row * a.ldx;
            const int lo = alone ? 0 : wave * share, hi = alone ? a.n : lo + share < a.n ? lo + share : a.n;
            f32x4 acc[MR];
#pragma unroll
            for (int k = 0; k < MR; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int c0 = lo; c0 < hi && (!alone || count); c0 += 512) {
                int cnt = 0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int c = c0 + 256 * h + 4 * lane;
                    f32x4 v = {0.f, 0.f, 0.f, 0.f};
                    if (c < hi) v = *(const f32x4*)(x + c);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint64_t some = __builtin_amdgcn_ballot_w64(v[e] != 0.f);
                        if (!some) continue;
                        const int at = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
                        if (v[e] != 0.f) {
                            l.cols[wave][at] = c + e;
                            l.vals[wave][at] = v[e];
                        }
                        cnt += __popcll(some);
                    }
                }
                __builtin_amdgcn_wave_barrier();
                for (int q = 0; q < cnt; q += UN) {
                    f32x4 p[UN][MR];
                    float xq[UN];
#pragma unroll
                    for (int i = 0; i < UN; ++i) {
                        const int at = q + i < cnt ? q + i : q;
                        xq[i] = q + i < cnt ? l.vals[wave][at] : 0.f;
                        const int col = __builtin_amdgcn_readfirstlane((int)l.cols[wave][at]);
                        __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.PhiT + (long long)col * a.ldm), 0, a.ldm * 4, kBufferFlags);
#pragma unroll
                        for (int k = 0; k < MR; ++k) p[i][k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, k * 1024, 0));
                    }
#pragma unroll
                    for (int i = 0; i < UN; ++i) {
                        if (q + i >= cnt) break;
#pragma unroll
                        for (int k = 0; k < MR; ++k)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[k][e] = fmaf(xq[i], p[i][k][e], acc[k][e]);
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
            const float* y = a.Y + row * a.ldY;
            float* out = a.R + row * a.ldm;
            if (alone) {
#pragma unroll
                for (int k = 0; k < MR; ++k) {
                    const int c = 256 * k + 4 * lane;
                    if (c >= a.ldm) continue;
                    f32x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = c + e < a.m ? y[c + e] - acc[k][e] : 0.f;
                    *(f32x4*)(out + c) = o;
                }
                continue;
            }
            __syncthreads();        // (uniform: every wavefront of the workgroup takes every shared row)
#pragma unroll
            for (int k = 0; k < MR; ++k) *(f32x4*)(l.part[wave] + 256 * k + 4 * lane) = acc[k];
            __syncthreads();
            for (int c = threadIdx.x; c < a.ldm; c += 256)
                out[c] = c < a.m ? y[c] - ((l.part[0][c] + l.part[1][c]) + (l.part[2][c] + l.part[3][c])) : 0.f;
        }
    }
}
// The float residual over all columns, or in its place the one above.
template <typename Epi, int MR>
struct EpiResidualEitherF32 : Epi {
    static constexpr bool kLate = true;
    SupportRule rule;
    ResidualSupportF32Args s;
    static constexpr size_t kLds = sizeof(ResidualSupportF32Lds<MR>);
    __device__ __forceinline__ void instead(void* lds) const {
        residual_support_f32<MR>(s, *(ResidualSupportF32Lds<MR>*)lds, blockIdx.x, gridDim.x);
    }
};

}  // namespace csat

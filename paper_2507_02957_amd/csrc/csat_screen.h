// Rows whose iterate is zero throughout.  For a measurement row y with |Phi^T y| <= lambda everywhere, x = 0 is ISTA's fixed point from the
// start (u = mu Phi^T y, |u| <= mu lambda = theta): every iterate is exactly zero, whatever the number of iterations.  Large calls
// with many such rows (short_video: four of five) find them with the first iteration's product, and the decoder runs the rows that are left,
// packed together.  The device decides: a sample of the rows first (every few rows; 1 to 2 % of such a call where all rows stay), then all.
//
// What it takes (short_video, 76 800 rows, of which 15 000 to 17 000 stay): the sample and the launches around it 45 us, bf16 operands of all rows 48, their product
// 122 (on 256 x 320 tiles; 156 on 256 x 256: its contraction is seven steps a tile), the lists 12, packing 39, C 47; the decoder runs 120 to 133 groups of
// rows instead of 600, 1.35 ms (a chain of 20 iterations) instead of 3.2. A forward 3.49 -> 1.75 ms; float, 19 200 rows 6.91 -> 2.31 (with the
// residual over the support); 205 824 rows, n = 1608, m = 752, one of a hundred left 9.7 -> 2.5.
//
// A row stays unless |mu Phi^T y| <= (1 - 2^-8) theta everywhere; NaN and infinities stay.  The decoder's own sums, in another order, then give zero
// too, as long as they differ by less than lambda / 256 (a few roundings of 2^-24 of sum |phi y|).  Below such a lambda (1e-4 of sum |phi y|) a coefficient that is
// the rounding of these sums may be left out; zero is as near to the exact value.
#pragma once
#include "csat_kernels.h"

namespace csat {

constexpr float kScreenMargin = 1.f - 1.f / 256;
// Words on the device: [0] 1 where the decoder takes the rows as they are, [1] 0, [2] the rows that are left (as a SupportRule with limit 0:
// sparse() where the rows are packed)
constexpr int kScreenWords = 4;

// The product's epilogue: Stay[r] = 1 where a row has an element above the bound.
struct EpiScreen {
    static constexpr bool kTile = true;
    static constexpr int kStageBytes = 0, kWideStageBytes = 0;
    static constexpr bool kRule = true, kRows = true;
    struct Pre {};
    struct Rule {
        const uint32_t* off;      // null: always
        __device__ __forceinline__ bool sparse() const { return off && *off != 0; }
    };
    uint8_t* Stay;
    float mu, bound;
    long long M; int N;
    Rule rule;
    __device__ __forceinline__ void mark(bool above, long long r, int lane) const {      // r: this lane's row
        const uint64_t b = __builtin_amdgcn_ballot_w64(above);
        if ((lane & 31) == 0 && (uint32_t)(lane >> 5 ? b >> 32 : b) != 0 && r < M) Stay[r] = 1;
    }
    __device__ __forceinline__ Pre begin(long long, long long, int) const { return {}; }
    __device__ __forceinline__ void half(int, long long r0, long long c0w, int lane, const f32x16 (&acc)[4], char*, const Pre&) const {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            bool above = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) above |= c0w + 32 * j + (lane & 31) < N && !(fabsf(mu * acc[j][v]) <= bound);
            mark(above, r0 + 8 * (v / 4) + 4 * (lane >> 5) + v % 4, lane);
        }
    }
    template <int TN>
    __device__ __forceinline__ Pre begin_wide(long long, long long, int) const { return {}; }
    template <int TN>
    __device__ __forceinline__ void whole_wide(long long r0w, long long c0w, int lane, const f32x16 (&acc)[2][TN], char*, const Pre&) const {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                bool above = false;
#pragma unroll
                for (int j = 0; j < TN; ++j) above |= c0w + 32 * j + (lane & 31) < N && !(fabsf(mu * acc[i][j][v]) <= bound);
                mark(above, r0w + 32 * i + 8 * (v / 4) + 4 * (lane >> 5) + v % 4, lane);
            }
    }
    __device__ __forceinline__ void flush(long long, long long, int, const char*, const Pre&) const {}
    __device__ __forceinline__ void rows(long long r0, long long c, const f32x16& acc) const {
#pragma unroll
        for (int v = 0; v < 16; ++v) mark(c < N && !(fabsf(mu * acc[v]) <= bound), r0 + TileRows::row(v), threadIdx.x & 63);
    }
};

static __global__ void screen_begin_kernel(uint32_t* words, uint32_t* stay, long long stay_words) {
    if (blockIdx.x == 0 && threadIdx.x < kScreenWords) words[threadIdx.x] = 0;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < stay_words; i += (long long)gridDim.x * blockDim.x) stay[i] = 0u;
}

// After the sample: packing off unless at most `most` of its rows stay.  Clears its marks.
static __global__ __launch_bounds__(1024) void screen_decide_kernel(uint32_t* words, uint32_t* stay, int sample, int most) {
    __shared__ int sum;
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    int n = 0;
    for (int i = threadIdx.x; i < (sample + 3) / 4; i += 1024) {
        n += __popc(stay[i]);
        stay[i] = 0u;
    }
    if (n) atomicAdd(&sum, n);
    __syncthreads();
    if (threadIdx.x == 0) words[0] = sum > most;
}

// Rows that stay, in order: counts of 1024 rows each, then their places (Place[r], -1 where r does not stay; List[place] = r).
// More than `most` rows: packing off after all.  And where V holds an infinity or NaN, whose products with the coefficients that are
// zero are NaN: its `pieces` are looked over by the workgroups behind the `blocks` that count, which then set `on`'s second word.
template <typename T>
__global__ __launch_bounds__(256) void screen_count_kernel(SupportRule on, const uint32_t* stay, long long rows, int* counts, int blocks, const uint4* V, long long pieces) {
    if (!on.sparse()) return;
    if ((int)blockIdx.x >= blocks) {
        if (holds_unbounded<T>(V, pieces, (long long)(blockIdx.x - blocks) * 256 + threadIdx.x, (long long)(gridDim.x - blocks) * 256)) ((uint32_t*)on.ctl)[1] = 1u;
        return;
    }
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;      // four rows
    int n = i * 4 < rows ? __popc(stay[i]) : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    __shared__ int part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}
// `words` is read by every block of the launch behind this one, not by this one's own (block 0 writes it): they go by `on`.
static __global__ __launch_bounds__(256) void screen_place_kernel(SupportRule on, uint32_t* next, const uint32_t* stay, long long rows, const int* counts, int* Place,
                                                                  int* List, int most) {
    const bool packed = on.sparse();
    __shared__ int before, total, waves[4];
    if (threadIdx.x == 0) before = total = 0;
    __syncthreads();
    if (packed) {
        int b = 0, t = 0;
        for (int i = threadIdx.x; i < (int)gridDim.x; i += 256) {
            t += counts[i];
            if (i < (int)blockIdx.x) b += counts[i];
        }
        if (b) atomicAdd(&before, b);
        if (t) atomicAdd(&total, t);
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        next[0] = !packed || total > most;
        next[1] = 0;
        next[2] = total;
    }
    if (!packed || total > most) return;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    const uint32_t s = i * 4 < rows ? stay[i] : 0u;
    const int n = __popc(s), lane = threadIdx.x & 63;
    int incl = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) waves[threadIdx.x >> 6] = incl;
    __syncthreads();
    int at = before + incl - n;
    for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) at += waves[w];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const long long r = i * 4 + e;
        if (r >= rows) break;
        const bool stays = (s >> (8 * e)) & 1;
        Place[r] = stays ? at : -1;
        if (stays) List[at++] = (int)r;
    }
}

// Rows of y into other layouts, a wavefront each: row i of the result is row List[i] (the last of them again up to whole 256 rows), or
// i * stride.  Sources and float results are row-major [ld] or, with `tiled`, accumulator tiles [tile of 32 rows][ld / 32][4][64] float4.
struct ScreenRowsArgs {
    const uint32_t* words;     // not null: only where the rows are packed; count rows of List
    const int* List; long long rows; int stride;
    const float* Y; long long ldY; int y_tiled;
    float* Yp; long long ldYp; int yp_tiled;       // or null; ldYp columns
    void* R; long long ldR; int r_bf16;            // or null; ldR columns, zero from m on
    int m;
};
__device__ __forceinline__ long long tiled_at(long long r, long long ld, int c) {      // element of (row r, column c)
    const int e = c & 3, h = (c >> 2) & 1, g = (c >> 3) & 3;
    return (((r >> 5) * (ld >> 5) + (c >> 5)) * 4 + g) * 256 + (h * 32 + (r & 31)) * 4 + e;
}
static __global__ __launch_bounds__(256) void screen_rows_kernel(ScreenRowsArgs a) {
    long long rows = a.rows, have = a.rows;
    if (a.words) {
        if (a.words[0]) return;
        if (a.List) {
            have = a.words[2];
            rows = (have + 255) / 256 * 256;
        }
    }
    const int lane = threadIdx.x & 63;
    for (long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); i < rows; i += (long long)gridDim.x * 4) {
        const long long k = i < have ? i : have - 1, r = a.List ? a.List[k] : k * a.stride;
        const long long width = a.Yp && a.ldYp > a.ldR ? a.ldYp : a.R ? a.ldR : a.ldYp;
        for (int c0 = 0; c0 < width; c0 += 512) {
            float y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int c = c0 + 64 * e + lane;
                y[e] = c < a.m ? a.Y[a.y_tiled ? tiled_at(r, a.ldY, c) : r * a.ldY + c] : 0.f;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int c = c0 + 64 * e + lane;
                if (a.Yp && c < a.ldYp) a.Yp[a.yp_tiled ? tiled_at(i, a.ldYp, c) : i * a.ldYp + c] = y[e];
                if (a.R && c < a.ldR) {
                    if (a.r_bf16) ((bf16_t*)a.R)[i * a.ldR + c] = f2bf(y[e]);
                    else ((float*)a.R)[i * a.ldR + c] = y[e];
                }
            }
        }
    }
}

// C = X V where the rows are packed: zeros for the rows that did not stay, for the others the non-zero coefficients' rows of V, a wavefront per
// row.  X [count, ldx] in T (bf16: the operand copy, the coefficients as the product over all columns takes them).  A decoder that gave
// up (*err): NaN.
template <typename T>
__global__ __launch_bounds__(256) void screen_finish_kernel(const uint32_t* words, const int* err, const int* Place, const T* X, long long ldx, const T* V, T* C, long long rows, int n_q,
                                                            int n, int d) {
    if (words[0]) return;
    constexpr int W = 16 / sizeof(T), kList = 64 * W;      // coefficients per lane and trip
    __shared__ uint32_t cols[4][kList];
    __shared__ float vals[4][kList];
    struct alignas(16) Piece { T v[W]; };
    struct alignas(4 * sizeof(T)) Four { T v[4]; };
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (long long r = (long long)blockIdx.x * 4 + wave; r < rows; r += (long long)gridDim.x * 4) {
        const int place = __builtin_amdgcn_readfirstlane(Place[r]);
        for (int d0 = 0; d0 < d; d0 += 256) {
            // four elements of a row of V per lane, as many rows side by side as the wavefront holds
            const int lanes = (d - d0 < 256 ? d - d0 : 256) / 4, side = 64 / lanes, mine = lane / lanes, c4 = d0 + 4 * (lane % lanes);
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
            if (*err) acc[0] = acc[1] = acc[2] = acc[3] = __uint_as_float(0x7fc00000u);
            else if (place >= 0) {
                const T* x = X + place * ldx;
                const T* v = V + r / n_q * n * (long long)d + c4;
                for (int c0 = 0; c0 < n; c0 += kList) {      // (rows of X are padded to whole pieces)
                    const int c = c0 + W * lane;
                    Piece p{};
                    if (c < ldx) p = *(const Piece*)(x + c);
                    int cnt = 0;
#pragma unroll
                    for (int j = 0; j < W; ++j) {
                        const float e = c + j < n ? Elem<T>::load(&p.v[j]) : 0.f;
                        const uint64_t some = __builtin_amdgcn_ballot_w64(e != 0.f);
                        if (!some) continue;
                        const int at = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
                        if (e != 0.f) {
                            cols[wave][at] = c + j;
                            vals[wave][at] = e;
                        }
                        cnt += __popcll(some);
                    }
                    __builtin_amdgcn_wave_barrier();
                    for (int q = 0; q < cnt; q += 8 * side) {
                        Four f[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int at = q + i * side + mine;
                            f[i] = *(const Four*)(v + (long long)cols[wave][at < cnt ? at : q] * d);
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int at = q + i * side + mine;
                            if (mine >= side || at >= cnt) continue;
                            const float xq = vals[wave][at];
#pragma unroll
                            for (int k = 0; k < 4; ++k) acc[k] = fmaf(xq, Elem<T>::load(&f[i].v[k]), acc[k]);
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                }
                // the sums that lie side by side
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float sum = acc[k];
                    for (int g = 1; g < side; ++g) sum += __shfl(acc[k], (lane % lanes) + g * lanes, 64);
                    acc[k] = sum;
                }
            }
            if (lane < lanes) {
                Four o;
#pragma unroll
                for (int k = 0; k < 4; ++k) Elem<T>::store(&o.v[k], acc[k]);
                *(Four*)(C + r * d + c4) = o;
            }
        }
    }
}

}  // namespace csat

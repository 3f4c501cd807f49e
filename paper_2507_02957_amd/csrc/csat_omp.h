// Orthogonal matching pursuit, the greedy decoder the paper names next to ISTA (introduction and
// limitations sections; it gives no details, so this is the standard algorithm).  Per row: k times
// pick the column of Phi most correlated with the residual (largest |phi_j^T r|, lowest index on a
// tie, never a column twice), refit the picked coefficients by least squares, update the residual.
//
// The correlations of all rows are one GEMM per pick (R Phi, the decoder's update product).  The
// least-squares refit is kept as an incrementally built QR factorisation per row (modified
// Gram-Schmidt): with the picked columns Phi_S = Q T (Q orthonormal, T upper triangular), the
// residual update is r <- r - (q^T r) q for the new q only, and the coefficients follow once at the
// end from T x = Q^T y.  One wavefront per row, lanes strided over m, fp32 throughout.
#pragma once
#include "csat_kernels.h"

namespace csat {

constexpr int kOmpMaxPicks = 32;     // registers of the finishing kernel hold one coefficient per pick
constexpr int kOmpMaxM = 1024;       // 16 values of an m-vector per lane

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// picks[r][it] = argmax_c |Cm[r][c]| over the columns not picked before (lowest index on a tie)
static __global__ __launch_bounds__(256) void omp_pick_kernel(const float* Cm, long long ldc, long long rows, int n, int* picks,
                                                       int k, int it) {
    const int lane = threadIdx.x & 63;
    const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const float* c = Cm + r * ldc;
    int* pk = picks + r * k;
    float best = -1.f;
    int bi = 0x7fffffff;
    const int mine = lane < it ? pk[lane] : -1;    // earlier picks, one per lane (it <= 32)
    // four columns per lane and step (rows of Cm are 16-byte aligned: ldc is a multiple of 4)
    for (int j4 = lane * 4; j4 < n; j4 += 256) {
        const f32x4 cv = __builtin_nontemporal_load((const f32x4*)(c + j4));      // read once: keep it out of the caches' way
        float a[4] = {fabsf(cv[0]), fabsf(cv[1]), fabsf(cv[2]), fabsf(cv[3])};
        for (int s = 0; s < it; ++s) {            // uniform trip count: only the picks made so far
            const int d = __builtin_amdgcn_readlane(mine, s) - j4;
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = d == e ? -2.f : a[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (j4 + e < n && a[e] > best) { best = a[e]; bi = j4 + e; }    // ascending index per lane: the first maximum stays
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ob = __shfl_xor(best, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    if (lane == 0) pk[it] = bi < n ? bi : 0;      // only reachable when every correlation is NaN
}

// Epilogue of the correlation product on the large-tile GEMM: instead of the correlations, the best column of each row
// within the wavefront's 128 (largest |c|, lowest index on a tie, earlier picks left out).  The update kernel takes the
// best of those.  The correlations (491 MB at 76 800 x 1600, m = 392) are neither written nor read back: a pick took
// 182 us of product and 92 us of search and takes 187 us; what bounds it now is the short contraction, whose seven steps
// per tile do not cover the tile's start and epilogue.
struct OmpCand { float val; int idx; };
struct EpiOmpBest {
    static constexpr bool kTile = true, kWhole = true;
    static constexpr int kPitch = 33 * 8;                       // 32 candidates and a pad against bank conflicts
    static constexpr int kStageBytes = 64 * kPitch + 64 * 16;
    struct Pre { uint4 ex; };                                   // columns of this block that row r0w + lane may not pick
    OmpCand* cand; int nseg;                                    // [M][nseg], one per 128 columns
    const int* picks; int k, it;                                // [M][k], `it` made so far
    long long M; int N;
    // (before the main loop: the reads of the earlier picks hide behind the first operands', eight at a time)
    __device__ __forceinline__ Pre begin(long long r0w, long long c0w, int lane) const {
        uint32_t ex[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const long long left = N - c0w - 32 * j;
            ex[j] = left >= 32 ? 0u : left <= 0 ? 0xffffffffu : 0xffffffffu << left;
        }
        const long long row = r0w + lane < M ? r0w + lane : M - 1;
        for (int s0 = 0; s0 < it; s0 += 8) {
            int p[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) p[s] = picks[row * k + (s0 + s < it ? s0 + s : 0)];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int q = p[s] - (int)c0w;
#pragma unroll
                for (int j = 0; j < 4; ++j) ex[j] |= (q >> 5) == j ? 1u << (q & 31) : 0u;
            }
        }
        return Pre{uint4{ex[0], ex[1], ex[2], ex[3]}};
    }
    __device__ __forceinline__ void whole(long long r0w, long long c0w, int lane, const f32x16 (&acc)[2][4], char* stage,
                                          const Pre& pre) const {
        if (r0w >= M || c0w >= N) return;                       // (uniform)
        const int li = lane & 31, lh = lane >> 5;
        const long long row = r0w + lane;
        uint4* mask = (uint4*)(stage + 64 * kPitch);
        mask[lane] = pre.ex;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int rr = 32 * i + 8 * (v / 4) + 4 * lh + (v % 4);
                const uint4 e = mask[rr];
                const uint32_t w[4] = {e.x, e.y, e.z, e.w};
                OmpCand b{-1.f, 0x7fffffff};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int c = (int)c0w + 32 * j + li;
                    const float a = (w[j] >> li) & 1u ? -2.f : fabsf(acc[i][j][v]);
                    if (a > b.val) b = OmpCand{a, c};
                }
                *(OmpCand*)(stage + rr * kPitch + li * 8) = b;
            }
        OmpCand b{-1.f, 0x7fffffff};
#pragma unroll
        for (int q = 0; q < 32; ++q) {
            const OmpCand o = *(const OmpCand*)(stage + lane * kPitch + q * 8);
            if (o.val > b.val || (o.val == b.val && o.idx < b.idx)) b = o;
        }
        if (row < M) cand[row * nseg + (c0w >> 7)] = b;
    }
    __device__ __forceinline__ void flush(long long, long long, int, const char*) const {}
};

// Adds the picked column to the row's factorisation and updates its residual.
//   PhiT [n, ldp]   columns of Phi as rows (element type T)
//   Qb [rows, k, mq]  orthonormal vectors, Tri [rows, k, k] the triangular factor (column `it` written here),
//   Z [rows, k]  q^T y,  Rf [rows, mq] fp32 residual (in/out),  Rop [rows, ldr] operand copy of it (pads zero)
// cand [rows, nseg]: the pick is the best of these (EpiOmpBest) and is written to picks here; null: picks holds it.
// MQ: values of an m-vector per lane, ceil(m / 64) rounded up to 4, 8 or 16.
template <typename T, int MQ>
__global__ __launch_bounds__(256) void omp_update_kernel(const T* PhiT, long long ldp, int m, const OmpCand* cand, int nseg,
                                                         int* picks, int k, int it, float* Qb, float* Tri, float* Z, float* Rf, int mq, T* Rop,
                                                         long long ldr, long long rows) {
    const int lane = threadIdx.x & 63;
    const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    int j;
    if (cand) {
        OmpCand b{-1.f, 0x7fffffff};
        for (int q = lane; q < nseg; q += 64) {
            const OmpCand o = cand[r * nseg + q];
            if (o.val > b.val) b = o;                   // ascending index per lane
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float ob = __shfl_xor(b.val, o, 64);
            const int oi = __shfl_xor(b.idx, o, 64);
            if (ob > b.val || (ob == b.val && oi < b.idx)) b = OmpCand{ob, oi};
        }
        j = b.val >= 0.f ? b.idx : 0;                   // (0: every correlation is NaN)
        if (lane == 0) picks[r * k + it] = j;
    } else {
        j = picks[r * k + it];
    }
    const T* col = PhiT + (long long)j * ldp;
    float* qrow = Qb + r * (long long)k * mq;
    float v[MQ];
#pragma unroll
    for (int i = 0; i < MQ; ++i) {
        const int l = lane + 64 * i;
        v[i] = l < m ? Elem<T>::load(col + l) : 0.f;
    }
    for (int s = 0; s < it; ++s) {
        const float* q = qrow + (long long)s * mq;
        float qv[MQ];
        float dot = 0.f;
#pragma unroll
        for (int i = 0; i < MQ; ++i) {
            const int l = lane + 64 * i;
            qv[i] = l < mq ? q[l] : 0.f;
            dot += qv[i] * v[i];
        }
        dot = wave_sum(dot);
        if (lane == 0) Tri[(r * k + s) * k + it] = dot;
#pragma unroll
        for (int i = 0; i < MQ; ++i) v[i] -= dot * qv[i];
    }
    float nn = 0.f;
#pragma unroll
    for (int i = 0; i < MQ; ++i) nn += v[i] * v[i];
    const float nrm = sqrtf(wave_sum(nn));
    const float inv = nrm > 0.f ? 1.f / nrm : 0.f;       // a column inside the span of the earlier picks adds nothing
    if (lane == 0) Tri[(r * k + it) * k + it] = nrm;
    float* res = Rf + r * mq;
    float zt = 0.f;
    float rv[MQ];
#pragma unroll
    for (int i = 0; i < MQ; ++i) {
        const int l = lane + 64 * i;
        v[i] *= inv;
        if (l < mq) qrow[(long long)it * mq + l] = v[i];
        rv[i] = l < mq ? res[l] : 0.f;
        zt += v[i] * rv[i];
    }
    zt = wave_sum(zt);
    if (lane == 0) Z[r * k + it] = zt;
#pragma unroll
    for (int i = 0; i < MQ; ++i) {
        const int l = lane + 64 * i;
        const float x = rv[i] - zt * v[i];
        if (l < mq) res[l] = x;
        if (l < ldr) Elem<T>::store(Rop + r * ldr + l, l < m ? x : 0.f);
    }
    for (int l = lane + 64 * MQ; l < ldr; l += 64) Elem<T>::store(Rop + r * ldr + l, 0.f);    // operand pads beyond the lanes' share
}

// Coefficients from T x = z by back substitution, scattered into X (zeroed beforehand); optional
// copy of the picks and C[r,:] = sum_s x_s V[head(r), pick_s, :].
template <typename T>
__global__ __launch_bounds__(256) void omp_finish_kernel(const float* Tri, const float* Z, const int* picks, int k, long long rows,
                                                         int n_q, int n, int d, float* X, int* picks_out, const T* V, T* C) {
    const int lane = threadIdx.x & 63;
    const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const float* tri = Tri + r * (long long)k * k;
    const int* pk = picks + r * k;
    // Lane s holds row s of the factor and the unknown x_s; from the last unknown on, each is broadcast and subtracted.
    // (With every lane running the whole substitution its k^2 / 2 loads came one after the other: 216 us on 76 800 rows of
    // eight picks.)
    const int row = lane < k ? lane : 0;
    float t[kOmpMaxPicks];
#pragma unroll
    for (int s = 0; s < kOmpMaxPicks; ++s) t[s] = s < k ? tri[row * k + (s >= row ? s : row)] : 0.f;
    float acc = lane < k ? Z[r * k + row] : 0.f, mine = 0.f;
    float x[kOmpMaxPicks];
#pragma unroll
    for (int s = kOmpMaxPicks - 1; s >= 0; --s) {
        x[s] = 0.f;
        if (s < k) {
            const float xs = t[s] > 0.f ? acc / t[s] : 0.f;          // (lane s: t[s] is the diagonal)
            x[s] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(xs), s));
            if (lane == s) mine = x[s];
            acc -= t[s] * x[s];
        }
    }
    const int my_pick = lane < k ? pk[lane] : 0;
    if (lane < k) {
        if (X) X[r * (long long)n + my_pick] = mine;
        if (picks_out) picks_out[r * k + lane] = my_pick;
    }
    if (C) {
        const T* v = V + (r / n_q) * (long long)n * d;
        for (int c = lane; c < d; c += 64) {
            float sum = 0.f;
#pragma unroll
            for (int s = 0; s < kOmpMaxPicks; ++s)
                if (s < k) sum += x[s] * Elem<T>::load(v + (long long)__builtin_amdgcn_readlane(my_pick, s) * d + c);
            Elem<T>::store(C + r * (long long)d + c, sum);
        }
    }
}

}  // namespace csat

// Orthogonal matching pursuit, the greedy decoder the paper names next to ISTA (introduction and
// limitations sections; it gives no details, so this is the standard algorithm).  Per row: k times
// pick the column of Phi most correlated with the residual (largest |phi_j^T r|, lowest index on a
// tie, never a column twice), refit the picked coefficients by least squares, update the residual.
//
// Two launches per pick: the correlations R Phi with each row's largest (bf16: omp_pick_product_kernel, or EpiOmpBest on the large-tile
// product; float: the product and omp_pick_kernel), and omp_update_kernel, which refits the picked coefficients and forms the next residual.
#pragma once
#include "csat_kernels.h"

namespace csat {

constexpr int kOmpMaxPicks = 32;     // registers of the finishing kernel hold one coefficient per pick
constexpr int kOmpMaxM = 1024;       // 16 values of an m-vector per lane

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

// ---- correlations and the pick, bf16 ----
// A wavefront holds the residuals of 32 rows as MFMA B operands, 16 registers per 64 values of m, and walks the columns of Phi
// in chunks of 32, which the workgroup's wavefronts share through LDS.  A chunk's correlations are an accumulator tile with a
// row's columns in two lanes' registers; the largest is kept in registers, a few elements of the chunk before behind each
// MFMA (three vector instructions an element: the columns a row may not pick come as lane masks in scalar registers), and
// nothing but one candidate per row leaves the kernel.  Two wavefronts per SIMD up to m = 512, one beyond.
// 76 800 rows, n = 1600, m = 392: 119 us a pick, 111 without masks (53 of it MFMA time, 28 the residuals' way into registers);
// as a 256 x 256 product with the search in its epilogue 187, its seven K steps too few to cover a tile's start and end.
// (64 rows a wavefront, one per SIMD, halve the LDS reads but push the sums into the accumulator file: 178 against 155 at
// that stage.)  The row blocks beyond whole rounds of the chip are cut into shares of n; the update takes the best of their
// candidates.
struct OmpCand { float val; int idx; };

// Epilogue of the correlation product on the large-tile GEMM, for m > 512 where its rounds of tiles take less time: the best column of
// each row within the wavefront's 128 (largest |c|, lowest index on a tie, earlier picks left out).  The update kernel takes the
// best of those.  Nine K steps and more cover a tile's start and the search; omp_pick_product_kernel has one wavefront per SIMD there.
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
    __device__ __forceinline__ void flush(long long, long long, int, const char*, const Pre&) const {}
};

// Columns that a row may not pick (picked before, or beyond n): [row tile of 32][chunk][32 words], a bit per row.  Word
// omp_taken_word(c) is column c of the chunk, so that words 2 v and 2 v + 1 are the lane mask of accumulator register v.
constexpr __host__ __device__ int omp_taken_word(int c) { return 2 * ((c >> 3) * 4 + (c & 3)) + ((c >> 2) & 1); }
struct OmpPickArgs {
    const bf16_t* PhiT; const bf16_t* R;     // [n, ldm], [rows, ldm], pads zero
    long long ldm, rows;
    const uint32_t* taken;
    OmpCand* cand;                           // [rows, splits]
    int n, nct;
    int whole, splits, group;                // row blocks that one workgroup takes all of n for; shares of n of the others, and how
                                             // many blocks follow each other before the next share
};
constexpr int omp_pick_waves(int KS) { return KS <= 8 ? 8 : 4; }                              // KS: m in 64s
constexpr int omp_pick_rows(int KS) { return omp_pick_waves(KS) * 32; }
constexpr int omp_pick_chunks(int KS) { return KS == 1 ? 4 : KS <= 3 ? 2 : 1; }               // per step
constexpr int omp_pick_per_cu(int KS) { return KS <= 2 ? 2 : 1; }                             // workgroups
constexpr int omp_pick_ring(int KS) { return KS <= 13 ? 3 : 2; }                              // steps in LDS
constexpr int omp_pick_stage_bytes(int KS) { return omp_pick_chunks(KS) * KS * 4096; }
constexpr size_t omp_pick_lds_bytes(int KS) { return (size_t)omp_pick_ring(KS) * omp_pick_stage_bytes(KS); }

static __global__ void omp_taken_init_kernel(uint32_t* taken, int n, int nct, long long total) {
    const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= total) return;
    const int w = (int)(id & 31), c = (w >> 3) * 8 + (w & 1) * 4 + ((w >> 1) & 3);      // omp_taken_word's inverse
    taken[id] = (int)((id >> 5) % nct) * 32 + c < n ? 0u : 0xffffffffu;
}

template <int KS>
__global__ __launch_bounds__(64 * omp_pick_waves(KS), omp_pick_waves(KS) / 4 * omp_pick_per_cu(KS)) void omp_pick_product_kernel(OmpPickArgs a) {
    constexpr int W = omp_pick_waves(KS), CPS = omp_pick_chunks(KS), NS = CPS * KS, STAGE = omp_pick_stage_bytes(KS),
                  RING = omp_pick_ring(KS);
    constexpr int SLOTS = KS == 1 ? 4 : 4 * KS - 4;             // pairs of MFMAs of a chunk that the search of the chunk before is spread over
    typedef uint64_t u64x8 __attribute__((ext_vector_type(8)));
    typedef const __attribute__((address_space(4))) u64x8* mask_ptr_t;
    extern __shared__ uint4 lds[];
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // groups of eight: the shares of a row block run on one XCD, one after the other: its residuals (256 rows are 230 KB at m = 392)
    // come from memory once and then from that L2
    int split = 0, splits = 1;
    long long block = blockIdx.x;
    if (block >= a.whole) {
        const int id = (int)(block - a.whole), slot_id = id / a.group;
        splits = a.splits;
        split = slot_id % splits;
        block = a.whole + (long long)(slot_id / splits) * a.group + id % a.group;
    }
    if (block * (W * 32) >= a.rows) return;                 // (the grid is padded to whole groups of row blocks)
    const long long tile = block * W + wave, row = tile * 32 + li;
    const int steps = (a.nct + CPS - 1) / CPS, share = (steps + splits - 1) / splits;
    const int s0 = split * share, s1 = s0 + share < steps ? s0 + share : steps;
    const uint32_t lds0 = (uint32_t)(size_t)(lds_ptr_t)lds;

    // Staging: a request brings 8 columns (rows of PhiT) x 64 values of m, wavefront w columns 8 (w % 4) on of every (W / 4)-th
    // slab; the 16-byte slot of a column is XORed with (column / 2) so that the fragment reads of consecutive columns fall in
    // different banks.
    constexpr int PAR = W / 4, RPW = (NS + PAR - 1) / PAR;       // requests per step of a wavefront (one less in the second half)
    const int half = wave >> 2, quarter = wave & 3, sr = quarter * 8 + (lane >> 3);
    const uint32_t soff = ((lane & 7) ^ ((sr >> 1) & 7)) * 16, ldb = (uint32_t)a.ldm * 2;
    const bool fewer = NS % PAR != 0 && half == PAR - 1;
    auto stage = [&](int step, uint32_t so, int i) {
        const int s = PAR * i + half;
        if (NS % PAR != 0 && s >= NS) return;
        int ch = step * CPS + s / KS;
        ch = ch < a.nct ? ch : a.nct - 1;
        const int last = a.n - 1 - 32 * ch;                      // columns beyond n: the last one (their bits in `taken` are set)
        const char* base = (const char*)a.PhiT + (long long)ch * 32 * ldb + (s % KS) * 128;
        __builtin_amdgcn_global_load_lds((glb_ptr_t)(base + ((uint32_t)(sr < last ? sr : last) * ldb + soff)),
                                         (lds_ptr_t)((char*)lds + so + s * 4096 + quarter * 1024), 16, 0, 0);
    };
    auto stage_all = [&](int step, uint32_t so) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) stage(step, so, i);
    };
    uint32_t ad[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) ad[g] = lds0 + li * 128 + ((2 * g + lh) ^ ((li >> 1) & 7)) * 16;

    bf16x8 rb[4 * KS];
    if (s0 < s1) stage_all(s0, 0);
    if (RING == 3 && s0 + 1 < s1) stage_all(s0 + 1, STAGE);
    const long long tiles = (a.rows + 31) / 32, rc = row < a.rows ? row : a.rows - 1;
    const mask_ptr_t taken = (mask_ptr_t)(const void*)(a.taken + (tile < tiles ? tile : tiles - 1) * a.nct * 32);
#pragma unroll
    for (int f = 0; f < 4 * KS; ++f) rb[f] = __builtin_bit_cast(bf16x8, *(const uint4*)(a.R + rc * a.ldm + f * 16 + lh * 8));
    float best = -1.f;
    int at = 0x7fffffff, off = -1;
    f32x16 u[2];                           // the correlations being formed, and those of the chunk before being searched
    u64x8 ex[2], exn[2];                   // ... and the rows that may not pick its columns (asked for a chunk ahead: a read from memory)
    int c0 = 0;
    // Elements [E0, E1) of the 16 of buffer b: register v is column 8 (v / 4) + 4 lh + v % 4, ascending columns so that the
    // first maximum stays.
    auto search = [&](auto bc, auto e0c, auto e1c) {
        constexpr int b = decltype(bc)::value, E0 = decltype(e0c)::value, E1 = decltype(e1c)::value;
#pragma unroll
        for (int v = E0; v < E1; ++v) {
            if (v == 0) off = -1;
            const float c = fabsf(u[b][v]);
            const bool larger = __builtin_amdgcn_inverse_ballot_w64(~ex[v / 8][v % 8] & __builtin_amdgcn_ballot_w64(c > best));
            best = larger ? c : best;
            off = larger ? 8 * (v / 4) + v % 4 : off;
            if (v == 15) at = off >= 0 ? c0 + 4 * lh + off : at;
        }
    };
    auto ask_taken = [&](int ch) {
        ch = ch < a.nct ? ch : a.nct - 1;
        exn[0] = taken[2 * ch];
        exn[1] = taken[2 * ch + 1];
    };
    auto take_taken = [&](int ch) {
        c0 = 32 * ch;
#pragma unroll
        for (int h = 0; h < 2; ++h) ex[h] = CPS > 1 && c0 >= a.n ? (u64x8)(~0ull) : exn[h];
    };
    // everything but the requests of the last step asked for has landed
    auto step_end = [&](bool requested) {
        if (RING == 3 && requested) {
            if (fewer) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NS / PAR) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RPW) : "memory");
        }
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto step_body = [&](int step, uint32_t so, uint32_t sn, auto pc) {
        constexpr int par = decltype(pc)::value;                 // of the step: its chunk c uses buffer (par CPS + c) % 2
        const bool more = step + RING - 1 < s1;
        u32x4 fr[2][4];
        auto fetch = [&](auto sc) {
            constexpr int s = decltype(sc)::value;
#pragma unroll
            for (int g = 0; g < 4; ++g) lds_read16<s * 4096>(fr[s & 1][g], ad[g] + so);
        };
        auto run = [&](auto self, auto sc) {
            constexpr int s = decltype(sc)::value;
            if constexpr (s < NS) {
                constexpr int c = s / KS, cur = (par * CPS + c) & 1;
                if constexpr (s + 1 < NS) fetch(std::integral_constant<int, s + 1>{});
                if (more) {                                      // (a ring of two waits for them at the step's end: early)
                    if (RING == 3 && s < RPW) stage(step + 2, sn, s);
                    if (RING == 2 && 2 * s < RPW) stage(step + 1, sn, 2 * s);
                    if (RING == 2 && 2 * s + 1 < RPW) stage(step + 1, sn, 2 * s + 1);
                }
                lds_wait<(s + 1 < NS ? 4 : 0)>(fr[s & 1][0], fr[s & 1][1], fr[s & 1][2], fr[s & 1][3]);
                auto slot = [&](auto gc) {
                    constexpr int g = decltype(gc)::value, i = (s % KS) * 4 + g;
                    f32x16 acc = u[cur];
                    if constexpr (i == 0)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
                    u[cur] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fr[s & 1][g]), rb[i], acc, 0, 0, 0);
                    if constexpr (i < SLOTS)
                        search(std::integral_constant<int, cur ^ 1>{}, std::integral_constant<int, i * 16 / SLOTS>{},
                               std::integral_constant<int, (i + 1) * 16 / SLOTS>{});
                    __builtin_amdgcn_sched_barrier(0);
                };
                if constexpr (s % KS == 0) ask_taken(step * CPS + c);
                slot(std::integral_constant<int, 0>{});
                slot(std::integral_constant<int, 1>{});
                slot(std::integral_constant<int, 2>{});
                if constexpr (KS > 1 && s % KS == KS - 1) take_taken(step * CPS + c);
                slot(std::integral_constant<int, 3>{});
                if constexpr (KS == 1) take_taken(step * CPS + c);
                self(self, std::integral_constant<int, s + 1>{});
            }
        };
        fetch(std::integral_constant<int, 0>{});
        run(run, std::integral_constant<int, 0>{});
        step_end(more);
    };
    ex[0] = ex[1] = ~0ull;                                       // nothing to search before the first chunk
#pragma unroll
    for (int v = 0; v < 16; ++v) u[1][v] = 0.f;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    uint32_t so = 0, sn = (RING - 1) * STAGE;                    // the step's slot, and the one that is free
    auto turn = [&] { sn = so; so = so + STAGE == RING * STAGE ? 0 : so + STAGE; };
    for (int step = s0; step < s1; step += 2) {
        step_body(step, so, sn, std::integral_constant<int, 0>{});
        turn();
        if (step + 1 < s1) {
            step_body(step + 1, so, sn, std::integral_constant<int, 1>{});
            turn();
        }
    }
    using E0 = std::integral_constant<int, 0>;
    using E1 = std::integral_constant<int, 16>;
    if (CPS % 2 == 0 || (s1 - s0) % 2 == 0) search(std::integral_constant<int, 1>{}, E0{}, E1{});
    else search(std::integral_constant<int, 0>{}, E0{}, E1{});
    const float ob = __shfl_xor(best, 32, 64);
    const int oa = __shfl_xor(at, 32, 64);
    if (ob > best || (ob == best && oa < at)) { best = ob; at = oa; }
    if (row < a.rows && lh == 0) a.cand[row * a.splits + split] = OmpCand{best, at};
}

// ---- refit and residual ----
// The least-squares refit is kept as an incrementally built QR factorisation per row (modified Gram-Schmidt): with the
// picked columns Phi_S = Q T (Q orthonormal, T upper triangular), the residual update is r <- r - (q^T r) q for the new q
// only, and the coefficients follow once at the end from T x = Q^T y.  One wavefront per row, lane l holds elements
// l + 64 i of an m-vector, fp32 throughout.
template <typename T>
struct OmpUpdateArgs {
    const T* PhiT; long long ldp;             // [n, ldp] columns of Phi as rows
    const T* PhiQ;                            // [n, 64, pitch] the same in the lanes' order, pads zero (omp_pack_columns_kernel); a single pick, or
                                              // stored vectors: null
    const float* Y;                           // [rows, m]
    const OmpCand* cand; int splits;          // the pick is the best of these and is written to picks; null: picks holds it
    long long rows_whole;                     // ... rows before this one have a single candidate
    int* picks; int k, it;                    // [rows, k]
    uint32_t* taken; int nct;                 // as in OmpPickArgs (omp_pick_product_kernel only)
    float* Tri; float* Z;                     // [rows, k, k] triangular factor (column `it` written here), [rows, k] q^T y
    float* Fac;                               // [rows, k (k + 1) / 2] the same factor by columns, with 1 / its diagonal (omp_update_kernel)
    float* Qb;                                // [rows, k, mq] orthonormal vectors (omp_update_stored_kernel)
    T* R; long long ldr;                      // [rows, ldr] residual as the next product's operand, pads zero
    long long rows; int m, mq;
};

// The sum over a wavefront, in the order of a butterfly over lane distances 32, 16, 8, 4, 2, 1 (after the first three the
// values repeat every eight lanes, so a rotation by four is that exchange).  The same bits in every lane: no addition is contracted
// with a product that v is (one value per lane, m <= 64), whose two lanes would round differently.
__device__ __forceinline__ float wave_sum(float v) {
#pragma clang fp contract(off)
    v += __shfl_xor(v, 32, 64);
    v += __shfl_xor(v, 16, 64);
#define CSAT_DPP(CTRL) __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xf, 0xf, false))
    v += CSAT_DPP(0x128);       // row_ror:8
    v += CSAT_DPP(0x124);       // row_ror:4
    v += CSAT_DPP(0x4e);        // quad_perm [2,3,0,1]
    v += CSAT_DPP(0xb1);        // quad_perm [1,0,3,2]
#undef CSAT_DPP
    return v;
}
__device__ __forceinline__ float omp_lane(float v, int l) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l)); }

// values a lane's piece of a column is padded to: whole 16-byte loads (8 bytes where that is all)
constexpr __host__ __device__ int omp_column_pitch(int MQ, int esize) { return MQ <= 4 ? 4 : esize == 2 ? (MQ + 7) / 8 * 8 : (MQ + 3) / 4 * 4; }
// dst[j][lane][i] = Phi[lane + 64 i][j], from PhiT [n, ldp]; a thread per (j, lane), total of them
template <typename T>
static __global__ void omp_pack_columns_kernel(const T* PhiT, long long ldp, int m, int pitch, T* dst, long long total) {
    const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= total) return;
    const T* src = PhiT + (id >> 6) * ldp;
    for (int i = 0; i < pitch; i += 4) {
        typename std::conditional<sizeof(T) == 4, uint4, ushort4>::type w;
        T v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int l = (int)(id & 63) + 64 * (i + e);
            v[e] = l < m ? src[l] : (T)0;
        }
        w = __builtin_bit_cast(decltype(w), v);
        *(decltype(w)*)(dst + id * pitch + i) = w;
    }
}
template <int MQ>
__device__ __forceinline__ void omp_load_column(const float* PhiQ, int j, int lane, float (&v)[MQ]) {
    constexpr int P = omp_column_pitch(MQ, 4);
    const float* p = PhiQ + ((long long)j * 64 + lane) * P;
#pragma unroll
    for (int i = 0; i < P; i += 4) {
        const f32x4 a = *(const f32x4*)(p + i);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < MQ) v[i + e] = a[e];
    }
}
template <int MQ>
__device__ __forceinline__ void omp_load_column(const bf16_t* PhiQ, int j, int lane, float (&v)[MQ]) {
    constexpr int P = omp_column_pitch(MQ, 2), W = P == 4 ? 2 : 4;
    typedef uint32_t words __attribute__((ext_vector_type(W)));
    const bf16_t* p = PhiQ + ((long long)j * 64 + lane) * P;
#pragma unroll
    for (int i = 0; i < P; i += 2 * W) {
        const words a = *(const words*)(p + i);
#pragma unroll
        for (int e = 0; e < 2 * W; ++e)
            if (i + e < MQ) v[i + e] = __uint_as_float(e % 2 ? a[e / 2] & 0xffff0000u : a[e / 2] << 16);
    }
}
template <typename T, int MQ>
__device__ __forceinline__ void omp_load_pick(const OmpUpdateArgs<T>& a, int j, int lane, float (&v)[MQ]) {
    if (a.PhiQ) return omp_load_column<MQ>(a.PhiQ, j, lane, v);
#pragma unroll
    for (int i = 0; i < MQ; ++i) v[i] = lane + 64 * i < a.m ? Elem<T>::load(a.PhiT + j * a.ldp + lane + 64 * i) : 0.f;
}
// The pick of this call, written where the next launches look for it.
template <typename T>
__device__ __forceinline__ int omp_take_pick(const OmpUpdateArgs<T>& a, long long r, int lane) {
    if (!a.cand) return a.picks[r * a.k + a.it];
    const int nc = r < a.rows_whole ? 1 : a.splits;
    const OmpCand none{-1.f, 0x7fffffff};
    OmpCand b = lane < nc ? a.cand[r * a.splits + lane] : none;
    for (int q = 64; q < nc; q += 64) {                 // (the first 64 outside, where their read overlaps the others: 84 -> 83 us, 76 800 rows, m = 392)
        const OmpCand o = q + lane < nc ? a.cand[r * a.splits + q + lane] : none;
        if (o.val > b.val) b = o;                       // ascending columns per lane
    }
    if (nc > 1) {                                       // largest value, lowest index on a tie
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float ob = __shfl_xor(b.val, o, 64);
            const int oi = __shfl_xor(b.idx, o, 64);
            if (ob > b.val || (ob == b.val && oi < b.idx)) b = OmpCand{ob, oi};
        }
    }
    const int j = __builtin_amdgcn_readfirstlane(b.val >= 0.f ? b.idx : 0);     // (0: every correlation is NaN)
    if (lane == 0) {
        a.picks[r * a.k + a.it] = j;
        if (a.taken && a.it + 1 < a.k) atomicOr(a.taken + ((r >> 5) * a.nct + (j >> 5)) * 32 + omp_taken_word(j & 31), 1u << (r & 31));
    }
    return j;
}
// The new column v against the rest r: norm, coefficient, and the residual operand.
template <typename T, int MQ>
__device__ __forceinline__ void omp_finish_update(const OmpUpdateArgs<T>& a, long long r, int lane, float (&v)[MQ], float (&rv)[MQ], float* q_out, float* r_out) {
    float nn = 0.f;
#pragma unroll
    for (int i = 0; i < MQ; ++i) nn += v[i] * v[i];
    const float nrm = sqrtf(wave_sum(nn));
    const float inv = nrm > 0.f ? 1.f / nrm : 0.f;       // a column inside the span of the earlier picks adds nothing
    float zt = 0.f;
#pragma unroll
    for (int i = 0; i < MQ; ++i) {
        v[i] *= inv;
        if (q_out && lane + 64 * i < a.mq) q_out[lane + 64 * i] = v[i];
        zt += v[i] * rv[i];
    }
    zt = wave_sum(zt);
    if (lane == 0) {
        a.Tri[(r * a.k + a.it) * a.k + a.it] = nrm;
        if (!q_out) a.Fac[r * (a.k * (a.k + 1) / 2) + a.it * (a.it + 1) / 2 + a.it] = inv;
        a.Z[r * a.k + a.it] = zt;
    }
    if (a.it + 1 == a.k) return;                         // no product follows
#pragma unroll
    for (int i = 0; i < MQ; ++i) {
        const int l = lane + 64 * i;
        const float x = l < a.m ? rv[i] - zt * v[i] : 0.f;
        if (r_out && l < a.m) r_out[l] = x;
        if (l < a.ldr) Elem<T>::store(a.R + r * a.ldr + l, x);
    }
    for (int l = lane + 64 * MQ; l < a.ldr; l += 64) Elem<T>::store(a.R + r * a.ldr + l, 0.f);    // operand pads beyond the lanes' share
}

// No orthonormal vector and no residual is stored: the wavefront has the earlier ones again from the picked columns
// (which the L2 holds) and the stored factor, by the operations that formed them, and the residual from y by the
// operations that updated it, so every bit is the same.  Up to KQ picks (their vectors are KQ x MQ registers).
// 76 800 rows, m = 392, eight picks: with both stored a pick moved 0.97 GB on average and took 208 us; 73 us here.
// What bounds it: y and the operand copy (0.18 GB), it^2 / 2 multiply-adds per element.
template <typename T, int MQ, int KQ>
__global__ __launch_bounds__(256) void omp_update_kernel(OmpUpdateArgs<T> a) {
    const int lane = threadIdx.x & 63;
    const long long r = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r >= a.rows) return;
    const int it = a.it, k = a.k;
    const int j = omp_take_pick(a, r, lane);
    const int mine = lane < it ? a.picks[r * k + lane] : 0;
    float* fac = a.Fac + r * (k * (k + 1) / 2);
    constexpr int NF = (KQ * (KQ - 1) / 2 + 63) / 64;      // factors of the earlier picks, 64 a register
    float f[NF];
#pragma unroll
    for (int e = 0; e < NF; ++e) f[e] = lane + 64 * e < it * (it + 1) / 2 ? fac[lane + 64 * e] : 0.f;
    const float z = lane < it ? a.Z[r * k + lane] : 0.f;
    float v[MQ], rv[MQ], q[KQ][MQ];
    omp_load_pick<T, MQ>(a, j, lane, v);
#pragma unroll
    for (int s = 0; s < KQ - 1; ++s)
        if (s < it) omp_load_column<MQ>(a.PhiQ, __builtin_amdgcn_readlane(mine, s), lane, q[s]);
#pragma unroll
    for (int i = 0; i < MQ; ++i) rv[i] = lane + 64 * i < a.m ? a.Y[r * a.m + lane + 64 * i] : 0.f;
    auto factor = [&](int s, int t) { const int id = s * (s + 1) / 2 + t; return omp_lane(f[id / 64], id % 64); };
#pragma unroll
    for (int s = 0; s < KQ - 1; ++s)
        if (s < it) {
#pragma unroll
            for (int t = 0; t < s; ++t) {
                const float dot = factor(s, t);
#pragma unroll
                for (int i = 0; i < MQ; ++i) q[s][i] -= dot * q[t][i];
            }
            const float inv = factor(s, s), zt = omp_lane(z, s);
#pragma unroll
            for (int i = 0; i < MQ; ++i) {
                q[s][i] *= inv;
                rv[i] -= zt * q[s][i];
            }
            float dot = 0.f;
#pragma unroll
            for (int i = 0; i < MQ; ++i) dot += q[s][i] * v[i];
            dot = wave_sum(dot);
            if (lane == 0) {
                a.Tri[(r * k + s) * k + it] = dot;
                fac[it * (it + 1) / 2 + s] = dot;
            }
#pragma unroll
            for (int i = 0; i < MQ; ++i) v[i] -= dot * q[s][i];
        }
    omp_finish_update<T, MQ>(a, r, lane, v, rv, nullptr, nullptr);
}

// More picks than that, or few rows: orthonormal vectors and (in Rf) residuals stored.
template <typename T, int MQ>
__global__ __launch_bounds__(256) void omp_update_stored_kernel(OmpUpdateArgs<T> a, float* Rf) {
    const int lane = threadIdx.x & 63;
    const long long r = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r >= a.rows) return;
    const int it = a.it, k = a.k, mq = a.mq;
    const int j = omp_take_pick(a, r, lane);
    float* qrow = a.Qb + r * (long long)k * mq;
    float v[MQ], rv[MQ];
    omp_load_pick<T, MQ>(a, j, lane, v);
    const float* res = it == 0 ? a.Y + r * a.m : Rf + r * mq;
#pragma unroll
    for (int i = 0; i < MQ; ++i) rv[i] = lane + 64 * i < a.m ? res[lane + 64 * i] : 0.f;
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
        if (lane == 0) a.Tri[(r * k + s) * k + it] = dot;
#pragma unroll
        for (int i = 0; i < MQ; ++i) v[i] -= dot * qv[i];
    }
    omp_finish_update<T, MQ>(a, r, lane, v, rv, qrow + (long long)it * mq, Rf + r * mq);
}

// Coefficients from T x = z by back substitution, scattered into X (zeroed beforehand); optional
// copy of the picks and C[r,:] = sum_s x_s V[head(r), pick_s, :].
// KM >= k: what the loops over the picks are unrolled to (76 800 rows of eight picks: 77 us at 32, 50 us at 8).
template <typename T, int KM>
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
    float t[KM];
#pragma unroll
    for (int s = 0; s < KM; ++s) t[s] = s < k ? tri[row * k + (s >= row ? s : row)] : 0.f;
    float acc = lane < k ? Z[r * k + row] : 0.f, mine = 0.f;
    float x[KM];
#pragma unroll
    for (int s = KM - 1; s >= 0; --s) {
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
            for (int s = 0; s < KM; ++s)
                if (s < k) sum += x[s] * Elem<T>::load(v + (long long)__builtin_amdgcn_readlane(my_pick, s) * d + c);
            Elem<T>::store(C + r * (long long)d + c, sum);
        }
    }
}

}  // namespace csat

// ISTA decoder for problems so small that the whole packed Phi fits the LDS of a compute unit and a 32-row tile's
// whole iterate fits the registers of one wavefront (bf16): one launch runs every iteration, and between the load of
// Phi at the start and the stores of the result at the end a wavefront touches neither barrier nor memory, except for
// the rows of y that each iteration's residual starts from.
//
// The arithmetic is the fused decoder's (csat_ista_fused.h), product by product in the same order, so the results are
// the same bits: per 32-column chunk U^T = Phi_chunk^T r^T (fragments read from LDS with the transposing load),
// x <- eta_theta(x + mu U) in registers, racc -= Phi_chunk x^T (the same fragments read plainly).
//
// What bounded these shapes on the streaming kernels was the chain of chunk steps: at three tiles of m a step has 12
// MFMAs (384 cycles) but took about 2000, for the barrier, the wait for the staged chunk, the memory round trip of the
// old iterate and the requests of the next step.  Here a step is the MFMAs, their LDS reads (1 KB each: four
// wavefronts at the full MFMA rate need the whole LDS bandwidth, the bound that is left) and the threshold.
// Measured, whole forward before -> after: image_text (26 304 rows, n = 274, m = 96, 20 iterations) 221 -> 103 us;
// 76 800 rows, n = 300, m = 128: 675 -> 386; 131 072 rows, n = 512, m = 32: 1778 -> 383; 1096 rows of image_text's
// kind: 150 -> 88; n = 500, m = 150 (the largest Phi that fits), 128 000 rows: 1028 -> 511.
#pragma once
#include "csat_gemm_f32.h"
#include "csat_ista_fused.h"

namespace csat {

struct IstaResidentArgs {
    const uint4* PhiPack;   // [nct][ista_fused_set_frags(MT)][64], as the fused decoder's
    const float* Y;         // [rows, ldy], ldy = 32 * MT, columns >= m zero
    bf16_t* Xb;             // [rows, ldxb] bf16 copy of the final iterate, zero beyond n, or null
    float* Xout;            // [rows, n] or null
    int* status;            // set to 0: this decoder cannot give up
    long long rows;
    int n, nct, ldy, ldxb, iters;
    int tiles_per_wg;       // wavefronts of a workgroup that own a tile (1, 2 or 4)
    float mu, theta;
};

constexpr size_t ista_resident_lds_bytes(int MT, int nct) { return (size_t)nct * 2 * MT * 1024; }
// Chunk count of the instance that takes nct chunks at MT tiles of m, 0 if there is none: Phi has to fit the 160 KB of
// LDS, the iterate and the residual the 512 registers.  (The instances are straight-line code over their chunks: with
// a count that is only known at run time the branches made the compiler spill hundreds of registers.  Chunks between
// the row's and the instance's multiply zeros.)
constexpr int ista_resident_chunks(int MT, int nct) {
    const int c = nct <= 3 ? 3 : nct <= 5 ? 5 : nct <= 7 ? 7 : nct <= 9 ? 9 : nct <= 12 ? 12 : nct <= 16 ? 16 : 0;
    return MT <= 8 && c * MT <= 80 ? c : 0;
}

// NCT: chunks of the instance (nct <= NCT)
template <int MT, int NCT>
__global__ __launch_bounds__(256, 1) void ista_resident_kernel(IstaResidentArgs a) {
    extern __shared__ uint4 lds[];
    constexpr int NF = 2 * MT, SETF = ista_fused_set_frags(MT), CHUNK = NF * 1024;
    constexpr int G = 2;                        // fragments per LDS wait
    const int lane = threadIdx.x & 63, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nct = a.nct;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.status = 0;

    for (int f = wave; f < nct * NF; f += 4)    // all of Phi, 1 KB per request
        __builtin_amdgcn_global_load_lds((glb_ptr_t)(a.PhiPack + ((long long)(f / NF) * SETF + f % NF) * 64 + lane),
                                         (lds_ptr_t)((char*)lds + f * 1024), 16, 0, 0);
    for (int f = nct * NF + wave; f < NCT * NF; f += 4) lds[f * 64 + lane] = uint4{0u, 0u, 0u, 0u};
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (wave >= a.tiles_per_wg) return;         // (no barrier below)
    const long long rt = (long long)blockIdx.x * a.tiles_per_wg + wave;
    if (rt * 32 >= a.rows) return;
    const long long row = rt * 32 + (lane & 31);
    const bool row_ok = row < a.rows;
    const float* yrow = a.Y + (row_ok ? row : a.rows - 1) * a.ldy + 4 * lh;      // rows past the end compute on a valid row
    const uint32_t lds0 = (uint32_t)(size_t)(lds_ptr_t)lds;
    const uint32_t nat16 = lds0 + frag_slot(lane & 31, lh) * 16;                 // see ista_fused_kernel
    const uint32_t tr8 = lds0 + ((lane >> 4) & 1) * (MT * 1024) + frag_slot(4 * lh + ((lane & 15) >> 2), lane & 1) * 16 +
                         ((lane >> 1) & 1) * 8;

    f32x16 x[NCT], racc[MT], u;
    bf16x8 rb[NF], xb[2];
#pragma unroll
    for (int i = 0; i < NCT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) x[i][v] = 0.f;
    auto load_y = [&]() {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 y4 = *(const f32x4*)(yrow + 32 * mt + 8 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) racc[mt][4 * g + e] = y4[e];
            }
    };
    auto boundary = [&]() {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            rb[2 * mt] = cvt8<0>(racc[mt], 1.f);
            rb[2 * mt + 1] = cvt8<8>(racc[mt], 1.f);
        }
    };

    // One step: GEMM-U of chunk `cu` (DO_U) with the threshold of chunk I (DO_T) between its MFMAs, then GEMM-R of
    // chunk I (DO_R).
    auto step = [&](auto do_u, auto do_t, auto do_r, auto ic, int cu) {
        constexpr bool DO_U = decltype(do_u)::value, DO_T = decltype(do_t)::value, DO_R = decltype(do_r)::value;
        constexpr int I = decltype(ic)::value;
        constexpr int NU = DO_U ? NF : 0, NR = DO_R ? NF : 0, NA = NU + NR, NG = (NA + G - 1) / G;
        constexpr int NTG = NU / G, EPG = NTG > 0 ? (16 + NTG - 1) / NTG : 16;
        const uint32_t baseA = tr8 + cu * CHUNK, baseB = nat16 + I * CHUNK;
        auto ops = [](int k) constexpr {
            int c = 0;
            for (int i = 0; i < G; ++i) c += (k * G + i < NU) ? 2 : (k * G + i < NA) ? 1 : 0;
            return c;
        };
        u32x4 fr[2][G];
        u32x2 ft[2][G][2];
        f32x16 un;
        auto fetch = [&](auto kc, auto jc) {
            constexpr int k = decltype(kc)::value, i = decltype(jc)::value, f = k * G + i;
            if constexpr (f < NU) {
                lds_read8_tr<(f >> 1) * 1024 + (f & 1) * 256>(ft[k & 1][i][0], baseA);
                lds_read8_tr<(f >> 1) * 1024 + (f & 1) * 256 + 128>(ft[k & 1][i][1], baseA);
            } else if constexpr (f < NA) lds_read16<(f - NU) * 1024>(fr[k & 1][i], baseB);
        };
        auto fetch_group = [&](auto self, auto kc, auto jc) {
            constexpr int i = decltype(jc)::value;
            if constexpr (i < G) {
                fetch(kc, jc);
                self(self, kc, std::integral_constant<int, i + 1>{});
            }
        };
        auto threshold = [&](int v) {
            float xv = soft_threshold(x[I][v] + a.mu * u[v], a.theta);
            asm volatile("" : "+v"(xv));           // keeps the arithmetic between the MFMAs it is written next to
            x[I][v] = xv;
        };
        auto operand = [&]() {
            if constexpr (DO_R) {
                xb[0] = cvt8<0>(x[I], -1.f);
                xb[1] = cvt8<8>(x[I], -1.f);
            }
        };
#pragma unroll
        for (int v = 0; v < 16; ++v) un[v] = 0.f;
        using Z_ = std::integral_constant<int, 0>;
        if constexpr (NG > 0) fetch_group(fetch_group, Z_{}, Z_{});
        if constexpr (DO_T && NTG == 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) threshold(v);
            operand();
        }
        auto group = [&](auto kc) {
            constexpr int k = decltype(kc)::value;
            constexpr int NEXT = (k + 1 < NG) ? ops(k + 1) : 0;
            if constexpr (k + 1 < NG) fetch_group(fetch_group, std::integral_constant<int, k + 1>{}, Z_{});
            lds_wait_n<NEXT>();
#pragma unroll
            for (int i = 0; i < G; ++i) {
                if (k * G + i < NU) lds_pin(ft[k & 1][i][0], ft[k & 1][i][1]);
                else if (k * G + i < NA) lds_pin(fr[k & 1][i]);
            }
            if constexpr (DO_T && NTG > 0 && k == NTG) operand();
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const int f = k * G + i;
                if (f < NU) {
                    const u32x4 fa = __builtin_shufflevector(ft[k & 1][i][0], ft[k & 1][i][1], 0, 1, 2, 3);
                    un = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa), rb[f], un, 0, 0, 0);
                } else if (f < NA) {
                    const int r = f - NU;
                    racc[r % MT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fr[k & 1][i]),
                                                                           xb[r / MT], racc[r % MT], 0, 0, 0);
                }
            }
            if constexpr (DO_T && NTG > 0 && k < NTG) {
#pragma unroll
                for (int e = 0; e < EPG; ++e)
                    if (k * EPG + e < 16) threshold(k * EPG + e);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto run = [&](auto self, auto kc) {
            constexpr int k = decltype(kc)::value;
            if constexpr (k < NG) {
                group(kc);
                self(self, std::integral_constant<int, k + 1>{});
            }
        };
        run(run, Z_{});
        if constexpr (DO_U) u = un;
    };

    using T_ = std::true_type;
    using F_ = std::false_type;
    auto chunks = [&](auto self, auto ic, auto do_r) {
        constexpr int I = decltype(ic)::value;
        if constexpr (I + 1 < NCT) {
            step(T_{}, T_{}, do_r, ic, I + 1);
            self(self, std::integral_constant<int, I + 1>{}, do_r);
        } else {
            step(F_{}, T_{}, do_r, ic, 0);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    load_y();
    boundary();
    for (int t = 0; t + 1 < a.iters; ++t) {
        load_y();
        step(T_{}, F_{}, F_{}, I0{}, 0);
        chunks(chunks, I0{}, T_{});
        boundary();
    }
    step(T_{}, F_{}, F_{}, I0{}, 0);
    chunks(chunks, I0{}, F_{});
    if (!row_ok) return;
#pragma unroll
    for (int i = 0; i < NCT; ++i)
        {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = 32 * i + 8 * g + 4 * lh;
                if (a.Xb && col < a.ldxb)      // (zero beyond n; the instance's chunks beyond the row's hold NaN where y is infinite)
                    *(uint2*)(a.Xb + row * a.ldxb + col) =
                        i < nct ? uint2{f2bf_pk(x[i][4 * g], x[i][4 * g + 1]), f2bf_pk(x[i][4 * g + 2], x[i][4 * g + 3])} : uint2{0u, 0u};
                if (a.Xout) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < a.n) a.Xout[row * (long long)a.n + col + e] = x[i][4 * g + e];
                }
            }
        }
    if (a.Xb)                                   // operand columns beyond the instance's chunks
        for (int col = 32 * NCT + 4 * lh; col < a.ldxb; col += 8) *(uint2*)(a.Xb + row * a.ldxb + col) = uint2{0u, 0u};
}


// ----------------------------------------------------------------------------------------
// The same for float problems, with Phi, the residual and the iterate as three bf16 parts each and six part products
// per product (csat_gemm_f32.h).  A workgroup of 4 wavefronts owns one 32-row tile: the wavefronts split the chunks of
// n (wavefront w takes chunks w, w + 4, ...), and once per iteration their partial sums of Phi x meet in LDS, one tile
// of m at a time, where every thread forms two elements of y - Phi x and writes their parts as the next operands.
// Splitting a tile over the four SIMDs matters because these launches have few tiles: 256 x 256 with m = 64 (8 tiles)
// took 20 products of two or eight workgroups each, 445 us a forward with the launches between them; now 106 us, 41 of
// them this kernel.  Errors against float64 are at most those of the float MFMA's products (the residual's sums meet in a
// fixed order).
// ----------------------------------------------------------------------------------------
struct IstaResidentF32Args {
    const float* Phi;       // [m, n]
    const float* Y; long long ldY;      // [rows, ldY]
    float* Xs; long long ldS;           // [rows, ldS] final iterate, zero beyond n, or null
    float* Xout;                        // [rows, n] or null
    int* status;
    long long rows;
    int m, n, nct, iters;
    float mu, theta;
};

constexpr size_t ista_resident_f32_lds_bytes(int MT, int nct) { return ((size_t)nct * 6 * MT + 16 + 6 * MT) * 1024; }
constexpr int kResidentF32MaxMT = 4;
// Chunks per wavefront of the instance that takes nct chunks at MT tiles of m (whose Phi must fit LDS), 0: none
constexpr int ista_resident_f32_chunks(int MT, int nct) {
    if (MT > kResidentF32MaxMT || ista_resident_f32_lds_bytes(MT, nct) > 160 * 1024) return 0;
    const int c = (nct + 3) / 4;
    return MT == 1 ? (c <= 3 ? 3 : 6) : MT == 2 ? 3 : 2;
}

// One tile in plain float arithmetic: infinities, NaN and the smallest numbers then come out as the float products give
// them (EpiIstaUpdate's threshold turns a NaN into 0).  The residuals are in LDS (32 x m floats), the iterate where the result goes.
static __device__ __noinline__ void resident_f32_plain(const IstaResidentF32Args& a, long long row0, float* r, int tid) {
    const int rows = a.rows - row0 < 32 ? (int)(a.rows - row0) : 32;
    float* X = a.Xs ? a.Xs + row0 * a.ldS : a.Xout + row0 * a.n;
    const long long ld = a.Xs ? a.ldS : a.n;
    for (int i = tid; i < rows * a.n; i += 256) X[(i / a.n) * ld + i % a.n] = 0.f;
    for (int i = tid; i < rows * (int)(ld - a.n); i += 256) X[(i / (ld - a.n)) * ld + a.n + i % (ld - a.n)] = 0.f;
    for (int t = 0; t < a.iters; ++t) {
        __syncthreads();
        for (int i = tid; i < rows * a.m; i += 256) {
            const int q = i / a.m, l = i % a.m;
            float s = 0.f;
            if (t > 0)
                for (int j = 0; j < a.n; ++j) s += a.Phi[(long long)l * a.n + j] * X[q * ld + j];
            r[i] = a.Y[(row0 + q) * a.ldY + l] - s;
        }
        __syncthreads();
        for (int i = tid; i < rows * a.n; i += 256) {
            const int q = i / a.n, j = i % a.n;
            float s = 0.f;
            for (int l = 0; l < a.m; ++l) s += a.Phi[(long long)l * a.n + j] * r[q * a.m + l];
            float u = a.mu * s;
            if (t > 0) u += X[q * ld + j];
            const float b = fabsf(u) - a.theta;
            X[q * ld + j] = b > 0.f ? copysignf(b, u) : 0.f;
        }
    }
    __syncthreads();
    if (a.Xs && a.Xout)
        for (int i = tid; i < rows * a.n; i += 256) a.Xout[row0 * a.n + i] = X[(i / a.n) * ld + i % a.n];
}

template <int MT, int CPW>
__global__ __launch_bounds__(256, 1) void ista_resident_f32_kernel(IstaResidentF32Args a) {
    extern __shared__ uint4 lds[];
    constexpr int NF = 2 * MT, PLANE = NF * 1024, CHUNK = 3 * PLANE;     // bytes of one part of a chunk, of a chunk
    const int tid = threadIdx.x, lane = tid & 63, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nct = a.nct;
    const long long row0 = (long long)blockIdx.x * 32, row = row0 + (lane & 31);
    const bool row_ok = row < a.rows;
    float* red = (float*)((char*)lds + nct * CHUNK);                     // [wavefront][group][lane] float4 of one tile of m
    uint4* op = (uint4*)((char*)red + 16 * 1024);                        // [part][fragment][lane]: the residual's operands
    if (blockIdx.x == 0 && tid == 0) *a.status = 0;

    bool special = false;          // an input that is not finite, or so large that its parts or sums may not be
    // Phi's parts as fragments (pack_phi_fragments_kernel's order)
    for (int p = tid; p < nct * NF * 64; p += 256) {
        const int slot = p & 63, f = (p >> 6) % NF, ct = (p >> 6) / NF;
        const int h = slot >> 5, l = 32 * (f % MT) + ((slot & 31) ^ (4 * h)), j0 = 32 * ct + 16 * (f / MT) + 4 * h;
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int j = j0 + 8 * (q >> 2) + (q & 3);
            v[q] = l < a.m && j < a.n ? a.Phi[(long long)l * a.n + j] : 0.f;
            special |= !(fabsf(v[q]) <= 1e18f);
        }
        uint32_t w[3][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) split3(v[2 * q], v[2 * q + 1], w[0][q], w[1][q], w[2][q]);
#pragma unroll
        for (int s = 0; s < 3; ++s)
            lds[(ct * CHUNK + s * PLANE) / 16 + f * 64 + slot] = uint4{w[s][0], w[s][1], w[s][2], w[s][3]};
    }

    // This thread's share of the residual: elements 2 half, 2 half + 1 of group g of lane `el`, for every tile of m
    const int half = tid & 1, el = (tid >> 1) & 31, eh = (tid >> 6) & 1, g0 = tid >> 7;      // groups g0, g0 + 2
    const long long erow = row0 + el < a.rows ? row0 + el : a.rows - 1;
    float y[MT][2][2];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int l = 32 * mt + 8 * (g0 + 2 * k) + 4 * eh + 2 * half + e;
                y[mt][k][e] = l < a.m ? a.Y[erow * a.ldY + l] : 0.f;
                special |= !(fabsf(y[mt][k][e]) <= 1e18f);
            }
    // Whether any thread of the workgroup says so, through `red` (the compiler's own vote would need LDS beyond the 160 KB
    // that the largest instance fills)
    auto any = [&](bool mine) {
        __syncthreads();
        if (tid == 0) *(volatile int*)red = 0;
        __syncthreads();
        if (mine) *(volatile int*)red = 1;
        __syncthreads();
        const bool r = *(volatile int*)red != 0;
        __syncthreads();
        return r;
    };
    if (any(special)) {
        resident_f32_plain(a, row0, (float*)lds, tid);
        return;
    }
    const uint32_t nat16 = frag_slot(lane & 31, lh) * 16;
    const uint32_t tr8 = ((lane >> 4) & 1) * (MT * 1024) + frag_slot(4 * lh + ((lane & 15) >> 2), lane & 1) * 16 + ((lane >> 1) & 1) * 8;

    f32x16 x[CPW], racc[MT], rcorr[MT];
    bf16x8 rb[3][NF];
#pragma unroll
    for (int i = 0; i < CPW; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) x[i][v] = 0.f;

    // residual operands from the partial sums (first: Phi x = 0)
    auto residual = [&](bool first) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (!first) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 s;
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[e] = racc[mt][4 * g + e] + rcorr[mt][4 * g + e];
                    *(f32x4*)(red + ((wave * 4 + g) * 64 + lane) * 4) = s;
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int g = g0 + 2 * k, ln = el + 32 * eh;
                float r0 = y[mt][k][0], r1 = y[mt][k][1];
                if (!first) {
                    float s0 = 0.f, s1 = 0.f;
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const float2 p = *(const float2*)(red + ((w * 4 + g) * 64 + ln) * 4 + 2 * half);
                        s0 += p.x; s1 += p.y;
                    }
                    r0 -= s0; r1 -= s1;
                }
                uint32_t w[3];
                split3(r0, r1, w[0], w[1], w[2]);
#pragma unroll
                for (int s = 0; s < 3; ++s) ((uint32_t*)(op + (s * NF + 2 * mt + (g >> 1)) * 64 + ln))[(g & 1) * 2 + half] = w[s];
            }
            __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int f = 0; f < NF; ++f) rb[s][f] = __builtin_bit_cast(bf16x8, op[(s * NF + f) * 64 + lane]);
    };

    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    typedef __attribute__((address_space(3))) const char* lds_bytes_t;
    const lds_bytes_t base = (lds_bytes_t)(lds_ptr_t)lds;
    auto read_t = [&](uint32_t off) {      // a fragment of Phi^T
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(base + off));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(base + off + 128));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // one product: five smaller ones into `corr`, the large one into `acc`
    auto product = [](const bf16x8 (&p)[3], const bf16x8& q0, const bf16x8& q1, const bf16x8& q2, f32x16& acc, f32x16& corr) {
        corr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[2], q0, corr, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[0], q0, acc, 0, 0, 0);
        corr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[0], q2, corr, 0, 0, 0);
        corr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[1], q1, corr, 0, 0, 0);
        corr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[1], q0, corr, 0, 0, 0);
        corr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[0], q1, corr, 0, 0, 0);
    };
    residual(true);
    for (int t = 0; t < a.iters; ++t) {
        const bool last = t + 1 == a.iters;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) racc[mt][v] = rcorr[mt][v] = 0.f;
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            const int ct = wave + 4 * i;
            if (ct >= nct) continue;             // uniform
            const uint32_t chunk = ct * CHUNK;
            f32x16 u, uc;
#pragma unroll
            for (int v = 0; v < 16; ++v) u[v] = uc[v] = 0.f;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                bf16x8 p[3];
#pragma unroll
                for (int s = 0; s < 3; ++s) p[s] = read_t(chunk + tr8 + s * PLANE + (f >> 1) * 1024 + (f & 1) * 256);
                product(p, rb[0][f], rb[1][f], rb[2][f], u, uc);
            }
            bf16x8 xp[3][2];
#pragma unroll
            for (int v = 0; v < 16; ++v) x[i][v] = soft_threshold(x[i][v] + a.mu * (u[v] + uc[v]), a.theta);
            if (last) continue;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                uint32_t w[3][4];
#pragma unroll
                for (int k = 0; k < 4; ++k) split3(x[i][8 * q + 2 * k], x[i][8 * q + 2 * k + 1], w[0][k], w[1][k], w[2][k]);
#pragma unroll
                for (int s = 0; s < 3; ++s) xp[s][q] = __builtin_bit_cast(bf16x8, uint4{w[s][0], w[s][1], w[s][2], w[s][3]});
            }
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    bf16x8 p[3];
#pragma unroll
                    for (int s = 0; s < 3; ++s)
                        p[s] = __builtin_bit_cast(bf16x8, lds[(chunk + nat16 + s * PLANE + (q * MT + mt) * 1024) / 16]);
                    product(p, xp[0][q], xp[1][q], xp[2][q], racc[mt], rcorr[mt]);
                }
        }
        if (!last) residual(false);
    }
    // An iterate or a residual that left the range of float (a step far too large) stays infinite or NaN in its row: NaN
    // parts make every later product of the row NaN.  A row of measurements so small that their parts lose bits has an
    // iterate as small.
    SplitSuspect suspect;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        if (wave + 4 * i >= nct) continue;
#pragma unroll
        for (int v = 0; v < 16; ++v) suspect.add(x[i][v]);
    }
    if (any(suspect.any())) {
        resident_f32_plain(a, row0, (float*)lds, tid);
        return;
    }
    if (!row_ok) return;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int ct = wave + 4 * i;
        if (ct >= nct) continue;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = 32 * ct + 8 * g + 4 * lh;
            if (a.Xs && col < a.ldS)             // (ldS is a multiple of 8, less than 32 beyond n)
                *(f32x4*)(a.Xs + row * a.ldS + col) = f32x4{x[i][4 * g], x[i][4 * g + 1], x[i][4 * g + 2], x[i][4 * g + 3]};
            if (a.Xout) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < a.n) a.Xout[row * (long long)a.n + col + e] = x[i][4 * g + e];
            }
        }
    }
}

}  // namespace csat

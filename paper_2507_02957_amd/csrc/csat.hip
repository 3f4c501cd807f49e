// C ABI of the CSAT forward pass (see include/csat.h): argument checks, workspace carving and
// kernel launches.  All arithmetic of the path lives in csat_kernels.h.
#include "csat.h"
#include "csat_kernels.h"
#include "csat_ista_fused.h"
#include "csat_ista_coop.h"
#include "csat_ista_resident.h"
#include "csat_omp.h"
#include "csat_fwht.h"
#include "csat_gemm_big.h"
#include "csat_gemm_f32.h"
#include "csat_gemm_deep.h"
#include "csat_attention.h"
#include "csat_attention_z.h"
#include "csat_measure.h"
#include "csat_support.h"
#include "csat_screen.h"
#include "csat_launch.h"
#include "csat_peaks.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <thread>
#include <vector>

using namespace csat;

namespace {

// Optional per-kernel timing: when enabled, a pair of HIP events brackets every launch on the
// caller's stream; csat_profile_read sums the elapsed times per kernel id.
struct Profiler {
    struct Span { int kid; hipEvent_t a, b; };
    bool on = false;
    std::vector<Span> spans;
    void begin(int kid, hipStream_t st) {
        if (!on) return;
        Span s{kid, nullptr, nullptr};
        if (hipEventCreate(&s.a) != hipSuccess || hipEventCreate(&s.b) != hipSuccess) return;
        (void)hipEventRecord(s.a, st);      // profiling is best effort: a failed record shows up as a failed read
        spans.push_back(s);
    }
    void end(hipStream_t st) {
        if (on && !spans.empty()) (void)hipEventRecord(spans.back().b, st);
    }
    void clear() {
        for (auto& s : spans) { (void)hipEventDestroy(s.a); (void)hipEventDestroy(s.b); }
        spans.clear();
    }
};

// Kernel-selection overrides (csat_set_option).  All zero = the library's own choices; a call's
// results and workspace needs never depend on anything but its arguments and these.
struct Options {
    int v[CSAT_OPT_COUNT] = {};
    int operator[](int k) const { return v[k]; }
};

struct Context {
    uint32_t magic;
    Profiler prof;
    Options opt;
    int decoder_kernel = -1;     // what the last decoder call on this context launched (csat_profile_decoder_kernel)
    int forms[CSAT_FORM_COUNT] = {};     // ... and the last call of any kind (csat_profile_launch_form)
};
constexpr uint32_t kMagic = 0x43534154u;   // "CSAT"

// Options of the call in progress on this thread (set by OptionScope at the top of every entry point
// that launches kernels; the defaults otherwise, e.g. in the host-only size queries).
const Options kDefaultOptions{};
thread_local const Options* tl_opt = &kDefaultOptions;
int tl_decoder_kernel_sink = -1;
thread_local int* tl_decoder_kernel = &tl_decoder_kernel_sink;
thread_local int tl_forms_sink[CSAT_FORM_COUNT];
thread_local int* tl_forms = tl_forms_sink;
struct OptionScope {
    const Options* prev;
    int *prev_kernel, *prev_forms;
    explicit OptionScope(void* ctx) : prev(tl_opt), prev_kernel(tl_decoder_kernel), prev_forms(tl_forms) {
        Context* c = static_cast<Context*>(ctx);
        tl_opt = &c->opt;
        tl_decoder_kernel = &c->decoder_kernel;
        if (tl_forms != c->forms) std::memset(c->forms, 0, sizeof c->forms);      // (a call within a call adds to it)
        tl_forms = c->forms;
    }
    ~OptionScope() { tl_opt = prev; tl_decoder_kernel = prev_kernel; tl_forms = prev_forms; }
};

inline long long round_up(long long v, long long a) { return (v + a - 1) / a * a; }
// bf16 round trip on the host (round to nearest even), for scalars the kernels must see as the element type does
inline uint16_t f2bf_host(float f) {
    uint32_t u;
    std::memcpy(&u, &f, 4);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
inline float bf2f_host(uint16_t h) {
    const uint32_t u = (uint32_t)h << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t esize(csat_dtype t) { return t == CSAT_BF16 ? 2 : 4; }

csat_status check_dims(const csat_dims* d) {
    if (!d) return CSAT_ERR_NULL;
    if (d->dtype != CSAT_F32 && d->dtype != CSAT_BF16) return CSAT_ERR_DTYPE;
    if (d->B <= 0 || d->H <= 0 || d->n_q <= 0 || d->n <= 0 || d->d <= 0 || d->m <= 0) return CSAT_ERR_SHAPE;
    if (d->m > d->n || (d->d % 8) != 0) return CSAT_ERR_SHAPE;
    if ((long long)d->B * d->H > 65535) return CSAT_ERR_SHAPE;
    if ((long long)d->B * d->H * d->n_q > 0x7fffffffLL) return CSAT_ERR_SHAPE;
    return CSAT_OK;
}
csat_status check_ctx(void* ctx) {
    if (!ctx) return CSAT_ERR_NULL;
    return static_cast<Context*>(ctx)->magic == kMagic ? CSAT_OK : CSAT_ERR_PARAM;
}

// Kernel-selection overrides of the call in progress (see csat_set_option in csat.h).
int decoder_choice() { const int o = (*tl_opt)[CSAT_OPT_DECODER]; return o == 1 || o == 2 ? o : 0; }   // 1: GEMM pair per iteration; 2: fused wherever it fits
int gemm_raster_choice() { return ((*tl_opt)[CSAT_OPT_RASTER] & 7) == 1 ? 0 : 1; }   // 0: column-fastest everywhere
// A row operand larger than the Infinity Cache, which a launch with XCD-owned column groups reads once per group:
// its loads carry the non-temporal hint, so that they displace less of what the launch re-reads.  Measured on
// long_video's update GEMM (A = 0.5 GB): 12.9 -> 12.2 ms per launch; a 20 MB operand (cross_modal) is better off
// cached (0.205 -> 0.219 ms with the hint), and so is the residual GEMM's 8.6 GB row operand, whose four column
// tiles share every row (7.2 -> 7.4 ms with it).  (Option bits 8 / 16: never / always, for measurements.)
bool stream_hint(long long bytes) {
    const int rx = (*tl_opt)[CSAT_OPT_RASTER];
    return (rx & 8) ? false : (rx & 16) ? true : bytes > (256LL << 20);
}
int lista_choice() { return (*tl_opt)[CSAT_OPT_LISTA] == 1 ? 1 : 0; }                // 1: element-wise epilogue
int hadamard_choice() { return (*tl_opt)[CSAT_OPT_HADAMARD] == 1 ? 1 : 0; }          // 1: iterate in LDS
int gemm_choice() { return (*tl_opt)[CSAT_OPT_GEMM] == 1 ? 1 : 0; }                  // 1: 128-wide kernel only

constexpr size_t kLdsPerWorkgroup = 160 * 1024;     // LDS of a gfx950 compute unit

// The fused decoder keeps its fp32 iterate either sparse in memory (per-lane masks: only non-zero float4
// are read and written) or dense (the whole iterate streams every iteration).  Sparse pays when the
// dense iterate is too large to stay cache-resident between iterations (short_video, 491 MB: 4.4 ms
// against 5.0 ms); on a small problem the masks only add latency (image_text, 30 MB: 0.23 ms against
// 0.19 ms).  CSAT_OPT_STATE overrides the choice (for comparing the two).
bool sparse_state(size_t dense_state_bytes) {
    const int o = (*tl_opt)[CSAT_OPT_STATE] & 3;
    if (o == 1) return false;
    if (o == 2) return true;
    return dense_state_bytes > ((size_t)128 << 20);
}

constexpr size_t kStaticScratchBytes = (size_t)48 << 20;      // csat_forward_static's workspace

// The decoders' rule for products over the support of the iterate (csat_support.h), its words in the workspace's status block.
int support_choice() { return (*tl_opt)[CSAT_OPT_SUPPORT]; }      // 1: never; 2: wherever a kernel exists
constexpr int kSupportWord = 8;
int screen_choice() { return (*tl_opt)[CSAT_OPT_SCREEN]; }        // 1: never; 2: wherever it applies
constexpr int kScreenWord = 16, kScreenSampleWord = 24;
// Of the sample's rows, the most that may stay: at most half the rows fit packed, of which the product over all rows makes sure.  45 % left, 13 104 rows, n = 11 744,
// m = 1024: 9.8 -> 7.5 ms.  The sample of about 1000 rows is off by 1.6 % now and then by three times that: at 0.45, 60 928 rows, n = 7616, m = 1024 with 42.7 % left
// took 27.5 ms instead of 14.5; where more than half stay after all, the product over all rows is lost, 3 % of 14 iterations.
constexpr double kScreenShare = 0.48;

// Largest m (in 32-wide tiles) the fused decoder takes.  Its residual accumulators need 16 registers per tile: up to
// 13 tiles they fit next to the operands of the two-chunk schedule; 14 to 16 tiles fill the accumulator file and run
// on the one-chunk schedule with 128-row workgroups (a few dozen spilled registers).  That still beats the large-tile
// GEMM pair when the launch has enough 128-row groups to occupy a good part of the chip (cross_modal, m = 512,
// 154 groups: 7.3 against 9.1 ms; short_video's shape at m = 512, 600 groups: 5.2 against 8.3 ms per forward), not
// below: a group's iterations are a chain, so the launch lasts as long with 40 groups as with 150 (cross_modal's rows
// with fewer heads, forward: 39 groups 6.5 against 3.8 ms, 97 groups 7.5 against 7.2, 121 groups 7.9 against 7.6).
constexpr int kFusedMaxMT = 16;
constexpr int kFused2MaxMT = 13;
constexpr long long kFusedWideMinGroups = 128;
// Polls (about 1 us apart) a unit of the fused decoder waits for the preceding segment of its rows, or a workgroup for the
// others of its tile, before it gives up; several seconds, against a whole launch of a few milliseconds.
// CSAT_OPT_FUSED_SPIN_LIMIT overrides it.
constexpr long long kFusedSpinLimit = 1ll << 22;

// Workspace layout: one carving shared by every entry point (each uses a subset), so one
// size query serves all four calls.
struct Workspace {
    long long ldn, ldm;      // padded leading dimensions of n- and m-long operand rows
    long long ldy;           // leading dimension of the fp32 measurement rows (multiple of 32)
    int MT, nct;             // 32-wide tiles along m and n (fused decoder)
    long long rows_pad;      // rows rounded up to the fused decoder's 128-row workgroups
    bool fused;              // the fused decoder runs this shape (it applies and is not overridden)
    int* Status;     // [64]  word 0: the ISTA decoder of the last call gave up (read by csat_decoder_status)
    uint4* PhiPack;  // [nct, ~2*MT, 64]  Phi as MFMA fragments for the fused decoder
    int* FusedSync;  // [2 + rows_pad/32]  unit counter, error flag and per-group progress of the fused decoder
    uint4* Hand;     // [rows_pad/128, 4, 2*MT, 64]  residual operands handed between segments of the fused decoder
    uint8_t* Mask;   // [rows_pad/32, nct or ldn/32, 64]  non-zero masks of the sparse fp32 state (bf16 mode)
    char* PhiP;   // [m, ldn]      Phi, operand layout
    char* PhiT;   // [n, ldm]      Phi^T
    char* KT;     // [BH, d, ldn]  K^T per head
    char* VT;     // [BH, d, ldn]  V^T per head
    char* Kc;     // [BH, m, d]
    char* Vc;     // [BH, m, d]
    bf16_t* KcHL; // [BH, m, 2d]   bf16 (hi | lo) split of K~ for the score contraction (bf16 mode)
    uint4* KcPack; // [BH, MT, parts * groups, 64]  K~ as MFMA fragments for the one-kernel compressed attention (d <= 128)
    char* VcT;    // [BH, d, ldm]
    float* A;     // [rows, ldy]   compressed attention rows (the decoder's measurements), zero padded
    char* R;      // [rows, ldm]   softmax / residual operand
    float* Xs;    // [rows, ldn]   decoder state ([rows_pad, 32*nct] in fragment order when fused)
    bf16_t* Xb;   // [rows, ldn]   bf16 operand copy of the state (bf16 mode)
    char* Z;      // [rows, d]
    int split;    // > 1: the residual product runs as this many partial products along K (few output tiles)
    float* SplitP;  // [split, rows, ldm]  their outputs
    int tile_split;  // > 1: workgroups per 32-row tile of the shared-tile decoder
    int* TileSync;   // [2 + 2 * tiles * tile_split]  ... their counter and flags
    f32x4* Xchg;     // [tiles, tile_split, 2, MT, 4, 64]  ... and their parts of the residual (in SplitP's place)
    size_t bytes;
    Profiler* prof;   // never null during a call
};

// Workgroups that share a 32-row tile of the shared-tile decoder (csat_ista_coop.h), each with its share of the columns: as
// many as make an iteration shortest by these fits to measured ones (us): a chunk 0.25 + 0.025 MT (two more for the
// pipeline's ramp), the exchange of the parts of the residual 1.5 + (0.4 + 0.035 MT) a member and up to 3 with the chip full of
// members.  20 iterations, one to sixteen members: 96 tiles, m = 392, n = 1600 612, 417 us; 30 tiles 591, 372, three 318, four 315,
// five 298, eight 346; 8 tiles four 282, five 267, six 274, twelve 333; n = 3000, m = 130, 10 tiles 763, 438, four 275, eight 217, twelve
// 213, sixteen 227; n = 2000, m = 224, 10 tiles 543, 324, four 224, eight 192, twelve 222; n = 16 384, m = 64, 8 tiles 2835, 1477, sixteen
// 305; n = 512, m = 392, 120 tiles 227, 247.
// Not for fewer than four iterations, whose sums so keep the order of the other decoders, nor to save less than
// kTileSplitMinUs of a call.
constexpr int kTileSplitMinIters = 4, kTileSplitMax = 16;
constexpr double kTileSplitMinUs = 20;
double coop_iteration_us(int MT, long long tiles, int nct, int members) {
    const double exchange = members == 1 ? 0 : 1.5 + members * (0.4 + 0.035 * MT) + (double)(tiles * members) / 256 * 3;
    return ((nct + members - 1) / members + 2) * (0.25 + 0.025 * MT) + exchange;
}
int coop_tile_split(int MT, long long tiles, int nct) {
    int best = 1;
    for (int g = 2; MT <= kCoopMaxMT && g <= kTileSplitMax && g * tiles <= 256 && g * 4 <= nct; ++g)
        if (coop_iteration_us(MT, tiles, nct, g) < coop_iteration_us(MT, tiles, nct, best)) best = g;
    return best;
}

Workspace carve(const csat_dims& d, char* base) {
    Workspace w{};
    const size_t e = esize(d.dtype);
    const long long BH = (long long)d.B * d.H, rows = BH * d.n_q;
    // bf16 operand rows are zero-padded to a multiple of 64 elements (the large-tile GEMM's K step)
    const long long kpad = d.dtype == CSAT_BF16 ? 64 : 8;
    w.ldn = round_up(d.n, kpad);
    w.ldm = round_up(d.m, kpad);
    w.ldy = round_up(d.m, 32);
    w.MT = (int)(w.ldy / 32);
    w.nct = (int)((d.n + 31) / 32);
    w.rows_pad = round_up(rows, 128);
    // The carving does not depend on the kernel-selection overrides: buffers that differ between the
    // fused decoder and the GEMM pair are sized for the larger of the two.
    const bool fused_ok = d.dtype == CSAT_BF16 && w.MT <= kFusedMaxMT && w.nct >= 3;
    const bool fused_pays = w.MT <= kFused2MaxMT || w.rows_pad / 128 >= kFusedWideMinGroups;
    w.fused = fused_ok && decoder_choice() != 1 && (fused_pays || decoder_choice() == 2);
    size_t off = 0;
    auto take = [&](size_t nbytes) {
        char* p = base + off;
        off += (size_t)round_up((long long)nbytes, 256);
        return p;
    };
    w.Status = (int*)take(256);
    w.PhiP = take((size_t)d.m * w.ldn * e);
    w.PhiT = take((size_t)d.n * w.ldm * e);
    w.KT = take((size_t)BH * d.d * w.ldn * e);
    w.VT = take((size_t)BH * d.d * w.ldn * e);
    w.Kc = take((size_t)BH * d.m * d.d * e);
    w.Vc = take((size_t)BH * d.m * d.d * e);
    w.KcHL = (bf16_t*)take(d.dtype == CSAT_BF16 ? (size_t)BH * d.m * d.d * 4 : 0);
    w.KcPack = (uint4*)take(d.d <= 128 ? (size_t)BH * w.MT * (d.dtype == CSAT_BF16 ? 2 * ((d.d + 15) / 16) : (d.d + 7) / 8) * 1024 : 0);
    w.VcT = take((size_t)BH * d.d * w.ldm * e);
    // (chunk count rounded up to even: the two-chunk schedule walks whole pairs, the odd one out is a zero chunk)
    w.PhiPack = (uint4*)take(fused_ok ? (size_t)((w.nct + 1) / 2 * 2) * ista_fused_set_frags(w.MT) * 1024 : 0);
    w.FusedSync = (int*)take(fused_ok ? (size_t)(2 + w.rows_pad / 32) * 4 : 0);
    w.Hand = (uint4*)take(fused_ok ? (size_t)(w.rows_pad / 128) * 4 * 2 * w.MT * 1024 : 0);
    // ldn >= 32 * nct, so the GEMM pair's mask and state sizes cover the fused decoder's
    w.Mask = (uint8_t*)take(d.dtype == CSAT_BF16 ? (size_t)(w.rows_pad / 32) * (w.ldn / 32) * 64 : 0);
    w.A = (float*)take((size_t)rows * w.ldy * 4);
    w.R = take((size_t)rows * w.ldm * e);
    w.Xs = (float*)take((size_t)w.rows_pad * w.ldn * 4);
    w.Xb = (bf16_t*)take(d.dtype == CSAT_BF16 ? (size_t)rows * w.ldn * 2 : 0);
    w.Z = take((size_t)rows * d.d * e);
    // A residual product with few 256 x 256 output tiles leaves most of the chip idle while each tile
    // walks the whole of K = n: split K so that tiles x parts comes close to the 256 CUs this is sized
    // for (parts divides the number of 64-wide K steps, at most 8).
    w.split = 1;
    if (d.dtype == CSAT_BF16 && rows >= 256 && w.ldm >= 128) {
        const long long tiles = ((rows + 255) / 256) * ((w.ldm + 255) / 256), ksteps = w.ldn / 64;
        for (int s = 2; s <= 8; ++s)
            if (ksteps % s == 0 && tiles * s <= 256) w.split = s;
    }
    // ... and the parts of the residual of the shared-tile decoder, where several workgroups share a tile: never both
    const long long tiles32 = (rows + 31) / 32;
    const size_t split_bytes = w.split > 1 ? (size_t)w.split * rows * w.ldm * 4 : 0;
    w.tile_split = fused_ok ? coop_tile_split(w.MT, tiles32, w.nct) : 1;
    const size_t before = off;
    auto parts = [&](size_t bytes) { return w.tile_split > 1 ? std::max(bytes, (size_t)tiles32 * w.tile_split * 2 * w.MT * 4096) : bytes; };
    w.SplitP = (float*)take(parts(split_bytes));
    w.TileSync = (int*)take(w.tile_split > 1 ? (size_t)(2 + 2 * tiles32 * w.tile_split) * 4 : 0);
    if (off > kStaticScratchBytes && before + round_up((long long)split_bytes, 256) <= (long long)kStaticScratchBytes) {   // (what fits the static array without still does)
        w.tile_split = 1;
        off = before;
        w.SplitP = (float*)take(split_bytes);
    }
    w.Xchg = (f32x4*)w.SplitP;
    w.bytes = off;
    return w;
}

#define HIP_TRY(expr)                                  \
    do {                                               \
        if ((expr) != hipSuccess) return CSAT_ERR_HIP; \
    } while (0)
#define CSAT_TRY(expr)                  \
    do {                                \
        csat_status s_ = (expr);        \
        if (s_ != CSAT_OK) return s_;   \
    } while (0)

// No option asks for a decoder, or for a property of one: any that does is honoured.
bool decoder_not_asked_for() {
    const Options& o = *tl_opt;
    return !(o[CSAT_OPT_DECODER] || o[CSAT_OPT_STATE] || o[CSAT_OPT_FUSED_SEGMENTS] || o[CSAT_OPT_FUSED_THIN] || o[CSAT_OPT_FUSED_SCHEDULE]);
}
// Whether the ISTA decoder keeps Phi in LDS and the iterate in registers (csat_ista_resident.h).  It has no wait to limit
// and no error record to preset: those options ask for a decoder that does.
bool decoder_options_free() {
    return decoder_not_asked_for() && !((*tl_opt)[CSAT_OPT_FUSED_SPIN_LIMIT] || (*tl_opt)[CSAT_OPT_INJECT_DECODER_ERROR]);
}
bool decoder_is_resident(const Workspace& w) {
    return decoder_options_free() && w.fused && ista_resident_chunks(w.MT, w.nct) != 0;      // (fused: bf16, and n > 64)
}
// CUs of the current device (persistent grids and work-distribution heuristics)
int cu_count() {
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) return 256;
        return v;
    }();
    return n;
}

// ... and its float form.  One iteration is one product: nothing to keep in LDS.  Every 32-row tile splits Phi anew, so two
// or three iterations of many tiles are better off on the products unless Phi is one tile of m (n = 64, m = 64, two
// iterations: 20 000 rows 42 us against 54 on the products, 80 000 rows 116 against 96, 200 000 rows 274 against 189, three
// iterations 333 against 282; m = 32: 64 against 86 and 135 against 158).
bool decoder_is_resident_f32(const csat_dims& d, const Workspace& w, int iters) {
    return d.dtype == CSAT_F32 && iters >= 2 && decoder_options_free() && gemm_choice() != 1 && ista_resident_f32_chunks(w.MT, w.nct) != 0 &&
           (iters >= 4 || w.MT == 1 || w.rows_pad / 32 <= 4ll * cu_count());
}

struct Timed {   // brackets the launches issued during its lifetime
    Profiler* p; hipStream_t st;
    Timed(const Workspace& w, int kid, hipStream_t s) : p(w.prof), st(s) { p->begin(kid, st); }
    ~Timed() { p->end(st); }
};

template <typename T, int BM, int BN, int WM, int WN, typename Epi>
csat_status launch_gemm(const GemmArgs& g, long long n_cover, int batch, const Epi& epi, hipStream_t st) {
    // n_cover >= N: columns the epilogue must visit (pads included)
    dim3 grid((unsigned)((g.M + BM - 1) / BM), (unsigned)((n_cover + BN - 1) / BN), (unsigned)batch);
    hipLaunchKernelGGL((gemm_nt_kernel<T, BM, BN, WM, WN, Epi>), grid, dim3(256), 0, st, g, epi);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

template <typename Epi, int WM, int WN, int KS, int TN = 4>
csat_status launch_gemm_big_shape(const GemmArgs& g, long long n_cover, int batch, const Epi& epi, hipStream_t st) {
    using S = BigGemmShape<Epi, WM, WN, KS, TN>;
    HIP_TRY(hipFuncSetAttribute((const void*)gemm_nt_bf16_big_kernel<Epi, WM, WN, KS, TN>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::kLdsBytes));
    const long long tm = (g.M + S::kRowsA - 1) / S::kRowsA, tn = (n_cover + S::kRowsB - 1) / S::kRowsB;
    GemmArgs gt = g;
    gt.a_kwrap = (int)tn;     // column tiles: the kernel walks a 1-D grid
    gt.raster = (tn <= 8 && batch == 1 && gemm_raster_choice() != 0) ? 1 : 0;
    // many column tiles, a multiple of 8: each XCD keeps a few column tiles' operand in its L2 (see the kernel)
    if (const int rx = (*tl_opt)[CSAT_OPT_RASTER], ro = rx & 7; tn >= 16 && tn % 8 == 0 && batch == 1 && ro != 1) {
        const int per_xcd = (int)(tn / 8);
        int cb = ro >= 2 ? 1 << (ro - 2) : 4;                  // (option values 2, 3, 4, 5: groups of 1, 2, 4, 8 for measurements)
        while (cb > 1 && per_xcd % cb != 0) cb >>= 1;
        gt.raster = 2 + (cb == 8 ? 3 : cb == 4 ? 2 : cb == 2 ? 1 : 0);
        if (stream_hint((long long)g.M * g.K * 2)) gt.raster |= kRasterStreamA;
    }
    const long long tiles = gt.raster == 1 ? (tm + 7) / 8 * 8 * tn : tm * tn;
    dim3 grid((unsigned)tiles, 1, (unsigned)batch);
    hipLaunchKernelGGL((gemm_nt_bf16_big_kernel<Epi, WM, WN, KS, TN>), grid, dim3(S::kThreads), S::kLdsBytes, st, gt, epi);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

// 256 x 256 x 64 tiles, 8 wavefronts.  (A 256 x 128 x 32 shape with two workgroups per CU, meant to
// run one workgroup's epilogue under the other's main loop, measured slower on every workload.)
template <typename Epi>
csat_status launch_gemm_big(const GemmArgs& g, long long n_cover, int batch, const Epi& epi, hipStream_t st) {
    return launch_gemm_big_shape<Epi, 4, 2, 64>(g, n_cover, batch, epi, st);
}

// 256 x 320 tiles where they take less of the CUs' time: a CU has one tile at a time, so that is whole rounds of tiles times
// their width, and a twelfth for the wider tile's loop.  A forward of 20 layers over 76 800 rows, n = 1600 (six rounds of 320 against nine of
// 256): 8.63 ms against 9.60; not where the rounds are as wide: 8 layers over 16 000 rows, n = 2000 (two, two) 1.51 against 1.43,
// 6 over 8000, n = 3500 (two, two) 1.32 against 1.17.
bool wide_tiles_pay(const GemmArgs& g, long long n_cover) {
    auto cost = [&](int width) {
        const long long tiles = (g.M + 255ll) / 256 * ((n_cover + width - 1) / width);
        return (tiles + cu_count() - 1) / cu_count() * width;
    };
    return cost(320) * 13 < cost(256) * 12;
}
template <typename Epi>
csat_status launch_gemm_big_lista(const GemmArgs& g, long long n_cover, const Epi& epi, hipStream_t st) {
    const bool wide = wide_tiles_pay(g, n_cover);
    tl_forms[CSAT_FORM_LISTA_TILE] = wide ? 320 : 256;
    if (wide) return launch_gemm_big_shape<Epi, 4, 2, 64, 5>(g, n_cover, 1, epi, st);
    return launch_gemm_big<Epi>(g, n_cover, 1, epi, st);
}

// Big bf16 problems whose operands are zero-padded to a multiple of 64 along K (every workspace
// operand is) go to the 256x256 kernel.  Otherwise: narrow-N problems (N <= 64) waste half of a
// 128-wide tile, so they get the 64-wide one.
template <typename T>
bool use_big_gemm(const GemmArgs& g, long long n_cover) {
    if (sizeof(T) != 2) return false;
    const long long Kp = round_up(g.K, 64);
    return Kp <= g.lda && Kp <= g.ldb && g.a_kwrap == 0 && g.M >= 256 && n_cover >= 128 && gemm_choice() != 1;
}

// float products (csat_gemm_f32.h)
template <typename Epi>
csat_status launch_gemm_f32(GemmArgs g, long long n_cover, int batch, const Epi& epi, hipStream_t st) {
    g.raster = (int)((n_cover + kF32TileN - 1) / kF32TileN);      // column tiles; row tiles in whole groups of eight
    const dim3 grid((unsigned)((g.M + 8 * kF32TileM - 1) / (8 * kF32TileM) * 8 * g.raster), 1, (unsigned)batch);
    hipLaunchKernelGGL((gemm_nt_f32_split_kernel<Epi>), grid, dim3(256), 0, st, g, epi);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

// Products that would be so few 128-wide tiles that most CUs had none go to small tiles, a workgroup each, whose wavefronts share the
// contraction (csat_gemm_deep.h): 32 x 32, or 64 x 64 in bf16 from two of the small ones per CU on.  Measurement of K and V (with its
// transposes), 128-wide against 32-wide (64-wide) tiles, us: float, n = 1600, m = 392, d = 64: one head 73.8, 21.0 (57.3), 12 heads (96 tiles of
// 128 x 64) 82.4, 58.2 (65.4), 48 heads (384) 142, 168; 64 heads of n = 300, m = 96 (128) 30.2, 30.3; bf16: 10 heads of
// n = 1571, m = 197, d = 80 (40) 41.2, 29.8 (30.1), 4 heads of n = 16 384, m = 1024, d = 80 (64) 247, 210 (160), 392 x 3072 over
// 3200 (96) equal, 16 heads of n = 4096, m = 512, d = 96 (128) 83.6, 121 (95.5).
template <typename T>
bool few_tiles(const GemmArgs& g, long long n_cover, int batch) {
    const long long wide = n_cover <= 64 ? 64 : 128, tiles = (g.M + 127ll) / 128 * ((n_cover + wide - 1) / wide) * batch;
    return tiles * 8 <= (sizeof(T) == 4 ? 3ll : 2ll) * cu_count() && gemm_choice() != 1;
}

template <typename T, int T32, bool SPLIT, typename Epi>
csat_status launch_gemm_deep(const GemmArgs& g, long long n_cover, int batch, const Epi& epi, hipStream_t st) {
    constexpr int BT = 32 * T32;
    const dim3 grid((unsigned)((g.M + BT - 1) / BT), (unsigned)((n_cover + BT - 1) / BT), (unsigned)batch);
    tl_forms[CSAT_FORM_SMALL_TILES] |= T32 | (SPLIT ? 4 : 0);
    hipLaunchKernelGGL((gemm_nt_deep_kernel<T, T32, SPLIT, Epi>), grid, dim3(64 * kDeepWaves), 0, st, g, epi);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

template <typename T, typename Epi>
csat_status gemm(const GemmArgs& g, long long n_cover, int batch, const Epi& epi, hipStream_t st) {
    if constexpr (sizeof(T) == 2) {
        const long long Kp = round_up(g.K, 64);
        if (use_big_gemm<T>(g, n_cover)) {
            GemmArgs gb = g;
            gb.K = (int)Kp;
            return launch_gemm_big<Epi>(gb, n_cover, batch, epi, st);
        }
    }
    if constexpr (!has_rows_epilogue<Epi>::value) {
        if (few_tiles<T>(g, n_cover, batch)) {
            if (sizeof(T) == 2 && (g.M + 31ll) / 32 * ((n_cover + 31) / 32) * batch > 2 * cu_count()) return launch_gemm_deep<T, 2, false, Epi>(g, n_cover, batch, epi, st);
            return launch_gemm_deep<T, 1, false, Epi>(g, n_cover, batch, epi, st);
        }
    }
    if (n_cover <= 64) return launch_gemm<T, 128, 64, 2, 2, Epi>(g, n_cover, batch, epi, st);
    return launch_gemm<T, 128, 128, 2, 2, Epi>(g, n_cover, batch, epi, st);
}

// The ISTA decoder's products and its synthesis: in float, on the bf16 matrix cores (csat_gemm_f32.h).  The measurement,
// the output product, the unrolled decoder's layers and matching pursuit's correlations stay on the float MFMA: no
// case spends its time on the first two, and what the last two amplify (a layer's S is not a contraction; a pick is a
// comparison) would move their outputs further than two correct float implementations are allowed to differ.  Narrow
// products over a contraction of one step stay there too: the split's start costs more than it saves (one iteration of
// 256 to 20 000 rows, n = 40 or 64, m = 8 or 32: 23 to 26.5 us against 25 to 28; n = 200 33 to 46 against 32 to 39).
// (Of few tiles too: what the split leaves out is largest beside a sum of one product, and that is what a sparse row's
// synthesis over at most 32 columns is.)
template <typename T, typename Epi>
csat_status decoder_gemm(const GemmArgs& g, long long n_cover, int batch, const Epi& epi, hipStream_t st) {
    if constexpr (sizeof(T) == 4) {
        if (gemm_choice() != 1 && (g.K > 32 || n_cover > 128)) {
            if constexpr (!has_rows_epilogue<Epi>::value) {
                if (few_tiles<T>(g, n_cover, batch)) return launch_gemm_deep<T, 1, true, Epi>(g, n_cover, batch, epi, st);
            }
            return launch_gemm_f32<Epi>(g, n_cover, batch, epi, st);
        }
    }
    return gemm<T>(g, n_cover, batch, epi, st);
}

template <typename TI, typename TO>
csat_status pack_rows(const TI* src, long long lds_, TO* dst, long long ldd, long long rows, int cols, hipStream_t st) {
    const int vec = lds_ % 4 == 0 && ldd % 4 == 0 && reinterpret_cast<uintptr_t>(src) % (4 * sizeof(TI)) == 0 &&
                    reinterpret_cast<uintptr_t>(dst) % (4 * sizeof(TO)) == 0;
    int lshift = 0;      // lanes per row: four columns each, at most a wavefront
    while (lshift < 6 && (4ll << lshift) < ldd) ++lshift;
    hipLaunchKernelGGL((pack_rows_kernel<TI, TO>), dim3((unsigned)(((rows << lshift) + 255) / 256), (unsigned)((ldd + kPackCols - 1) / kPackCols)), dim3(256), 0, st,
                       src, lds_, dst, ldd, rows, cols, vec, lshift);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

template <typename T>
csat_status transpose_pack(const T* src, T* dst, long long ldd, int batch, int R, int Cc, hipStream_t st, const T* src2 = nullptr) {
    const int one = batch;      // batches of src; as many of src2 behind them
    if (src2) batch *= 2;
    dim3 grid((unsigned)((ldd + 31) / 32), (unsigned)((Cc + 31) / 32), (unsigned)batch);
    hipLaunchKernelGGL((transpose_pack_kernel<T>), grid, dim3(32, 8), 0, st, src, src2, one, (long long)R * Cc, dst, ldd,
                       (long long)Cc * ldd, R, Cc);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

csat_status fill_zero(void* p, size_t bytes, hipStream_t st) {   // bytes multiple of 4
    long long words = (long long)(bytes / 4);
    if (words == 0) return CSAT_OK;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, (uint32_t*)p, words);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

// ---------------------------------------------------------------------------------------
// Stage drivers on prepared operands (typed by the element type T).
// ---------------------------------------------------------------------------------------

// Operand copies of Phi: row-major padded (measurement GEMM; generic decoder's residual GEMM),
// transposed (generic decoder's update GEMM) or MFMA fragments (fused decoder).
template <typename T>
csat_status prepare_phi(const csat_dims& d, const Workspace& w, const T* Phi, bool for_measure, int decoder_iters,
                        hipStream_t st) {
    const bool for_decoder = decoder_iters > 0 && !decoder_is_resident_f32(d, w, decoder_iters);
    Timed tm(w, CSAT_K_LAYOUT, st);
    const bool generic = for_decoder && !w.fused;
    if (for_measure || generic) CSAT_TRY((pack_rows<T, T>(Phi, d.n, (T*)w.PhiP, w.ldn, d.m, d.n, st)));
    if (generic) CSAT_TRY(transpose_pack<T>(Phi, (T*)w.PhiT, w.ldm, 1, d.m, d.n, st));
    if constexpr (sizeof(T) == 2) {
        if (for_decoder && w.fused) {
            const int nct2 = (w.nct + 1) / 2 * 2;
            long long total = (long long)nct2 * ista_fused_set_frags(w.MT) * 64;
            hipLaunchKernelGGL(pack_phi_fragments_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                               (const bf16_t*)Phi, d.m, d.n, w.MT, nct2, w.PhiPack);
            HIP_TRY(hipGetLastError());
        }
    }
    return CSAT_OK;
}

// Whether the measurement runs as the one kernel that reads K and V as they are (csat_measure.h): bf16, d of
// one or two 64-wide tiles, one matrix for both products.
template <typename T>
bool measure_is_direct(const csat_dims& d, bool separate) {
    return sizeof(T) == 2 && !separate && (d.d == 64 || d.d == 128) && (*tl_opt)[CSAT_OPT_MEASURE] != 1;
}
// The synthesis straight from V as the caller holds it ([n, d] per head): the measurement kernel with the head's rows
// of the bf16 iterate as its row operand (csat_measure.h), no transposed copy of V.  bf16 with d = 64 or 128.
template <typename T>
bool synthesis_is_direct(const csat_dims& d) {
    return sizeof(T) == 2 && (d.d == 64 || d.d == 128) && (*tl_opt)[CSAT_OPT_SYNTHESIS] != 2;
}
// ... and whether it reads Phi as the caller holds it (rows 16-byte aligned), so that no operand copy is needed
// (phi_is_operand: the caller's Phi has the layout of that copy; float only, bf16's rows are padded to 64)
template <typename T>
bool phi_is_operand(const csat_dims& d, const void* Phi) { return sizeof(T) == 4 && d.n % 8 == 0 && aligned16(Phi); }
template <typename T>
bool measure_reads_raw_phi(const csat_dims& d, bool separate) { return measure_is_direct<T>(d, separate) && d.n % 8 == 0; }

// Kc = Phi_K K, Vc = Phi V (+ transposed copy of Vc when VcT != nullptr).  vt_ready: the caller needs no transposed
// copy of V in w.VT afterwards (the one-kernel path then makes none).  w.PhiP holds Phi (= Phi_V) on
// entry and on return; a separate key matrix PhiK (raw, caller layout) borrows it for the K product.
// *kc_packed (optional) reports whether K~'s (hi | lo) fragments for the one-kernel attention were written too.
// v_packed (optional): the caller will run the one-kernel attention with its own output product; *v_packed then
// reports that the VcT buffer holds V~ as that product's fragments instead of the transpose.
template <typename T>
csat_status run_measure(const csat_dims& d, const Workspace& w, const T* K, const T* V, T* Kc, T* Vc, T* VcT,
                        bool vt_ready, bool split_k, hipStream_t st, const T* PhiK = nullptr,
                        const T* PhiV = nullptr, bool want_v = true, bool* kc_packed = nullptr,
                        bool* v_packed = nullptr) {
    const bool separate = PhiK && PhiK != PhiV;
    const int BH = d.B * d.H;
    if (kc_packed) *kc_packed = false;
    if (v_packed) *v_packed = false;
    if constexpr (sizeof(T) == 2) {
        // one matrix for both products and d of one or two 64-wide tiles: both products in one launch, straight
        // from K and V as they are, with every copy of K~ and V~ the next stage reads (csat_measure.h)
        if (measure_is_direct<T>(d, separate)) {
            if (!vt_ready) {
                Timed tm(w, CSAT_K_LAYOUT, st);
                CSAT_TRY(transpose_pack<T>(V, (T*)w.VT, w.ldn, BH, d.n, d.d, st));
            }
            Timed tm(w, CSAT_K_MEASURE, st);
            MeasureDirectArgs a{};
            // Phi as the caller holds it where its rows are 16-byte aligned, else the zero-padded operand copy
            const bool raw = PhiV && measure_reads_raw_phi<T>(d, separate);
            a.Phi = raw ? (const bf16_t*)PhiV : (const bf16_t*)w.PhiP;
            a.ldp = raw ? d.n : w.ldn;
            a.ncols = raw ? d.n : (int)w.ldn;
            a.K = (const bf16_t*)K; a.V = (const bf16_t*)V; a.strideX = (long long)d.n * d.d;
            a.m = d.m; a.n = d.n; a.MT = w.MT;
            a.Kc = (bf16_t*)Kc;
            a.KcHL = split_k ? w.KcHL : nullptr;
            a.KcPack = split_k && kc_packed ? w.KcPack : nullptr;
            a.Vc = want_v ? (bf16_t*)Vc : nullptr;
            const bool frags = v_packed && VcT && want_v && (*tl_opt)[CSAT_OPT_MEASURE] != 2;
            a.VcT = frags ? nullptr : (bf16_t*)VcT; a.ldm = w.ldm;
            a.VPack = frags ? (uint4*)VcT : nullptr;        // (MT * 32 <= ldm: the fragments fit the transpose's buffer)
            if (frags) *v_packed = true;
            a.heads = BH;
            a.blocks_per_head = want_v ? (w.MT + 1) / 2 : (w.MT + 3) / 4;
            const dim3 grid((unsigned)(8 * ((BH + 7) / 8) * a.blocks_per_head));
            // 64 rows of K and V per step; two steps in flight, four for long contractions (measured on the five
            // workloads: 26 us either way at n = 1600, 221 against 247 us at n = 4096, 238 against 285 at n = 16384)
#define MD(DT, KS, PD, KG)                                                                                            \
    do {                                                                                                              \
        if (want_v) hipLaunchKernelGGL((measure_direct_kernel<DT, KS, PD, true, KG>), grid, dim3(256 * KG), 0, st, a);  \
        else hipLaunchKernelGGL((measure_direct_kernel<DT, KS, PD, false, KG>), grid, dim3(256 * KG), 0, st, a);        \
    } while (0)
            const bool deep = d.n >= 4096;
            // No more workgroups than CUs: two groups of wavefronts split the contraction (csat_measure.h).  They walk n in
            // rounds of 512 rows (d = 64) or 256 (d = 128), one group in rounds of 128, or 256 from n = 4096 on, so a
            // round that is mostly empty can cost more than they save: d = 64, 48 heads, m = 256: n = 512 8.0 us with one
            // group and 8.5 with two, 700 12.3 and 13.9, 1024 12.1 and 11.5, 1600 17.1 and 17.6, 2048 20.0 and 17.6, 8192 61.8 and
            // 51.3; d = 128, 12 heads, m = 256: n = 512 12.2 and 10.5, 1600 29.3 and 22.6.  With more heads than half the CUs
            // memory is the bound (d = 64, 256 heads, m = 64: n = 700 13.4 and 16.7, 4096 42.4 and 44.6).
            const bool rounds_full = d.d == 128 ? d.n >= 512 : d.n >= 2048 || (d.n >= 1024 && (d.n - 1) % 512 >= 384);
            const bool two = (long long)BH * a.blocks_per_head <= cu_count() && 2 * BH <= cu_count() && rounds_full;
            if (d.d == 64) { if (two) MD(2, 64, 4, 2); else if (deep) MD(2, 64, 4, 1); else MD(2, 64, 2, 1); }
            else { if (two) MD(4, 32, 4, 2); else if (deep) MD(4, 64, 4, 1); else MD(4, 64, 2, 1); }
#undef MD
            HIP_TRY(hipGetLastError());
            if (kc_packed) *kc_packed = a.KcPack != nullptr;
            return CSAT_OK;
        }
    }
    // Both products in one launch (and both transposes) where they share the matrix and the copies are adjacent: small
    // problems are bound by launches of a few workgroups (256 x 256, m = 64 in float: a launch of each kind less, 18 us).
    const bool pair_t = !separate && want_v && 2ll * BH <= 65535 && w.VT == w.KT + (size_t)BH * d.d * w.ldn * sizeof(T);
    // The products of 128-wide tiles run three workgroups per CU, so what one launch saves or costs is in how full the last
    // round is (cost of a round of one, two and three per CU: 1.6 : 2.2 : 3, from float, d = 128, n = 1024): 48 heads, m = 1024 (384
    // workgroups each) 231 us against 304 with two launches, 128 heads, m = 392 (512 each) 392 against 356, 256 heads (1024) n = 512
    // 382 against 412.  64-wide tiles (d <= 64): one launch is never slower.
    auto rounds = [](long long tiles) {
        const long long cus = cu_count(), rest = tiles % (3 * cus);
        return tiles / (3 * cus) * 30 + (rest == 0 ? 0 : rest <= cus ? 16 : rest <= 2 * cus ? 22 : 30);
    };
    const long long tiles = (long long)BH * ((d.m + 127) / 128) * ((d.d + 127) / 128);
    const bool pair = pair_t && (d.d <= 64 || rounds(2 * tiles) <= 2 * rounds(tiles));
    // Phi as the caller holds it where that is the operand layout already
    const void* A = PhiV && !separate && phi_is_operand<T>(d, PhiV) ? (const void*)PhiV : w.PhiP;
    {
        Timed tm(w, CSAT_K_LAYOUT, st);
        CSAT_TRY(transpose_pack<T>(K, (T*)w.KT, w.ldn, BH, d.n, d.d, st, pair_t ? V : nullptr));
        // (vt_ready says what the caller needs afterwards; the V product below reads the transposed copy either way)
        if (!pair_t && (!vt_ready || want_v)) CSAT_TRY(transpose_pack<T>(V, (T*)w.VT, w.ldn, BH, d.n, d.d, st));
        if (VcT && w.ldm > d.m) CSAT_TRY(fill_zero(VcT, (size_t)BH * d.d * w.ldm * sizeof(T), st));
    }
    if (separate) {
        Timed tl(w, CSAT_K_LAYOUT, st);
        CSAT_TRY((pack_rows<T, T>(PhiK, d.n, (T*)w.PhiP, w.ldn, d.m, d.n, st)));
    }
    Timed tm(w, CSAT_K_MEASURE, st);
    GemmArgs g{A, w.ldn, 0, w.KT, w.ldn, (long long)d.d * w.ldn, d.m, d.d, d.n, 0};
    const EpiStore<T> ev{Vc, d.d, (long long)d.m * d.d, VcT, w.ldm, (long long)d.d * w.ldm, 1.f, d.m, d.d};
    if (pair) {
        if constexpr (sizeof(T) == 2) {
            if (split_k)
                return gemm<T>(g, d.d, 2 * BH, EpiPair<EpiMeasureSplit, EpiStore<T>>{{(bf16_t*)Kc, w.KcHL, d.m, d.d}, ev, BH}, st);
        }
        return gemm<T>(g, d.d, 2 * BH, EpiPair<EpiStore<T>, EpiStore<T>>{{Kc, d.d, (long long)d.m * d.d, nullptr, 0, 0, 1.f, d.m, d.d}, ev, BH}, st);
    }
    if constexpr (sizeof(T) == 2) {
        if (split_k) {
            EpiMeasureSplit ek{(bf16_t*)Kc, w.KcHL, d.m, d.d};
            CSAT_TRY((gemm<T>(g, d.d, BH, ek, st)));
        }
    }
    if (sizeof(T) != 2 || !split_k) {
        EpiStore<T> ek{Kc, d.d, (long long)d.m * d.d, nullptr, 0, 0, 1.f, d.m, d.d};
        CSAT_TRY((gemm<T>(g, d.d, BH, ek, st)));
    }
    if (separate) CSAT_TRY((pack_rows<T, T>(PhiV, d.n, (T*)w.PhiP, w.ldn, d.m, d.n, st)));
    if (!want_v) return CSAT_OK;      // (V~ only feeds the compressed output Z: a forward without Z does not need it)
    g.Bt = w.VT;
    CSAT_TRY((gemm<T>(g, d.d, BH, ev, st)));
    return CSAT_OK;
}

// Whether the one-kernel attention keeps all of a head's K~ fragments (ns per tile of m, mt tiles) in LDS and all
// score tiles of a row block in registers: one sweep over m instead of two.
bool attention_single_sweep(int mt, int ns) {
    return mt <= 16 && (size_t)attention_mtp(mt, true) * ns * 1024 <= (size_t)kAttnMaxLdsBytes;
}

// ... and whether V~'s fragments for the kernel's own output product (bf16, d = 64 or 128, K~ as the (hi | lo)
// pair) fit into LDS next to K~'s
bool attention_packed_v_fits(int mt, int d) {
    const int ns = 2 * (d / 16);
    return attention_single_sweep(mt, ns) && (size_t)attention_mtp(mt, true) * (ns + d / 16) * 1024 <= (size_t)kAttnLdsBytes;
}

// Compressed attention in one kernel (csat_attention.h; d <= 128) behind a small kernel that packs K~ as
// MFMA fragments.  Ksrc: K~ rows [BH][m][kparts * d] (the plain matrix, or the bf16 (hi | lo) pair).
// A may be null when only Z is wanted.
template <typename T>
csat_status launch_attention_fused(const csat_dims& d, const Workspace& w, const T* Q, const T* Ksrc, int kparts,
                                   const T* VcT, float* A, long long ldA, T* P, T* Z, T* ZT, hipStream_t st,
                                   bool kc_packed = false, bool v_packed = false, bool a_tiled = false) {
    constexpr int GK = sizeof(T) == 2 ? 16 : 8;          // contraction depth of one fragment
    const int BH = d.B * d.H;
    AttentionArgs a{};
    a.ng = (d.d + GK - 1) / GK;
    a.ns = kparts * a.ng;
    a.Q = Q; a.strideQ = (long long)d.n_q * d.d;
    a.Kf = w.KcPack;
    // (fragments of V~ only come from the one-kernel measurement: bf16, d = 64 or 128; ZT is not produced from them)
    a.VcT = v_packed ? nullptr : VcT; a.ldv = w.ldm; a.strideV = (long long)d.d * w.ldm;
    a.Vf = v_packed ? (const uint4*)VcT : nullptr;
    a.A = A; a.ldA = ldA; a.a_tiled = a_tiled ? 1 : 0;
    a.P = P; a.ldP = w.ldm;
    a.Z = Z;
    a.ZT = ZT; a.ldT = sizeof(T) == 2 ? 2 * w.ldn : w.ldn; a.strideT = (long long)d.d * a.ldT;
    a.n_q = d.n_q; a.m = d.m; a.d = d.d;
    a.scale_log2e = 1.4426950408889634f / sqrtf((float)d.d);
    a.tiles_per_head = (d.n_q + 31) / 32;
    const int mt = w.MT;
    const bool single = attention_single_sweep(mt, a.ns);
    // Rounds of one row tile per wavefront: with all of K~ in LDS a workgroup amortises its staging over several
    // rounds; take the count that needs the fewest passes of the grid over the chip (ties: fewer rounds).
    int nw = attention_waves(attention_mtp(mt, single), v_packed ? 2 : 0);
    // Fewer wavefronts per workgroup, down to two, while there is no more than a workgroup per CU: eight row tiles of one head are
    // otherwise one CU's work.  Stage call with A~ and Z, eight, four, two, one wavefronts, us: float, 1 x 256 rows, m = 64 30.4, 22.9,
    // 20.8, 20.4; 16 x 300, m = 128, d = 32 38.6, 28.0, 25.1, 23.7; 12 x 1600, m = 392 (four at most) -, 75.6, 95.7, 119; 192 x 120,
    // m = 73 43.1, 41.7, 51.8, 43.3; bf16, 10 x 333, m = 197, d = 80 54.0, 43.9, 39.3, 38.9; 4 x 300, m = 1024 135, 84.8, 70.9, 68.0;
    // 64 x 500, m = 100 32.9, 29.1, 33.2, 45.8; 128 x 300, m = 128 37.3, 40.7, 39.7, 47.9.
    while (nw > 2 && (long long)BH * ((a.tiles_per_head + nw / 2 - 1) / (nw / 2)) <= cu_count()) nw /= 2;
    a.waves = nw;
    tl_forms[CSAT_FORM_ATTENTION_WAVES] = nw;
    a.rounds = 1;
    if (single) {
        const int cus = cu_count();
        long long best = -1;
        for (int r = 1; r <= 8; ++r) {
            const long long wgs = (long long)BH * ((a.tiles_per_head + nw * r - 1) / (nw * r));
            const long long cost = (wgs + cus - 1) / cus * (4 * r + 1);      // + 1: the staging, about a quarter of a round
            if (best < 0 || cost < best) { best = cost; a.rounds = r; }
        }
    }
    a.wg_per_head = (a.tiles_per_head + nw * a.rounds - 1) / (nw * a.rounds);
    // LDS for all the tiles the kernel instance holds (slots of tiles beyond m are zeroed, not skipped)
    const int mtp = attention_mtp(mt, single);
    size_t lds_bytes = (size_t)mtp * a.ns * 1024;
    a.v_lds = -1;
    if (a.Vf) {      // V~'s fragments next to K~'s (single sweep; the caller made sure the CU's LDS holds both)
        const size_t vbytes = (size_t)mtp * (d.d / 16) * 1024;
        if (!single || lds_bytes + vbytes > (size_t)kAttnLdsBytes) return CSAT_ERR_SHAPE;
        a.v_lds = mtp * a.ns;
        lds_bytes += vbytes;
    }
    if (!kc_packed) {
        Timed tm(w, CSAT_K_SCORES, st);
        const long long total = (long long)BH * mt * a.ns * 64;
        hipLaunchKernelGGL((pack_kc_fragments_kernel<T>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, Ksrc,
                           (long long)kparts * d.d, d.m, d.d, kparts, mt, a.ng, w.KcPack, total);
        HIP_TRY(hipGetLastError());
    }
    const unsigned grid = (unsigned)(BH * a.wg_per_head);
    const bool want_z = Z || ZT;
    Timed tm(w, CSAT_K_SOFTMAX, st);
    if (sizeof(T) == 2) {
        // (those kernels store whole tiles only)
        if (want_z && a.Vf && ((A && (ldA % 4 != 0 || ldA < 32 * mt)) || (P && w.ldm < 32 * mt))) return CSAT_ERR_SHAPE;
        if (want_z && a.Vf) HIP_TRY(d.d == 64 ? attention_fused_launch_bf16_z2(mt, single, a, grid, lds_bytes, st)
                                              : attention_fused_launch_bf16_z3(mt, single, a, grid, lds_bytes, st));
        else HIP_TRY(want_z ? attention_fused_launch_bf16_z1(mt, single, a, grid, lds_bytes, st)
                            : attention_fused_launch_bf16_z0(mt, single, a, grid, lds_bytes, st));
    }
    else HIP_TRY(want_z ? attention_fused_launch_f32_z1(mt, single, a, grid, lds_bytes, st)
                        : attention_fused_launch_f32_z0(mt, single, a, grid, lds_bytes, st));
    return CSAT_OK;
}

// Whether the compressed attention runs as the one kernel: d <= 128 unless overridden; a head with fewer than 8 row
// tiles and more than 32 KB of K~ fragments cannot amortise keeping K~ in LDS (cross-attention with a short query
// side: 85 us against 44 us measured at 77 queries, m = 512) and takes the three kernels.
template <typename T>
bool attention_is_fused(const csat_dims& d, const Workspace& w, bool split_k) {
    const int attn_opt = (*tl_opt)[CSAT_OPT_ATTENTION];
    const int frag_depth = sizeof(T) == 2 ? 16 : 8;
    const bool short_side = (d.n_q + 31) / 32 < 8 &&
                            (long long)w.MT * (sizeof(T) == 2 && split_k ? 2 : 1) * ((d.d + frag_depth - 1) / frag_depth) > 32;
    return d.d <= 128 && attn_opt != 1 && (attn_opt == 2 || !short_side);
}

// Whether a call that wants Z but not A~ takes the kernel that never stores A~ (csat_attention_z.h): bf16, d a multiple
// of 32 up to 128.  parts: 2 where K~ comes as its (hi | lo) pair.  A short query side is one workgroup per head that walks
// all of m, where the three kernels spread m over workgroups; that shows at d = 128, whose workgroups have a CU each
// (kAttnZChain fragments per tile of m and more), with few heads.  Stage call, d = 128, m = 1024, one query: 4 heads 30 us
// against 35 without A~, 48 heads 39 against 42, 192 heads 99 against 98; 33 queries 33 and 35, 65 queries 36 and 36, 300 queries
// 69 and 37; m = 512, one query: 24 and 23.  As a pair, m = 1024, 4 heads: one query 53 and 58, 200 queries 61 and 65, 300
// queries 101 and 67.  At d = 32 to 96 nothing like it (one query, m = 1024: d = 64 26 and 24, d = 96 30 and 31).
constexpr long long kAttnZChain = 384;
template <typename T>
bool attention_z_applies(const csat_dims& d, int parts) {
    if (sizeof(T) != 2 || d.d % 32 != 0 || d.d > 128 || (*tl_opt)[CSAT_OPT_ATTENTION] != 0) return false;
    const long long chain = (d.m + 31) / 32 * (long long)(parts + 1) * (d.d / 16);
    return !(d.d == 128 && chain >= kAttnZChain && (long long)d.B * d.H <= 48 && d.n_q <= (parts == 2 ? 255 : 64));
}
// Z and / or ZT (see run_attention) without A~.  Ksrc: K~ rows [BH][m][kparts * d]; Vc: V~ rows.  kc_packed / v_packed: their
// fragments are in w.KcPack / w.VcT already.
template <typename T>
csat_status run_attention_z(const csat_dims& d, const Workspace& w, const T* Q, const T* Ksrc, int kparts, bool kc_packed,
                            const T* Vc, bool v_packed, T* Z, T* ZT, hipStream_t st) {
    const int BH = d.B * d.H;
    AttentionZArgs a{};
    a.Q = (const bf16_t*)Q;
    a.Kf = w.KcPack;
    a.Vf = (const uint4*)w.VcT;
    a.Z = (bf16_t*)Z; a.ZT = (bf16_t*)ZT;
    a.ldT = 2 * w.ldn; a.strideT = (long long)d.d * a.ldT;
    a.n_q = d.n_q; a.m = d.m; a.MT = w.MT;
    a.scale_log2e = 1.4426950408889634f / sqrtf((float)d.d);
    a.shift = 8.f;
    for (long long v = 1; v < d.m; v *= 2) a.shift += 1.f;
    a.tiles_per_head = (d.n_q + 31) / 32;
    if (!kc_packed || !v_packed) {
        Timed tm(w, CSAT_K_LAYOUT, st);
        const long long nk = kc_packed ? 0 : (long long)BH * w.MT * kparts * (d.d / 16) * 64;
        const long long nv = v_packed ? 0 : (long long)BH * w.MT * (d.d / 16) * 64;
        hipLaunchKernelGGL(pack_kv_fragments_kernel, dim3((unsigned)((nk + nv + 255) / 256)), dim3(256), 0, st, (const bf16_t*)Ksrc,
                           (const bf16_t*)Vc, d.m, d.d, kparts, w.MT, w.KcPack, (uint4*)w.VcT, nk, nv);
        HIP_TRY(hipGetLastError());
    }
    // All of a head's fragments in LDS where they fit; a workgroup then works through several rounds of one row tile
    // per wavefront, as many as need the fewest passes of the grid over the chip (a round's time per tile of m: a
    // quarter of the staging's; ties: fewer rounds).  Else two tiles of m at a time, one round.
    const int slot = attention_z_slot_bytes(d.d, kparts), slots = (w.MT + kAttnZTiles - 1) / kAttnZTiles;
    const bool resident = (long long)slot * slots <= (long long)kLdsPerWorkgroup;
    const size_t lds_bytes = (size_t)slot * (resident ? slots : 2);
    const int per_cu = d.d <= 64 && 2 * lds_bytes <= kLdsPerWorkgroup ? 2 : 1;
    a.rounds = 1;
    if (resident) {
        const long long slots_on_chip = (long long)cu_count() * per_cu;
        long long best = -1;
        for (int r = 1; r <= 8; ++r) {
            const long long wgs = (long long)BH * ((a.tiles_per_head + kAttnZWaves * r - 1) / (kAttnZWaves * r));
            const long long cost = (wgs + slots_on_chip - 1) / slots_on_chip * (4 * r + 1);
            if (best < 0 || cost < best) { best = cost; a.rounds = r; }
        }
    }
    a.wg_per_head = (a.tiles_per_head + kAttnZWaves * a.rounds - 1) / (kAttnZWaves * a.rounds);
    Timed tm(w, CSAT_K_SOFTMAX, st);
    HIP_TRY(attention_z_launch(d.d, kparts, resident, a, (unsigned)(BH * a.wg_per_head), lds_bytes, st));
    return CSAT_OK;
}

// A = softmax(Q Kc^T / sqrt(d)) (float, [rows, m]); P = operand copy [rows, ldm];
// Z = A Vc when Z != nullptr (needs VcT)
// ZT != nullptr (with Z possibly null): also the transposed output per head, [BH, d, ldn] in fp32 mode,
// [BH, d, 2*ldn] as a bf16 (hi | lo) pair in bf16 mode; ZT must be zeroed beforehand.
template <typename T>
csat_status run_attention(const csat_dims& d, const Workspace& w, const T* Q, const T* Kc, const T* VcT,
                          float* A, long long ldA, T* P, T* Z, bool split_k, hipStream_t st, T* ZT = nullptr,
                          bool kc_packed = false, bool v_packed = false, bool a_tiled = false) {
    const int BH = d.B * d.H;
    const long long rows = (long long)BH * d.n_q;
    const int attn_opt = (*tl_opt)[CSAT_OPT_ATTENTION];
    // With Z requested (the stage call, the column-wise reading, a caller that wants Z) and more than four tiles of m,
    // the one kernel's own output product, which reads V~ per wavefront, measured slower than a product kernel behind it
    // (short_video, stage call: 158 us in one kernel, 115 us as three kernels; image_text, three tiles: 33 against 39):
    // there the one kernel writes A~ and its operand copy, and Z comes from the product kernel below.  A~ is the same
    // whether Z is requested or not.
    // (With V~ as the product's fragments, written by the one-kernel measurement, the one kernel's own product reads
    // them with one coalesced load per MFMA and is the faster again.)
    const bool wide_z = (Z || ZT) && w.MT > 4 && attn_opt != 2 && P != nullptr && !v_packed;
    bool have_a = false;
    if (attention_is_fused<T>(d, w, split_k)) {
        const bool hl = sizeof(T) == 2 && split_k;                 // contract against the (hi | lo) pair of K~
        const T* Ksrc = hl ? (const T*)w.KcHL : Kc;
        const bool packed = kc_packed && hl;
        if (!wide_z) return launch_attention_fused<T>(d, w, Q, Ksrc, hl ? 2 : 1, VcT, A, ldA, P, Z, ZT, st, packed, v_packed, a_tiled);
        if (a_tiled) return CSAT_ERR_SHAPE;      // (the caller asks for tiles only where the one launch does everything)
        CSAT_TRY(launch_attention_fused<T>(d, w, Q, Ksrc, hl ? 2 : 1, VcT, A, ldA, P, (T*)nullptr, (T*)nullptr, st, packed));
        have_a = true;
    }
    if (!have_a) {      // scores with the scale fused, then the row softmax
        GemmArgs g{Q, d.d, (long long)d.n_q * d.d, Kc, d.d, (long long)d.m * d.d, d.n_q, d.m, d.d, 0};
        if (sizeof(T) == 2 && split_k) {   // [Q | Q] against [K~hi | K~lo]
            g.Bt = w.KcHL; g.ldb = 2 * d.d; g.strideB = (long long)d.m * 2 * d.d; g.K = 2 * d.d;
            g.a_kwrap = d.d / 8;
        }
        EpiStore<float> es{A, ldA, (long long)d.n_q * ldA, nullptr, 0, 0, 1.f / sqrtf((float)d.d), d.n_q, d.m};
        {
            Timed tm(w, CSAT_K_SCORES, st);
            CSAT_TRY((gemm<T>(g, d.m, BH, es, st)));
        }
        {
            Timed tm(w, CSAT_K_SOFTMAX, st);
            if (d.m <= 512)
                hipLaunchKernelGGL((softmax_rows_kernel<T, 8>), dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, A, ldA, rows,
                                   d.m, P, w.ldm);
            else
                hipLaunchKernelGGL((softmax_rows_kernel<T, 16>), dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, A, ldA, rows,
                                   d.m, P, w.ldm);
            HIP_TRY(hipGetLastError());
        }
    }
    if (Z || ZT) {
        Timed tm(w, CSAT_K_OUTPUT, st);
        GemmArgs gz{P, w.ldm, (long long)d.n_q * w.ldm, VcT, w.ldm, (long long)d.d * w.ldm, d.n_q, d.d, d.m, 0};
        if constexpr (sizeof(T) == 2) {
            if (ZT) {
                EpiStoreSplitT ez{(bf16_t*)Z, d.d, (long long)d.n_q * d.d, (bf16_t*)ZT, 2 * w.ldn, (long long)d.d * 2 * w.ldn,
                                  d.n_q, d.d};
                return gemm<T>(gz, d.d, BH, ez, st);
            }
        }
        EpiStore<T> ez{Z, d.d, (long long)d.n_q * d.d, ZT, w.ldn, (long long)d.d * w.ldn, 1.f, d.n_q, d.d};
        CSAT_TRY((gemm<T>(gz, d.d, BH, ez, st)));
    }
    return CSAT_OK;
}

// Segments per group for the fused decoder: G groups of whole length take ceil(G / P) rounds on P
// CUs, units of 1/S of the length ceil(G S / P) / S; each segment start costs a pipeline refill and
// a hand-over.  `overhead`: that cost as a share of a whole-length group.  Measured on short_video (20 iterations of
// 50 chunks, 1.5 ms per group): about 30 us per hand-over, most of it the agent-scope release fence, which writes back
// the whole L2 (the state of the 32 compute units behind it): the time of about 20 chunk steps.  (Without the fences
// - results then unreliable - five segments took 3.36 ms against 3.59; handing the state over through system-scope
// accesses instead, written through and read from memory, no fences, gave the same results bit for bit and cost as
// much in every step, waiting for the write-through stores, as it saved at the hand-overs.)
int fused_segments(long long groups, int iters, int cus, double overhead) {
    if (groups <= cus) return 1;
    int best = 1;
    double best_cost = 1e300;
    for (int s = 1; s <= 8 && s <= iters; ++s) {
        const double rounds = (double)((groups * s + cus - 1) / cus) / s;
        const double cost = rounds * (1.0 + overhead * s);
        if (cost < best_cost - 1e-12) { best_cost = cost; best = s; }
    }
    return best;
}

// Which fused decoder kernel a launch gets: 0 / 1 one chunk per step with dense / sparse state, 2 one 32-row tile per
// workgroup, 3 / 4 two chunks per step with dense / sparse state, 6 one 32-row tile shared by eight wavefronts.  iters only
// decides between 2 and 6.
int fused_variant(int MT, long long rows_pad, int nct, int iters) {
    const int cus = cu_count();
    // Few rows: eight wavefronts share a tile, one tile per CU at a time (csat_ista_coop.h).  A CU's 128-row group takes
    // about as long as two such tiles at thirteen tiles of m (0.59 against 1.08 us a chunk) and as three at three (0.24
    // against 0.7), so the line is at one tile per CU, two up to four tiles of m.  Measured, forward of 10 iterations:
    // m = 392, 300 tiles 682 against 631 us on groups; m = 192, 256 tiles 190 against 202 (with a single wavefront per
    // tile), 512 tiles 334 against 329; m = 90, 384 tiles 195 against 285, 512 tiles 234 against 312; m = 40, 304 tiles
    // 114 against 182, 608 tiles 207 against 190; m = 128, n = 1600, 512 tiles 350 against 486.  Not for two or
    // three iterations over an iterate larger than the Infinity Cache: that is bound by memory, and one wavefront per tile
    // leaves more of it to the loads (n = 16 384, 256 tiles, m = 200: two iterations 1053 us with a wavefront per tile, 1315 with
    // eight, three 1477 and 1655, ten 0.9 of the time with eight; at 256 MB, n = 8192, two 0.87).
    const bool streams = iters <= 3 && (long long)rows_pad * nct * 128 > 256ll << 20;
    if (decoder_not_asked_for() && MT <= kCoopMaxMT && rows_pad / 32 <= (MT <= 4 ? 2 : 1) * cus && !(streams && rows_pad / 32 <= cus)) return 6;
    // (one 32-row tile per workgroup; 14 tiles of m and more: only when forced)
    const bool thin = rows_pad / 32 <= cus && (*tl_opt)[CSAT_OPT_FUSED_THIN] != 1;
    int variant = thin ? 2 : (sparse_state((size_t)rows_pad * nct * 32 * 4) ? 1 : 0);
    // 128-row workgroups on rows of at least five chunks and three tiles of m: two chunks per step (the schedule
    // looks two steps ahead, and spreads each threshold over more than one group of MFMAs)
    // and works in whole pairs of chunks: an odd chunk count is padded with a zero chunk, not worth it for short rows
    // (image_text, 9 chunks: 0.207 ms against 0.190 ms on the one-chunk schedule)
    if (!thin && nct >= 5 && (nct % 2 == 0 || nct >= 21) && MT >= 3 && MT <= kFused2MaxMT && (*tl_opt)[CSAT_OPT_FUSED_SCHEDULE] != 1) variant += 3;
    return variant;
}

// The synthesis C = X V inside the two-chunk decoder's last iteration (csat_ista_fused2.h): bf16, d = 64, whole
// 32-row tiles per head, and V's fragments must fit the buffer of V^T they replace.
bool synthesis_in_decoder(const csat_dims& d, const Workspace& w) {
    if (!w.fused || decoder_is_resident(w) || d.dtype != CSAT_BF16 || d.d != 64 || d.n_q % 32 != 0 || (*tl_opt)[CSAT_OPT_SYNTHESIS] >= 1) return false;
    const int v = fused_variant(w.MT, w.rows_pad, w.nct, 0);
    if (v != 3 && v != 4) return false;
    return (long long)((w.nct + 1) / 2 * 2) * 32 <= w.ldn;
}

csat_status launch_ista_resident(const csat_dims& d, const Workspace& w, IstaResidentArgs a, hipStream_t st) {
    const long long tiles = (a.rows + 31) / 32;
    const int cus = cu_count();
    a.tiles_per_wg = tiles <= cus ? 1 : tiles <= 2ll * cus ? 2 : 4;
    const unsigned grid = (unsigned)((tiles + a.tiles_per_wg - 1) / a.tiles_per_wg);
    *tl_decoder_kernel = 5;
    switch (w.MT * 100 + ista_resident_chunks(w.MT, w.nct)) {
#define CSAT_RESIDENT_CASE(MT_, NCT_) case MT_ * 100 + NCT_: HIP_TRY(ista_resident_launch_##MT_##_##NCT_(a, grid, st)); return CSAT_OK;
        CSAT_RESIDENT_INSTANCES(CSAT_RESIDENT_CASE)
#undef CSAT_RESIDENT_CASE
    }
    return CSAT_ERR_SHAPE;
}

hipError_t launch_fused_variant(int MT, int variant, const IstaFusedArgs& a, unsigned grid, hipStream_t st) {
    switch (MT) {
#define CSAT_FUSED_CASE(N) case N: return ista_fused_launch_mt##N(variant, a, grid, st);
        CSAT_FUSED_CASE(1) CSAT_FUSED_CASE(2) CSAT_FUSED_CASE(3) CSAT_FUSED_CASE(4)
        CSAT_FUSED_CASE(5) CSAT_FUSED_CASE(6) CSAT_FUSED_CASE(7) CSAT_FUSED_CASE(8)
        CSAT_FUSED_CASE(9) CSAT_FUSED_CASE(10) CSAT_FUSED_CASE(11) CSAT_FUSED_CASE(12)
        CSAT_FUSED_CASE(13) CSAT_FUSED_CASE(14) CSAT_FUSED_CASE(15) CSAT_FUSED_CASE(16)
#undef CSAT_FUSED_CASE
    }
    return hipErrorInvalidValue;
}

csat_status launch_ista_fused(int MT, IstaFusedArgs a, long long rows_pad, hipStream_t st) {
    const int cus = cu_count();
    const int variant = fused_variant(MT, rows_pad, a.nct, a.iters);
    const bool thin = variant == 2;
    a.groups = variant == 6 ? (int)((a.rows + 31) / 32) : (int)(rows_pad / (thin ? 32 : 128));
    const int nct_real = a.nct;
    if (variant >= 3 && variant != 6) a.nct = (a.nct + 1) / 2 * 2;
    // A dense-ish iterate larger than the Infinity Cache streams through once per iteration: its accesses carry the
    // non-temporal hint on the one-chunk schedule (cross_modal: 7.97 -> 7.30 ms per launch; nothing to gain where the
    // iterate is sparse or cache-resident).  CSAT_OPT_STATE + 4 / + 8: always / never.
    {
        const int so = (*tl_opt)[CSAT_OPT_STATE];
        a.state_stream = (so & 8) ? 0 : (so & 4) ? 1 : (rows_pad * (long long)a.nct * 32 * 4 > (256ll << 20));
    }
    a.segs = fused_segments(a.groups, a.iters, cus, 20.0 / ((double)a.iters * nct_real));
    // The two-chunk kernel cuts the group-iterations of the launch into one equal share per CU instead (each group cut
    // at most once; see the kernel), unless a segment count is asked for.
    a.tape = 0;
    if (variant >= 3 && variant != 6 && a.groups > cus) a.tape = cus;
    if (a.packed) {      // (its rows, and so its groups and shares, are the device's)
        a.segs = 1;
        HIP_TRY(launch_fused_variant(MT, variant, a, (unsigned)(a.groups < cus ? a.groups : cus), st));
        return CSAT_OK;
    }
    if (const int v = (*tl_opt)[CSAT_OPT_FUSED_SEGMENTS]; v >= 1 && v <= a.iters) { a.segs = v; a.tape = 0; }
    else if (v < 0 && variant >= 3) a.tape = -v < a.groups ? -v : a.groups;       // (tests: shares on small launches)
    if ((*tl_opt)[CSAT_OPT_FUSED_SPIN_LIMIT] != 0) a.spin_limit = (*tl_opt)[CSAT_OPT_FUSED_SPIN_LIMIT] < 0 ? 0 : (*tl_opt)[CSAT_OPT_FUSED_SPIN_LIMIT];
    // (a.sync was cleared together with the status word: run_ista)
    const long long units = a.tape > 0 ? a.tape : (long long)a.groups * a.segs;
    const unsigned grid = (unsigned)(variant == 6 ? a.groups * a.tile_split : units < cus ? units : cus);
    *tl_decoder_kernel = variant;
    if (variant == 6) tl_forms[CSAT_FORM_DECODER_MEMBERS] = a.tile_split;
    HIP_TRY(launch_fused_variant(MT, variant, a, grid, st));
    return CSAT_OK;
}

// Clears the rule's words.
csat_status support_begin(const Workspace& w, hipStream_t st) {
    hipLaunchKernelGGL(set_word_kernel, dim3(1), dim3(64), 0, st, w.Status, 0, (uint32_t*)w.Status + kSupportWord, 3ll);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}
// Counts what the first threshold left (its mask bytes, whole 16-byte pieces), and looks V over (in bf16, of v_bytes) where given.
csat_status support_count(const Workspace& w, const uint8_t* mask, long long bytes, hipStream_t st, const uint32_t* screen = nullptr, float scale = 0.f, long long rows = 0,
                          const void* V = nullptr, long long v_bytes = 0) {
    const long long chunks = bytes / 16;
    // (V may be longer than the masks: 18 432 rows, n = 96, d = 96, its 3.5 MB by the masks' nine workgroups 30 us of a call of 780)
    hipLaunchKernelGGL(support_count_kernel, dim3((unsigned)std::min<long long>((std::max(chunks, v_bytes / 16) + 1023) / 1024, cu_count())), dim3(256), 0, st, (const uint4*)mask, chunks,
                       (uint32_t*)w.Status + kSupportWord, screen, scale, rows, (const uint4*)V, v_bytes / 16);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

// Whether the large-tile decoder's residual may go over the support of the iterate, which the device decides: not where the
// product over all columns takes less than about 40 us (its operations at 1.2 PFLOP/s).
// (A byte for every four rows lies in K's transposed copy, which the decoder does not read.)
bool residual_support_applies(const csat_dims& d, long long rows, int iters) {
    if (support_choice() == 1 || iters < 2 || d.m > 1024 || d.n > 65536) return false;
    if (rows / 4 >= (long long)d.B * d.H * d.d * d.n * 2 || rows / 4 * d.n >= (1ll << 32)) return false;
    return support_choice() == 2 || (double)rows * d.n * d.m > 2.4e10;
}
// ... in a launch of its own, with more wavefronts than in the product's place, where a launch that returns at once is below 1 % of an
// iteration (the product over all columns about 200 us).
bool residual_support_apart(const csat_dims& d, long long rows) { return (double)rows * d.n * d.m > 1.2e11; }
// ... and up to which density: non-zero float4 (four rows of a column) that the first iteration may leave to every four rows.  Forward over
// all columns against over the support, us.  Apart: 205 824 rows, n = 1608, m = 752, 11 iterations: 2 a quad 14 910, 9750; 18 14 990, 12 490;
// 38 976 rows, n = 9744, m = 1024, 31 iterations: 10 54 400, 29 900; 142 54 100, 38 900; 394 54 700, 50 700; 13 104 rows, n = 11 744: 100 9940,
// 7360; 368 10 100, 9850.  In the product's place: 28 544 rows, n = 1824, m = 745, 31 iterations: none 7160, 3820; 5 7170, 5960; 22 7210, 7780; 48 000
// rows: 45 12 130, 14 390; few rows, whose longest lists end the launch: 8192 rows, n = 2048, m = 600, 20 iterations: 4 1660, 1450; 10 1670,
// 1750; 4272 rows, n = 6496, 36 iterations: 24 5850, 5640; 78 5860, 6950; 3432 rows, n = 13 713, 9 iterations: 50 3890, 2590; 392 3900, 4880; 9000 rows,
// n = 5000, m = 1024, 20 iterations: 37 4960, 4710; 142 5000, 6650.  A short product leaves less to win: of its steps (columns times rounds of tiles) the masks
// and rows take about 1650 in any case, and below 1500 columns, of many rows, the density where both are as quick goes with the square of the steps (70 shapes, of which
// some turn at half or at four times that density, as their coefficients lie in few rows or in all): 12 800 rows, n = 2000, m = 1000: 2 2940, 2600; 14 2940, 3550; 15 600 rows, n = 2400,
// m = 800: 6.5 3425, 3140; 15 168 rows, n = 3008, m = 1024: 6 4290, 3880; 25 4330, 4650; 22 232 rows, n = 1582, m = 766, 16 iterations: 7 3180, 2710; 27
// 3190, 3520; 30 624 rows, n = 1425, m = 953: 3 3430, 3190; 10 3460, 3820.  Not where rows are packed: 29 112 rows, n = 1961, m = 840, 14 of them
// packed: 20 1710, 1240.
double residual_support_limit(const csat_dims& d, const Workspace& w, long long rows, bool packed) {
    if (support_choice() == 2) return 4294967295.0;
    const double quads = rows / 4.0 * d.n;
    if (residual_support_apart(d, rows)) return quads / 64;
    const double share = rows >= 12288 ? 128 : 270;
    if (packed || w.split > 1) return quads / share;
    const double steps = d.n * (double)(((rows + 255) / 256 * ((w.ldm + 255) / 256) + cu_count() - 1) / cu_count());
    const double least = d.n >= 1500 ? (double)rows * d.n * d.m / (1.75e5 * std::max(steps - 1650, 50.0)) : std::pow(50000 / steps, 2);
    return quads / std::max(share, least);
}

// ... and the float decoder's, in the product's place (rows that take a few microseconds each, however short Phi's columns are: not below m = 256, where
// the product is as quick), and up to which share of the iterate.  Forward over all columns against over the support, us: 19 200 rows,
// n = 1600, m = 392, 20 iterations: 0.023 3010, 2460; 0.025 3220, 2950; 0.029 3710, 3720; 0.036 7060, 7110; few rows, whose longest lists end the launch:
// 4000 rows, n = 3000, m = 400: 0.012 3840, 4070; 7536 rows, n = 1120, m = 300, 41 iterations: 0.0015 4510, 4340; 0.006 4510, 4730; 16 384 rows,
// n = 2048, m = 178, 29 iterations: 0.006 6050, 7460.
bool residual_support_f32_applies(const csat_dims& d, long long rows, int iters) {
    if (support_choice() == 1 || iters < 2 || d.m > 1024 || gemm_choice() == 1 || (d.m <= 32 && d.n <= 128) || d.n <= 32 || rows * d.n >= (1ll << 32)) return false;
    return support_choice() == 2 || (d.m >= 256 && (double)rows * d.n * d.m > 2e9 && (iters - 1.0) * rows * d.n * d.m > 6.5e10);      // (a millisecond of products: 20 us)
}
double residual_support_f32_limit(const csat_dims& d, long long rows) {
    if (support_choice() == 2) return 4294967295.0;
    return (double)rows * d.n * (rows >= 12288 ? 0.025 : 0.002);
}

// Rows without a coefficient left out of the decoder, the others packed (csat_screen.h).  The packed rows take half of what all rows
// have, so at most half of them may stay; their y goes into the other half of the iterate's buffer, the lists into K's transposed copy.
struct ScreenPlan {
    const uint32_t* words = nullptr;      // null: not for this call
    const int* Place = nullptr;
    const float* Y = nullptr; long long ldY = 0;
};
// The sample and the launches that return at once take 40 to 60 us: not where the decoder takes less than about 2.5 ms (its operations at
// 1 PFLOP/s, 0.12 in float).  X where the caller wants it stays with the decoder over all rows.
bool screen_applies(const csat_dims& d, const Workspace& w, const void* X, const void* V, const void* C, int iters) {
    const long long rows = (long long)d.B * d.H * d.n_q, BH = (long long)d.B * d.H;
    if (screen_choice() == 1 || X || !V || !C || iters < 2 || rows < 1024 || gemm_choice() == 1) return false;
    if (BH * d.d * w.ldn * (long long)esize(d.dtype) < 10 * rows + 16384) return false;
    if (d.dtype == CSAT_BF16) {
        if (!w.fused && (w.ldm < 128 || d.n < 128)) return false;
        if (w.fused && (decoder_is_resident(w) || !decoder_options_free() || d.n < 128)) return false;
        const int v = w.fused ? fused_variant(w.MT, w.rows_pad, w.nct, iters) : 3;
        if (v != 3 && v != 4) return false;
    } else if (decoder_is_resident_f32(d, w, iters) || (d.m <= 32 && d.n <= 128)) {
        return false;
    }
    return screen_choice() == 2 || 4.0 * iters * rows * d.n * d.m > (d.dtype == CSAT_BF16 ? 2.5e12 : 3e11);
}
csat_status screen_rows(const ScreenRowsArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(screen_rows_kernel, dim3((unsigned)std::min<long long>((a.rows + 3) / 4, 8ll * cu_count())), dim3(256), 0, st, a);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}
template <typename T>
csat_status screen(const csat_dims& d, const Workspace& w, const T* Phi, const T* V, const float* Y, long long ldY, bool y_tiled, float mu, float theta, ScreenPlan* plan, hipStream_t st) {
    constexpr bool kBf16 = sizeof(T) == 2;
    const long long rows = (long long)d.B * d.H * d.n_q, stay_bytes = round_up(rows, 16), blocks = (rows + 1023) / 1024;
    char* at = w.KT;
    uint8_t* stay = (uint8_t*)at;
    int* counts = (int*)(at += round_up(stay_bytes, 256));
    int* Place = (int*)(at += round_up(blocks * 4, 256));
    int* List = (int*)(at += round_up(rows * 4, 256));
    uint32_t *sample_words = (uint32_t*)w.Status + kScreenSampleWord, *words = (uint32_t*)w.Status + kScreenWord;
    Timed tm(w, CSAT_K_LAYOUT, st);
    hipLaunchKernelGGL(screen_begin_kernel, dim3((unsigned)std::min<long long>((stay_bytes / 4 + 255) / 256, cu_count())), dim3(256), 0, st, sample_words, (uint32_t*)stay, stay_bytes / 4);
    HIP_TRY(hipGetLastError());
    // the fused decoder has neither operand of the product; the others have the first residual
    if (w.fused) CSAT_TRY(transpose_pack<T>(Phi, (T*)w.PhiT, w.ldm, 1, d.m, d.n, st));
    // every so many rows, and no divisor of a head's: rows of one place in their heads are often alike
    long long stride = std::max<long long>(1, rows / std::max<long long>(512, rows / 64));
    while (std::gcd(stride, (long long)d.n_q) != 1) ++stride;
    const long long sample = rows / stride;
    ScreenRowsArgs ra{nullptr, nullptr, sample, (int)stride, Y, ldY, y_tiled, nullptr, 0, 0, w.R, w.ldm, kBf16, d.m};
    if (w.fused) CSAT_TRY(screen_rows(ra, st));
    auto product = [&](long long M, long long lda, const uint32_t* off) -> csat_status {
        GemmArgs g{w.R, lda, 0, w.PhiT, w.ldm, 0, (int)M, d.n, d.m, 0};
        const EpiScreen e{stay, mu, theta * kScreenMargin, M, d.n, {off}};
        if constexpr (kBf16) {
            g.K = (int)round_up(g.K, 64);
            const bool wide = wide_tiles_pay(g, d.n);
            tl_forms[CSAT_FORM_SCREEN_TILE] = wide ? 320 : 256;      // (of all rows: the sample's comes first)
            if (wide) return launch_gemm_big_shape<EpiScreen, 4, 2, 64, 5>(g, d.n, 1, e, st);
            return launch_gemm_big(g, d.n, 1, e, st);
        } else {
            return launch_gemm_f32(g, d.n, 1, e, st);
        }
    };
    CSAT_TRY(product(sample, w.fused ? w.ldm : w.ldm * stride, nullptr));
    hipLaunchKernelGGL(screen_decide_kernel, dim3(1), dim3(1024), 0, st, sample_words, (uint32_t*)stay, (int)sample, screen_choice() == 2 ? (int)sample : (int)(sample * kScreenShare));
    HIP_TRY(hipGetLastError());
    const SupportRule on{sample_words, 0};
    if (w.fused) {
        ra.words = sample_words;
        ra.rows = rows;
        ra.stride = 1;
        CSAT_TRY(screen_rows(ra, st));
    }
    CSAT_TRY(product(rows, w.ldm, sample_words));
    // whole 256 rows of packed y behind the first half of the iterate, whose rows may be shorter than y's (m close to n, in float: 8 and 32 the multiples)
    float* Yp = w.Xs + w.rows_pad / 2 * w.ldn;
    const long long most = std::min(rows / 2, w.rows_pad / 2 * w.ldn / w.ldy) - 256;
    const long long v_pieces = (long long)d.B * d.H * d.n * d.d * (long long)sizeof(T) / 16;
    hipLaunchKernelGGL((screen_count_kernel<T>), dim3((unsigned)(blocks + std::min<long long>((v_pieces + 1023) / 1024, 4ll * cu_count()))), dim3(256), 0, st, on, (const uint32_t*)stay,
                       rows, counts, (int)blocks, (const uint4*)V, v_pieces);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(screen_place_kernel, dim3((unsigned)blocks), dim3(256), 0, st, on, words, (const uint32_t*)stay, rows, counts, Place, List, (int)most);
    HIP_TRY(hipGetLastError());
    CSAT_TRY(screen_rows(ScreenRowsArgs{words, List, rows, 1, Y, ldY, y_tiled, Yp, w.ldy, y_tiled, w.fused ? nullptr : w.R, w.fused ? 0 : w.ldm, kBf16, d.m}, st));
    *plan = ScreenPlan{words, Place, Yp, w.ldy};
    return CSAT_OK;
}
// C of the packed rows, and zeros for the others (behind the synthesis over all rows, which writes C too)
template <typename T>
csat_status screen_finish(const csat_dims& d, const Workspace& w, const ScreenPlan& plan, const T* V, T* C, hipStream_t st) {
    if (!plan.words) return CSAT_OK;
    const long long rows = (long long)d.B * d.H * d.n_q;
    Timed tm(w, CSAT_K_SYNTHESIS, st);
    hipLaunchKernelGGL((screen_finish_kernel<T>), dim3((unsigned)std::min<long long>((rows + 3) / 4, 16ll * cu_count())), dim3(256), 0, st, plan.words, w.Status, plan.Place,
                       sizeof(T) == 2 ? (const T*)w.Xb : (const T*)w.Xs, w.ldn, V, C, rows, d.n_q, d.n, d.d);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

// ISTA on rows of Y (float, leading dimension ldY).  Generic decoder: w.R must already hold Y in
// operand layout (the first residual, since x^0 = 0); the final state is left in w.Xs (float mode)
// or w.Xb (bf16 mode).  Fused decoder (bf16, m <= 512): Y must be w.A-style rows with
// ldY == w.ldy and zero pads; the final iterate is left in w.Xb.
template <typename T>
csat_status run_ista(const csat_dims& d, const Workspace& w, const T* Phi, const float* Y, long long ldY, float lambda, float mu,
                     int iters, float* Xout, hipStream_t st, const T* Vsyn = nullptr, T* Csyn = nullptr, bool y_tiled = false, const ScreenPlan& plan = {}) {
    constexpr bool kBf16 = sizeof(T) == 2;
    const long long rows = (long long)d.B * d.H * d.n_q;
    const float theta = mu * lambda;
    if constexpr (kBf16) {
        if (decoder_is_resident(w)) {
            Timed tm(w, CSAT_K_UPDATE, st);
            return launch_ista_resident(d, w, IstaResidentArgs{w.PhiPack, Y, w.Xb, Xout, w.Status, rows, d.n, w.nct, (int)ldY, (int)w.ldn, iters, 1, mu, theta}, st);
        }
    }
    if constexpr (!kBf16) {
        if (decoder_is_resident_f32(d, w, iters)) {
            *tl_decoder_kernel = 5;
            Timed tm(w, CSAT_K_UPDATE, st);
            HIP_TRY(ista_resident_f32_launch(w.MT, IstaResidentF32Args{Phi, Y, ldY, w.Xs, w.ldn, Xout, w.Status, rows, d.m, d.n, w.nct, iters, mu, theta},
                                             (unsigned)((rows + 31) / 32), st));
            return CSAT_OK;
        }
    }
    // word 0 of the status block: set by the fused decoder when its bounded wait gives up
    // (and, in the same launch, the fused decoder's unit counter and progress words: 2 + one per group of 32 rows at most)
    const long long tiles = (rows + 31) / 32;
    const bool shared = w.fused && w.tile_split > 1 && iters >= kTileSplitMinIters && tiles * w.tile_split <= cu_count() &&
                        iters * (coop_iteration_us(w.MT, tiles, w.nct, 1) - coop_iteration_us(w.MT, tiles, w.nct, w.tile_split)) >= kTileSplitMinUs &&
                        fused_variant(w.MT, w.rows_pad, w.nct, iters) == 6;
    int* sync = shared ? w.TileSync : w.FusedSync;
    const long long sync_words = !w.fused ? 0 : shared ? 2 + 2 * tiles * w.tile_split : 2 + w.rows_pad / 32;
    hipLaunchKernelGGL(set_word_kernel, dim3((unsigned)(sync_words > 256 ? (sync_words + 255) / 256 : 1)), dim3(256), 0, st, w.Status,
                       (w.fused && (*tl_opt)[CSAT_OPT_INJECT_DECODER_ERROR]) ? 1 : 0, (uint32_t*)sync, sync_words);
    HIP_TRY(hipGetLastError());
    *tl_decoder_kernel = -1;
    if (w.fused) {
        IstaFusedArgs a{w.PhiPack, Y, w.Xs, w.Mask, w.Xb, Xout, rows, d.n, w.nct, (int)ldY, (int)w.ldn, iters, mu, theta,
                        0, 1, sync, w.Hand, w.Status, kFusedSpinLimit};
        a.tile_split = shared ? w.tile_split : 1;
        a.xchg = w.Xchg;
        // Vsyn (the caller checked synthesis_in_decoder): C = X V in the kernel's last iteration, from V's fragments in
        // the buffer of V^T; no bf16 copy of the iterate then
        a.y_tiled = y_tiled ? 1 : 0;
        const bool syn = Vsyn && Csyn;
        if (syn) {
            Timed tm(w, CSAT_K_LAYOUT, st);
            const int nct2 = (w.nct + 1) / 2 * 2;
            const long long total = (long long)d.B * d.H * nct2 * 256;
            hipLaunchKernelGGL(pack_v_fragments_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                               (const bf16_t*)Vsyn, d.n, nct2, total, (uint4*)w.VT);
            HIP_TRY(hipGetLastError());
            a.Xb = nullptr;
            a.Vf = (const uint4*)w.VT; a.C = (bf16_t*)Csyn; a.n_q = d.n_q;
        }
        // the kernel writes the bf16 copy in whole 32-column chunks; operand rows are padded further
        // (the GEMM reads them; the synthesis straight from V stops at column n)
        if (!syn && !synthesis_is_direct<T>(d) && w.ldn > (long long)w.nct * 32) CSAT_TRY(fill_zero(w.Xb, (size_t)rows * w.ldn * 2, st));
        {
            Timed tm(w, CSAT_K_UPDATE, st);
            a.screen = plan.words;
            if (plan.words) {      // one of the two returns at once
                IstaFusedArgs p = a;
                p.packed = 1;
                p.Y = plan.Y;
                p.Vf = nullptr; p.C = nullptr; p.Xb = w.Xb;
                CSAT_TRY(launch_ista_fused(w.MT, p, w.rows_pad, st));
            }
            CSAT_TRY(launch_ista_fused(w.MT, a, w.rows_pad, st));
        }
        // a decoder that gave up leaves part of the iterate unwritten: make that visible in the outputs
        // (NaN in X and, through the synthesis product, in C) as well as in csat_decoder_status
        hipLaunchKernelGGL(poison_on_error_kernel, dim3(256), dim3(256), 0, st, w.Status, (uint32_t*)Xout,
                           Xout ? rows * (long long)d.n : 0ll, syn ? (uint32_t*)Csyn : (uint32_t*)w.Xb,
                           syn ? rows * (long long)d.d / 2 : rows * w.ldn / 2);
        HIP_TRY(hipGetLastError());
        return CSAT_OK;
    }
    // large tiles throughout: the iterate has its masks
    const size_t support_same = plan.words ? (size_t)(round_up(rows, 256) * 9 + 8192 + rows / 128) / 256 * 256 : 0;      // (behind the lists)
    SupportRule rule;
    if constexpr (kBf16) {
        const GemmArgs gr{nullptr, w.ldn, 0, nullptr, w.ldn, 0, (int)rows, d.m, d.n, 0}, gu{nullptr, w.ldm, 0, nullptr, w.ldm, 0, (int)rows, d.n, d.m, 0};
        if (residual_support_applies(d, rows, iters) && use_big_gemm<T>(gr, w.ldm) && use_big_gemm<T>(gu, w.ldn) &&
            (w.split > 1 || (ldY % 4 == 0 && aligned16(Y)))) {
            rule.ctl = (const uint32_t*)w.Status + kSupportWord;
            rule.limit = (uint32_t)std::min(4294967295.0, residual_support_limit(d, w, rows, false));
            CSAT_TRY(support_begin(w, st));
        }
    }
    if constexpr (!kBf16) {
        if (residual_support_f32_applies(d, rows, iters) && (plan.words || support_choice() == 2)) {      // (packed rows, above all: few tiles of a long contraction)
            rule.ctl = (const uint32_t*)w.Status + kSupportWord;
            rule.limit = (uint32_t)std::min(4294967295.0, residual_support_f32_limit(d, rows));
            CSAT_TRY(support_begin(w, st));
        }
    }
    for (int t = 0; t < iters; ++t) {
        if (t > 0) {   // residual r = y - Phi x
            GemmArgs g{kBf16 ? (const void*)w.Xb : (const void*)w.Xs, w.ldn, 0, w.PhiP, w.ldn, 0, 0, d.m, d.n, 0};
            g.M = (int)rows;
            g.screen = plan.words;
            Timed tm(w, CSAT_K_RESIDUAL, st);
            auto residual_f32 = [&]() -> csat_status {
                if constexpr (!kBf16) {
                    if (t == 1) {
                        hipLaunchKernelGGL(support_count_f32_kernel, dim3((unsigned)std::min<long long>((rows + 7) / 8, cu_count())), dim3(256), 0, st, w.Xs, w.ldn, rows, d.n, 8,
                                           (uint32_t*)w.Status + kSupportWord, plan.words, (const float*)w.PhiT, d.n * w.ldm);
                        HIP_TRY(hipGetLastError());
                    }
                    const EpiResidual<float> er{Y, ldY, (float*)w.R, w.ldm, rows, d.m, plan.Y, plan.ldY};
                    const ResidualSupportF32Args sf{w.Xs, w.ldn, (const float*)w.PhiT, (int)w.ldm, Y, ldY, (float*)w.R, rows, d.n, d.m, plan.words, plan.Y, plan.ldY};
                    auto launch = [&](auto mr) {
                        constexpr int MR = decltype(mr)::value;
                        if (!plan.words) return launch_gemm_f32(g, w.ldm, 1, EpiResidualEitherF32<EpiResidual<float>, MR>{er, rule, sf}, st);
                        return launch_gemm_f32(g, w.ldm, 1, EpiResidualEitherF32<EpiScreened<EpiResidual<float>>, MR>{{er}, rule, sf}, st);
                    };
                    if (w.ldm <= 256) return launch(std::integral_constant<int, 1>{});
                    if (w.ldm <= 512) return launch(std::integral_constant<int, 2>{});
                    return launch(std::integral_constant<int, 4>{});
                }
                return CSAT_OK;
            };
            const ResidualSupportArgs sa{w.Mask, (const f32x4*)w.Xs, w.ldn / 32, (const bf16_t*)w.PhiT, (int)w.ldm, Y, ldY, (bf16_t*)w.R, (uint8_t*)w.KT + support_same, rows, d.m, t == 1, plan.words, plan.Y, plan.ldY};
            auto launch_residual = [&](const auto& epi, const GemmArgs& ga, int parts) -> csat_status {
                using Epi = std::decay_t<decltype(epi)>;
                tl_forms[CSAT_FORM_RESIDUAL] = parts + (rule.ctl && parts == 1 && residual_support_apart(d, rows) ? 16 : 0);
                if (!rule.ctl) return launch_gemm_big(ga, w.ldm, parts, epi, st);
                auto launch = [&](auto mr) -> csat_status {
                    constexpr int MR = decltype(mr)::value;
                    if (tl_forms[CSAT_FORM_RESIDUAL] < 16) return launch_gemm_big(ga, w.ldm, parts, EpiResidualEither<Epi, MR>{epi, rule, sa}, st);
                    hipLaunchKernelGGL(residual_support_kernel<MR>, dim3((unsigned)std::min<long long>((rows + 15) / 16, 4ll * cu_count())), dim3(256), 0, st, rule, sa);
                    HIP_TRY(hipGetLastError());
                    return launch_gemm_big(ga, w.ldm, parts, EpiResidualEither<Epi, 0>{epi, rule, sa}, st);
                };
                const long long regs = (w.ldm + 63) / 64;      // the instance whose 64 MR elements hold a row
                if (regs <= 8) return launch(std::integral_constant<int, 8>{});
                if (regs <= 10) return launch(std::integral_constant<int, 10>{});
                if (regs <= 12) return launch(std::integral_constant<int, 12>{});
                return launch(std::integral_constant<int, 16>{});
            };
            if (kBf16 && rule.ctl && t == 1)
                CSAT_TRY(support_count(w, w.Mask, (rows + 31) / 32 * (w.ldn / 32) * 64, st, plan.words,
                                       (float)(residual_support_limit(d, w, rows, false) / residual_support_limit(d, w, rows, true)), rows));
            if (!kBf16 && rule.ctl) {
                CSAT_TRY(residual_f32());
            } else if (w.split > 1 && use_big_gemm<T>(g, w.ldm)) {     // partial products along K, then r = y - their sum
                GemmArgs gs = g;
                gs.K = (int)(w.ldn / w.split);
                gs.strideA = gs.strideB = gs.K;
                const EpiStorePart ep{{w.SplitP, w.ldm, rows * w.ldm, nullptr, 0, 0, 1.f, (int)rows, d.m}};
                if (plan.words) CSAT_TRY(launch_residual(EpiScreened<EpiStorePart>{ep}, gs, w.split));
                else CSAT_TRY(launch_residual(ep, gs, w.split));
                const long long total = rows * w.ldm;
                hipLaunchKernelGGL(residual_reduce_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, Y, ldY,
                                   w.SplitP, w.split, rows * w.ldm, (bf16_t*)w.R, w.ldm, rows, d.m, rule, plan.words, plan.Y, plan.ldY);
                HIP_TRY(hipGetLastError());
            } else if (use_big_gemm<T>(g, w.ldm) && ldY % 4 == 0 && aligned16(Y)) {
                const EpiResidualTiled er{Y, ldY, (bf16_t*)w.R, w.ldm, rows, d.m, plan.Y, plan.ldY};
                g.K = (int)round_up(g.K, 64);
                if (plan.words) CSAT_TRY(launch_residual(EpiScreened<EpiResidualTiled>{er}, g, 1));
                else CSAT_TRY(launch_residual(er, g, 1));
            } else {
                EpiResidual<T> er{Y, ldY, (T*)w.R, w.ldm, rows, d.m, plan.Y, plan.ldY};
                if (plan.words) CSAT_TRY((decoder_gemm<T>(g, w.ldm, 1, EpiScreened<EpiResidual<T>>{er}, st)));
                else CSAT_TRY((decoder_gemm<T>(g, w.ldm, 1, er, st)));
            }
        }
        GemmArgs g{w.R, w.ldm, 0, w.PhiT, w.ldm, 0, (int)rows, d.n, d.m, 0};
        g.screen = plan.words;
        Timed tm(w, CSAT_K_UPDATE, st);
        if (use_big_gemm<T>(g, w.ldn)) {   // large-tile kernel: state in accumulator order
            EpiIstaUpdateTiled eu{(f32x4*)w.Xs, w.ldn / 32, w.Mask, w.Xb, w.ldn, (t == iters - 1) ? Xout : nullptr,
                                  mu, theta, rows, d.n, t == 0, t > 0 && t < iters - 1 ? rule : SupportRule{}};      // (the synthesis reads the last copy)
            g.K = (int)round_up(g.K, 64);
            if (plan.words) CSAT_TRY(launch_gemm_big(g, w.ldn, 1, EpiScreened<EpiIstaUpdateTiled>{eu}, st));
            else CSAT_TRY(launch_gemm_big(g, w.ldn, 1, eu, st));
            continue;
        }
        EpiIstaUpdate eu{w.Xs, kBf16 ? w.Xb : nullptr, w.ldn, (t == iters - 1) ? Xout : nullptr,
                         mu, theta, rows, d.n, t == 0};
        if (plan.words) CSAT_TRY((decoder_gemm<T>(g, w.ldn, 1, EpiScreened<EpiIstaUpdate>{eu}, st)));
        else CSAT_TRY((decoder_gemm<T>(g, w.ldn, 1, eu, st)));
    }
    return CSAT_OK;
}

// C = X V per head from the decoder state; V: as the caller holds it, or nullptr when only w.VT (its transpose) is there
template <typename T>
csat_status run_synthesis(const csat_dims& d, const Workspace& w, T* C, hipStream_t st, const T* V = nullptr, SupportRule rule = {}) {
    constexpr bool kBf16 = sizeof(T) == 2;
    const int BH = d.B * d.H;
    if constexpr (kBf16) {
        if (V && synthesis_is_direct<T>(d)) {
            MeasureDirectArgs a{};
            a.Phi = w.Xb; a.ldp = w.ldn; a.strideA = (long long)d.n_q * w.ldn;
            a.ncols = (int)round_up(d.n, 8);         // (the operand's columns from n on are zero)
            a.K = (const bf16_t*)V; a.V = nullptr; a.strideX = (long long)d.n * d.d;
            a.m = d.n_q; a.n = d.n; a.MT = (d.n_q + 31) / 32;
            a.Kc = (bf16_t*)C;
            a.heads = BH;
            a.blocks_per_head = (a.MT + 3) / 4;
            a.rule = rule;
            const dim3 grid((unsigned)(8 * ((BH + 7) / 8) * a.blocks_per_head));
            Timed tm(w, CSAT_K_SYNTHESIS, st);
            const bool deep = d.n >= 4096;
            if (d.d == 64) {
                if (deep) hipLaunchKernelGGL((measure_direct_kernel<2, 64, 4, false>), grid, dim3(256), 0, st, a);
                else hipLaunchKernelGGL((measure_direct_kernel<2, 64, 2, false>), grid, dim3(256), 0, st, a);
            } else {
                if (deep) hipLaunchKernelGGL((measure_direct_kernel<4, 64, 4, false>), grid, dim3(256), 0, st, a);
                else hipLaunchKernelGGL((measure_direct_kernel<4, 64, 2, false>), grid, dim3(256), 0, st, a);
            }
            HIP_TRY(hipGetLastError());
            return CSAT_OK;
        }
    }
    GemmArgs g{kBf16 ? (const void*)w.Xb : (const void*)w.Xs, w.ldn, (long long)d.n_q * w.ldn,
               w.VT, w.ldn, (long long)d.d * w.ldn, d.n_q, d.d, d.n, 0};
    EpiStore<T> ec{C, d.d, (long long)d.n_q * d.d, nullptr, 0, 0, 1.f, d.n_q, d.d};
    Timed tm(w, CSAT_K_SYNTHESIS, st);
    if (rule.ctl) return decoder_gemm<T>(g, d.d, BH, EpiRuled<EpiStore<T>>{ec, rule}, st);
    return decoder_gemm<T>(g, d.d, BH, ec, st);
}

template <typename T>
csat_status measure_t(const csat_dims& d, const Workspace& w, const void* PhiK, const void* Phi, const void* K,
                      const void* V, void* Kc, void* Vc, hipStream_t st) {
    const bool separate = PhiK && PhiK != Phi;
    CSAT_TRY(prepare_phi<T>(d, w, (const T*)Phi, !(measure_reads_raw_phi<T>(d, separate) || (!separate && phi_is_operand<T>(d, Phi))), 0, st));
    return run_measure<T>(d, w, (const T*)K, (const T*)V, (T*)Kc, (T*)Vc, nullptr, measure_is_direct<T>(d, separate), false, st, (const T*)PhiK,
                          (const T*)Phi);
}

template <typename T>
csat_status attention_t(const csat_dims& d, const Workspace& w, const void* Q, const void* Kc, const void* Vc,
                        float* A, void* Z, hipStream_t st) {
    const int BH = d.B * d.H;
    if (!A && attention_z_applies<T>(d, 1))
        return run_attention_z<T>(d, w, (const T*)Q, (const T*)Kc, 1, false, (const T*)Vc, false, (T*)Z, (T*)nullptr, st);
    {
        Timed tm(w, CSAT_K_LAYOUT, st);
        CSAT_TRY(transpose_pack<T>((const T*)Vc, (T*)w.VcT, w.ldm, BH, d.m, d.d, st));
    }
    return run_attention<T>(d, w, (const T*)Q, (const T*)Kc, (const T*)w.VcT, A ? A : w.A, A ? (long long)d.m : w.ldy, (T*)w.R, (T*)Z, false, st);
}

template <typename T>
csat_status recover_t(const csat_dims& d, const Workspace& w, const float* Y, const void* Phi, float lambda,
                      float mu, int iters, float* X, const void* V, void* C, hipStream_t st) {
    const int BH = d.B * d.H;
    const long long rows = (long long)BH * d.n_q;
    const bool want_c = V && C;
    if (iters == 0) {
        if (X) CSAT_TRY(fill_zero(X, (size_t)rows * d.n * 4, st));
        if (want_c) CSAT_TRY(fill_zero(C, (size_t)rows * d.d * sizeof(T), st));
        return CSAT_OK;
    }
    CSAT_TRY(prepare_phi<T>(d, w, (const T*)Phi, false, iters, st));
    {
        Timed tm(w, CSAT_K_LAYOUT, st);
        if (w.fused) CSAT_TRY((pack_rows<float, float>(Y, d.m, w.A, w.ldy, rows, d.m, st)));
        else if (!decoder_is_resident_f32(d, w, iters)) CSAT_TRY((pack_rows<float, T>(Y, d.m, (T*)w.R, w.ldm, rows, d.m, st)));
        if (want_c && !synthesis_is_direct<T>(d)) CSAT_TRY(transpose_pack<T>((const T*)V, (T*)w.VT, w.ldn, BH, d.n, d.d, st));
    }
    ScreenPlan plan;
    const float* y = w.fused ? w.A : Y;
    const long long ld = w.fused ? w.ldy : (long long)d.m;
    if (want_c && screen_applies(d, w, X, V, C, iters)) CSAT_TRY(screen<T>(d, w, (const T*)Phi, (const T*)V, y, ld, false, mu, mu * lambda, &plan, st));
    CSAT_TRY(run_ista<T>(d, w, (const T*)Phi, y, ld, lambda, mu, iters, X, st, nullptr, nullptr, false, plan));
    if (want_c) CSAT_TRY(run_synthesis<T>(d, w, (T*)C, st, (const T*)V, SupportRule{plan.words, 0}));
    return screen_finish<T>(d, w, plan, (const T*)V, (T*)C, st);
}

template <typename T>
csat_status forward_t(const csat_dims& d, const Workspace& w, const void* Q, const void* K, const void* V,
                      const void* PhiK, const void* Phi, float lambda, float mu, int iters, void* C, void* Z,
                      float* X, hipStream_t st) {
    const bool separate = PhiK && PhiK != Phi;
    CSAT_TRY(prepare_phi<T>(d, w, (const T*)Phi, !(measure_reads_raw_phi<T>(d, separate) || (!separate && phi_is_operand<T>(d, Phi))), iters, st));
    const bool need_z = Z || iters == 0;
    T* zdst = (iters == 0) ? (T*)C : (T*)Z;
    bool kc_packed = false, v_packed = false;
    const bool direct = measure_is_direct<T>(d, separate);
    // no decoder: A~ is not wanted
    const bool z_only = iters == 0 && attention_z_applies<T>(d, 2);
    // (then nothing reads V^T: the one-kernel measurement takes V as it is)
    const bool syn = iters > 0 && synthesis_in_decoder(d, w) && direct;
    CSAT_TRY(run_measure<T>(d, w, (const T*)K, (const T*)V, (T*)w.Kc, (T*)w.Vc, need_z && (direct || !z_only) ? (T*)w.VcT : nullptr,
                            syn || synthesis_is_direct<T>(d), true, st, (const T*)PhiK, (const T*)Phi, need_z, &kc_packed,
                            // (the two-sweep form of the kernel leaves Z to a product GEMM: with the product's registers
                            // on top it spills; long_video 4.0 ms against 1.2)
                            z_only || (attention_is_fused<T>(d, w, true) && attention_packed_v_fits(w.MT, d.d)) ? &v_packed : nullptr));
    if (z_only) {
        CSAT_TRY(run_attention_z<T>(d, w, (const T*)Q, (const T*)w.KcHL, 2, kc_packed, (const T*)w.Vc, v_packed, zdst, (T*)nullptr, st));
        if (Z) HIP_TRY(hipMemcpyAsync(Z, C, (size_t)d.B * d.H * d.n_q * d.d * sizeof(T), hipMemcpyDeviceToDevice, st));
        return CSAT_OK;
    }
    // the operand copy of A~ feeds the Z product as a GEMM and the GEMM-pair decoder; the fused decoder reads A~ itself
    T* pcopy = ((need_z && !v_packed) || !(w.fused || decoder_is_resident_f32(d, w, iters))) ? (T*)w.R : nullptr;
    // A~ in accumulator tiles between the attention kernel and the two-chunk decoder: both then move whole 1 KB pieces
    // per instruction instead of 16-byte pieces of 32 rows.  Needs whole 32-row tiles per head and the forms of the two
    // kernels that support it (single sweep with the scores kept in the accumulator file; the two-chunk decoder).
    bool y_tiled = false;
    if constexpr (sizeof(T) == 2) {
        y_tiled = iters > 0 && w.fused && !decoder_is_resident(w) && d.n_q % 32 == 0 && (*tl_opt)[CSAT_OPT_Y_LAYOUT] != 1 &&
                  (fused_variant(w.MT, w.rows_pad, w.nct, iters) == 3 || fused_variant(w.MT, w.rows_pad, w.nct, iters) == 4) && attention_is_fused<T>(d, w, true) &&
                  attention_single_sweep(w.MT, 2 * ((d.d + 15) / 16)) &&
                  (v_packed || (!need_z && attention_mtp(w.MT, true) == 13));
    }
    CSAT_TRY(run_attention<T>(d, w, (const T*)Q, (const T*)w.Kc, (const T*)w.VcT, w.A, w.ldy, pcopy,
                              need_z ? zdst : nullptr, true, st, nullptr, kc_packed, v_packed, y_tiled));
    if (iters == 0) {
        if (Z) HIP_TRY(hipMemcpyAsync(Z, C, (size_t)d.B * d.H * d.n_q * d.d * sizeof(T), hipMemcpyDeviceToDevice, st));
        return CSAT_OK;
    }
    ScreenPlan plan;
    if (screen_applies(d, w, X, V, C, iters)) CSAT_TRY(screen<T>(d, w, (const T*)Phi, (const T*)V, w.A, w.ldy, y_tiled, mu, mu * lambda, &plan, st));
    CSAT_TRY(run_ista<T>(d, w, (const T*)Phi, w.A, w.ldy, lambda, mu, iters, X, st, syn ? (const T*)V : nullptr, syn ? (T*)C : nullptr, y_tiled, plan));
    if (!syn) CSAT_TRY(run_synthesis<T>(d, w, (T*)C, st, (const T*)V, SupportRule{plan.words, 0}));
    return screen_finish<T>(d, w, plan, (const T*)V, (T*)C, st);
}

// Column-wise decode (n_q == n): the decoder's problems are the d feature columns of Z per head.
// Its buffers are a second carving, for the same shape with d rows per head, placed after the main
// one, followed by the transposed Z and the decoded columns.
csat_dims rd_dims(const csat_dims& d) {
    csat_dims r = d;
    r.n_q = d.d;
    return r;
}
struct RdExtra { char* ZT; float* Xout; size_t bytes; };
RdExtra carve_rd_extra(const csat_dims& d, const Workspace& wr, char* base) {
    const long long rows = (long long)d.B * d.H * d.d;
    const size_t zt = (size_t)round_up(rows * wr.ldn * 4, 256);   // a bf16 (hi | lo) pair or one float per element
    return RdExtra{base, (float*)(base + zt), zt + (size_t)round_up(rows * (long long)d.n * 4, 256)};
}

template <typename T>
csat_status forward_rd_t(const csat_dims& d, const Workspace& w, const Workspace& wr, const RdExtra& x, const void* Q,
                         const void* K, const void* V, const void* PhiK, const void* Phi, float lambda, float mu,
                         int iters, void* C, void* Z, hipStream_t st) {
    constexpr bool kBf16 = sizeof(T) == 2;
    const int BH = d.B * d.H;
    const long long rows = (long long)BH * d.d;          // decoder problems
    const csat_dims dr = rd_dims(d);
    CSAT_TRY(prepare_phi<T>(d, w, (const T*)Phi, true, 0, st));
    const bool direct = measure_is_direct<T>(d, PhiK && PhiK != Phi), z_only = attention_z_applies<T>(d, 2);
    bool kc_packed = false, v_packed = false;
    CSAT_TRY(run_measure<T>(d, w, (const T*)K, (const T*)V, (T*)w.Kc, (T*)w.Vc, direct || !z_only ? (T*)w.VcT : nullptr,
                            direct, true, st, (const T*)PhiK, (const T*)Phi, true, z_only ? &kc_packed : nullptr, z_only ? &v_packed : nullptr));
    // the compressed block's output (and its transpose ZT): nothing here reads A~
    auto attention = [&](T* Zdst, T* ZTdst) -> csat_status {
        if (z_only) return run_attention_z<T>(d, w, (const T*)Q, (const T*)w.KcHL, 2, kc_packed, (const T*)w.Vc, v_packed, Zdst, ZTdst, st);
        return run_attention<T>(d, w, (const T*)Q, (const T*)w.Kc, (const T*)w.VcT, w.A, w.ldy, (T*)w.R, Zdst, true, st, ZTdst);
    };
    if (iters == 0) {
        CSAT_TRY(attention((T*)C, (T*)nullptr));
        if (Z) HIP_TRY(hipMemcpyAsync(Z, C, (size_t)BH * d.n * d.d * sizeof(T), hipMemcpyDeviceToDevice, st));
        return CSAT_OK;
    }
    const long long ldzt = kBf16 ? 2 * w.ldn : w.ldn;
    CSAT_TRY(fill_zero(x.ZT, (size_t)rows * ldzt * sizeof(T), st));
    CSAT_TRY(attention((T*)Z, (T*)x.ZT));
    {   // Y^T [m, rows] = Phi Z^T per column, stored transposed as the decoder's measurement rows
        CSAT_TRY(fill_zero(wr.A, (size_t)rows * wr.ldy * 4, st));
        GemmArgs g{w.PhiP, w.ldn, 0, x.ZT, ldzt, 0, d.m, (int)rows, kBf16 ? (int)(2 * w.ldn) : d.n, kBf16 ? (int)(w.ldn / 8) : 0};
        EpiStore<float> ey{nullptr, 0, 0, wr.A, wr.ldy, 0, 1.f, d.m, (int)rows};
        Timed tm(w, CSAT_K_MEASURE, st);
        CSAT_TRY((gemm<T>(g, rows, 1, ey, st)));
    }
    CSAT_TRY(prepare_phi<T>(dr, wr, (const T*)Phi, false, iters, st));
    if (!wr.fused && !decoder_is_resident_f32(dr, wr, iters)) {
        Timed tm(w, CSAT_K_LAYOUT, st);
        CSAT_TRY((pack_rows<float, T>(wr.A, wr.ldy, (T*)wr.R, wr.ldm, rows, d.m, st)));
    }
    CSAT_TRY(run_ista<T>(dr, wr, (const T*)Phi, wr.A, wr.ldy, lambda, mu, iters, x.Xout, st));
    {   // C[b,h,j,k] = decoded column k at token j
        Timed tm(w, CSAT_K_SYNTHESIS, st);
        dim3 grid((unsigned)((d.d + 31) / 32), (unsigned)((d.n + 31) / 32), (unsigned)BH);
        hipLaunchKernelGGL((transpose_cast_kernel<T>), grid, dim3(32, 8), 0, st, x.Xout, (T*)C, d.d, d.n);
        HIP_TRY(hipGetLastError());
    }
    return CSAT_OK;
}

// Buffers of the unrolled (LISTA) decoder, carved after the main workspace.
struct ListaExtra {
    char* D;        // [n, ldn]     S - I, operand layout
    float* W;       // [rows_pad, ldn]  B y (row-major, or in accumulator order on the large-tile path)
    float* StateF;  // [rows_pad, ldn]  fp32 iterate (bf16 mode; in fp32 mode the operand buffers are the iterate)
    uint8_t* Mask;  // [rows_pad/32, ldn/32, 64]  non-zero float4 pieces of the iterate (large-tile path)
    char* Op[2];    // [rows, ldn]  GEMM operand of the current / next layer
    size_t bytes;
};
ListaExtra carve_lista(const csat_dims& d, const Workspace& w, char* base) {
    const long long rows = (long long)d.B * d.H * d.n_q;
    const size_t e = esize(d.dtype);
    ListaExtra x{};
    size_t off = 0;
    auto take = [&](size_t nbytes) {
        char* p = base + off;
        off += (size_t)round_up((long long)nbytes, 256);
        return p;
    };
    x.D = take((size_t)d.n * w.ldn * e);
    x.W = (float*)take((size_t)w.rows_pad * w.ldn * 4);
    x.StateF = (float*)take(d.dtype == CSAT_BF16 ? (size_t)w.rows_pad * w.ldn * 4 : 0);
    x.Mask = (uint8_t*)take(d.dtype == CSAT_BF16 ? (size_t)(w.rows_pad / 32) * (w.ldn / 32) * 64 : 0);
    x.Op[0] = take((size_t)rows * w.ldn * e);
    x.Op[1] = take((size_t)rows * w.ldn * e);
    x.bytes = off;
    return x;
}

// Whether the layers behind the first may run over the support of their iterate, which the device decides: not where they
// take less than about 400 us in all (20 us a layer and its operations at 0.9 PFLOP/s), 2 to 3 % of which the counting and the launches
// that return at once would take.  S - I transposed takes the place of the second operand buffer.
bool lista_support_applies(const csat_dims& d, long long rows, int iters) {
    if (support_choice() == 1 || iters < 2 || iters > kSupportMaxLayers || d.n > kListaSupportMaxN || rows < d.n || rows / 4 * d.n >= (1ll << 32)) return false;
    return support_choice() == 2 || (iters - 1) * (20.0 + (double)rows * d.n * d.n / 4.5e8) > 400.0;
}
// ... and up to which density: non-zero float4 (four rows of a column) that the first layer may leave to every four rows.  Over
// all columns against over the support, us: n = 1600, 76 800 rows, 20 layers: 9 a quad 8760, 2540; 25 8920, 4150; 77 9260, 8000; 288 10 820, 19 060;
// n = 2500, 20 000 rows, 10 layers: 39 2985, 2070; 80 3040, 3260; n = 700, 44 800 rows, 20 layers: 24 2270, 1120; 56 2450, 1720; 139
// 2720, 2970; fewer rows, whose longest lists end the launch: n = 700, 5600 rows, 8 layers: 52 299, 311; n = 2048, 8192 rows, 10 layers: 10 772, 470; 20
// 750, 630; 43 740, 880; n = 4096 (its matrix far beyond an L2), 16 384 rows, 10 layers: 23 4590, 4960; 57 4600, 7570; short rows, whose layers take as long
// as their launches: n = 416, 6656 rows, 16 layers: 271 a quad 488, 468; 402 493, 772; n = 278, 34 656 rows, 38 layers: 118 1720, 1600; 218 1780, 2550; of those
// shorter than 128 float4 a quad are no limit, but a share of their columns, all of few rows' and two in five where rows are many: n = 116, 4704 rows, 24 layers: 101 510,
// 300; n = 94, 16 416 rows, 27 layers: 78 606, 565; n = 146, 22 912 rows, 35 layers: 63 910, 670; 116 930, 1100; n = 96, 18 432 rows, 25 layers:
// 95 572, 810; n = 108, 95 056 rows, 27 layers: 37 1340, 1170; 60 1350, 1620; 94 1360, 2680; few long rows: n = 3052, 12 712 rows, 11 layers:
// 1.5 2480, 1805; 13 2520, 3510; n = 2163, 2192 rows, 39 layers: 6 2600, 2380; 17 2600, 3390.
double lista_support_limit(const csat_dims& d, long long rows) {
    if (support_choice() == 2) return 4294967295.0;
    if (d.n <= 512) return rows / 4.0 * std::min(128.0, std::max(0.4, std::min(1.0, 15000.0 / rows)) * d.n);
    return rows / 4.0 * (d.n > 3328 || (d.n > 2048 && rows < 16384) ? 12 : rows >= 16384 ? 48 : 24);
}
// ... and not where thresholds fall far below the first layer's: its count then says nothing of the coefficients that the later layers leave.  Over
// all columns against over the support, us (first layer's float4 a quad; the lowest threshold, of the first): 76 800 rows, n = 1600, 20 layers:
// (9, 0.6) 8670, 2880; (0.4, 0.25) 8750, 4130; (25, 0.4) 9300, 8340; (25, 0.2) 10 300, 20 650; (9, 0.016) 11 080, 87 490; 44 800 rows, n = 700: (24, 0.6)
// 2220, 1150; (56, 0.4) 2630, 2800; (56, 0.2) 2800, 5370.  (An S that makes the iterate grow is not looked for: with a random matrix of norm 2 added
// to short_video's, 8600 and 10 080; reports of the rows on the way, by which the launch could give up, cost 2 % of every other call.)
constexpr float kListaSupportFall = 0.25f;
bool lista_thresholds_fall(const float* thetas, int iters) {
    for (int t = 1; t < iters; ++t)
        if (thetas[t] < kListaSupportFall * thetas[0]) return true;
    return false;
}
template <typename T>
csat_status lista_t(const csat_dims& d, const Workspace& w, const ListaExtra& x, const float* Y, const void* S,
                    const void* Bw, const float* thetas, int iters, float* X, const void* V, void* C, hipStream_t st) {
    constexpr bool kBf16 = sizeof(T) == 2;
    const int BH = d.B * d.H;
    const long long rows = (long long)BH * d.n_q;
    const bool want_c = V && C;
    if (iters == 0) {
        if (X) CSAT_TRY(fill_zero(X, (size_t)rows * d.n * 4, st));
        if (want_c) CSAT_TRY(fill_zero(C, (size_t)rows * d.d * sizeof(T), st));
        return CSAT_OK;
    }
    // bf16 problems large enough for the 256-wide kernel take tile-level epilogues
    const bool tiled = kBf16 && use_big_gemm<T>(GemmArgs{nullptr, w.ldn, 0, nullptr, w.ldn, 0, (int)rows, d.n, d.n, 0}, w.ldn) &&
                       use_big_gemm<T>(GemmArgs{nullptr, w.ldm, 0, nullptr, w.ldm, 0, (int)rows, d.n, d.m, 0}, w.ldn) &&
                       lista_choice() != 1;
    SupportRule rule;
    if (tiled && lista_support_applies(d, rows, iters) && (support_choice() == 2 || !lista_thresholds_fall(thetas, iters))) {
        rule.ctl = (const uint32_t*)w.Status + kSupportWord;
        rule.limit = (uint32_t)std::min(4294967295.0, lista_support_limit(d, rows));
        CSAT_TRY(support_begin(w, st));
    }
    {
        Timed tm(w, CSAT_K_LAYOUT, st);
        CSAT_TRY((pack_rows<T, T>((const T*)Bw, d.m, (T*)w.PhiT, w.ldm, d.n, d.m, st)));
        const long long total = (long long)d.n * w.ldn;
        hipLaunchKernelGGL((sub_identity_pack_kernel<T>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                           (const T*)S, d.n, (T*)x.D, w.ldn, rule.ctl ? (uint32_t*)w.Status + kSupportWord + 1 : nullptr);
        HIP_TRY(hipGetLastError());
        CSAT_TRY((pack_rows<float, T>(Y, d.m, (T*)w.R, w.ldm, rows, d.m, st)));
        if (want_c && !synthesis_is_direct<T>(d)) CSAT_TRY(transpose_pack<T>((const T*)V, (T*)w.VT, w.ldn, BH, d.n, d.d, st));
        // alpha^(0) = 0
        if (!tiled) CSAT_TRY(fill_zero(x.Op[0], (size_t)rows * w.ldn * sizeof(T), st));
        if (kBf16 && !tiled) CSAT_TRY(fill_zero(x.StateF, (size_t)rows * w.ldn * 4, st));
    }
    {   // W = B y for every row (tiled: and the first layer, alpha = eta(W))
        GemmArgs g{w.R, w.ldm, 0, w.PhiT, w.ldm, 0, (int)rows, d.n, d.m, 0};
        Timed tm(w, CSAT_K_RESIDUAL, st);
        if (tiled) {
            EpiListaFirstTiled ew{{(f32x4*)x.StateF, w.ldn / 32, x.Mask, (bf16_t*)x.Op[1], w.ldn, iters == 1 ? X : nullptr, 1.f, thetas[0], rows, d.n, 1},
                                  iters == 1 ? nullptr : (f32x4*)x.W};
            g.K = (int)round_up(g.K, 64);
            CSAT_TRY(launch_gemm_big_lista(g, w.ldn, ew, st));
        } else {
            EpiStore<float> ew{x.W, w.ldn, 0, nullptr, 0, 0, 1.f, (int)rows, d.n};
            CSAT_TRY((gemm<T>(g, d.n, 1, ew, st)));
        }
    }
    if constexpr (kBf16) {
        if (rule.ctl) {
            Timed tm(w, CSAT_K_LAYOUT, st);
            CSAT_TRY(support_count(w, x.Mask, (rows + 31) / 32 * (w.ldn / 32) * 64, st, nullptr, 0.f, 0, want_c ? V : nullptr, want_c ? (long long)BH * d.n * d.d * 2 : 0));
            hipLaunchKernelGGL(support_transpose_kernel, dim3((unsigned)((w.ldn + 63) / 64), (unsigned)((d.n + 63) / 64)), dim3(256), 0, st, rule,
                               (const bf16_t*)x.D, (bf16_t*)x.Op[0], d.n, (int)w.ldn);
            HIP_TRY(hipGetLastError());
        }
    }
    for (int t = tiled ? 1 : 0; t < iters; ++t) {
        char* cur = x.Op[t & 1];
        char* nxt = x.Op[(t + 1) & 1];
        GemmArgs g{cur, w.ldn, 0, x.D, w.ldn, 0, (int)rows, d.n, d.n, 0};
        if (tiled) {    // accumulators start from W; the iterate is kept like the ISTA decoder's (sparse, accumulator order)
            EpiListaUpdateTiled eu{{(f32x4*)x.StateF, w.ldn / 32, x.Mask, (bf16_t*)nxt, w.ldn,
                                    (t == iters - 1) ? X : nullptr, 1.f, thetas[t], rows, d.n, 0},
                                   (const f32x4*)x.W, rule};
            g.K = (int)round_up(g.K, 64);
            Timed tm(w, CSAT_K_UPDATE, st);
            CSAT_TRY(launch_gemm_big_lista(g, w.ldn, eu, st));
            continue;
        }
        EpiListaUpdate eu{kBf16 ? x.StateF : (const float*)cur, kBf16 ? x.StateF : (float*)nxt, w.ldn, x.W,
                          kBf16 ? (bf16_t*)nxt : nullptr, (t == iters - 1) ? X : nullptr, thetas[t], rows, d.n};
        Timed tm(w, CSAT_K_UPDATE, st);
        CSAT_TRY((gemm<T>(g, w.ldn, 1, eu, st)));
    }
    if (want_c) {
        Workspace wf = w;          // the synthesis reads the final operand buffer
        if (kBf16) wf.Xb = (bf16_t*)x.Op[iters & 1];
        else wf.Xs = (float*)x.Op[iters & 1];
        CSAT_TRY(run_synthesis<T>(d, wf, (T*)C, st, (const T*)V, rule));
    }
    if constexpr (kBf16) {
        if (rule.ctl) {      // (behind the synthesis, which not every shape's kernel leaves out: C is written last here)
            ListaSupportArgs a{rule, (const f32x4*)x.W, w.ldn / 32, (const bf16_t*)x.Op[0], (int)w.ldn, X, (const bf16_t*)V, want_c ? (bf16_t*)C : nullptr,
                               rows, d.n_q, d.n, d.d, iters, {}};
            std::copy(thetas, thetas + iters, a.theta);
            Timed tm(w, CSAT_K_UPDATE, st);
            HIP_TRY(lista_support_launch(a, (unsigned)((rows + 3) / 4), st));
        }
    }
    return CSAT_OK;
}

// Buffers of the matching-pursuit decoder, carved after the main workspace.
struct OmpExtra {
    float* Cm;     // [rows, ldn]    correlations of the current residuals with every column; or, where the pick is taken
                   //                with the product, its candidates [rows, splits]
    uint32_t* taken;  // [row tiles of 32, nct, 32]  columns that a row may not pick, a bit per row (bf16)
    float* Tri;    // [rows, k, k]   triangular factor
    float* Fac;    // [rows, k (k + 1) / 2]  ... by columns, with 1 / its diagonal (held vectors)
    float* Z;      // [rows, k]      Q^T y
    int* picks;    // [rows, k]
    bool stored;   // the update stores the orthonormal vectors (omp_stores_vectors)
    char* PhiQ;    // [n, 64, pitch]  columns of Phi in the update's order: held vectors, more than one pick
    float* Rf;     // [rows, mq]     fp32 residuals and ...
    float* Qb;     // [rows, k, mq]  ... orthonormalised picked columns: stored vectors
    int mq, MQ;    // m in whole 64s; values of an m-vector per lane of the update
    size_t bytes;
};
// Picks whose orthonormal vectors the update keeps in registers: 128 registers at most; at one value per lane (m <= 64) reading them
// back is cheaper than forming more than eight again (float, 8192 rows, n = 64, m = 32, 16 picks: 361 us against 341).
constexpr int omp_held_picks(int MQ) { return MQ == 1 || MQ == 16 ? 8 : 16; }
// Held vectors need Phi's columns packed first, a pass over all of Phi for the few columns that few rows pick.  Vectors are stored
// instead, also of fewer picks, where their buffers are no larger than the packed columns and the packing takes longer than it
// saves: in bf16 a launch of 4 us and 1.3 ps an element against MQ (0.5 + 0.18 k) us (fits); in float few rows gain nothing from
// held vectors.  Calls, held and stored, us: float, n = 16 384, m = 1024, 256 rows, 4 picks 599, 557; n = 2048, m = 1000, one row, 2
// picks 58, 52; bf16, n = 16 384, m = 1024, 512 rows, 2 picks 125, 117, 64 rows, 8 picks 255, 273; n = 1600, m = 392, 64 rows, 4 picks
// 64, 68; n = 16 384, m = 64, 512 rows, 8 picks 123, 116.
bool omp_stores_vectors(const csat_dims& d, int MQ, int mq, int k, size_t packed_bytes) {
    if (k > omp_held_picks(MQ)) return true;
    if (k == 1 || (size_t)d.B * d.H * d.n_q * (k + 1) * mq * 4 > packed_bytes) return false;
    return d.dtype == CSAT_F32 || 4 + 1.3e-6 * d.n * d.m > MQ * (0.5 + 0.18 * k);
}
OmpExtra carve_omp(const csat_dims& d, const Workspace& w, int k, char* base) {
    const long long rows = (long long)d.B * d.H * d.n_q;
    OmpExtra x{};
    x.mq = (int)round_up(d.m, 64);
    x.MQ = x.mq <= 512 ? x.mq / 64 : 16;
    const size_t packed_bytes = (size_t)d.n * 64 * omp_column_pitch(x.MQ, (int)esize(d.dtype)) * esize(d.dtype);
    x.stored = omp_stores_vectors(d, x.MQ, x.mq, k, packed_bytes);
    size_t off = 0;
    auto take = [&](size_t nbytes) {
        char* p = base + off;
        off += (size_t)round_up((long long)nbytes, 256);
        return p;
    };
    x.Cm = (float*)take((size_t)rows * w.ldn * 4);
    x.taken = (uint32_t*)take(d.dtype == CSAT_BF16 ? (size_t)((rows + 31) / 32) * w.nct * 128 : 0);
    x.Tri = (float*)take((size_t)rows * k * k * 4);
    x.Fac = (float*)take(x.stored ? 0 : (size_t)rows * (k * (k + 1) / 2) * 4);
    x.Z = (float*)take((size_t)rows * k * 4);
    x.picks = (int*)take((size_t)rows * k * 4);
    x.PhiQ = take(x.stored || k == 1 ? 0 : packed_bytes);
    x.Rf = (float*)take(x.stored ? (size_t)rows * x.mq * 4 : 0);
    x.Qb = (float*)take(x.stored ? (size_t)rows * k * x.mq * 4 : 0);
    // (a workspace for more picks holds fewer ones too, also where those pack the columns)
    const int held = omp_held_picks(x.MQ);
    x.bytes = k > held ? std::max(off, carve_omp(d, w, held, base).bytes) : off;
    return x;
}

constexpr int kOmpMaxSplits = 128;    // (at most a chunk of 32 columns each: a candidate is 8 bytes, a row of Cm four a column)
constexpr int kOmpPickStart = 4;      // a workgroup's start, its residuals' way from memory or L2, in steps
// Row blocks that run whole, as many as fill the chip evenly, and the shares of n that the others are cut into, as many as need the
// fewest passes over the chip.  76 800 rows, n = 1600, m = 392 (300 blocks of 50 steps): every block in three shares 137 us, 256
// whole and 44 in five 119.  The shares of a block run on one XCD unless they take fewer passes spread over all: a few blocks would
// leave whole XCDs idle.
// Returns the steps that one place on the chip then walks.
long long omp_pick_plan(OmpPickArgs& a) {
    const int KS = (int)(a.ldm / 64), steps = (a.nct + omp_pick_chunks(KS) - 1) / omp_pick_chunks(KS);
    const long long blocks = (a.rows + omp_pick_rows(KS) - 1) / omp_pick_rows(KS), slots = (long long)cu_count() * omp_pick_per_cu(KS);
    a.whole = (int)(blocks / slots * slots);
    a.splits = 1;
    a.group = 8;
    long long best = -1;
    for (int s = 1; s <= kOmpMaxSplits && s <= steps; ++s) {
        const long long cut = blocks - a.whole, here = ((cut + 7) / 8 * s + slots / 8 - 1) / (slots / 8), spread = (cut * s + slots - 1) / slots;
        const long long cost = std::min(here, spread) * ((steps + s - 1) / s + kOmpPickStart);
        if (best < 0 || cost < best) { best = cost; a.splits = s; a.group = here <= spread ? 8 : (int)cut; }
    }
    return a.whole / slots * (steps + kOmpPickStart) + best;
}
// Above m = 512 the kernel has room for one wavefront per SIMD, and what it has over the 256 x 256 tiles is only that it needs no whole
// rounds of them.  The line is where a round of tiles, in units of a step's time per 64 of m, is 60 + 26 / 3 of m in 64s (fits to 210
// products of n = 1100 to 16 384, 256 to 65 536 rows; none it sends the wrong way costs more than 8 %).  A pick, the columns passing and tiles, us:
// n = 1100, m = 640: 256 rows 13, 26; 16 384 rows 47, 49; n = 4096, m = 768: 1024 rows 21, 28; 4096 rows 49, 32; 65 536 rows 623, 450;
// n = 16 384, m = 1024: 256 rows 22, 33; 1024 rows 54, 38; 16 384 rows 647, 526.
bool omp_pick_on_tiles(const GemmArgs& g, int n, long long pick_steps) {
    const long long KS = g.ldb / 64, tiles = (g.M + 255ll) / 256 * ((n + 255ll) / 256);
    return KS > 8 && use_big_gemm<bf16_t>(g, n) && (tiles + cu_count() - 1) / cu_count() * (180 + 26 * KS) < 3 * pick_steps * KS;
}
csat_status launch_omp_pick(const OmpPickArgs& a, hipStream_t st) {
    const int KS = (int)(a.ldm / 64);
    const long long blocks = (a.rows + omp_pick_rows(KS) - 1) / omp_pick_rows(KS);
    const dim3 grid((unsigned)(a.whole + (blocks - a.whole + a.group - 1) / a.group * a.group * a.splits));
    const size_t lds = omp_pick_lds_bytes(KS);
    tl_forms[CSAT_FORM_OMP_SHARES] = a.splits;
    switch (KS) {
#define CSAT_OMP_PICK(N)                                                                                                       \
    case N:                                                                                                                    \
        HIP_TRY(hipFuncSetAttribute((const void*)omp_pick_product_kernel<N>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
        hipLaunchKernelGGL((omp_pick_product_kernel<N>), grid, dim3(64 * omp_pick_waves(N)), lds, st, a);                          \
        break;
        CSAT_OMP_PICK(1) CSAT_OMP_PICK(2) CSAT_OMP_PICK(3) CSAT_OMP_PICK(4) CSAT_OMP_PICK(5) CSAT_OMP_PICK(6) CSAT_OMP_PICK(7) CSAT_OMP_PICK(8)
        CSAT_OMP_PICK(9) CSAT_OMP_PICK(10) CSAT_OMP_PICK(11) CSAT_OMP_PICK(12) CSAT_OMP_PICK(13) CSAT_OMP_PICK(14) CSAT_OMP_PICK(15) CSAT_OMP_PICK(16)
#undef CSAT_OMP_PICK
        default: return CSAT_ERR_SHAPE;
    }
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

template <typename T>
csat_status launch_omp_update(const OmpUpdateArgs<T>& a, int MQ, bool stored, float* Rf, hipStream_t st) {
    const dim3 grid((unsigned)((a.rows + 3) / 4)), block(256);
    const int form = stored ? 2 : a.it < 8 ? 0 : 1;
    tl_forms[CSAT_FORM_OMP_REFIT] = stored ? 2 : 1;
    switch (MQ) {
#define CSAT_OMP_UPDATE(M)                                                                                             \
    case M:                                                                                                           \
        if (form == 2) hipLaunchKernelGGL((omp_update_stored_kernel<T, M>), grid, block, 0, st, a, Rf);                \
        else if (form == 0 || omp_held_picks(M) == 8) hipLaunchKernelGGL((omp_update_kernel<T, M, 8>), grid, block, 0, st, a); \
        else hipLaunchKernelGGL((omp_update_kernel<T, M, omp_held_picks(M)>), grid, block, 0, st, a);                   \
        break;
        CSAT_OMP_UPDATE(1) CSAT_OMP_UPDATE(2) CSAT_OMP_UPDATE(3) CSAT_OMP_UPDATE(4) CSAT_OMP_UPDATE(5) CSAT_OMP_UPDATE(6) CSAT_OMP_UPDATE(7) CSAT_OMP_UPDATE(8)
        CSAT_OMP_UPDATE(16)
#undef CSAT_OMP_UPDATE
        default: return CSAT_ERR_SHAPE;
    }
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

template <typename T>
csat_status omp_t(const csat_dims& d, const Workspace& w, const OmpExtra& x, const float* Y, const void* Phi, int k,
                  float* X, int* picks, const void* V, void* C, hipStream_t st) {
    const int BH = d.B * d.H;
    const long long rows = (long long)BH * d.n_q;
    const bool want_c = V && C;
    if (X) CSAT_TRY(fill_zero(X, (size_t)rows * d.n * 4, st));
    if (k == 0) {
        if (want_c) CSAT_TRY(fill_zero(C, (size_t)rows * d.d * sizeof(T), st));
        return CSAT_OK;
    }
    const bool in_product = sizeof(T) == 2 && gemm_choice() != 1;
    OmpCand* cand = in_product ? (OmpCand*)x.Cm : nullptr;
    GemmArgs g{w.R, w.ldm, 0, w.PhiT, w.ldm, 0, (int)rows, d.n, d.m, 0};
    OmpPickArgs p{(const bf16_t*)w.PhiT, (const bf16_t*)w.R, w.ldm, rows, x.taken, cand, d.n, w.nct, 0, 1, 8};
    const bool on_tiles = in_product && omp_pick_on_tiles(g, d.n, omp_pick_plan(p));
    tl_forms[CSAT_FORM_OMP_PICK] = on_tiles ? 3 : in_product ? 2 : 1;
    if (on_tiles) {
        g.K = (int)round_up(g.K, 64);
        p.whole = 0;
        p.splits = (d.n + 127) / 128;
    }
    {
        Timed tm(w, CSAT_K_LAYOUT, st);
        CSAT_TRY(transpose_pack<T>((const T*)Phi, (T*)w.PhiT, w.ldm, 1, d.m, d.n, st));
        CSAT_TRY((pack_rows<float, T>(Y, d.m, (T*)w.R, w.ldm, rows, d.m, st)));        // r = y
        const int pitch = omp_column_pitch(x.MQ, (int)sizeof(T));
        const long long total = (long long)d.n * 64;
        if (k > 1 && !x.stored) hipLaunchKernelGGL((omp_pack_columns_kernel<T>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, (const T*)w.PhiT, w.ldm, d.m,
                           pitch, (T*)x.PhiQ, total);
        HIP_TRY(hipGetLastError());
        if (in_product && !on_tiles) {
            const long long words = (rows + 31) / 32 * w.nct * 32;
            hipLaunchKernelGGL(omp_taken_init_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, x.taken, d.n, w.nct, words);
            HIP_TRY(hipGetLastError());
        }
    }
    OmpUpdateArgs<T> u{(const T*)w.PhiT, w.ldm, k > 1 && !x.stored ? (const T*)x.PhiQ : nullptr, Y, cand, p.splits, (long long)p.whole * omp_pick_rows((int)(w.ldm / 64)), x.picks, k, 0, on_tiles ? nullptr : x.taken, w.nct, x.Tri, x.Z, x.Fac, x.Qb, (T*)w.R, w.ldm, rows, d.m, x.mq};
    for (int it = 0; it < k; ++it) {
        u.it = it;
        if (on_tiles) {
            Timed tm(w, CSAT_K_UPDATE, st);
            CSAT_TRY(launch_gemm_big(g, d.n, 1, EpiOmpBest{cand, p.splits, x.picks, k, it, rows, d.n}, st));
        } else if (in_product) {
            Timed tm(w, CSAT_K_UPDATE, st);
            CSAT_TRY(launch_omp_pick(p, st));
        } else {
            {
                Timed tm(w, CSAT_K_UPDATE, st);
                EpiStoreStream ec{x.Cm, w.ldn, (int)rows, d.n};
                CSAT_TRY((gemm<T>(g, d.n, 1, ec, st)));
            }
            Timed tm(w, CSAT_K_RESIDUAL, st);
            hipLaunchKernelGGL(omp_pick_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, x.Cm, w.ldn, rows, d.n, x.picks, k, it);
            HIP_TRY(hipGetLastError());
        }
        Timed tm(w, CSAT_K_RESIDUAL, st);
        CSAT_TRY(launch_omp_update<T>(u, x.MQ, x.stored, x.Rf, st));
    }
    Timed tm(w, CSAT_K_SYNTHESIS, st);
#define CSAT_OMP_FINISH(KM)                                                                                                          \
    hipLaunchKernelGGL((omp_finish_kernel<T, KM>), dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, x.Tri, x.Z, x.picks, k, rows, d.n_q, \
                       d.n, d.d, X, picks, want_c ? (const T*)V : nullptr, want_c ? (T*)C : nullptr)
    if (k <= 8) CSAT_OMP_FINISH(8);
    else if (k <= 16) CSAT_OMP_FINISH(16);
    else CSAT_OMP_FINISH(kOmpMaxPicks);
#undef CSAT_OMP_FINISH
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

template <typename T>
csat_status hadamard_t(const csat_dims& d, const Workspace& w, const float* Y, long long ldY, const int* rows_of_h,
                       const signed char* signs, float lambda, float mu, int iters, float* X, const void* V, void* C,
                       hipStream_t st) {
    constexpr bool kBf16 = sizeof(T) == 2;
    const int BH = d.B * d.H;
    const long long rows = (long long)BH * d.n_q;
    const bool want_c = V && C;
    if (iters == 0) {
        if (X) CSAT_TRY(fill_zero(X, (size_t)rows * d.n * 4, st));
        if (want_c) CSAT_TRY(fill_zero(C, (size_t)rows * d.d * sizeof(T), st));
        return CSAT_OK;
    }
    int N = 1, logN = 0;
    while (N < d.n) { N *= 2; ++logN; }
    float scale = 1.f / sqrtf((float)d.m);
    if (kBf16) scale = bf2f_host(f2bf_host(scale));       // the explicit matrix would hold this value
    HadamardArgs a{Y, ldY, rows_of_h, signs, X, want_c ? (kBf16 ? (void*)w.Xb : (void*)w.Xs) : nullptr, w.ldn, rows,
                   d.n, d.m, N, logN, iters, mu, mu * lambda, scale};
    const bool in_regs = N >= 512 && hadamard_choice() != 1;      // the iterate in registers (two values per thread at least)
    const size_t lds_bytes = ista_hadamard_lds_bytes(N, d.m), reg_lds = (size_t)(fwht_pad(N) + 1 + 2 * d.m) * 4;
    if ((in_regs ? reg_lds : lds_bytes) > kLdsPerWorkgroup) return CSAT_ERR_SHAPE;     // the documented limit
    const size_t row_lds = (size_t)(fwht_pad(N) + 1) * 4;                              // (what the kernel with the iterate in registers uses of it)
    {
        Timed tm(w, CSAT_K_LAYOUT, st);
        if (want_c && !synthesis_is_direct<T>(d)) CSAT_TRY(transpose_pack<T>((const T*)V, (T*)w.VT, w.ldn, BH, d.n, d.d, st));
    }
    {
        Timed tm(w, CSAT_K_UPDATE, st);
        const long long cap = (long long)cu_count() * 16;
        const dim3 grid((unsigned)(rows < cap ? rows : cap));
#define CSAT_HADAMARD_LAUNCH(NT_)                                                                                     \
    do {                                                                                                              \
        HIP_TRY(hipFuncSetAttribute((const void*)ista_hadamard_kernel<T, NT_>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                    (int)lds_bytes));                                                                 \
        hipLaunchKernelGGL((ista_hadamard_kernel<T, NT_>), grid, dim3(NT_), lds_bytes, st, a);                         \
    } while (0)
#define CSAT_HADAMARD_REG_LAUNCH(NT_, VPT_)                                                                              \
    do {                                                                                                              \
        HIP_TRY(hipFuncSetAttribute((const void*)ista_hadamard_reg_kernel<T, NT_, VPT_>,                              \
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)row_lds));                       \
        hipLaunchKernelGGL((ista_hadamard_reg_kernel<T, NT_, VPT_>), grid, dim3(NT_), row_lds, st, a, inv);           \
    } while (0)
        if (in_regs) {
            int* inv = (int*)w.PhiT;                   // N ints; the stored-matrix operands are not used on this path
            hipLaunchKernelGGL(hadamard_inverse_fill_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, inv, N);
            hipLaunchKernelGGL(hadamard_inverse_scatter_kernel, dim3((unsigned)((d.m + 255) / 256)), dim3(256), 0, st,
                               rows_of_h, d.m, N, inv);
            // threads per row: N/16 where that is a whole wavefront, so that a pass can take four butterfly
            // stages (16 values per thread) and a transform needs about log2 N / 4 barriers
            if (N == 512) CSAT_HADAMARD_REG_LAUNCH(64, 8);
            else if (N == 1024) CSAT_HADAMARD_REG_LAUNCH(64, 16);
            else if (N == 2048) CSAT_HADAMARD_REG_LAUNCH(128, 16);
            else if (N == 4096) CSAT_HADAMARD_REG_LAUNCH(256, 16);
            else if (N == 8192) CSAT_HADAMARD_REG_LAUNCH(512, 16);
            else CSAT_HADAMARD_REG_LAUNCH(512, 32);
        }
        else if (N <= 2048) CSAT_HADAMARD_LAUNCH(256);
        else if (N <= 4096) CSAT_HADAMARD_LAUNCH(512);
        else CSAT_HADAMARD_LAUNCH(1024);
#undef CSAT_HADAMARD_REG_LAUNCH
#undef CSAT_HADAMARD_LAUNCH
        HIP_TRY(hipGetLastError());
    }
    if (want_c) CSAT_TRY(run_synthesis<T>(d, w, (T*)C, st, (const T*)V));
    return CSAT_OK;
}

// K~ and V~ by transforms (no stored Phi)
template <typename T>
csat_status measure_hadamard_t(const csat_dims& d, const int* rows_of_h, const signed char* signs, const void* K,
                               const void* V, void* Kc, void* Vc, Profiler* prof, hipStream_t st, bf16_t* KcHL = nullptr) {
    constexpr bool kBf16 = sizeof(T) == 2;
    constexpr int CB = 16 / (int)sizeof(T);
    const int BH = d.B * d.H;
    int N = 1, logN = 0;
    while (N < d.n) { N *= 2; ++logN; }
    float scale = 1.f / sqrtf((float)d.m);
    if (kBf16) scale = bf2f_host(f2bf_host(scale));       // the explicit matrix would hold this value
    const size_t col_bytes = (size_t)(fwht_pad(N) + 1) * 4;
    int held = (int)((kLdsPerWorkgroup - 8192) / col_bytes);
    if (held < 1 || BH > 65535) return CSAT_ERR_SHAPE;
    held = held > CB ? CB : held;
    const size_t lds_bytes = held * col_bytes;
    const dim3 grid((unsigned)((d.d + CB - 1) / CB), (unsigned)BH);
    Workspace w{};
    w.prof = prof;
    Timed tm(w, CSAT_K_MEASURE, st);
#define CSAT_MEASURE_HADAMARD(NT_)                                                                                      \
    do {                                                                                                              \
        HIP_TRY(hipFuncSetAttribute((const void*)measure_hadamard_kernel<T, NT_>,                                     \
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes));                     \
        hipLaunchKernelGGL((measure_hadamard_kernel<T, NT_>), grid, dim3(NT_), lds_bytes, st, (const T*)K, (T*)Kc,    \
                           rows_of_h, signs, d.n, d.d, d.m, N, logN, scale, held, KcHL);                              \
        hipLaunchKernelGGL((measure_hadamard_kernel<T, NT_>), grid, dim3(NT_), lds_bytes, st, (const T*)V, (T*)Vc,    \
                           rows_of_h, signs, d.n, d.d, d.m, N, logN, scale, held, (bf16_t*)nullptr);                  \
    } while (0)
    if (N <= 2048) CSAT_MEASURE_HADAMARD(256);
    else if (N <= 4096) CSAT_MEASURE_HADAMARD(512);
    else CSAT_MEASURE_HADAMARD(1024);
#undef CSAT_MEASURE_HADAMARD
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

// The whole block with the structured matrix: measurement and decoder by transforms, no stored Phi.
template <typename T>
csat_status forward_hadamard_t(const csat_dims& d, const Workspace& w, const void* Q, const void* K, const void* V,
                               const int* rows_of_h, const signed char* signs, float lambda, float mu, int iters, void* C,
                               void* Z, float* X, hipStream_t st) {
    constexpr bool kBf16 = sizeof(T) == 2;
    const int BH = d.B * d.H;
    CSAT_TRY(measure_hadamard_t<T>(d, rows_of_h, signs, K, V, w.Kc, w.Vc, w.prof, st, kBf16 ? w.KcHL : nullptr));
    const bool need_z = Z || iters == 0;
    T* zdst = (iters == 0) ? (T*)C : (T*)Z;
    if (iters == 0 && attention_z_applies<T>(d, 2)) {
        CSAT_TRY(run_attention_z<T>(d, w, (const T*)Q, (const T*)w.KcHL, 2, false, (const T*)w.Vc, false, zdst, (T*)nullptr, st));
    } else {
        if (need_z) {
            Timed tm(w, CSAT_K_LAYOUT, st);
            CSAT_TRY(transpose_pack<T>((const T*)w.Vc, (T*)w.VcT, w.ldm, BH, d.m, d.d, st));
        }
        CSAT_TRY(run_attention<T>(d, w, (const T*)Q, (const T*)w.Kc, (const T*)w.VcT, w.A, w.ldy, need_z ? (T*)w.R : nullptr,
                                  need_z ? zdst : nullptr, true, st));
    }
    if (iters == 0) {
        if (Z) HIP_TRY(hipMemcpyAsync(Z, C, (size_t)BH * d.n_q * d.d * sizeof(T), hipMemcpyDeviceToDevice, st));
        return CSAT_OK;
    }
    return hadamard_t<T>(d, w, w.A, w.ldy, rows_of_h, signs, lambda, mu, iters, X, V, C, st);
}

// The column-wise reading with the structured matrix: compressed block as in forward_hadamard_t, Y = Phi Z by
// transforms on Z's feature columns, the transform-based decoder on those B*H*d problems, columns back to C.
template <typename T>
csat_status forward_rd_hadamard_t(const csat_dims& d, const Workspace& w, const Workspace& wr, const RdExtra& x,
                                  const void* Q, const void* K, const void* V, const int* rows_of_h,
                                  const signed char* signs, float lambda, float mu, int iters, void* C, void* Z,
                                  hipStream_t st) {
    constexpr bool kBf16 = sizeof(T) == 2;
    const int BH = d.B * d.H;
    const long long rows = (long long)BH * d.d;          // decoder problems
    const csat_dims dr = rd_dims(d);
    CSAT_TRY(measure_hadamard_t<T>(d, rows_of_h, signs, K, V, w.Kc, w.Vc, w.prof, st, kBf16 ? w.KcHL : nullptr));
    auto attention = [&](T* Zdst, T* ZTdst) -> csat_status {      // (nothing here reads A~)
        if (attention_z_applies<T>(d, 2))
            return run_attention_z<T>(d, w, (const T*)Q, (const T*)w.KcHL, 2, false, (const T*)w.Vc, false, Zdst, ZTdst, st);
        {
            Timed tm(w, CSAT_K_LAYOUT, st);
            CSAT_TRY(transpose_pack<T>((const T*)w.Vc, (T*)w.VcT, w.ldm, BH, d.m, d.d, st));
        }
        return run_attention<T>(d, w, (const T*)Q, (const T*)w.Kc, (const T*)w.VcT, w.A, w.ldy, (T*)w.R, Zdst, true, st, ZTdst);
    };
    if (iters == 0) {
        CSAT_TRY(attention((T*)C, (T*)nullptr));
        if (Z) HIP_TRY(hipMemcpyAsync(Z, C, (size_t)BH * d.n * d.d * sizeof(T), hipMemcpyDeviceToDevice, st));
        return CSAT_OK;
    }
    const long long ldzt = kBf16 ? 2 * w.ldn : w.ldn;
    CSAT_TRY(fill_zero(x.ZT, (size_t)rows * ldzt * sizeof(T), st));
    CSAT_TRY(attention((T*)Z, (T*)x.ZT));
    int N = 1, logN = 0;
    while (N < d.n) { N *= 2; ++logN; }
    float scale = 1.f / sqrtf((float)d.m);
    if (kBf16) scale = bf2f_host(f2bf_host(scale));
    {
        const size_t lds_bytes = (size_t)(fwht_pad(N) + 1) * 4;
        const long long cap = (long long)cu_count() * 16;
        const dim3 grid((unsigned)(rows < cap ? rows : cap));
        Timed tm(w, CSAT_K_MEASURE, st);
#define CSAT_MEASURE_COLUMNS(NT_)                                                                                       \
    do {                                                                                                              \
        HIP_TRY(hipFuncSetAttribute((const void*)measure_columns_hadamard_kernel<T, NT_>,                             \
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes));                     \
        hipLaunchKernelGGL((measure_columns_hadamard_kernel<T, NT_>), grid, dim3(NT_), lds_bytes, st, (const T*)x.ZT,  \
                           ldzt, kBf16 ? w.ldn : 0ll, rows_of_h, signs, wr.A, wr.ldy, rows, d.n, d.m, N, logN, scale);  \
    } while (0)
        if (N <= 2048) CSAT_MEASURE_COLUMNS(256);
        else if (N <= 4096) CSAT_MEASURE_COLUMNS(512);
        else CSAT_MEASURE_COLUMNS(1024);
#undef CSAT_MEASURE_COLUMNS
        HIP_TRY(hipGetLastError());
    }
    CSAT_TRY(hadamard_t<T>(dr, wr, wr.A, wr.ldy, rows_of_h, signs, lambda, mu, iters, x.Xout, nullptr, nullptr, st));
    {   // C[b,h,j,k] = decoded column k at token j
        Timed tm(w, CSAT_K_SYNTHESIS, st);
        dim3 grid((unsigned)((d.d + 31) / 32), (unsigned)((d.n + 31) / 32), (unsigned)BH);
        hipLaunchKernelGGL((transpose_cast_kernel<T>), grid, dim3(32, 8), 0, st, x.Xout, (T*)C, d.d, d.n);
        HIP_TRY(hipGetLastError());
    }
    return CSAT_OK;
}

csat_status check_ws(void* ctx, const csat_dims* dims, void* workspace, size_t workspace_bytes, Workspace* w) {
    if (!workspace) return CSAT_ERR_WORKSPACE;
    if (!aligned16(workspace)) return CSAT_ERR_ALIGN;
    *w = carve(*dims, (char*)workspace);
    w->prof = &static_cast<Context*>(ctx)->prof;
    return workspace_bytes >= w->bytes ? CSAT_OK : CSAT_ERR_WORKSPACE;
}

// The transform-based decoder keeps a row's transform buffer and measurements in LDS: checked by the entry
// points before anything is launched (hadamard_t computes the same sizes for its launch).
bool hadamard_fits_lds(int n, int m) {
    int N = 1;
    while (N < n) N *= 2;
    const bool in_regs = N >= 512 && hadamard_choice() != 1;
    const size_t need = in_regs ? (size_t)(fwht_pad(N) + 1 + 2 * m) * 4 : ista_hadamard_lds_bytes(N, m);
    return need <= kLdsPerWorkgroup;
}

// Scratch of csat_forward_static: the workspace of a small problem, held in the code object's own device memory
// so that the call allocates nothing.  Every device the library is used on holds its own copy until the process ends.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's copy of `scratch` (looked up once per device, with that device current).
csat_status static_scratch(void** out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return CSAT_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return CSAT_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return CSAT_OK;
}

}  // namespace

extern "C" {

csat_status csat_create(void** ctx) {
    if (!ctx) return CSAT_ERR_NULL;
    Context* c = new (std::nothrow) Context{kMagic, {}};
    if (!c) return CSAT_ERR_PARAM;
    *ctx = c;
    return CSAT_OK;
}

csat_status csat_destroy(void* ctx) {
    CSAT_TRY(check_ctx(ctx));
    Context* c = static_cast<Context*>(ctx);
    c->magic = 0;
    c->prof.clear();
    delete c;
    return CSAT_OK;
}

const char* csat_status_string(csat_status s) {
    switch (s) {
        case CSAT_OK: return "ok";
        case CSAT_ERR_NULL: return "a required pointer is NULL";
        case CSAT_ERR_SHAPE: return "bad shape (non-positive dimension, m > n, d not a multiple of 8, or B*H > 65535)";
        case CSAT_ERR_DTYPE: return "unsupported dtype";
        case CSAT_ERR_ALIGN: return "pointer not 16-byte aligned";
        case CSAT_ERR_WORKSPACE: return "workspace missing or too small";
        case CSAT_ERR_PARAM: return "bad parameter (lambda < 0, step <= 0, iters < 0, or invalid context)";
        case CSAT_ERR_HIP: return "HIP runtime error";
        case CSAT_ERR_TIMEOUT: return "the decoder's bounded wait gave up; the outputs of that call are invalid";
    }
    return "unknown status";
}

csat_status csat_workspace_bytes(const csat_dims* dims, int iters, size_t* bytes) {
    CSAT_TRY(check_dims(dims));
    if (!bytes) return CSAT_ERR_NULL;
    if (iters < 0) return CSAT_ERR_PARAM;
    size_t total = carve(*dims, nullptr).bytes;
    if (dims->n_q == dims->n) {   // room for the column-wise decode as well
        const Workspace wr = carve(rd_dims(*dims), nullptr);
        total += wr.bytes + carve_rd_extra(*dims, wr, nullptr).bytes;
    }
    *bytes = total;
    return CSAT_OK;
}

// Word k of the SplitMix64 sequence started at `seed` (the state advances by a fixed odd constant, so any word
// can be formed on its own), then its output mix.
static inline uint64_t phi_word(uint64_t seed, uint64_t k) {
    uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

csat_status csat_phi_fill(int kind, unsigned long long seed, int m, int n, float* phi_host) {
    if (!phi_host) return CSAT_ERR_NULL;
    if (m <= 0 || n <= 0) return CSAT_ERR_SHAPE;
    if (kind != CSAT_PHI_GAUSSIAN && kind != CSAT_PHI_RADEMACHER) return CSAT_ERR_PARAM;
    const double scale = 1.0 / std::sqrt((double)m), two_pi = 6.283185307179586476925286766559;
    const long long total = (long long)m * n;
    for (long long i = 0; i < total; ++i) {
        const uint64_t w1 = phi_word(seed, 2 * (uint64_t)i), w2 = phi_word(seed, 2 * (uint64_t)i + 1);
        double v;
        if (kind == CSAT_PHI_RADEMACHER) {
            v = (w1 >> 63) ? -1.0 : 1.0;
        } else {      // Box-Muller: u1 in (0, 1], u2 in [0, 1), 53 bits each
            const double u1 = ((double)(w1 >> 11) + 1.0) * 0x1p-53, u2 = (double)(w2 >> 11) * 0x1p-53;
            v = std::sqrt(-2.0 * std::log(u1)) * std::cos(two_pi * u2);
        }
        phi_host[i] = (float)(v * scale);
    }
    return CSAT_OK;
}

csat_status csat_phi_opnorm2(const float* phi, int m, int n, double* L) {
    if (!phi || !L) return CSAT_ERR_NULL;
    if (m <= 0 || n <= 0) return CSAT_ERR_SHAPE;
    // power iteration on G = Phi Phi^T (m x m, formed once in double; rows of G shared out over host threads,
    // every entry summed in the same order whatever the thread count)
    std::vector<double> G((size_t)m * m, 0.0);
    unsigned hw = std::thread::hardware_concurrency();
    const int nthreads = (int)std::max(1u, std::min(hw ? hw : 1u, std::min(16u, (unsigned)m)));
    auto gram_rows = [&](int t) {
        constexpr int JB = 8;                      // rows of Phi kept hot against row i
        for (int i = t; i < m; i += nthreads) {
            const float* a = phi + (size_t)i * n;
            for (int j0 = i; j0 < m; j0 += JB) {
                const int jn = std::min(JB, m - j0);
                double s[JB] = {};
                for (int k = 0; k < n; ++k) {
                    const double ak = (double)a[k];
                    for (int jj = 0; jj < jn; ++jj) s[jj] += ak * (double)phi[(size_t)(j0 + jj) * n + k];
                }
                for (int jj = 0; jj < jn; ++jj) G[(size_t)i * m + j0 + jj] = s[jj];
            }
        }
    };
    if (nthreads == 1) {
        gram_rows(0);
    } else {
        std::vector<std::thread> pool;
        for (int t = 0; t < nthreads; ++t) pool.emplace_back(gram_rows, t);
        for (auto& th : pool) th.join();
    }
    for (int i = 0; i < m; ++i)
        for (int j = i + 1; j < m; ++j) G[(size_t)j * m + i] = G[(size_t)i * m + j];
    std::vector<double> v(m), w(m);
    for (int i = 0; i < m; ++i) v[i] = 1.0 + 0.37 * std::sin(1.0 + 1.7 * i);   // generic start vector
    double lam = 0.0;
    for (int it = 0; it < 200000; ++it) {
        double nrm = 0.0;
        for (int i = 0; i < m; ++i) {
            double s = 0.0;
            const double* g = &G[(size_t)i * m];
            for (int j = 0; j < m; ++j) s += g[j] * v[j];
            w[i] = s;
            nrm += s * s;
        }
        nrm = std::sqrt(nrm);
        if (nrm == 0.0) { lam = 0.0; break; }
        double rq = 0.0, vv = 0.0;
        for (int i = 0; i < m; ++i) { rq += v[i] * w[i]; vv += v[i] * v[i]; }
        double newlam = rq / vv;
        for (int i = 0; i < m; ++i) v[i] = w[i] / nrm;
        bool done = std::fabs(newlam - lam) <= 1e-15 * std::fabs(newlam) && it > 8;
        lam = newlam;
        if (done) break;
    }
    *L = lam;
    return CSAT_OK;
}

csat_status csat_peak_copy(void* ctx, const void* src, void* dst, size_t bytes, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    if (!src || !dst) return CSAT_ERR_NULL;
    if (bytes == 0 || bytes % 16 != 0) return CSAT_ERR_SHAPE;
    if (!aligned16(src) || !aligned16(dst)) return CSAT_ERR_ALIGN;
    const long long words = (long long)(bytes / 16);
    const long long want = (words + 255) / 256;
    const unsigned grid = (unsigned)std::min<long long>(want, (long long)cu_count() * 16);
    hipLaunchKernelGGL(peak_copy_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, (const uint4*)src, (uint4*)dst,
                       words);
    HIP_TRY(hipGetLastError());
    return CSAT_OK;
}

csat_status csat_peak_mfma(void* ctx, float* out, size_t out_bytes, int iters, double* flops, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    if (!out || !flops) return CSAT_ERR_NULL;
    if (iters <= 0) return CSAT_ERR_PARAM;
    if (!aligned16(out)) return CSAT_ERR_ALIGN;
    const unsigned grid = (unsigned)cu_count() * 2;      // two wavefronts per SIMD
    if (out_bytes < (size_t)grid * 256 * sizeof(float)) return CSAT_ERR_WORKSPACE;
    hipLaunchKernelGGL(peak_mfma_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, out, iters);
    HIP_TRY(hipGetLastError());
    *flops = (double)grid * 4 * (double)iters * kPeakMfmaPerIter * kPeakMfmaFlopsEach;
    return CSAT_OK;
}

csat_status csat_peak_mfma_issue(void* ctx, float* out, size_t out_bytes, int iters, int valu_per_mfma, int lds_reads_per_mfma,
                                 double* flops, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    if (!out || !flops) return CSAT_ERR_NULL;
    if (iters <= 0) return CSAT_ERR_PARAM;
    if (!aligned16(out)) return CSAT_ERR_ALIGN;
    const unsigned grid = (unsigned)cu_count();          // one wavefront per SIMD
    if (out_bytes < (size_t)grid * 256 * sizeof(float)) return CSAT_ERR_WORKSPACE;
    auto launch = [&](auto kernel) -> csat_status {
        HIP_TRY(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPeakIssueLdsBytes));
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), kPeakIssueLdsBytes, (hipStream_t)stream, out, iters);
        HIP_TRY(hipGetLastError());
        return CSAT_OK;
    };
    const int key = valu_per_mfma * 10 + lds_reads_per_mfma;
    switch (key) {
#define CSAT_ISSUE_CASE(KV, KL) case KV * 10 + KL: CSAT_TRY(launch(peak_issue_kernel<KV, KL>)); break;
        CSAT_ISSUE_CASE(0, 0) CSAT_ISSUE_CASE(3, 0) CSAT_ISSUE_CASE(6, 0) CSAT_ISSUE_CASE(9, 0) CSAT_ISSUE_CASE(12, 0)
        CSAT_ISSUE_CASE(0, 1) CSAT_ISSUE_CASE(3, 1) CSAT_ISSUE_CASE(6, 1) CSAT_ISSUE_CASE(0, 2)
#undef CSAT_ISSUE_CASE
        default: return CSAT_ERR_PARAM;
    }
    *flops = (double)grid * 4 * (double)iters * 8 * kPeakMfmaFlopsEach;
    return CSAT_OK;
}

csat_status csat_profile_enable(void* ctx, int on) {
    CSAT_TRY(check_ctx(ctx));
    Profiler& p = static_cast<Context*>(ctx)->prof;
    p.clear();
    p.on = on != 0;
    return CSAT_OK;
}

csat_status csat_profile_decoder_kernel(void* ctx, int* kernel) {
    CSAT_TRY(check_ctx(ctx));
    if (!kernel) return CSAT_ERR_NULL;
    *kernel = static_cast<Context*>(ctx)->decoder_kernel;
    return CSAT_OK;
}

csat_status csat_profile_launch_form(void* ctx, int form, int* value) {
    CSAT_TRY(check_ctx(ctx));
    if (!value) return CSAT_ERR_NULL;
    if (form < 0 || form >= CSAT_FORM_COUNT) return CSAT_ERR_PARAM;
    *value = static_cast<Context*>(ctx)->forms[form];
    return CSAT_OK;
}

csat_status csat_profile_read(void* ctx, int kernel_id, double* total_ms, int* launches) {
    CSAT_TRY(check_ctx(ctx));
    if (!total_ms || !launches) return CSAT_ERR_NULL;
    if (kernel_id < 0 || kernel_id >= CSAT_K_COUNT) return CSAT_ERR_PARAM;
    Profiler& p = static_cast<Context*>(ctx)->prof;
    double tot = 0.0;
    int cnt = 0;
    for (auto& s : p.spans) {
        if (s.kid != kernel_id) continue;
        float ms = 0.f;
        HIP_TRY(hipEventSynchronize(s.b));
        HIP_TRY(hipEventElapsedTime(&ms, s.a, s.b));
        tot += ms;
        ++cnt;
    }
    *total_ms = tot;
    *launches = cnt;
    return CSAT_OK;
}

#define DISPATCH(d, call_f32, call_bf16) ((d).dtype == CSAT_BF16 ? (call_bf16) : (call_f32))

csat_status csat_measure_kv(void* ctx, const csat_dims* dims, const void* PhiK, const void* PhiV, const void* K,
                            const void* V, void* Kc, void* Vc, void* workspace, size_t workspace_bytes,
                            void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!PhiK || !PhiV || !K || !V || !Kc || !Vc) return CSAT_ERR_NULL;
    if (!aligned16(PhiK) || !aligned16(PhiV) || !aligned16(K) || !aligned16(V) || !aligned16(Kc) || !aligned16(Vc))
        return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, measure_t<float>(*dims, w, PhiK, PhiV, K, V, Kc, Vc, st),
                    measure_t<bf16_t>(*dims, w, PhiK, PhiV, K, V, Kc, Vc, st));
}

csat_status csat_measure(void* ctx, const csat_dims* dims, const void* Phi, const void* K, const void* V,
                         void* Kc, void* Vc, void* workspace, size_t workspace_bytes, void* stream) {
    return csat_measure_kv(ctx, dims, Phi, Phi, K, V, Kc, Vc, workspace, workspace_bytes, stream);
}

csat_status csat_compressed_attention(void* ctx, const csat_dims* dims, const void* Q, const void* Kc,
                                      const void* Vc, float* A, void* Z, void* workspace, size_t workspace_bytes,
                                      void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!Q || !Kc || !Vc || !Z) return CSAT_ERR_NULL;
    if (!aligned16(Q) || !aligned16(Kc) || !aligned16(Vc) || !aligned16(A) || !aligned16(Z)) return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, attention_t<float>(*dims, w, Q, Kc, Vc, A, Z, st),
                    attention_t<bf16_t>(*dims, w, Q, Kc, Vc, A, Z, st));
}

csat_status csat_recover(void* ctx, const csat_dims* dims, const float* Y, const void* Phi, float lambda,
                         float step, int iters, float* X, const void* V, void* C, void* workspace,
                         size_t workspace_bytes, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!Y || !Phi) return CSAT_ERR_NULL;
    if (!X && !(V && C)) return CSAT_ERR_NULL;
    if (!(lambda >= 0.f) || !(step > 0.f) || !std::isfinite(step) || !std::isfinite(lambda) || iters < 0)
        return CSAT_ERR_PARAM;
    if (!aligned16(Y) || !aligned16(Phi) || !aligned16(X) || !aligned16(V) || !aligned16(C)) return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, recover_t<float>(*dims, w, Y, Phi, lambda, step, iters, X, V, C, st),
                    recover_t<bf16_t>(*dims, w, Y, Phi, lambda, step, iters, X, V, C, st));
}

csat_status csat_forward(void* ctx, const csat_dims* dims, const void* Q, const void* K, const void* V,
                         const void* Phi, float lambda, float step, int iters, void* C, void* Z, float* X,
                         void* workspace, size_t workspace_bytes, void* stream) {
    return csat_forward_kv(ctx, dims, Q, K, V, Phi, Phi, lambda, step, iters, C, Z, X, workspace, workspace_bytes,
                           stream);
}

csat_status csat_forward_kv(void* ctx, const csat_dims* dims, const void* Q, const void* K, const void* V,
                            const void* PhiK, const void* Phi, float lambda, float step, int iters, void* C,
                            void* Z, float* X, void* workspace, size_t workspace_bytes, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!Q || !K || !V || !PhiK || !Phi || !C) return CSAT_ERR_NULL;
    if (!aligned16(PhiK)) return CSAT_ERR_ALIGN;
    if (!(lambda >= 0.f) || !(step > 0.f) || !std::isfinite(step) || !std::isfinite(lambda) || iters < 0)
        return CSAT_ERR_PARAM;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(Phi) || !aligned16(C) || !aligned16(Z) ||
        !aligned16(X))
        return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, forward_t<float>(*dims, w, Q, K, V, PhiK, Phi, lambda, step, iters, C, Z, X, st),
                    forward_t<bf16_t>(*dims, w, Q, K, V, PhiK, Phi, lambda, step, iters, C, Z, X, st));
}

csat_status csat_forward_rd(void* ctx, const csat_dims* dims, const void* Q, const void* K, const void* V,
                            const void* Phi, float lambda, float step, int iters, void* C, void* Z,
                            void* workspace, size_t workspace_bytes, void* stream) {
    return csat_forward_rd_kv(ctx, dims, Q, K, V, Phi, Phi, lambda, step, iters, C, Z, workspace, workspace_bytes,
                              stream);
}

csat_status csat_forward_rd_kv(void* ctx, const csat_dims* dims, const void* Q, const void* K, const void* V,
                               const void* PhiK, const void* Phi, float lambda, float step, int iters, void* C,
                               void* Z, void* workspace, size_t workspace_bytes, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (dims->n_q != dims->n) return CSAT_ERR_SHAPE;
    if (!Q || !K || !V || !PhiK || !Phi || !C) return CSAT_ERR_NULL;
    if (!aligned16(PhiK)) return CSAT_ERR_ALIGN;
    if (!(lambda >= 0.f) || !(step > 0.f) || !std::isfinite(step) || !std::isfinite(lambda) || iters < 0)
        return CSAT_ERR_PARAM;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(Phi) || !aligned16(C) || !aligned16(Z))
        return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    const csat_dims dr = rd_dims(*dims);
    Workspace wr = carve(dr, (char*)workspace + w.bytes);
    wr.prof = w.prof;
    wr.Status = w.Status;      // one status block per workspace: the column-wise decoder reports there as well
    const RdExtra x = carve_rd_extra(*dims, wr, (char*)workspace + w.bytes + wr.bytes);
    if (workspace_bytes < w.bytes + wr.bytes + x.bytes) return CSAT_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, forward_rd_t<float>(*dims, w, wr, x, Q, K, V, PhiK, Phi, lambda, step, iters, C, Z, st),
                    forward_rd_t<bf16_t>(*dims, w, wr, x, Q, K, V, PhiK, Phi, lambda, step, iters, C, Z, st));
}

csat_status csat_lista_workspace_bytes(const csat_dims* dims, int iters, size_t* bytes) {
    CSAT_TRY(check_dims(dims));
    if (!bytes) return CSAT_ERR_NULL;
    if (iters < 0) return CSAT_ERR_PARAM;
    const Workspace w = carve(*dims, nullptr);
    *bytes = w.bytes + carve_lista(*dims, w, nullptr).bytes;
    return CSAT_OK;
}

csat_status csat_recover_lista(void* ctx, const csat_dims* dims, const float* Y, const void* S, const void* Bw,
                               const float* thetas, int iters, float* X, const void* V, void* C, void* workspace,
                               size_t workspace_bytes, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!Y || !S || !Bw) return CSAT_ERR_NULL;
    if (!X && !(V && C)) return CSAT_ERR_NULL;
    if (iters < 0 || (iters > 0 && !thetas)) return iters < 0 ? CSAT_ERR_PARAM : CSAT_ERR_NULL;
    for (int t = 0; t < iters; ++t)
        if (!(thetas[t] >= 0.f) || !std::isfinite(thetas[t])) return CSAT_ERR_PARAM;
    if (!aligned16(Y) || !aligned16(S) || !aligned16(Bw) || !aligned16(X) || !aligned16(V) || !aligned16(C))
        return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    const ListaExtra x = carve_lista(*dims, w, (char*)workspace + w.bytes);
    if (workspace_bytes < w.bytes + x.bytes) return CSAT_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, lista_t<float>(*dims, w, x, Y, S, Bw, thetas, iters, X, V, C, st),
                    lista_t<bf16_t>(*dims, w, x, Y, S, Bw, thetas, iters, X, V, C, st));
}

csat_status csat_omp_workspace_bytes(const csat_dims* dims, int k, size_t* bytes) {
    CSAT_TRY(check_dims(dims));
    if (!bytes) return CSAT_ERR_NULL;
    if (k < 0 || k > kOmpMaxPicks || k > dims->m) return CSAT_ERR_PARAM;
    if (dims->m > kOmpMaxM) return CSAT_ERR_SHAPE;
    const Workspace w = carve(*dims, nullptr);
    *bytes = w.bytes + carve_omp(*dims, w, k, nullptr).bytes;
    return CSAT_OK;
}

csat_status csat_recover_omp(void* ctx, const csat_dims* dims, const float* Y, const void* Phi, int k, float* X,
                             int* picks, const void* V, void* C, void* workspace, size_t workspace_bytes,
                             void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!Y || !Phi) return CSAT_ERR_NULL;
    if (!X && !picks && !(V && C)) return CSAT_ERR_NULL;
    if (k < 0 || k > kOmpMaxPicks || k > dims->m) return CSAT_ERR_PARAM;
    if (dims->m > kOmpMaxM) return CSAT_ERR_SHAPE;
    if (!aligned16(Y) || !aligned16(Phi) || !aligned16(X) || !aligned16(picks) || !aligned16(V) || !aligned16(C))
        return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    const OmpExtra x = carve_omp(*dims, w, k, (char*)workspace + w.bytes);
    if (workspace_bytes < w.bytes + x.bytes) return CSAT_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, omp_t<float>(*dims, w, x, Y, Phi, k, X, picks, V, C, st),
                    omp_t<bf16_t>(*dims, w, x, Y, Phi, k, X, picks, V, C, st));
}

csat_status csat_recover_hadamard(void* ctx, const csat_dims* dims, const float* Y, const int* rows_of_h,
                                  const signed char* signs, float lambda, float step, int iters, float* X,
                                  const void* V, void* C, void* workspace, size_t workspace_bytes, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!Y || !rows_of_h || !signs) return CSAT_ERR_NULL;
    if (!X && !(V && C)) return CSAT_ERR_NULL;
    if (!(lambda >= 0.f) || !(step > 0.f) || !std::isfinite(step) || !std::isfinite(lambda) || iters < 0)
        return CSAT_ERR_PARAM;
    if (dims->n > kFwhtMaxN) return CSAT_ERR_SHAPE;
    if (!aligned16(Y) || !aligned16(X) || !aligned16(V) || !aligned16(C)) return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    if (!hadamard_fits_lds(dims->n, dims->m)) return CSAT_ERR_SHAPE;
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, hadamard_t<float>(*dims, w, Y, dims->m, rows_of_h, signs, lambda, step, iters, X, V, C, st),
                    hadamard_t<bf16_t>(*dims, w, Y, dims->m, rows_of_h, signs, lambda, step, iters, X, V, C, st));
}

csat_status csat_forward_hadamard(void* ctx, const csat_dims* dims, const void* Q, const void* K, const void* V,
                                  const int* rows_of_h, const signed char* signs, float lambda, float step, int iters,
                                  void* C, void* Z, float* X, void* workspace, size_t workspace_bytes, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!Q || !K || !V || !rows_of_h || !signs || !C) return CSAT_ERR_NULL;
    if (!(lambda >= 0.f) || !(step > 0.f) || !std::isfinite(step) || !std::isfinite(lambda) || iters < 0)
        return CSAT_ERR_PARAM;
    if (dims->n > kFwhtMaxN) return CSAT_ERR_SHAPE;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(C) || !aligned16(Z) || !aligned16(X))
        return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    if (iters > 0 && !hadamard_fits_lds(dims->n, dims->m)) return CSAT_ERR_SHAPE;
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims,
                    forward_hadamard_t<float>(*dims, w, Q, K, V, rows_of_h, signs, lambda, step, iters, C, Z, X, st),
                    forward_hadamard_t<bf16_t>(*dims, w, Q, K, V, rows_of_h, signs, lambda, step, iters, C, Z, X, st));
}

csat_status csat_forward_rd_hadamard(void* ctx, const csat_dims* dims, const void* Q, const void* K, const void* V,
                                     const int* rows_of_h, const signed char* signs, float lambda, float step,
                                     int iters, void* C, void* Z, void* workspace, size_t workspace_bytes,
                                     void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (dims->n_q != dims->n || dims->n > kFwhtMaxN) return CSAT_ERR_SHAPE;
    if (!Q || !K || !V || !rows_of_h || !signs || !C) return CSAT_ERR_NULL;
    if (!(lambda >= 0.f) || !(step > 0.f) || !std::isfinite(step) || !std::isfinite(lambda) || iters < 0)
        return CSAT_ERR_PARAM;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(C) || !aligned16(Z)) return CSAT_ERR_ALIGN;
    Workspace w;
    OptionScope scope(ctx);
    CSAT_TRY(check_ws(ctx, dims, workspace, workspace_bytes, &w));
    const csat_dims dr = rd_dims(*dims);
    Workspace wr = carve(dr, (char*)workspace + w.bytes);
    wr.prof = w.prof;
    wr.Status = w.Status;
    const RdExtra x = carve_rd_extra(*dims, wr, (char*)workspace + w.bytes + wr.bytes);
    if (workspace_bytes < w.bytes + wr.bytes + x.bytes) return CSAT_ERR_WORKSPACE;
    if (iters > 0 && !hadamard_fits_lds(dims->n, dims->m)) return CSAT_ERR_SHAPE;
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims,
                    forward_rd_hadamard_t<float>(*dims, w, wr, x, Q, K, V, rows_of_h, signs, lambda, step, iters, C, Z, st),
                    forward_rd_hadamard_t<bf16_t>(*dims, w, wr, x, Q, K, V, rows_of_h, signs, lambda, step, iters, C, Z, st));
}

csat_status csat_measure_hadamard(void* ctx, const csat_dims* dims, const int* rows_of_h, const signed char* signs,
                                  const void* K, const void* V, void* Kc, void* Vc, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!rows_of_h || !signs || !K || !V || !Kc || !Vc) return CSAT_ERR_NULL;
    if (dims->n > kFwhtMaxN) return CSAT_ERR_SHAPE;
    if (!aligned16(K) || !aligned16(V) || !aligned16(Kc) || !aligned16(Vc)) return CSAT_ERR_ALIGN;
    Profiler* prof = &static_cast<Context*>(ctx)->prof;
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, measure_hadamard_t<float>(*dims, rows_of_h, signs, K, V, Kc, Vc, prof, st),
                    measure_hadamard_t<bf16_t>(*dims, rows_of_h, signs, K, V, Kc, Vc, prof, st));
}

csat_status csat_set_option(void* ctx, int key, int value) {
    CSAT_TRY(check_ctx(ctx));
    if (key < 0 || key >= CSAT_OPT_COUNT) return CSAT_ERR_PARAM;
    static_cast<Context*>(ctx)->opt.v[key] = value;
    return CSAT_OK;
}

csat_status csat_decoder_status(void* ctx, const void* workspace, void* stream) {
    CSAT_TRY(check_ctx(ctx));
    if (!aligned16(workspace)) return CSAT_ERR_ALIGN;
    void* base = const_cast<void*>(workspace);
    if (!base) CSAT_TRY(static_scratch(&base));          // NULL: the scratch of csat_forward_static on this device
    int word = 0;
    HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
    // the status block is the first piece of every carving, word 0 the decoder's error flag
    HIP_TRY(hipMemcpy(&word, base, sizeof(int), hipMemcpyDeviceToHost));
    return word == 0 ? CSAT_OK : CSAT_ERR_TIMEOUT;
}

csat_status csat_static_workspace_bytes(size_t* bytes) {
    if (!bytes) return CSAT_ERR_NULL;
    *bytes = kStaticScratchBytes;
    return CSAT_OK;
}

csat_status csat_forward_static(void* ctx, const csat_dims* dims, const void* Q, const void* K, const void* V,
                                const void* Phi, float lambda, float step, int iters, void* C, void* Z, float* X,
                                void* stream) {
    CSAT_TRY(check_ctx(ctx));
    CSAT_TRY(check_dims(dims));
    if (!Q || !K || !V || !Phi || !C) return CSAT_ERR_NULL;
    if (!(lambda >= 0.f) || !(step > 0.f) || !std::isfinite(step) || !std::isfinite(lambda) || iters < 0)
        return CSAT_ERR_PARAM;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(Phi) || !aligned16(C) || !aligned16(Z) ||
        !aligned16(X))
        return CSAT_ERR_ALIGN;
    OptionScope scope(ctx);
    // the row-wise block needs the main carving only
    if (carve(*dims, nullptr).bytes > kStaticScratchBytes) return CSAT_ERR_WORKSPACE;
    void* base = nullptr;
    CSAT_TRY(static_scratch(&base));
    Workspace w = carve(*dims, (char*)base);
    Profiler off;            // event creation allocates: launches of this call are never bracketed
    w.prof = &off;
    hipStream_t st = (hipStream_t)stream;
    return DISPATCH(*dims, forward_t<float>(*dims, w, Q, K, V, Phi, Phi, lambda, step, iters, C, Z, X, st),
                    forward_t<bf16_t>(*dims, w, Q, K, V, Phi, Phi, lambda, step, iters, C, Z, X, st));
}

}  // extern "C"

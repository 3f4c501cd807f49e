// Launchers of the kernel families that are compiled as translation units of their own (one per
// instantiation group, so that they build in parallel and a change to one family recompiles only it).
// Each returns the HIP error of its launch.
#pragma once
#include <hip/hip_runtime.h>

namespace csat {

struct IstaFusedArgs;
struct IstaResidentArgs;
struct IstaResidentF32Args;
struct AttentionArgs;
struct AttentionZArgs;
struct ListaSupportArgs;

// Fused ISTA decoder for MT tiles of m (csat_ista_fused.h, csat_ista_fused2.h).  variant: 0 dense state, 1 sparse
// state, 2 one 32-row tile per workgroup (thin); 3 and 4: dense and sparse state on the two-chunk schedule; 6:
// one 32-row tile shared by eight wavefronts (csat_ista_coop.h, MT <= 13).  One function per MT, defined by csat_tu_ista_fused.hip
// compiled with -DCSAT_TU_MT=<MT>.
#define CSAT_DECLARE_FUSED(MT_) \
    hipError_t ista_fused_launch_mt##MT_(int variant, const IstaFusedArgs& a, unsigned grid, hipStream_t st);
CSAT_DECLARE_FUSED(1) CSAT_DECLARE_FUSED(2) CSAT_DECLARE_FUSED(3) CSAT_DECLARE_FUSED(4) CSAT_DECLARE_FUSED(5)
CSAT_DECLARE_FUSED(6) CSAT_DECLARE_FUSED(7) CSAT_DECLARE_FUSED(8) CSAT_DECLARE_FUSED(9) CSAT_DECLARE_FUSED(10)
CSAT_DECLARE_FUSED(11) CSAT_DECLARE_FUSED(12) CSAT_DECLARE_FUSED(13) CSAT_DECLARE_FUSED(14) CSAT_DECLARE_FUSED(15)
CSAT_DECLARE_FUSED(16)
#undef CSAT_DECLARE_FUSED

// ISTA decoder with Phi in LDS and the iterate in registers (csat_ista_resident.h): one function per instance
// (tiles of m, chunks of n), defined by csat_tu_ista_resident.hip.
#define CSAT_RESIDENT_INSTANCES(F)                                                                                       \
    F(1, 3) F(2, 3) F(3, 3) F(4, 3) F(5, 3) F(6, 3) F(7, 3) F(8, 3) F(1, 5) F(2, 5) F(3, 5) F(4, 5) F(5, 5) F(6, 5) F(7, 5) \
    F(8, 5) F(1, 7) F(2, 7) F(3, 7) F(4, 7) F(5, 7) F(6, 7) F(7, 7) F(8, 7) F(1, 9) F(2, 9) F(3, 9) F(4, 9) F(5, 9) F(6, 9) \
    F(7, 9) F(8, 9) F(1, 12) F(2, 12) F(3, 12) F(4, 12) F(5, 12) F(6, 12) F(1, 16) F(2, 16) F(3, 16) F(4, 16) F(5, 16)
#define CSAT_DECLARE_RESIDENT(MT_, NCT_) hipError_t ista_resident_launch_##MT_##_##NCT_(const IstaResidentArgs& a, unsigned grid, hipStream_t st);
CSAT_RESIDENT_INSTANCES(CSAT_DECLARE_RESIDENT)
#undef CSAT_DECLARE_RESIDENT
hipError_t ista_resident_f32_launch(int MT, const IstaResidentF32Args& a, unsigned grid, hipStream_t st);

// Compressed attention in one kernel (csat_attention.h) for mt_total tiles of m; `single`: all of K~ is kept in
// registers and LDS at once.  One function per element type and per "with the output product", defined by
// csat_tu_attention.hip compiled with -DCSAT_TU_BF16=<0|1> -DCSAT_TU_Z=<0|1>.
hipError_t attention_fused_launch_f32_z0(int mt_total, bool single, const AttentionArgs& a, unsigned grid, size_t lds_bytes, hipStream_t st);
hipError_t attention_fused_launch_f32_z1(int mt_total, bool single, const AttentionArgs& a, unsigned grid, size_t lds_bytes, hipStream_t st);
hipError_t attention_fused_launch_bf16_z0(int mt_total, bool single, const AttentionArgs& a, unsigned grid, size_t lds_bytes, hipStream_t st);
hipError_t attention_fused_launch_bf16_z1(int mt_total, bool single, const AttentionArgs& a, unsigned grid, size_t lds_bytes, hipStream_t st);
// ... with the output product from V~ as packed fragments (a.Vf), d = 64 (z2) or 128 (z3)
hipError_t attention_fused_launch_bf16_z2(int mt_total, bool single, const AttentionArgs& a, unsigned grid, size_t lds_bytes, hipStream_t st);
hipError_t attention_fused_launch_bf16_z3(int mt_total, bool single, const AttentionArgs& a, unsigned grid, size_t lds_bytes, hipStream_t st);

// Compressed attention without A~ (csat_attention_z.h): bf16, d a multiple of 32 up to 128; parts: 2 where K~ comes as
// its (hi | lo) pair; resident: all of a head's fragments in LDS.
hipError_t attention_z_launch(int d, int parts, bool resident, const AttentionZArgs& a, unsigned grid, size_t lds_bytes, hipStream_t st);

// The unrolled decoder over the support of its iterate (csat_support.h), n <= kListaSupportMaxN, a workgroup per four rows.
constexpr int kListaSupportMaxN = 4096;
hipError_t lista_support_launch(const ListaSupportArgs& a, unsigned grid, hipStream_t st);

}  // namespace csat

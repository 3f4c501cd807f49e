// Translation unit of the compressed attention without A~ (csat_attention_z.h).
#include "csat_attention_z.h"
#include "csat_launch.h"

namespace csat {

hipError_t attention_z_launch(int d, int parts, bool resident, const AttentionZArgs& a, unsigned grid, size_t lds_bytes, hipStream_t st) {
    auto launch = [&](auto kernel) -> hipError_t {
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * kAttnZWaves), lds_bytes, st, a);
        return hipGetLastError();
    };
#define CSAT_ATTN_Z(NZ_, PARTS_) (resident ? launch(attention_z_kernel<NZ_, PARTS_, true>) : launch(attention_z_kernel<NZ_, PARTS_, false>))
    switch (d / 32 * 4 + parts) {
        case 5: return CSAT_ATTN_Z(1, 1);
        case 6: return CSAT_ATTN_Z(1, 2);
        case 9: return CSAT_ATTN_Z(2, 1);
        case 10: return CSAT_ATTN_Z(2, 2);
        case 13: return CSAT_ATTN_Z(3, 1);
        case 14: return CSAT_ATTN_Z(3, 2);
        case 17: return CSAT_ATTN_Z(4, 1);
        case 18: return CSAT_ATTN_Z(4, 2);
    }
#undef CSAT_ATTN_Z
    return hipErrorInvalidValue;
}

}  // namespace csat

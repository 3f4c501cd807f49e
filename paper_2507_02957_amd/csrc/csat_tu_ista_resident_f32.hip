// Translation unit of the LDS-resident float ISTA decoder (csat_ista_resident.h).
#include "csat_ista_resident.h"
#include "csat_launch.h"

namespace csat {

hipError_t ista_resident_f32_launch(int MT, const IstaResidentF32Args& a, unsigned grid, hipStream_t st) {
    const size_t lds_bytes = ista_resident_f32_lds_bytes(MT, a.nct);
    auto launch = [&](auto kernel) -> hipError_t {
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), lds_bytes, st, a);
        return hipGetLastError();
    };
    switch (MT * 10 + ista_resident_f32_chunks(MT, a.nct)) {
        case 13: return launch(ista_resident_f32_kernel<1, 3>);
        case 16: return launch(ista_resident_f32_kernel<1, 6>);
        case 23: return launch(ista_resident_f32_kernel<2, 3>);
        case 32: return launch(ista_resident_f32_kernel<3, 2>);
        case 42: return launch(ista_resident_f32_kernel<4, 2>);
    }
    return hipErrorInvalidValue;
}

}  // namespace csat

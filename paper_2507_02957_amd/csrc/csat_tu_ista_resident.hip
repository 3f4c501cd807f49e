// Translation unit of one instance of the LDS-resident ISTA decoder: compile with -DCSAT_TU_MT=<tiles of m>
// -DCSAT_TU_NCT=<chunks of n>, the pairs of CSAT_RESIDENT_INSTANCES in csat_launch.h.
#include "csat_ista_resident.h"
#include "csat_launch.h"

#if !defined(CSAT_TU_MT) || !defined(CSAT_TU_NCT)
#error "compile with -DCSAT_TU_MT=<tiles of m> -DCSAT_TU_NCT=<chunks of n>"
#endif
#define CSAT_NAME2(a, b) ista_resident_launch_##a##_##b
#define CSAT_NAME(a, b) CSAT_NAME2(a, b)

namespace csat {

hipError_t CSAT_NAME(CSAT_TU_MT, CSAT_TU_NCT)(const IstaResidentArgs& a, unsigned grid, hipStream_t st) {
    const auto kernel = ista_resident_kernel<CSAT_TU_MT, CSAT_TU_NCT>;
    const size_t lds_bytes = ista_resident_lds_bytes(CSAT_TU_MT, CSAT_TU_NCT);
    const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), lds_bytes, st, a);
    return hipGetLastError();
}

}  // namespace csat

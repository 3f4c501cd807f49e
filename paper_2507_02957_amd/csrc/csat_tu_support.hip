// Translation unit of the decoders over the support of a sparse iterate (csat_support.h).
#include "csat_support.h"
#include "csat_launch.h"

namespace csat {

hipError_t lista_support_launch(const ListaSupportArgs& a, unsigned grid, hipStream_t st) {
    const size_t lds = (size_t)a.tiles_n * 32 * 16;
    auto launch = [&](auto kernel) -> hipError_t {
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), lds, st, a);
        return hipGetLastError();
    };
    const int regs = (a.n + 63) / 64;      // the smallest instance whose 64 R columns hold a row
#define CSAT_LISTA_SUPPORT(R_) if (regs <= R_) return launch(lista_support_kernel<R_>);
    CSAT_LISTA_SUPPORT(4) CSAT_LISTA_SUPPORT(8) CSAT_LISTA_SUPPORT(12) CSAT_LISTA_SUPPORT(16) CSAT_LISTA_SUPPORT(20)
    CSAT_LISTA_SUPPORT(26) CSAT_LISTA_SUPPORT(32) CSAT_LISTA_SUPPORT(40) CSAT_LISTA_SUPPORT(52) CSAT_LISTA_SUPPORT(64)
#undef CSAT_LISTA_SUPPORT
    return hipErrorInvalidValue;
}

}  // namespace csat

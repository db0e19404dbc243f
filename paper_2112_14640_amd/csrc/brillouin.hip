// Brillouin launches by precision; each precision is a translation unit of its own.
#include "kernels.h"

namespace dirac {

int launch_brillouin_fp64(const StencilArgs& a, hipStream_t st);
int launch_brillouin_fp32(const StencilArgs& a, hipStream_t st);
int launch_brillouin_bf16(const StencilArgs& a, hipStream_t st);

int launch_brillouin(const StencilArgs& a, hipStream_t st) {
    switch (a.prec) {
        case DIRAC_FP64: return launch_brillouin_fp64(a, st);
        case DIRAC_FP32: return launch_brillouin_fp32(a, st);
        case DIRAC_BF16: return launch_brillouin_bf16(a, st);
    }
    return DIRAC_EINVAL;
}

}  // namespace dirac

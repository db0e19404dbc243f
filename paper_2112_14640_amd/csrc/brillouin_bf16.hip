#include "brillouin_kernels.h"

namespace dirac {

int launch_brillouin_bf16(const StencilArgs& a, hipStream_t st) { return launch_prec<PrecBF16>(a, st); }

}  // namespace dirac

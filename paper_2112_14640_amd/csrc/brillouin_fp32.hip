#include "brillouin_kernels.h"

namespace dirac {

int launch_brillouin_fp32(const StencilArgs& a, hipStream_t st) { return launch_prec<PrecF32>(a, st); }

}  // namespace dirac

#include "brillouin_kernels.h"

namespace dirac {

int launch_brillouin_fp64(const StencilArgs& a, hipStream_t st) { return launch_prec<PrecF64>(a, st); }

}  // namespace dirac

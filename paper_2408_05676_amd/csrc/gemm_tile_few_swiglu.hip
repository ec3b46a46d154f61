// Gate/up projection of 17..80 rows with the SwiGLU epilogue: instantiations.
#include "gemm_tile_few.h"

namespace laser {

void launch_few_swiglu(const GemmTileArgs& t, bool f16, int ncu, hipStream_t stream) {
    if (f16) launch<GEPI_SWIGLU, true, true>(t, ncu, 1, 1, stream);
    else launch<GEPI_SWIGLU, true, false>(t, ncu, 1, 1, stream);
}

}  // namespace laser

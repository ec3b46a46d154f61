// Projections of 17..80 rows with a float output (QKV, O, down): instantiations.
#include "gemm_tile_few.h"

namespace laser {

int launch_few_f32(const GemmTileArgs& t, bool f16, int ncu, int want_split, int max_split, hipStream_t stream) {
    if (t.Xlo) return f16 ? launch<GEPI_F32, true, true>(t, ncu, want_split, max_split, stream) : launch<GEPI_F32, true, false>(t, ncu, want_split, max_split, stream);
    return f16 ? launch<GEPI_F32, false, true>(t, ncu, want_split, max_split, stream) : launch<GEPI_F32, false, false>(t, ncu, want_split, max_split, stream);
}

}  // namespace laser

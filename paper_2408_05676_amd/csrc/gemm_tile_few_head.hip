// Output head of 17..80 rows, two-entry lists (head.hip): the tiled product of one row tile with the statistics epilogue, 128
// columns a workgroup (250 workgroups at a vocabulary of 32000).
#include "gemm_tile_few.h"

namespace laser {

template <bool WF16>
static void go_rows(const GemmTileArgs& t, hipStream_t stream) {
    for_index<2, 6>([&](auto wmc) {
        constexpr int wm = decltype(wmc)::value;
        if ((t.M + 15) / 16 == wm) go<GEPI_HEAD2, false, WF16, wm, 2, 4>(t, 1, stream);
    });
}

void launch_few_head(const GemmTileArgs& t, bool f16, hipStream_t stream) {
    if (f16) go_rows<true>(t, stream);
    else go_rows<false>(t, stream);
}

}  // namespace laser

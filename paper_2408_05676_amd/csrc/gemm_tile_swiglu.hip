// Many-row gate/up projection with the SwiGLU epilogue: tile choice and instantiations.
#include "gemm_tile_plan.h"

namespace laser {

template <bool SPLIT, bool WF16>
static void go(const GemmTileArgs& t, int ncu, hipStream_t stream) {
    constexpr auto& shapes = [] () -> auto& { if constexpr (SPLIT) return kTileSplit; else return kTilePlain; }();
    constexpr int nv = !WF16 ? (SPLIT ? kTileSplitCommon : kTilePlainCommon) : (int)(sizeof(shapes) / sizeof(shapes[0]));
    const GemmTilePlan pl = gemm_tile_plan(shapes, nv, t, true, SPLIT, ncu, 1, 1);
    for_index<0, nv>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        if (pl.v == v) gemm_tile_go<GEPI_SWIGLU, SPLIT, WF16, shapes[v].wm, shapes[v].wn>(t, 1, stream);
    });
}

void launch_tile_swiglu(const GemmTileArgs& t, bool f16, int ncu, hipStream_t stream) {
    if (!on_16_byte_grid(t.W) || (!f16 && (size_t)t.N * t.Kd * 2 >= (3ull << 30))) return launch_off_grid_swiglu(t, stream);
    if (t.Xlo) { if (f16) go<true, true>(t, ncu, stream); else go<true, false>(t, ncu, stream); }
    else { if (f16) go<false, true>(t, ncu, stream); else go<false, false>(t, ncu, stream); }
}

}  // namespace laser

// Many-row projections with a float output (QKV, O, down): tile choice and instantiations.
#include "gemm_tile_plan.h"

namespace laser {

template <bool SPLIT, bool WF16>
static int go(const GemmTileArgs& t, int ncu, int want_split, int max_split, hipStream_t stream) {
    constexpr auto& shapes = [] () -> auto& { if constexpr (SPLIT) return kTileSplit; else return kTilePlain; }();
    constexpr int nv = !WF16 ? (SPLIT ? kTileSplitCommon : kTilePlainCommon) : (int)(sizeof(shapes) / sizeof(shapes[0]));
    const GemmTilePlan pl = gemm_tile_plan(shapes, nv, t, false, SPLIT, ncu, want_split, max_split);
    for_index<0, nv>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        if (pl.v == v) gemm_tile_go<GEPI_F32, SPLIT, WF16, shapes[v].wm, shapes[v].wn>(t, pl.S, stream);
    });
    return pl.S;
}

int launch_tile_f32(const GemmTileArgs& t, bool f16, int ncu, int want_split, int max_split, hipStream_t stream) {
    if (!on_16_byte_grid(t.W)) return launch_off_grid_f32(t, ncu, want_split, max_split, stream);
    if (t.Xlo) return f16 ? go<true, true>(t, ncu, want_split, max_split, stream) : go<true, false>(t, ncu, want_split, max_split, stream);
    return f16 ? go<false, true>(t, ncu, want_split, max_split, stream) : go<false, false>(t, ncu, want_split, max_split, stream);
}

}  // namespace laser

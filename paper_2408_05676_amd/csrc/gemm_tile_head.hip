// Many-row output head: the tiled product with the statistics epilogue.
#include "gemm_tile_plan.h"

namespace laser {

template <int EPI, bool WF16>
static void go(const GemmTileArgs& t, int ncu, hipStream_t stream) {
    constexpr int nv = EPI == GEPI_HEAD2 && WF16 ? (int)(sizeof(kTileHead) / sizeof(kTileHead[0])) : kTileHeadCommon;
    const GemmTilePlan pl = gemm_tile_plan(kTileHead, nv, t, false, false, ncu, 1, 1);
    for_index<0, nv>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        if (pl.v == v) gemm_tile_go<EPI, false, WF16, kTileHead[v].wm, kTileHead[v].wn>(t, 1, stream);
    });
}

void launch_tile_head(const GemmTileArgs& t, bool f16, int ncu, hipStream_t stream) {
    if (!on_16_byte_grid(t.W)) return launch_off_grid_head(t, stream);
    if (t.hp.topk <= 2) { if (f16) go<GEPI_HEAD2, true>(t, ncu, stream); else go<GEPI_HEAD2, false>(t, ncu, stream); }
    else { if (f16) go<GEPI_HEAD, true>(t, ncu, stream); else go<GEPI_HEAD, false>(t, ncu, stream); }
}

}  // namespace laser

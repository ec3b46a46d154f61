// Projections of 17..80 activation rows: the tiled product of gemm_tile.h with ONE row tile and its columns dealt to three
// or four waves, so that the weights (bf16, widened in registers) are streamed once.
//
// What bounds it: the rows' way into the compute units. A stage of 72 rows in two planes is 20 KB beside 8, 12 or 16 KB of
// weights, and loads into LDS pass about 50 bytes per ns and compute unit, whatever the tile (taking the matrix
// instructions out changes nothing, taking out the rows' loads gives 30 % at 96 workgroups). With 256 workgroups the
// weights of QKV at the 7B width stream at 4.4 TB/s between start and end. Against the kernel of gemm_mid.h, which stages
// the rows through registers with a barrier per step, us at 72 rows (N x K) inside a step: 12288 x 4096 39.9 -> 30.9,
// 4096 x 4096 15.1 -> 13.5, 4096 x 11008 26.0 -> 23.0, gate/up 2 x 11008 x 4096 68.3 -> 50.6; 6144 x 2048 14.8 -> 12.9,
// 2048 x 2048 7.9 -> 7.8, 2048 x 5632 9.4 -> 8.9, gate/up 2 x 5632 x 2048 24.2 -> 23.3. Tried beside it, alone in a loop: two
// waves sharing columns and two the reduction (a third less LDS reading) was within 2 % of this everywhere but the last
// (21.8 against 23.2).
#include <algorithm>

#include "gemm_tile_plan.h"

namespace laser {

namespace {

struct FewShape { int wn, nwn; };                       // 16-column fragments per wave, waves
constexpr FewShape kFewF32[] = {{2, 3}, {2, 4}, {1, 4}};
constexpr FewShape kFewSwiglu[] = {{2, 3}, {2, 4}};     // gate and up fragments come in pairs

constexpr int few_stages(int wm, FewShape s, bool split) {
    int ns = s.wn == 1 ? 5 : split && s.nwn == 4 ? 3 : 4;
    while (ns > 2 && gemm_tile_lds(wm * 16, s.wn * 16 * s.nwn, ns, split) > 163840) --ns;
    return ns;
}

// Of three tiles the best or within 7 % of it at 72 and 80 rows of both widths; with 24 rows the narrowest is up to 22 % better
// than the one taken (O 8.8 against 10.7 us, down 18.8 against 21.3). Microseconds of a launch: 0.02 per kilobyte a workgroup stages and 4 for its start and end, one workgroup
// per compute unit at a time, never less than the weights take from memory; a reduction part is written and read again.
template <int N>
GemmTilePlan few_plan(const FewShape (&shapes)[N], const GemmTileArgs& t, bool swiglu, int ncu, int want_split, int max_split) {
    GemmTilePlan best{0, 1};
    double best_cost = 1e300;
    const int nk = t.Kd / GT_BK, bm = (t.M + 15) / 16 * 16;
    if (want_split > 0 && (nk % want_split || want_split > max_split)) want_split = 1;
    for (int v = 0; v < N; ++v) {
        if (t.want_tile > 0 && t.want_tile <= N && v != t.want_tile - 1) continue;
        const int bn = shapes[v].wn * 16 * shapes[v].nwn, bf = swiglu ? bn / 2 : bn;
        const long tiles = (t.N + bf - 1) / bf;
        const double stage = 0.02 * (gemm_tile_lds(bm, bn, 1, t.Xlo != nullptr) / 1024);
        for (int S = 1; S <= max_split; S *= 2) {
            if (want_split > 0 ? S != want_split : (nk % S || (S > 1 && nk / S < 4))) continue;
            const long rounds = (tiles * S + ncu - 1) / ncu;
            const double stream = (double)t.N * t.Kd * (swiglu ? 4 : 2) / 5.0e6 + 4.0;
            const double cost = std::max((double)rounds * (nk / S * stage + 4.0), stream) + (S - 1) * (8.0 * t.M * t.N / 4.0e6);
            if (cost < best_cost) { best_cost = cost; best = GemmTilePlan{v, S}; }
        }
    }
    return best;
}

template <int EPI, bool SPLIT, int WM, int WN, int NWN>
void go(GemmTileArgs t, int S, hipStream_t stream) {
    constexpr int BF = EPI == GEPI_SWIGLU ? WN * 8 * NWN : WN * 16 * NWN;
    t.tiles_m = 1;
    t.tiles_n = (t.N + BF - 1) / BF * S;
    t.ksplit = S;
    const unsigned grid = 8u * (unsigned)((t.tiles_n + 7) / 8);
    hipLaunchKernelGGL((gemm_tile_kernel<EPI, WM, WN, 1, NWN, few_stages(WM, FewShape{WN, NWN}, SPLIT), SPLIT, false>), dim3(grid), dim3(64 * NWN), 0, stream, t);
}

template <int EPI, bool SPLIT>
int launch(const GemmTileArgs& t, int ncu, int want_split, int max_split, hipStream_t stream) {
    constexpr auto& shapes = [] () -> auto& { if constexpr (EPI == GEPI_SWIGLU) return kFewSwiglu; else return kFewF32; }();
    constexpr int nv = (int)(sizeof(shapes) / sizeof(shapes[0]));
    const GemmTilePlan pl = few_plan(shapes, t, EPI == GEPI_SWIGLU, ncu, want_split, max_split);
    for_index<2, 6>([&](auto wmc) {
        constexpr int wm = decltype(wmc)::value;
        if ((t.M + 15) / 16 == wm)
            for_index<0, nv>([&](auto vc) {
                constexpr int v = decltype(vc)::value;
                if (pl.v == v) go<EPI, SPLIT, wm, shapes[v].wn, shapes[v].nwn>(t, pl.S, stream);
            });
    });
    return pl.S;
}

}  // namespace

int launch_few_f32(const GemmTileArgs& t, int ncu, int want_split, int max_split, hipStream_t stream) {
    return t.Xlo ? launch<GEPI_F32, true>(t, ncu, want_split, max_split, stream) : launch<GEPI_F32, false>(t, ncu, want_split, max_split, stream);
}

void launch_few_swiglu(const GemmTileArgs& t, int ncu, hipStream_t stream) { launch<GEPI_SWIGLU, true>(t, ncu, 1, 1, stream); }

}  // namespace laser

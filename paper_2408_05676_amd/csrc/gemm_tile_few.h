// Projections of 17..80 activation rows: the tiled product of gemm_tile.h with ONE row tile and its columns dealt to three
// or four waves, so that the weights are streamed once (from the fp16 copy; bf16, widened in registers, without one).
//
// What bounds it: the lines a compute unit has in flight. Alone, a compute unit loads 115 bytes per ns of rows that its L2
// holds and 45 of weights from memory, and a mixture takes the sum of both times, however many loads are in flight and
// whichever waves make them; beyond 195 compute units the weights' part is memory's 6.2 TB/s. A stage of 72 rows in two planes
// is 20 KB beside 8, 12 or 16 KB of weights. Row-major weights stream 20 % slower (gemm_tile.h): with the copy, us inside a step
// at 72 rows, 7B: gate/up 49.5 -> 45.1, QKV 30.5 -> 27.1, down 23.2 -> 20.3, O 12.9 -> 13.0; 24 rows: gate/up 42 -> 31.8;
// 1B at 72 rows: gate/up 23.8 -> 21.9. Tried: weights touched ahead by scalar loads (2.7 bytes per ns), waves that load only
// rows or only weights, cache policies (no difference or slower). Tried earlier, alone in a loop: two waves sharing columns and
// two the reduction (a third less LDS reading) was within 2 % of this.
#pragma once

#include <algorithm>

#include "gemm_tile_plan.h"

namespace laser {

namespace {

struct FewShape { int wn, nwn; };                       // 16-column fragments per wave, waves
constexpr FewShape kFewF32[] = {{2, 3}, {2, 4}, {1, 4}};
constexpr FewShape kFewSwiglu[] = {{2, 3}, {2, 4}, {2, 2}};     // gate and up fragments come in pairs

constexpr int few_stages(int wm, FewShape s, bool split) {
    int ns = s.wn == 1 ? 5 : split && s.nwn == 4 ? 3 : 4;
    while (ns > 2 && gemm_tile_lds(wm * 16, s.wn * 16 * s.nwn, ns, split) > 163840) --ns;
    return ns;
}

// Microseconds of a launch: per kilobyte a workgroup stages 0.0095 for rows and for weights 0.032, or more from 195 workgroups on,
// where memory is what they wait for; 4 for its start and end, one workgroup per compute unit at a time; a reduction part is
// written and read again. (One rate for both sent 24 rows to too few workgroups: at the 7B width QKV 22.5 us, now 18.8, O
// 10.2 -> 8.7, down 18.3 -> 16.7; down of 48 rows 22.3 -> 18.6.)
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
        for (int S = 1; S <= max_split; S *= 2) {
            if (want_split > 0 ? S != want_split : (nk % S || (S > 1 && nk / S < 4))) continue;
            const long rounds = (tiles * S + ncu - 1) / ncu;
            const double w_kb = std::max(0.032, 0.164e-3 * (double)std::min((long)ncu, tiles * S));
            const double stage = 0.0095 * (bm * (t.Xlo ? 2 : 1) / 8) + w_kb * (bn / 8);
            const double cost = (double)rounds * (nk / S * stage + 4.0) + (S - 1) * (8.0 * t.M * t.N / 4.0e6);
            if (cost < best_cost) { best_cost = cost; best = GemmTilePlan{v, S}; }
        }
    }
    return best;
}

template <int EPI, bool SPLIT, bool WF16, int WM, int WN, int NWN>
void go(GemmTileArgs t, int S, hipStream_t stream) {
    constexpr int BF = EPI == GEPI_SWIGLU ? WN * 8 * NWN : WN * 16 * NWN;
    t.tiles_m = 1;
    t.tiles_n = (t.N + BF - 1) / BF * S;
    t.ksplit = S;
    const unsigned grid = 8u * (unsigned)((t.tiles_n + 7) / 8);
    hipLaunchKernelGGL((gemm_tile_kernel<EPI, WM, WN, 1, NWN, few_stages(WM, FewShape{WN, NWN}, SPLIT), SPLIT, WF16>), dim3(grid), dim3(64 * NWN), 0, stream, t);
}

template <int EPI, bool SPLIT, bool WF16>
int launch(const GemmTileArgs& t, int ncu, int want_split, int max_split, hipStream_t stream) {
    constexpr auto& shapes = [] () -> auto& { if constexpr (EPI == GEPI_SWIGLU) return kFewSwiglu; else return kFewF32; }();
    constexpr int nv = (int)(sizeof(shapes) / sizeof(shapes[0]));
    const GemmTilePlan pl = few_plan(shapes, t, EPI == GEPI_SWIGLU, ncu, want_split, max_split);
    for_index<2, 6>([&](auto wmc) {
        constexpr int wm = decltype(wmc)::value;
        if ((t.M + 15) / 16 == wm)
            for_index<0, nv>([&](auto vc) {
                constexpr int v = decltype(vc)::value;
                if (pl.v == v) go<EPI, SPLIT, WF16, wm, shapes[v].wn, shapes[v].nwn>(t, pl.S, stream);
            });
    });
    return pl.S;
}

}  // namespace

}  // namespace laser

// Which tile of gemm_tile.h a launch takes, and the launch itself (gemm_tile_*.hip hold the instantiations).
#pragma once

#include "gemm_tile.h"

namespace laser {

struct GemmTileShape { int wm, wn; };                   // 16-row and 16-column fragments per wave; 2 x 2 waves per workgroup
// Tiles of 96 .. 352 rows and 64 .. 256 columns: for most row counts one of them covers the rows with little padding AND
// gives a number of units that fills the compute units evenly ({4, 6}: gate/up of 256 rows at the 7B width has 230 units of it
// and took 172 of {4, 8}, 60.6 us -> 52.9). The first entries also exist for bf16 weights.
constexpr GemmTileShape kTilePlain[] = {{3, 4}, {4, 4}, {5, 4}, {6, 6}, {11, 6}, {5, 2}, {3, 8}, {4, 8}, {5, 8}, {6, 4}, {8, 4}, {8, 8}, {11, 4}, {4, 6}};
constexpr GemmTileShape kTileSplit[] = {{3, 4}, {4, 4}, {5, 4}, {6, 6}, {3, 6}, {4, 6}, {5, 6}, {6, 4}, {8, 4}};
// The head's record is 128 columns: wn = 8. {8, 8} spills 72 bytes a lane in its two-entry epilogue (no other tile uses
// scratch); the 1024-row head at a vocabulary of 128256 takes 1.00 ms with it.
constexpr GemmTileShape kTileHead[] = {{4, 8}, {6, 8}, {3, 8}, {8, 8}};
constexpr int kTilePlainCommon = 5, kTileSplitCommon = 4, kTileHeadCommon = 2;

constexpr int gemm_tile_stages(int wm, int wn, bool split) {     // ring depth: what fits in the 160 KB, at most 4
    int ns = 4;
    while (ns > 2 && gemm_tile_lds(wm * 32, wn * 32, ns, split) > 163840) --ns;
    return ns;
}

template <int J, int N, class F>
inline void for_index(F&& f) {                          // static_for on the host
    if constexpr (J < N) { f(std::integral_constant<int, J>{}); for_index<J + 1, N>(f); }
}

struct GemmTilePlan { int v, S; };

// One workgroup per compute unit at a time. Cycles of a reduction step of one workgroup: its matrix instructions (16 each) plus
// 17 for each kilobyte it stages; 8000 for a workgroup's start and epilogue; a reduction part more costs a write
// and a read of the output. Against every tile in turn at 96, 136, 256, 352, 512 and 704 rows of the 7B and 1B widths the one
// taken is the best or within 10 % of it in all 48 products (QKV at 704 rows 118.7 us of 118.7 .. 168, gate/up 107.6 of 107.6 ..
// 179, down at 352 rows 45.4, 8 tiles of 44.0 .. 51 beside it, at 512 rows 55.7 of 51.8 .. 76).
template <int NV>
inline GemmTilePlan gemm_tile_plan(const GemmTileShape (&shapes)[NV], int nv, const GemmTileArgs& t, bool swiglu, bool split, int ncu,
                                   int want_split, int max_split) {
    GemmTilePlan best{0, 1};
    double best_cost = 1e300;
    const int nk = t.Kd / GT_BK;
    if (want_split > 0 && (nk % want_split || want_split > max_split)) want_split = 1;
    for (int v = 0; v < nv; ++v) {
        if (t.want_tile > 0 && t.want_tile <= nv && v != t.want_tile - 1) continue;
        const int bm = shapes[v].wm * 32, bn = shapes[v].wn * 32, bf = swiglu ? bn / 2 : bn;
        const long tiles = (long)((t.M + bm - 1) / bm) * ((t.N + bf - 1) / bf);
        const double step = 2.0 * shapes[v].wm * shapes[v].wn * 16 * (split ? 2 : 1) + 17.0 * (gemm_tile_lds(bm, bn, 1, split) / 1024);
        for (int S = 1; S <= max_split; S *= 2) {
            if (want_split > 0 ? S != want_split : (nk % S || (S > 1 && nk / S < 4))) continue;
            const long rounds = (tiles * S + ncu - 1) / ncu;
            const double cost = (double)rounds * (nk / S * step + 8000.0) + (S - 1) * (8.0 * t.M * t.N / 1900.0);
            if (cost < best_cost) { best_cost = cost; best = GemmTilePlan{v, S}; }
        }
    }
    return best;
}

template <int EPI, bool SPLIT, bool WF16, int WM, int WN>
inline void gemm_tile_go(GemmTileArgs t, int S, hipStream_t stream) {
    constexpr int BF = EPI == GEPI_SWIGLU ? WN * 16 : WN * 32;
    t.tiles_m = (t.M + WM * 32 - 1) / (WM * 32);
    t.tiles_n = (t.N + BF - 1) / BF * S;
    t.ksplit = S;
    const unsigned grid = 8u * (unsigned)((t.tiles_m * t.tiles_n + 7) / 8);
    hipLaunchKernelGGL((gemm_tile_kernel<EPI, WM, WN, 2, 2, gemm_tile_stages(WM, WN, SPLIT), SPLIT, WF16>), dim3(grid), dim3(256), 0, stream, t);
}

// t: W, X, Xlo, M, N, Kd and the output; f16: W is fp16. Returns the number of reduction parts stored at t.outf.
int launch_tile_f32(const GemmTileArgs& t, bool f16, int ncu, int want_split, int max_split, hipStream_t stream);
void launch_tile_swiglu(const GemmTileArgs& t, bool f16, int ncu, hipStream_t stream);
// The same for 17..80 rows (gemm_tile_few.hip); SwiGLU takes split activations.
int launch_few_f32(const GemmTileArgs& t, bool f16, int ncu, int want_split, int max_split, hipStream_t stream);
void launch_few_swiglu(const GemmTileArgs& t, bool f16, int ncu, hipStream_t stream);
// topk <= 2
void launch_few_head(const GemmTileArgs& t, bool f16, hipStream_t stream);
void launch_tile_head(const GemmTileArgs& t, bool f16, int ncu, hipStream_t stream);
// The same for t.W bf16 off the 16-byte grid, more than 80 rows (gemm_off_grid.hip).
int launch_off_grid_f32(const GemmTileArgs& t, int ncu, int want_split, int max_split, hipStream_t stream);
void launch_off_grid_swiglu(const GemmTileArgs& t, hipStream_t stream);
void launch_off_grid_head(const GemmTileArgs& t, hipStream_t stream);

// Loads into LDS need it: the library's own buffers and copies are on the grid, a caller's weights and rows may not be.
inline bool on_16_byte_grid(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace laser

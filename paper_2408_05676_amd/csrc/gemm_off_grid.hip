// More than 80 rows with bf16 weights off the 16-byte grid (option f16_copies = 0 and a caller's buffer that starts off it): the
// tiled product with its operands staged through registers, which takes any address; loads into LDS do not.
//
// Workgroup tile 128 x 128, 256 threads = 2 x 2 waves of 64 x 64, each wave 2 x 2 v_mfma_f32_32x32x16_f16 tiles; two
// workgroups per compute unit hide each other's staging. Three stages in flight: the global loads of step kt + 2
// (registers), the conversion and LDS write of step kt + 1 (between the matrix instructions), the multiplication of step
// kt out of one of two LDS buffers; one workgroup barrier per step. A step of four layers of the 7B width, us, off
// the grid / on it with gemm_tile.h: 96 rows 985 / 800, 144 rows 1168 / 876, 352 rows 1937 / 1292, 704 rows 2973 / 2168 (80
// rows at a time on gemm_mid.h: 2085, 2103, 4680 and 8518). Tried instead: the tiles of gemm_tile.h with the weights through
// registers, one workgroup per compute unit: 1142, 1455, 2338 and 5713 us (one stage in flight does not cover the way to
// memory; the wide tiles spill).
//
// v_mfma_f32_32x32x16_f16, wave64, lane l, g = l / 32:
//   A: lane holds A[row = l % 32][k = 8 g .. 8 g + 7];  B: lane holds B[k = 8 g .. 8 g + 7][col = l % 32]
//   D: lane holds D[row = 8 (i / 4) + 4 g + i % 4][col = l % 32], i = 0..15
#include "gemm_tile_plan.h"

namespace laser {

namespace {

typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int GM_BM = 128;

__device__ inline float16_t mfma_32x32x16(const Frag8& a, const Frag8& b, float16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a.v, b.v, c, 0, 0, 0);
}

constexpr int off_grid_step(bool split) { return split ? 32 : 64; }      // reduction step

// weight row behind tile column j (0..BN-1) of n-tile tn
template <int EPI, int BN>
__device__ inline int w_row(const GemmTileArgs& a, int tn, int j) {
    if (EPI == GEPI_SWIGLU) {
        // columns of a wave: [32 gate | 32 up] of the same 32 features, so that one lane holds both
        const int wn = j >> 6, ct = (j >> 5) & 1, c = j & 31;
        return (ct ? a.N : 0) + tn * 64 + wn * 32 + c;
    }
    return tn * BN + j;
}

// BN = 128: 2 x 2 waves of 64 x 64. BN = 64 (narrow outputs, where 128-column tiles would leave CUs
// without work): 2 x 2 waves of 64 x 32. The SwiGLU epilogue needs BN = 128.
// SPLIT: the activations come as two fp16 planes; every weight fragment meets both (second accumulator
// set, folded in with the factor 2^-12 at the end). The reduction step drops to 32 so that the third
// LDS tile still leaves room for two workgroups per CU.
template <int EPI, int BN, bool SPLIT>
__global__ __launch_bounds__(256, 2) void gemm_off_grid_kernel(GemmTileArgs a) {
    static_assert(BN == 128 || (BN == 64 && EPI != GEPI_SWIGLU), "tile width");
    constexpr int GM_BK = off_grid_step(SPLIT);
    // LDS rows. Single-plane kernel: 64 + 8 halves, the padding spreads 16-byte reads of consecutive rows over the banks.
    // Split kernel (step 32): padded 80-byte rows left a third of the LDS-active cycles in bank conflicts (hardware
    // counter), so its rows are unpadded 64 bytes and the four 16-byte chunks of row r sit at chunk ^ ((r >> 2) & 3):
    // 16 consecutive rows at one logical chunk, and 4 rows x 4 chunks of a staging write, each touch 16 distinct
    // 16-byte bank groups.
    constexpr bool SWZ = SPLIT;
    constexpr int GM_LD = SWZ ? GM_BK : GM_BK + 8;
    constexpr int CH = GM_BK / 8;            // 16-byte chunks per tile row and k-step
    constexpr int RPT = 256 / CH;            // rows staged per pass of the 256 threads
    constexpr int ST = GM_BM / RPT;          // passes over the activation rows
    constexpr int STB = BN / RPT;            // passes over the weight rows
    constexpr int WN = BN / 2;               // columns per wave
    constexpr int NJ = WN / 32;              // 32-column MFMA tiles per wave
    constexpr int D = (SPLIT && BN == 128) ? 2 : (SPLIT ? 4 : 2);   // the split 128-column kernel has no registers for a deeper ring
    __shared__ __attribute__((aligned(16))) uint16_t sA[2][GM_BM][GM_LD];
    __shared__ __attribute__((aligned(16))) uint16_t sB[2][BN][GM_LD];
    __shared__ __attribute__((aligned(16))) uint16_t sAl[SPLIT ? 2 : 1][SPLIT ? GM_BM : 1][SPLIT ? GM_LD : 8];
    // ---- XCD-aware tile order, longest tiles first ----
    // n-tile tn belongs to XCD tn % 8 (consecutive workgroup ids go round-robin over the XCDs). Inside an XCD the
    // workgroups come in dispatch order: first every FULL m-tile of every owned n-tile (m fastest, so the m-tiles
    // that share a weight tile run together and hit it in L2), then the ragged last m-tiles, whose dead waves make
    // them finish in about half the time: issued last they fill the tail of the launch.
    const int xcd = blockIdx.x % 8, li = blockIdx.x / 8;
    const int nt_x = (a.tiles_n - xcd + 7) / 8;                 // n-tiles owned by this XCD
    const bool ragged = a.M % GM_BM != 0 && a.tiles_m > 1;
    const int full_m = ragged ? a.tiles_m - 1 : a.tiles_m;
    if (li >= nt_x * a.tiles_m) return;
    int tn, tm;
    if (li < nt_x * full_m) { tn = xcd + 8 * (li / full_m); tm = li % full_m; }
    else { tn = xcd + 8 * (li - nt_x * full_m); tm = a.tiles_m - 1; }
    const int kpart = tn % a.ksplit;          // (n-tile, reduction part) pairs were dealt out as one index
    tn /= a.ksplit;

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int lr = lane & 31, lg = lane >> 5;

    // global -> LDS staging: thread t moves chunk t % CH of rows t / CH + RPT i of both operands
    const int srow = tid / CH, sk = (tid % CH) * 8;
    const int skw = SWZ ? ((tid % CH) ^ ((srow >> 2) & 3)) * 8 : sk;       // LDS column of this thread's chunk (RPT is a multiple of 16)
    const uint16_t* xa[ST];
    const uint16_t* xl[ST];
    const uint16_t* wb[STB];
#pragma unroll
    for (int i = 0; i < ST; ++i) {
        int row = tm * GM_BM + srow + RPT * i;
        row = row < a.M ? row : a.M - 1;
        xa[i] = a.X + (size_t)row * a.Kd + sk;
        xl[i] = SPLIT ? a.Xlo + (size_t)row * a.Kd + sk : nullptr;
    }
#pragma unroll
    for (int i = 0; i < STB; ++i) {
        int wr = w_row<EPI, BN>(a, tn, srow + RPT * i);
        const int wmax = (EPI == GEPI_SWIGLU ? 2 * a.N : a.N) - 1;
        wr = wr < wmax ? wr : wmax;
        wb[i] = a.W + (size_t)wr * a.Kd + sk;
    }
    // head epilogue: thread t will own half of row t / 2; its candidate list is fetched now, under the main loop
    int hc_b = 0, hc_n = 0, hc_x0 = -1;
    if constexpr (EPI == GEPI_HEAD) {
        const int grow = tm * GM_BM + (tid >> 1);
        if (grow < a.M) { hc_b = a.hp.cand_beg[grow]; hc_n = a.hp.cand_cnt[grow]; }
        hc_x0 = hc_n > 0 ? a.hp.cand_x[hc_b] : -1;
    }
    float16_t acc[2][NJ];
    float16_t acl[SPLIT ? 2 : 1][SPLIT ? NJ : 1];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc[i][j][e] = 0.f;
                if constexpr (SPLIT) acl[i][j][e] = 0.f;
            }

    // a wave whose 64 rows all lie past M (ragged last m-tile) stages and synchronises but multiplies nothing
    const bool dead = __builtin_amdgcn_readfirstlane(tm * GM_BM + wm * 64) >= a.M;

    // Register ring of D k-steps. The element type must be a native vector: an array of HIP's uint4
    // (a struct) that is only copied as a whole is not promoted to registers and lands in scratch.
    u32x4 ra[D][ST], rb[D][STB], rl[D][SPLIT ? ST : 1];
    const int nk = a.Kd / GM_BK / a.ksplit;  // the host guarantees Kd % (GM_BK * ksplit) == 0
    {
        const int k0 = kpart * nk * GM_BK;
#pragma unroll
        for (int i = 0; i < ST; ++i) { xa[i] += k0; if constexpr (SPLIT) xl[i] += k0; }
#pragma unroll
        for (int i = 0; i < STB; ++i) wb[i] += k0;
    }
    float* const outf = a.outf ? a.outf + (size_t)kpart * a.M * a.N : nullptr;
    auto gload = [&](auto slot_c, int kt) {
        constexpr int slot = decltype(slot_c)::value;
        kt = kt < nk ? kt : nk - 1;          // unconditional, clamped: a load under a branch would be waited for at once
#pragma unroll
        for (int i = 0; i < ST; ++i) ra[slot][i] = *reinterpret_cast<const u32x4*>(xa[i] + kt * GM_BK);
        if constexpr (SPLIT) {
#pragma unroll
            for (int i = 0; i < ST; ++i) rl[slot][i] = *reinterpret_cast<const u32x4*>(xl[i] + kt * GM_BK);
        }
#pragma unroll
        for (int i = 0; i < STB; ++i) rb[slot][i] = *reinterpret_cast<const u32x4a2*>(wb[i] + kt * GM_BK);
    };
    // Software pipeline over k-steps: while step kt is multiplied out of LDS buffer kt % 2, the registers that
    // hold step kt + 1 are converted and written to the other buffer in pieces BETWEEN the matrix instructions
    // of the same basic block (so the vector ALU and LDS-write work hides behind the matrix pipe instead of
    // preceding it), and the global loads of step kt + 2 are in flight. One workgroup barrier per step: it
    // publishes buffer (kt + 1) % 2 and guarantees that every wave has finished reading buffer kt % 2 before
    // the next step overwrites it.
    constexpr int NKK = GM_BK / 16;
    auto stage_piece = [&](auto slot_c, int buf, int kk, unsigned keep) {       // piece kk (of NKK) of one k-step
        constexpr int slot = decltype(slot_c)::value;
#pragma unroll
        for (int i = 0; i < ST; ++i)
            if (i * NKK / ST == kk) {
                *reinterpret_cast<u32x4*>(&sA[buf][srow + RPT * i][skw]) = ra[slot][i] & keep;
                if constexpr (SPLIT) *reinterpret_cast<u32x4*>(&sAl[buf][srow + RPT * i][skw]) = rl[slot][i] & keep;
            }
#pragma unroll
        for (int i = 0; i < STB; ++i)
            if (i * NKK / STB == kk) {
                Frag8 fw;
                fw.v4 = rb[slot][i];
                bf16x8_to_f16x8(fw);
                *reinterpret_cast<u32x4*>(&sB[buf][srow + RPT * i][skw]) = fw.v4;
            }
    };
    auto multiply_piece = [&](int buf, int kk) {
        Frag8 fa[2], fb[NJ];
        // LDS column of this lane's fragment (every row offset above lr is a multiple of 32)
        const int fc = SWZ ? ((kk * 2 + lg) ^ ((lr >> 2) & 3)) * 8 : kk * 16 + lg * 8;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            fa[i].v4 = *reinterpret_cast<const u32x4*>(&sA[buf][wm * 64 + i * 32 + lr][fc]);
#pragma unroll
        for (int i = 0; i < NJ; ++i)
            fb[i].v4 = *reinterpret_cast<const u32x4*>(&sB[buf][wn * WN + i * 32 + lr][fc]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj) acc[i][jj] = mfma_32x32x16(fa[i], fb[jj], acc[i][jj]);
        if constexpr (SPLIT) {
            Frag8 fl[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                fl[i].v4 = *reinterpret_cast<const u32x4*>(&sAl[buf][wm * 64 + i * 32 + lr][fc]);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) acl[i][jj] = mfma_32x32x16(fl[i], fb[jj], acl[i][jj]);
        }
    };
    static_assert(D % 2 == 0, "slot j of the unrolled loop must map to LDS buffer j & 1");
    static_for<0, D>([&](auto sc) { gload(sc, decltype(sc)::value); });
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) stage_piece(std::integral_constant<int, 0>{}, 0, kk, 0xFFFFFFFFu);
    __syncthreads();
    // The whole loop exists twice (live and dead waves) so that neither body contains a branch: with a branch
    // inside, the conversions common to both arms are hoisted in front of it and run before, not between, the
    // matrix instructions.
    // Steps are taken in groups of D (D register slots, two LDS buffers). If the step count is not a multiple
    // of D the last group multiplies steps that do not exist: they are staged as zeros, which only that
    // group's code pays for (the mask costs a vector instruction per staged register).
    auto run = [&](auto dead_c) {
        constexpr bool kDead = decltype(dead_c)::value;
        auto pairs = [&](int kt_begin, int kt_end, auto mask_c) {
            constexpr bool kMask = decltype(mask_c)::value;
            for (int kt0 = kt_begin; kt0 < kt_end; kt0 += D) {
                static_for<0, D>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;      // step kt lives in LDS buffer j & 1; registers slot j are free
                    constexpr int jn = (j + 1) % D;             // slot that holds step kt + 1
                    const int kt = kt0 + j;
                    gload(jc, kt + D);
                    __builtin_amdgcn_sched_barrier(0);
                    const unsigned keep = (!kMask || kt + 1 < nk) ? 0xFFFFFFFFu : 0u;
#pragma unroll
                    for (int kk = 0; kk < NKK; ++kk) {
                        if constexpr (!kDead) multiply_piece(j & 1, kk);
                        stage_piece(std::integral_constant<int, jn>{}, jn & 1, kk, keep);
                    }
                    __syncthreads();
                });
            }
        };
        const int full_end = nk - nk % D;                // whole groups of D steps need no mask
        pairs(0, full_end, std::false_type{});
        if (nk % D) pairs(full_end, nk, std::true_type{});
    };
    if (dead) run(std::true_type{});
    else run(std::false_type{});
    if constexpr (SPLIT) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] += acl[i][j][e] * kLoInv;
    }
    if constexpr (EPI == GEPI_HEAD) {
        // ---- output-head epilogue: the tile goes through LDS in two halves of 64 columns (the staging buffer of the
        // activations is free after the loop's last barrier and holds 128 rows x 65 floats), where thread t owns half a
        // row (row t / 2, 32 of the 64 columns) and folds it into its running statistics; ids ascend per thread.
        static_assert(BN == 128 && !SPLIT, "the head epilogue is written for 128-column single-plane tiles");
        static_assert(sizeof(sA) >= GM_BM * 65 * sizeof(float), "the activation staging buffer must hold half a tile of floats");
        float* sC = reinterpret_cast<float*>(&sA[0][0][0]);
        const int trow = tid >> 1, part = tid & 1;
        const int grow = tm * GM_BM + trow;
        RowStat st;
        st.init();
        const int kt = a.hp.topk;                       // 1..KT
        float thr_v = -INFINITY;                        // the list's kt-th entry: what a value has to beat to enter
        int thr_i = 0x7FFFFFFF;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (wn == h) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            sC[(wm * 64 + i * 32 + 8 * (e >> 2) + 4 * lg + (e & 3)) * 65 + j * 32 + lr] = acc[i][j][e];
            }
            __syncthreads();
            const int n0 = tn * BN + h * 64 + part * 32;
            const float* src = sC + trow * 65 + part * 32;
            if (grow < a.M) {
                // 32 columns at once, without data-dependent branches on the common path: their maximum and its first
                // position, the sum of exponentials against the new running maximum, and the few values that beat the
                // list's kt-th entry (kt = the call's k: deeper list entries are never needed for "rank < k")
                float vals[32];
#pragma unroll
                for (int c = 0; c < 32; ++c) vals[c] = (n0 + c < a.N) ? src[c] : -INFINITY;
                float mloc = vals[0];
#pragma unroll
                for (int c = 1; c < 32; ++c) mloc = fmaxf(mloc, vals[c]);
                int cloc = 31;
#pragma unroll
                for (int c = 30; c >= 0; --c) cloc = vals[c] == mloc ? c : cloc;
                const float m_new = fmaxf(st.mx, mloc);
                float ssum = 0.f;
                if (m_new != -INFINITY) {
#pragma unroll
                    for (int c = 0; c < 32; ++c) ssum += __expf(vals[c] - m_new);          // exp(-inf) = 0 for columns past N
                    st.sum = st.sum * __expf(st.mx - m_new) + ssum;
                }
                if (mloc > st.mx) st.arg = n0 + cloc;                                      // ids ascend per thread: earlier ties stay
                st.mx = m_new;
                if (hc_x0 >= n0 && hc_x0 < n0 + 32) a.hp.cand_lx[hc_b] = src[hc_x0 - n0];
                for (int c = 1; c < hc_n; ++c) {                                         // further children of a tree node
                    const int x = a.hp.cand_x[hc_b + c];
                    if (x >= n0 && x < n0 + 32) a.hp.cand_lx[hc_b + c] = src[x - n0];
                }
#pragma unroll
                for (int c = 0; c < 32; ++c) {
                    if (n0 + c < a.N && before(vals[c], n0 + c, thr_v, thr_i)) {
                        st.push_top(vals[c], n0 + c);
#pragma unroll
                        for (int j = 0; j < KT; ++j) if (j == kt - 1) { thr_v = st.tv[j]; thr_i = st.ti[j]; }
                    }
                }
                if (a.hp.logits_dbg) {
#pragma unroll
                    for (int c = 0; c < 32; ++c) if (n0 + c < a.N) a.hp.logits_dbg[(size_t)grow * a.N + n0 + c] = vals[c];
                }
            }
            __syncthreads();
        }
        st.merge_from_lane(1);
        if (part == 0 && grow < a.M) st.store(a.hp, grow, tn);
        return;
    }
    // ---- epilogue: lane holds column lr of each 32-wide tile, rows 8 (e / 4) + 4 lg + e % 4 ----
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = tm * GM_BM + wm * 64 + i * 32 + 8 * (e >> 2) + 4 * lg + (e & 3);
            if (row >= a.M) continue;
            if (EPI == GEPI_SWIGLU) {
                const int feat = tn * 64 + wn * 32 + lr;
                if (feat < a.N) {
                    const float gt = acc[i][0][e], up = acc[i][NJ - 1][e];
                    a.outh[(size_t)row * a.N + feat] = f32_to_f16(gt / (1.f + __expf(-gt)) * up);
                }
            } else {
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int col = tn * BN + wn * WN + j * 32 + lr;
                    if (col < a.N) outf[(size_t)row * a.N + col] = acc[i][j][e];
                }
            }
        }
    }
}

// Reduction parts for a launch of `tiles` 128 x 128 tiles. Two workgroups share a compute unit ("slots") and a launch takes
// ceil(units / slots) rounds; a lone workgroup on a compute unit runs at about 0.6 of the shared time. S parts are S times as
// many units of 1/S the length; each costs one more pass of the output through memory.
int choose_parts(long tiles, int steps, long out_elems, int slots) {
    int best = 1;
    double best_cost = 1e30;
    for (int S = 1; S <= 4; S *= 2) {
        if (steps % S || steps / S < 8) continue;
        if (S > 2 && out_elems > (4L << 20)) continue;
        const long units = tiles * S;
        const double rounds = units <= slots / 2 ? 0.6 : (double)((units + slots - 1) / slots);
        const double cost = rounds / S + 0.04 * (S - 1);
        if (cost < best_cost - 1e-9) { best_cost = cost; best = S; }
    }
    return best;
}

template <int EPI, int BN, bool SPLIT>
void go(GemmTileArgs t, int S, hipStream_t stream) {
    constexpr int BF = EPI == GEPI_SWIGLU ? BN / 2 : BN;
    t.tiles_m = (t.M + GM_BM - 1) / GM_BM;
    t.tiles_n = (t.N + BF - 1) / BF * S;
    t.ksplit = S;
    const unsigned grid = 8u * (unsigned)((t.tiles_n + 7) / 8 * t.tiles_m);      // 8 x the largest share of an XCD
    hipLaunchKernelGGL((gemm_off_grid_kernel<EPI, BN, SPLIT>), dim3(grid), dim3(256), 0, stream, t);
}

}  // namespace

int launch_off_grid_f32(const GemmTileArgs& t, int ncu, int want_split, int max_split, hipStream_t stream) {
    const int steps = t.Kd / off_grid_step(t.Xlo != nullptr);
    const long tiles = (long)((t.M + GM_BM - 1) / GM_BM) * ((t.N + 127) / 128);
    int S = want_split ? want_split : choose_parts(tiles, steps, (long)t.M * t.N, 2 * ncu);
    if (steps % S || S > max_split) S = 1;
    // narrow outputs: 128-column tiles would leave compute units without work, 64-column tiles double the count
    const bool narrow = S == 1 && tiles * 4 < (long)ncu * 5;
    if (t.Xlo) { if (narrow) go<GEPI_F32, 64, true>(t, S, stream); else go<GEPI_F32, 128, true>(t, S, stream); }
    else { if (narrow) go<GEPI_F32, 64, false>(t, S, stream); else go<GEPI_F32, 128, false>(t, S, stream); }
    return S;
}

void launch_off_grid_swiglu(const GemmTileArgs& t, hipStream_t stream) {
    if (t.Xlo) go<GEPI_SWIGLU, 128, true>(t, 1, stream);
    else go<GEPI_SWIGLU, 128, false>(t, 1, stream);
}

void launch_off_grid_head(const GemmTileArgs& t, hipStream_t stream) { go<GEPI_HEAD, 128, false>(t, 1, stream); }

}  // namespace laser

// LDS-tiled matrix-core GEMM for many activation rows (more than the weight-streaming kernels take):
//   Y[M][N] = X[M][Kd] * W[N][Kd]^T,  X fp16 (one or two planes), W fp16 or bf16, fp32 accumulate.
#pragma once

#include "head_part.h"
#include "mfma.h"

namespace laser {

typedef unsigned u32x4a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef float float4a4_t __attribute__((ext_vector_type(4), aligned(4)));   // a caller's buffer may be aligned to its elements only

struct GemmTileArgs {
    const uint16_t* W;      // [N][Kd] bf16, or (WF16 kernels) the same values widened to fp16 and laid out by the 32 reduction
                            // elements of a fragment: [Kd / 32][N][32] (SwiGLU: 2F rows, gate rows then up rows; N = F)
    const uint16_t* X;      // [M][Kd] fp16
    const uint16_t* Xlo;    // [M][Kd] low plane of split activations (x = X + Xlo / 4096), SPLIT kernels only
    int M, N, Kd;
    int tiles_m, tiles_n;   // tiles_n counts BN-column tiles (SwiGLU: BN / 2 features), times ksplit
    int ksplit;             // > 1: the reduction is cut into ksplit equal parts, each a unit of its own that STORES its
                            // partial result at outf + part * M * N (the consumer adds the parts in a fixed order)
    float* outf;            // GEPI_F32: [ksplit][M][N]
    uint16_t* outh;         // GEPI_SWIGLU: [M][N] fp16
    HeadPart hp{};          // GEPI_HEAD*: where the per-(row, chunk) statistics go (chunk = the WN * 16 columns of a wave)
    uint32_t lo_off = 0;    // Xlo - X in bytes, for the tiles of 17..80 rows
    int want_tile = 0;      // for the host: 1 + the entry of the tile table to take, 0: chosen by the rule
};

// GEPI_HEAD: the output head. Logits are not stored: each row's columns of a wave are reduced to one record of partial
// statistics (head_part.h). GEPI_HEAD2: the same with two-entry candidate lists (calls with k <= 2).
enum { GEPI_F32, GEPI_SWIGLU, GEPI_HEAD, GEPI_HEAD2 };

constexpr int GT_BK = 64;   // reduction step: a staged row is one 128-byte line

// LDS bytes of a ring of ns stages
constexpr int gemm_tile_lds(int bm, int bn, int ns, bool split) { return (bn + bm * (split ? 2 : 1)) * GT_BK * 2 * ns; }

__device__ inline void mfma_acc(const Frag8& w, const Frag8& x, float4_t& c) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(w.v), "v"(x.v));
}
__device__ inline void mfma_acc_v(const Frag8& w, const Frag8& x, float4_t& c) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(c) : "v"(w.v), "v"(x.v));
}

template <int EPI, int WM, int WN, int NWM, int NWN, int NS, bool SPLIT, bool WF16>
__global__ __launch_bounds__(64 * NWM * NWN, (NWM * NWN + 3) / 4)
void gemm_tile_kernel(GemmTileArgs a) {
    constexpr int NW = NWM * NWN, BM = WM * 16 * NWM, BN = WN * 16 * NWN, BK = GT_BK;
    constexpr int SBYTES = gemm_tile_lds(BM, BN, 1, SPLIT);
    constexpr int PIECES = SBYTES / 1024;                    // 1 KB of staged rows: what one load instruction moves
    constexpr int CH = BK / 8, RPP = 64 / CH;                // 16-byte chunks per staged row, rows per piece
    constexpr int LPS = (PIECES + NW - 1) / NW;              // load instructions per wave and stage
    static_assert(SBYTES * NS <= 163840, "LDS");
    static_assert((NS - 2) * LPS < 64 && NS >= 2, "the wait counter has six bits");
    __shared__ __attribute__((aligned(1024))) char lds[SBYTES * NS];

    // XCD x takes an equal share of the units (n-tile major, m fastest)
    const int units = a.tiles_m * a.tiles_n, per = (units + 7) / 8;
    const int li = blockIdx.x / 8, unit = (blockIdx.x % 8) * per + li;
    if (li >= per || unit >= units) return;
    int tn = unit / a.tiles_m;
    const int tm = unit % a.tiles_m;
    const int kpart = tn % a.ksplit;
    tn /= a.ksplit;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / NWN, wn = wave % NWN;
    const int lr = lane & 15, lg = lane >> 4;

    const int nk = a.Kd / BK / a.ksplit;                  // the host guarantees Kd % (BK * ksplit) == 0
    const size_t k0 = (size_t)kpart * nk * BK;
    const uint32_t ldb = (uint32_t)a.Kd * 2;                 // bytes per row

    // ---- staging plan: wave w moves pieces w, w + NW, ...; lane l of a piece moves one 16-byte chunk of row l / CH ----
    // Rows are unpadded; chunk c of row r sits at c ^ swz(r), so that the 16 rows a fragment read touches at one logical
    // chunk lie in 16 distinct 16-byte bank groups.
    auto swz = [](int row) { return (row / (16 / CH)) & (CH - 1); };
    // Steps of a weight row are next to each other in a row-major matrix; in the widened copy the rows of half a step are, so
    // that the workgroups, which walk the steps together, read one stretch of memory at a time: alone, 256 workgroups with 96
    // rows each read 5.0 TB/s of a row-major matrix in pieces of 128 bytes and 6.2 TB/s of the copy. A piece of the copy is
    // half a step of 16 rows, and a stage holds the halves one after the other, rows of 64 bytes.
    constexpr int CW = WF16 ? BK / 16 : CH, RPW = 64 / CW;   // chunks per staged weight row, rows per weight piece
    auto swzw = [](int row) { return (row / (16 / CW)) & (CW - 1); };
    const uint32_t ldw = WF16 ? BK : ldb;
    const uint32_t wstep = WF16 ? (uint32_t)a.N * (EPI == GEPI_SWIGLU ? 2 : 1) * (BK * 2) : BK * 2;
    constexpr int WPW = BN / RPP / NW;                       // weight pieces per wave: load j of a wave is a weight piece iff j < WPW
    static_assert(WPW * RPP * NW == BN, "every wave's loads change from weights to rows at the same j");
    // likewise from rows to their low plane, where the rows' pieces divide by the waves; else the plane is reached by an offset
    constexpr bool LOWB = SPLIT && BM / RPP % NW == 0;
    constexpr int XPW = LOWB ? WPW + BM / RPP / NW : LPS;
    uint32_t voff[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        int p = wave + j * NW;
        p = p < PIECES ? p : PIECES - 1;                     // surplus requests repeat the last piece (same bytes, same place)
        if (j < WPW) {
            const int half = WF16 ? p / (BN / 16) : 0, row = (WF16 ? p % (BN / 16) : p) * RPW + lane / CW;
            const int c = (lane % CW) ^ swzw(row);            // the chunk that lives in this slot of the swizzled row
            // SwiGLU: the 16-row fragments alternate gate, up of the same 16 features
            int r0 = 0, r = row;
            if (EPI == GEPI_SWIGLU) { r0 = (row >> 5) * 16; r = row & 15; }
            const int left = a.N - 1 - tn * (EPI == GEPI_SWIGLU ? BN / 2 : BN);
            r = r0 + r < left ? r0 + r : left;               // (rows past the last repeat it)
            const uint32_t up = EPI == GEPI_SWIGLU && (row & 16) ? (uint32_t)a.N * ldw : 0;
            voff[j] = up + (uint32_t)r * ldw + c * 16 + half * (wstep / 2);
        } else {
            const int row = p * RPP + lane / CH;
            const int c = (lane % CH) ^ swz(row);
            const bool low = SPLIT && p * RPP >= BN + BM;
            int xr = row - BN - (low ? BM : 0);
            xr = tm * BM + xr < a.M ? xr : a.M - 1 - tm * BM;
            voff[j] = (uint32_t)xr * ldb + c * 16 + (low && !LOWB ? a.lo_off : 0);
        }
    }
    // Addresses of the stage being requested (moved on by a step once per stage), and the place of the wave's first piece in
    // LDS. A request is then four instructions; with a 64-bit address and an LDS address made for each it was about fourteen,
    // and the matrix instructions behind it waited. Both together, us inside a step at the 7B width: 704 rows QKV 119 -> 109,
    // gate/up 108 -> 100, down 68 -> 63, O 49 -> 45; 256 rows QKV 49 -> 45.5, down 36.7 -> 33.6.
    uint64_t wbase = (uint64_t)(uintptr_t)a.W + (uint64_t)tn * (EPI == GEPI_SWIGLU ? BN / 2 : BN) * ldw + (uint64_t)kpart * nk * wstep;
    uint64_t xbase = (uint64_t)(uintptr_t)(a.X + (size_t)tm * BM * a.Kd + k0);
    uint64_t lbase = LOWB ? (uint64_t)(uintptr_t)(a.Xlo + (size_t)tm * BM * a.Kd + k0) : 0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds + wave * 1024;
    const uint32_t last = lds0 + (PIECES - 1 - wave) * 1024;                 // (p = PIECES - 1)
    uint32_t lslot = 0;                                                     // LDS offset of the slot being filled
    // Load j of the stage being requested. m0 = the piece's LDS byte address, one wait state before its use. The compiler warns that m0
    // is a reserved register which it does not preserve around the statement: nothing else in this kernel uses it.
    auto issue = [&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const uint64_t base = j < WPW ? wbase : j < XPW ? xbase : lbase;
        const u32x4 srd{(uint32_t)base, (uint32_t)(base >> 32), 0xFFFFFFFFu, 0x00020000u};
        const uint32_t vo = voff[j], at = (PIECES % NW != 0 && j == LPS - 1 && wave + j * NW >= PIECES ? last : lds0 + j * NW * 1024) + lslot;
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %2, 0 offen lds" ::"v"(vo), "s"(at), "s"(srd) : "memory", "m0");
    };
    // On to the next stage. Requests past the last step repeat it: nobody reads what they bring, but the counts stay uniform.
    int kreq = 0;
    auto next_stage = [&] {
        ++kreq;
        wbase += kreq < nk ? wstep : 0;
        xbase += kreq < nk ? BK * 2 : 0;
        if constexpr (LOWB) lbase += kreq < nk ? BK * 2 : 0;
        lslot = lslot + SBYTES < SBYTES * NS ? lslot + SBYTES : 0;
    };

    float4_t acc[WM][WN];
    float4_t acl[SPLIT ? WM : 1][SPLIT ? WN : 1];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
            if constexpr (SPLIT) acl[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
        }

    Frag8 fw[2][WN], fx[2][WM], fl[2][SPLIT ? WM : 1];
    // fragment addresses: the row part of the swizzle depends on the lane only
    uint32_t ow[2], ox[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint32_t ch = (uint32_t)(((s * 4 + lg) ^ swz(lr)) * 16);
        ow[s] = (uint32_t)(wn * WN * 16 + lr) * (CW * 16) + (WF16 ? s * BN * CW * 16 + ((lg ^ swzw(lr)) * 16) : ch);
        ox[s] = (uint32_t)(BN + wm * WM * 16 + lr) * (BK * 2) + ch;
    }
    // fragment r of substep s: the wave's weight fragments, then its activation fragments (high plane, low plane)
    constexpr int NREAD = WN + WM * (SPLIT ? 2 : 1), NMUL = WM * WN * (SPLIT ? 2 : 1);
    auto read_frag = [&](auto sc, auto rc, int slot) {
        constexpr int s = decltype(sc)::value, r = decltype(rc)::value;
        if constexpr (r < WN) {
            fw[s][r].v4 = *reinterpret_cast<const u32x4*>(lds + slot * SBYTES + ow[s] + r * 16 * CW * 16);
        } else {
            constexpr int i = SPLIT ? (r - WN) / 2 : r - WN;
            constexpr bool low = SPLIT && ((r - WN) & 1);
            const u32x4 v = *reinterpret_cast<const u32x4*>(lds + slot * SBYTES + ox[s] + ((low ? BM : 0) + i * 16) * BK * 2);
            if constexpr (low) fl[s][i].v4 = v;
            else fx[s][i].v4 = v;
        }
    };
    // Multiplies substep s and reads the fragments of substep rs (of ring slot rslot) meanwhile, one read between every
    // few matrix instructions. The accumulators are pinned to the accumulation registers by assembly: left to itself
    // the compiler moves them back and forth between the register files inside the loop.
    // The loads L0 .. L1-1 of another stage are spread over the same instructions: in a burst they hold up the matrix
    // instructions behind them, about 32 cycles each.
    auto multiply_read = [&](auto sc, auto rsc, int rslot, auto l0c, auto l1c) {
        constexpr int s = decltype(sc)::value, L0 = decltype(l0c)::value, L1 = decltype(l1c)::value;
        if constexpr (!WF16) {
#pragma unroll
            for (int j = 0; j < WN; ++j) bf16x8_to_f16x8(fw[s][j]);
            // Vector write -> matrix read takes two wait states, which the compiler keeps for its own matrix instructions only.
            // Every fragment is an operand of the statements up to the wait, so no conversion can be moved behind it.
#pragma unroll
            for (int j = 0; j + 1 < WN; ++j) asm volatile("" : "+v"(fw[s][j].v4));
            asm volatile("s_nop 1" : "+v"(fw[s][WN - 1].v4));
        }
        static_for<0, NMUL>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            constexpr int i = m / (WN * (SPLIT ? 2 : 1)), q = m % (WN * (SPLIT ? 2 : 1)), j = q % WN;
            constexpr int r0 = m * NREAD / NMUL, r1 = (m + 1) * NREAD / NMUL;
            static_for<r0, r1>([&](auto rc) { read_frag(rsc, rc, rslot); });
            constexpr int l0 = L0 + (2 * m * (L1 - L0) + NMUL) / (2 * NMUL), l1 = L0 + (2 * (m + 1) * (L1 - L0) + NMUL) / (2 * NMUL);   // between the reads
            static_for<l0, l1>([&](auto jc) { issue(jc); });
            constexpr bool inv = i * WN * (SPLIT ? 2 : 1) + q >= 64;      // there are 256 accumulation registers: the rest sit in vector registers
            if constexpr (SPLIT && q >= WN) { if constexpr (inv) mfma_acc_v(fw[s][j], fl[s][i], acl[i][j]); else mfma_acc(fw[s][j], fl[s][i], acl[i][j]); }
            else { if constexpr (inv) mfma_acc_v(fw[s][j], fx[s][i], acc[i][j]); else mfma_acc(fw[s][j], fx[s][i], acc[i][j]); }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto sync = [&] {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * LPS) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using L0 = C0;
    using LA = std::integral_constant<int, LPS>;
    // A stage is two matrix-instruction steps. In the middle of stage kt: wait for stage kt + 1 and for everybody's last
    // reads of stage kt's slot, then request stage kt + NS into that slot. A ring of three stages or more spreads its
    // requests over both halves, a ring of two takes the half right after the wait (the other half would be too late).
    using LH = std::integral_constant<int, NS >= 3 ? (LPS + 1) / 2 : LPS>;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) { static_for<0, LPS>([&](auto jc) { issue(jc); }); next_stage(); }
    static_for<0, LH::value>([&](auto jc) { issue(jc); });
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * LPS + LH::value) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_for<0, NREAD>([&](auto rc) { read_frag(C0{}, rc, 0); });
    int slot = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const int nslot = slot + 1 < NS ? slot + 1 : 0;
        multiply_read(C0{}, C1{}, slot, LH{}, LA{});             // the rest of stage kt + NS - 1
        next_stage();
        sync();
        multiply_read(C1{}, C0{}, nslot, L0{}, LH{});            // stage kt + NS
        slot = nslot;
    }
    // The surplus requests must not land in a later workgroup's LDS; the last matrix instructions must have written. Reads of
    // the results in the source stay behind the wait; register copies of the compiler's own might not, which
    // test_matrix_waits.py looks for in the code as built.
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    static_for<0, NMUL>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        constexpr int i = m / (WN * (SPLIT ? 2 : 1)), q = m % (WN * (SPLIT ? 2 : 1)), j = q % WN;
        float4_t& c = (SPLIT && q >= WN) ? acl[SPLIT ? i : 0][SPLIT ? j : 0] : acc[i][j];
        if constexpr (m >= 64) asm volatile("" : "+v"(c));
        else asm volatile("" : "+a"(c));
    });
    if constexpr (SPLIT) {
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] += acl[i][j][e] * kLoInv;
    }

    // ---- epilogue: lane holds columns 4 lg .. 4 lg + 3 of every 16-column fragment, row lr of every 16-row fragment ----
    if constexpr (EPI == GEPI_HEAD || EPI == GEPI_HEAD2) {
        constexpr int KD = EPI == GEPI_HEAD2 ? 2 : KT;
        const int chunk = tn * NWN + wn;
        if (chunk >= a.hp.chunks) return;
        const int n0 = tn * BN + wn * WN * 16 + 4 * lg;
        const int kt = a.hp.topk < KD ? a.hp.topk : KD;
        const bool whole = tn * BN + (wn + 1) * WN * 16 <= a.N;
        // The rows' first candidates, two round trips for all of them: fetched row by row they also waited for the stores of the
        // row before. The rest is read by the few lanes that hold one of the tokens, or rows with several.
        int x0[WM], several = 0;
        {
            int cb[WM], cn[WM];
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                const int row = tm * BM + (wm * WM + i) * 16 + lr, rowc = row < a.M ? row : a.M - 1;
                cb[i] = a.hp.cand_beg[rowc];
                cn[i] = row < a.M ? a.hp.cand_cnt[rowc] : 0;
            }
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                const int x = a.hp.cand_x[cb[i]];                // (a row without candidates names a place that exists)
                x0[i] = cn[i] > 0 ? x : -1;
                several |= (cn[i] > 1 ? 1 : 0) << i;
            }
        }
        static_for<0, WM>([&](auto ic) {                     // (a loop this long is not unrolled by itself, and acc must not be indexed at run time)
            constexpr int i = decltype(ic)::value;
            const int row = tm * BM + (wm * WM + i) * 16 + lr;
            RowStatT<KD> st;
            st.init();
            float v[WN * 4];
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[j * 4 + e] = acc[i][j][e];
            if (!whole) {
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[j * 4 + e] = n0 + j * 16 + e < a.N ? v[j * 4 + e] : -INFINITY;
            }
            // maximum, its id and the second largest value in one pass, four instructions an element
            float mx = -INFINITY, second = -INFINITY;
            int at = 0x7FFFFFFF - n0;                        // ids relative to n0
#pragma unroll
            for (int q = 0; q < WN * 4; ++q) {
                if constexpr (KD == 2) second = __builtin_amdgcn_fmed3f(v[q], mx, second);
                at = v[q] > mx ? q / 4 * 16 + q % 4 : at;    // ids ascend: earlier ties stay
                mx = fmaxf(mx, v[q]);
            }
            float sum = 0.f;
            if (mx != -INFINITY) {
#pragma unroll
                for (int q = 0; q < WN * 4; ++q) sum += __expf(v[q] - mx);
            }
            st.mx = mx; st.sum = sum; st.arg = n0 + at;
            bool plain = false;
            if constexpr (KD == 2) plain = __ballot(!(second < mx && second > -INFINITY)) == 0;
            if (plain) {
                // two different finite values head the list of every lane: the second one's id is where it first stands
                int at2 = 0;
#pragma unroll
                for (int q = WN * 4 - 1; q >= 0; --q) at2 = v[q] == second ? q / 4 * 16 + q % 4 : at2;
                st.tv[0] = mx; st.ti[0] = n0 + at;
                st.tv[KD - 1] = second; st.ti[KD - 1] = n0 + at2;
            } else {
                float thr_v = -INFINITY;
                int thr_i = 0x7FFFFFFF;
#pragma unroll
                for (int q = 0; q < WN * 4; ++q) {
                    const int n = n0 + q / 4 * 16 + q % 4;
                    if (n < a.N && before(v[q], n, thr_v, thr_i)) {
                        st.push_top(v[q], n);
#pragma unroll
                        for (int t = 0; t < KD; ++t) if (t == kt - 1) { thr_v = st.tv[t]; thr_i = st.ti[t]; }
                    }
                }
            }
            auto mine = [&](int x) { const int o = x - n0; return o >= 0 && o < WN * 16 && (o & 15) < 4; };
            if (x0[i] >= 0 && (mine(x0[i]) || ((several >> i) & 1))) {
                const int cb = a.hp.cand_beg[row], cn = a.hp.cand_cnt[row];
                for (int c = 0; c < cn; ++c) {
                    const int x = a.hp.cand_x[cb + c];
                    if (mine(x)) {
#pragma unroll
                        for (int q = 0; q < WN * 4; ++q)
                            if (x - n0 == q / 4 * 16 + q % 4) a.hp.cand_lx[cb + c] = v[q];
                    }
                }
            }
            if (a.hp.logits_dbg && row < a.M) {
#pragma unroll
                for (int j = 0; j < WN; ++j)
                    if (n0 + j * 16 < a.N)                                   // N is a multiple of 16
                        *reinterpret_cast<float4a4_t*>(a.hp.logits_dbg + (size_t)row * a.N + n0 + j * 16) = float4a4_t{v[j * 4], v[j * 4 + 1], v[j * 4 + 2], v[j * 4 + 3]};
            }
            st.merge_from_lane(16);
            st.merge_from_lane(32);
            if (lg == 0 && row < a.M) st.store(a.hp, row, chunk);
        });
        return;
    }
    float* const outf = a.outf + (size_t)kpart * a.M * a.N;
#pragma unroll
    for (int i = 0; i < WM; ++i) {
        const int row = tm * BM + (wm * WM + i) * 16 + lr;
        if (row >= a.M) continue;
        if constexpr (EPI == GEPI_SWIGLU) {
            static_assert(WN % 2 == 0, "gate and up fragments come in pairs");
#pragma unroll
            for (int j = 0; j < WN; j += 2) {
                const int feat = tn * (BN / 2) + (wn * WN + j) * 8 + 4 * lg;
                if (feat >= a.N) continue;                   // N is a multiple of 16
                Frag4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float gt = acc[i][j][e], up = acc[i][j + 1 < WN ? j + 1 : j][e];
                    o.h[e] = f32_to_f16(gt / (1.f + __expf(-gt)) * up);
                }
                *reinterpret_cast<u32x2*>(a.outh + (size_t)row * a.N + feat) = o.v2;
            }
        } else {
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                const int col = tn * BN + (wn * WN + j) * 16 + 4 * lg;
                if (col >= a.N) continue;
                *reinterpret_cast<float4_t*>(outf + (size_t)row * a.N + col) = acc[i][j];
            }
        }
    }
}

}  // namespace laser

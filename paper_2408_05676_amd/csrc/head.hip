// Fused output head + acceptance (Sec. 3.4 Eq. 7-8; greedy Eq. 4; correction rule of Sec. 2.1). Logits are never
// stored (unless a debug buffer is passed): every kernel that produces them reduces them at once to per-(row,
// vocabulary chunk) partial statistics (head_part.h); accept_rows_kernel merges a row's chunks and ranks the row's
// candidates, and accept_scan_kernel walks the nodes of a sequence.
//
// Pass 1, by row count M = B*(K+1):
//   M <= 16   lm_head_kernel: every wavefront owns a contiguous chunk of the vocabulary, streams those rows of the
//             head matrix once through the matrix cores against all verified rows and keeps the running statistics
//             in registers (chunk = wavefront).
//   M <= 80   the head matrix is read once. k <= 2: the tiled GEMM with one row tile (chunk = a wave's 32 columns). Longer lists, or
//             operands off the 16-byte grid: the kernel of gemm_mid.h with its head epilogue (chunk = workgroup, 64 or 128
//             vocabulary entries, a quarter of the lists to keep and to merge). Head alone, us, k = 2 / 5: 72 rows x 32000 at a
//             width of 2048 tiled 51 / 90, gemm_mid.h 54 / 78; 72 rows x 128256 at 4096 290 / 445 and 334 / 427; 17 rows x
//             32000 at 2048 44 / 66 and 45 / 61.
//   more      the LDS-tiled matrix-core GEMM of gemm_tile.h with its head epilogue (chunk = a wave's 128 columns); rows off
//             the 16-byte grid are copied onto it first (1024 rows at a 128 k vocabulary: 943..958 us, on the grid 942..952).
// Pass 2: a wavefront per row merges the per-chunk partials. The draft's rank is the number of partial-list entries
// ordered before it; if a chunk hides an entry that precedes the draft, that chunk already contributes
// >= LASER_MAX_TOPK >= k listed ones, so "rank < k" is exact. A wavefront per sequence then examines the nodes
// and emits accepted drafts plus the correction token.
#include <cmath>
#include <mutex>

#include "gemm_tile_plan.h"
#include "gemm_skinny.h"
#include "gemm_mid.h"
#include "state.h"

namespace laser {

constexpr int kHeadStreamMaxRows = 16;   // up to here lm_head_kernel; beyond, a GEMM with the head epilogue
constexpr int kHeadMidMaxRows = 80;      // up to here that GEMM streams the head matrix once; beyond, the tiled one

struct HeadArgs {
    const uint16_t* W; const uint16_t* H; int M, V, d, tiles_per_wave;
    HeadPart hp;
};

// One wavefront per sequence (lane i = node i): the candidates of every row. Node i of the pseudo-sequence (token
// tokens[b][i]) is a candidate of its parent's row (row parent + 1; row 0 is the pending token's): for a chain, node i
// of row i. Candidates of a row are stored next to each other, in pseudo-sequence order; nodes past n_nodes[b] and
// tokens outside the vocabulary are no candidates (node_cand = -1: never accepted).
__global__ __launch_bounds__(64) void head_cands_kernel(const int32_t* tokens, const int32_t* parent, const int32_t* n_nodes, int B, int K, int vocab,
                                                        int32_t* cand_beg, int32_t* cand_cnt, int32_t* cand_x, int32_t* node_cand, float* cand_lx) {
    __shared__ int prow[LASER_MAX_DRAFT + 1];          // parent row of node i, -1: no candidate
    __shared__ int cnt[LASER_MAX_DRAFT + 1], beg[LASER_MAX_DRAFT + 1];
    const int b = blockIdx.x, i = threadIdx.x, R = K + 1;
    int nn = n_nodes[b];
    nn = nn < 0 ? 0 : (nn > K ? K : nn);
    int x = -1, pr = -1;
    if (i < K) {
        x = tokens[(size_t)b * K + i];
        if (i < nn && x >= 0 && x < vocab) pr = tree_parent_of(parent, b, K, i, nn) + 1;
    }
    if (i < R) cnt[i] = 0;
    prow[i] = pr;
    __syncthreads();
    if (pr >= 0) atomicAdd(&cnt[pr], 1);
    __syncthreads();
    if (i == 0) {
        int off = b * K;
        for (int r = 0; r < R; ++r) { beg[r] = off; off += cnt[r]; }
    }
    __syncthreads();
    if (i < R) { cand_beg[(size_t)b * R + i] = beg[i]; cand_cnt[(size_t)b * R + i] = cnt[i]; }
    if (i < K) {
        int c = -1;
        if (pr >= 0) {
            int before_me = 0;                          // earlier nodes below the same row keep their order
            for (int j = 0; j < i; ++j) before_me += prow[j] == pr ? 1 : 0;
            c = beg[pr] + before_me;
            cand_x[c] = x;
            cand_lx[c] = -INFINITY;
        }
        node_cand[(size_t)b * K + i] = c;
    }
}

template <int MB>
__global__ __launch_bounds__(256) void lm_head_kernel(HeadArgs a) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int chunk = blockIdx.x * 4 + wave;
    if (chunk >= a.hp.chunks) return;
    const int ntiles = a.V / 16;
    const int t0 = chunk * a.tiles_per_wave, t1 = min(ntiles, t0 + a.tiles_per_wave);
    const int row0 = blockIdx.y * MB * 16;

    RowStat st[MB];
    int cb[MB], cn[MB], x0[MB];           // the row's candidates; the first one's token is kept in a register
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        st[mb].init();
        const int row = row0 + mb * 16 + r;
        cb[mb] = row < a.M ? a.hp.cand_beg[row] : 0;
        cn[mb] = row < a.M ? a.hp.cand_cnt[row] : 0;
        x0[mb] = cn[mb] > 0 ? a.hp.cand_x[cb[mb]] : -1;
    }
    for (int t = t0; t < t1; ++t) {
        float4_t acc[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = float4_t{0.f, 0.f, 0.f, 0.f};
        wave_gemm_tile<MB, false>(a.W + (size_t)t * 16 * a.d, (size_t)a.d, a.H, nullptr, a.d, a.M, row0, 0, a.d, acc);
        const int n = t * 16 + 4 * g;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) st[mb].add(acc[mb][i], n + i);
            auto pick = [&](int c) { return c == 0 ? acc[mb][0] : c == 1 ? acc[mb][1] : c == 2 ? acc[mb][2] : acc[mb][3]; };
            if (x0[mb] >= n && x0[mb] < n + 4) a.hp.cand_lx[cb[mb]] = pick(x0[mb] - n);
            for (int c = 1; c < cn[mb]; ++c) {                   // further children of a tree node
                const int x = a.hp.cand_x[cb[mb] + c];
                if (x >= n && x < n + 4) a.hp.cand_lx[cb[mb] + c] = pick(x - n);
            }
            const int row = row0 + mb * 16 + r;
            if (a.hp.logits_dbg && row < a.M)
                *reinterpret_cast<float4*>(a.hp.logits_dbg + (size_t)row * a.V + n) =
                    make_float4(acc[mb][0], acc[mb][1], acc[mb][2], acc[mb][3]);
        }
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        st[mb].merge_from_lane(16);
        st[mb].merge_from_lane(32);
        const int row = row0 + mb * 16 + r;
        if (g == 0 && row < a.M) st[mb].store(a.hp, row, chunk);
    }
}

struct AcceptArgs {
    const float* hp_max; const float* hp_sum; const int32_t* hp_arg; const float* hp_topv; const int32_t* hp_topi;
    const int32_t* cand_beg; const int32_t* cand_cnt; const int32_t* cand_x; const float* cand_lx; const int32_t* node_cand;
    const int32_t* tokens; const int32_t* parent; const int32_t* n_nodes;      // parent == NULL: a chain
    int M, B, K, chunks, topk, mode; float p;
    float* row_mx; float* row_sum; int32_t* row_arg; int32_t* cand_rank;       // between the two kernels
    int32_t* accept_len; int32_t* out_tokens; int32_t* accept_path;            // accept_path may be NULL
};

// Pass 2a, a wavefront per row: the row's chunks are merged (softmax statistics, arg-max) and every candidate of the
// row gets its rank, the number of vocabulary entries ahead of it. A chunk's list is read only when the chunk's
// largest entry is ahead of one of the candidates (otherwise nothing in the chunk is).
constexpr int kCandPass = 4;          // candidates ranked per pass over a row's chunks
__global__ __launch_bounds__(256) void accept_rows_kernel(AcceptArgs a) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= a.M) return;
    const int cb = a.cand_beg[row], cn = a.cand_cnt[row];
    for (int c0 = 0; c0 < (cn > 0 ? cn : 1); c0 += kCandPass) {
        int x[kCandPass];
        float lx[kCandPass];
#pragma unroll
        for (int j = 0; j < kCandPass; ++j) {
            const bool have = c0 + j < cn;
            x[j] = have ? a.cand_x[cb + c0 + j] : -1;
            lx[j] = have ? a.cand_lx[cb + c0 + j] : -INFINITY;
        }
        float mx = -INFINITY, sum = 0.f;
        int arg = 0x7FFFFFFF, ahead[kCandPass] = {0, 0, 0, 0};
        // A lane's records, eight requested at a time: one by one, the 1000 chunks of 72 rows at a vocabulary of 32000 were
        // sixteen round trips in a row (22.4 us; 18.8 with the lists still read one by one, 16.86 so).
        constexpr int kRec = 8;
        for (int c1 = lane; c1 < a.chunks; c1 += 64 * kRec) {
            float vm[kRec], vs[kRec];
            int va[kRec];
#pragma unroll
            for (int u = 0; u < kRec; ++u) {
                const int c = c1 + 64 * u < a.chunks ? c1 + 64 * u : c1;
                const size_t o = (size_t)row * a.chunks + c;
                vm[u] = a.hp_max[o]; vs[u] = a.hp_sum[o]; va[u] = a.hp_arg[o];
            }
#pragma unroll
            for (int u = 0; u < kRec; ++u) {
                if (c1 + 64 * u >= a.chunks) break;
                const float cm = vm[u], cs = vs[u];
                const int ca = va[u];
                const float M = fmaxf(mx, cm);
                sum = sum * __expf(mx - M) + cs * __expf(cm - M);
                if (before(cm, ca, mx, arg)) arg = ca;
                mx = M;
            }
            // records whose list may hold entries ahead of a candidate; the first two entries of all of them together as well
            uint32_t open = 0;
#pragma unroll
            for (int u = 0; u < kRec; ++u)
#pragma unroll
                for (int j = 0; j < kCandPass; ++j)
                    open |= (c1 + 64 * u < a.chunks && x[j] >= 0 && va[u] != x[j] && before(vm[u], va[u], lx[j], x[j]) ? 1u : 0u) << u;
            if (!open) continue;
            float2 tv[kRec];
            int2 ti[kRec];
#pragma unroll
            for (int u = 0; u < kRec; ++u) {
                const size_t o = ((size_t)row * a.chunks + (((open >> u) & 1u) ? c1 + 64 * u : c1)) * KT;
                tv[u] = *reinterpret_cast<const float2*>(a.hp_topv + o);
                ti[u] = *reinterpret_cast<const int2*>(a.hp_topi + o);
            }
            auto count = [&](float v, int i) {
#pragma unroll
                for (int j = 0; j < kCandPass; ++j) ahead[j] += (x[j] >= 0 && i != x[j] && before(v, i, lx[j], x[j])) ? 1 : 0;
            };
#pragma unroll
            for (int u = 0; u < kRec; ++u)
                if ((open >> u) & 1u) {
                    count(tv[u].x, ti[u].x);
                    if (a.topk > 1) count(tv[u].y, ti[u].y);                // (a record holds topk entries, possibly no more)
                    for (int t = 2; t < a.topk && t < KT; ++t) {
                        const size_t o = ((size_t)row * a.chunks + c1 + 64 * u) * KT + t;
                        count(a.hp_topv[o], a.hp_topi[o]);
                    }
                }
        }
        for (int off = 32; off > 0; off >>= 1) {
            const float omx = __shfl_xor(mx, off), osum = __shfl_xor(sum, off);
            const int oarg = __shfl_xor(arg, off);
#pragma unroll
            for (int j = 0; j < kCandPass; ++j) ahead[j] += __shfl_xor(ahead[j], off);
            const float M = fmaxf(mx, omx);
            if (M != -INFINITY) sum = sum * __expf(mx - M) + osum * __expf(omx - M);
            if (before(omx, oarg, mx, arg)) arg = oarg;
            mx = M;
        }
        if (lane == 0) {
            if (c0 == 0) { a.row_mx[row] = mx; a.row_sum[row] = sum; a.row_arg[row] = arg; }
#pragma unroll
            for (int j = 0; j < kCandPass; ++j)
                if (c0 + j < cn) a.cand_rank[cb + c0 + j] = ahead[j];
        }
    }
}

// Pass 2b, a wavefront per sequence, lane i = node i: a node is verified iff its parent is and its token passes the rule
// against its parent's row; the deepest verified node -- the first one among equally deep -- ends the accepted branch,
// and the branch's tokens plus the arg-max of its last row are emitted (Sec. 3.4; Sec. 2.1 for the correction token).
// For a chain this is the longest accepted prefix. Bound by dependent loads: the nodes' own are made by all lanes at
// once, and the walk down the tree -- the nodes verified in turn t are those of depth t -- runs on lane masks.
__global__ __launch_bounds__(64) void accept_scan_kernel(AcceptArgs a) {
    static_assert(LASER_MAX_DRAFT < 64, "a lane per node and one for the correction token");
    const int b = blockIdx.x, i = threadIdx.x, R = a.K + 1;
    int nn = a.n_nodes[b];
    nn = nn < 0 ? 0 : (nn > a.K ? a.K : nn);
    int par = -1, tok = -1;
    bool ok = false;
    if (i < nn) {
        par = tree_parent_of(a.parent, b, a.K, i, nn);
        tok = a.tokens[(size_t)b * a.K + i];
        const int c = a.node_cand[(size_t)b * a.K + i];
        const int prow = b * R + par + 1;
        const float mx = a.row_mx[prow], sum = a.row_sum[prow];
        if (c >= 0) {
            const int rank = a.cand_rank[c];
            const float q = __expf(a.cand_lx[c] - mx) / sum;
            const bool in_k = rank < a.topk, above = q > a.p, top1 = rank == 0;
            ok = a.mode == LASER_MODE_RV ? (in_k && above)
               : a.mode == LASER_MODE_RV_OR_TOP1 ? (top1 || (in_k && above))
               : a.mode == LASER_MODE_TOPK_ONLY ? in_k : (top1 || above);
        }
    }
    unsigned long long last = __ballot(ok && par < 0);                // the verified nodes of one depth
    int depth = 0;
    while (last) {                                                     // a parent comes before its children: at most nn turns
        ++depth;
        const unsigned long long now = __ballot(ok && par >= 0 && ((last >> par) & 1ull));
        if (!now) break;
        last = now;
    }
    const int best = depth ? __ffsll(last) - 1 : -1;
    int out = -1, path = -1;
    for (int j = depth - 1, n = best; j >= 0; --j) {
        const int t = __shfl(tok, n);
        if (i == j) { out = t; path = n; }
        n = __shfl(par, n);
    }
    if (i == depth) out = a.row_arg[b * R + best + 1];
    if (i == 0) a.accept_len[b] = depth;
    if (i < R) a.out_tokens[(size_t)b * R + i] = out;
    if (a.accept_path && i < a.K) a.accept_path[(size_t)b * a.K + i] = path;
}

// Device buffers of the head: the rows' candidate lists, and per (row, vocabulary chunk) the partial statistics that
// pass 1 leaves for the acceptance kernels, and the per-row results between those two.
struct HeadBufs {
    int32_t* cand_beg; int32_t* cand_cnt; int32_t* cand_x; int32_t* node_cand; float* cand_lx;
    float* hp_max; float* hp_sum; int32_t* hp_arg; float* hp_topv; int32_t* hp_topi;
    float* row_mx; float* row_sum; int32_t* row_arg; int32_t* cand_rank;
};

// Chunks per row of the pass-1 kernel a row count takes (the partial arrays must hold rows x this many records).
static int head_chunks_for(const Model* m, int M) {
    if (M <= kHeadStreamMaxRows) return m->head_chunks;
    if (M <= kHeadMidMaxRows && m->d.d_model % kGemmKStep == 0)
        return (m->d.vocab + 31) / 32;                             // at most: the tiled form's waves of 32 columns
    return (m->d.vocab + 127) / 128;
}
// The records a call may need: the most over all row counts.
size_t head_records(const Model* m) {
    const size_t R = m->d.max_rows;
    size_t n = R * (size_t)head_chunks_for(m, kHeadMidMaxRows + 1);
    for (int M : {kHeadStreamMaxRows, kHeadMidMaxRows}) n = std::max(n, std::min<size_t>(R, M) * head_chunks_for(m, M));
    return n;
}

// Rows off the 16-byte grid onto it, for loads into LDS; n8: groups of eight values.
__global__ __launch_bounds__(256) void copy_rows_kernel(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, size_t n8) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n8) *reinterpret_cast<u32x4*>(dst + i * 8) = *reinterpret_cast<const u32x4a2*>(src + i * 8);
}

// candidates -> pass 1 -> acceptance. Allocates nothing up to 80 rows. tokens / parent / n_nodes: the drafts as a pseudo-sequence
// (parent == NULL: a chain, n_nodes = draft_len). few16: the fp16 copy of the head matrix for 17..80 rows and k <= 2, or NULL for
// the caller's own matrix.
static int run_head_bufs(Model* m, const uint16_t* few16, const uint16_t* h, const int32_t* tokens, const int32_t* parent, const int32_t* n_nodes, int B, int K,
                         int topk, float p, int mode, int32_t* accept_len, int32_t* out_tokens, int32_t* accept_path, float* logits_dbg,
                         const HeadBufs& hb, hipStream_t stream) {
    const int M = B * (K + 1), V = m->d.vocab, dm = m->d.d_model;
    hipLaunchKernelGGL(head_cands_kernel, dim3(B), dim3(64), 0, stream, tokens, parent, n_nodes, B, K, V,
                       hb.cand_beg, hb.cand_cnt, hb.cand_x, hb.node_cand, hb.cand_lx);
    HeadPart hp{hb.cand_beg, hb.cand_cnt, hb.cand_x, hb.cand_lx, hb.hp_max, hb.hp_sum, hb.hp_arg, hb.hp_topv, hb.hp_topi, 0, topk, logits_dbg};
    if (M <= kHeadStreamMaxRows) {
        const int ntiles = V / 16;
        const int tpw = (ntiles + 1023) / 1024;
        hp.chunks = m->head_chunks;
        HeadArgs a{m->d.wlm, h, M, V, dm, tpw, hp};
        dim3 grid((unsigned)((m->head_chunks + 3) / 4), 1u);         // at most 16 rows: one row tile
        hipLaunchKernelGGL(lm_head_kernel<1>, grid, dim3(256), 0, stream, a);
    } else if (M <= kHeadMidMaxRows && topk <= 2 && m->mid_waves == 0 && (few16 || on_16_byte_grid(m->d.wlm)) && on_16_byte_grid(h)) {
        hp.chunks = (V + 31) / 32;
        GemmTileArgs t{few16 ? few16 : m->d.wlm, h, nullptr, M, V, dm, 0, 0, 1, nullptr, nullptr, hp};
        launch_few_head(t, few16 != nullptr, stream);
    } else if (M <= kHeadMidMaxRows && dm % kGemmKStep == 0) {
        const GemmMidPlan pl = gemm_mid_plan(M, V, dm, 1, false, 0);
        hp.chunks = (V / 16 + pl.NW - 1) / pl.NW;                     // = workgroups of the launch
        GemmMidArgs t{m->d.wlm, h, nullptr, M, V, dm, nullptr, nullptr, nullptr, hp};
        launch_gemm_mid<EPI_HEAD, false>(t, pl, stream);
    } else {
        hp.chunks = (V + 127) / 128;
        if (m->f16_copies && !m->w16[4]) {         // first many-row head: widen the head matrix to fp16 once
            if (const int rc = widen_copies(m, kHeadMatrix, stream)) return rc;
        }
        if (!on_16_byte_grid(h)) {
            const size_t n8 = (size_t)M * dm / 8;
            hipLaunchKernelGGL(copy_rows_kernel, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, stream, h, m->xn, n8);
            h = m->xn;
        }
        int ncu = 0;
        LASER_HIP_CHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, 0));
        GemmTileArgs t{m->w16[4] ? m->w16[4] : m->d.wlm, h, nullptr, M, V, dm, 0, 0, 1, nullptr, nullptr, hp};
        t.want_tile = m->tile;
        launch_tile_head(t, m->w16[4] != nullptr, ncu, stream);
    }
    AcceptArgs aa{hb.hp_max, hb.hp_sum, hb.hp_arg, hb.hp_topv, hb.hp_topi, hb.cand_beg, hb.cand_cnt, hb.cand_x, hb.cand_lx, hb.node_cand,
                  tokens, parent, n_nodes, M, B, K, hp.chunks, topk, mode, p, hb.row_mx, hb.row_sum, hb.row_arg, hb.cand_rank,
                  accept_len, out_tokens, accept_path};
    hipLaunchKernelGGL(accept_rows_kernel, dim3((M + 3) / 4), dim3(256), 0, stream, aa);
    hipLaunchKernelGGL(accept_scan_kernel, dim3(B), dim3(64), 0, stream, aa);
    LASER_HIP_CHECK(hipGetLastError());
    return LASER_OK;
}

// few_copy: a step's own head, which up to 80 rows takes the copy that the step has made. The head alone (laser_verify_head)
// reads the caller's matrix at every call there, allocates nothing and waits for nothing.
int run_head(Model* m, bool few_copy, const uint16_t* h, const int32_t* tokens, const int32_t* parent, const int32_t* n_nodes, int B, int K,
             int topk, float p, int mode, int32_t* accept_len, int32_t* out_tokens, int32_t* accept_path, float* logits_dbg,
             hipStream_t stream) {
    HeadBufs hb{m->cand_beg, m->cand_cnt, m->cand_x, m->node_cand, m->cand_lx, m->hp_max, m->hp_sum, m->hp_arg, m->hp_topv, m->hp_topi,
                m->row_mx, m->row_sum, m->row_arg, m->cand_rank};
    return run_head_bufs(m, few_copy ? m->w16[4] : nullptr, h, tokens, parent, n_nodes, B, K, topk, p, mode, accept_len, out_tokens, accept_path, logits_dbg, hb, stream);
}

// ---- the head without any allocation ------------------------------------------------------------------------
// The partial statistics live in a file-scope device array instead of the model handle's workspace. Each GPU holds
// its own copy of the array at its own address: the address is taken once per device with that device current.
constexpr int kStaticRows = kHeadStreamMaxRows;      // rows one call may verify
constexpr int kStaticChunks = 1024;                  // vocabulary chunks (laser_model_create never makes more)
struct HeadScratch {
    float hp_max[kStaticRows * kStaticChunks];
    float hp_sum[kStaticRows * kStaticChunks];
    int32_t hp_arg[kStaticRows * kStaticChunks];
    float hp_topv[kStaticRows * kStaticChunks * KT];
    int32_t hp_topi[kStaticRows * kStaticChunks * KT];
    int32_t cand_beg[kStaticRows], cand_cnt[kStaticRows], cand_x[kStaticRows], node_cand[kStaticRows];
    float cand_lx[kStaticRows];
    float row_mx[kStaticRows], row_sum[kStaticRows];
    int32_t row_arg[kStaticRows], cand_rank[kStaticRows];
};
static __device__ __align__(256) unsigned char scratch[sizeof(HeadScratch)];      // 1.19 MiB per GPU, for the life of the process

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices];             // device address of `scratch` on each GPU, once known

static int head_scratch(HeadScratch** out) {
    int dev = -1;
    LASER_HIP_CHECK(hipGetDevice(&dev));
    LASER_REQUIRE(dev >= 0 && dev < kMaxDevices, LASER_E_LIMIT, "device ordinal %d beyond %d", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        LASER_HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        LASER_REQUIRE(ptr != nullptr, LASER_E_HIP, "hipGetSymbolAddress returned no address for the head scratch");
        g_scratch_ptr[dev] = ptr;
    }
    *out = reinterpret_cast<HeadScratch*>(g_scratch_ptr[dev]);
    return LASER_OK;
}

int run_head_static(Model* m, const uint16_t* h, const int32_t* drafts, const int32_t* draft_len, int B, int K,
                    int topk, float p, int mode, int32_t* accept_len, int32_t* out_tokens, hipStream_t stream) {
    const int M = B * (K + 1);
    LASER_REQUIRE(M <= kStaticRows, LASER_E_LIMIT, "B*(K+1) = %d rows exceed the %d this entry point verifies per call", M, kStaticRows);
    LASER_REQUIRE(m->head_chunks <= kStaticChunks, LASER_E_LIMIT, "vocabulary of %d needs %d chunks, the static scratch holds %d",
                  m->d.vocab, m->head_chunks, kStaticChunks);
    HeadScratch* sc = nullptr;
    int rc = head_scratch(&sc);
    if (rc) return rc;
    // Nothing in the array has to start at zero: head_cands_kernel rewrites the candidate lists of the call's rows, and
    // lm_head_kernel overwrites every (row, chunk) record that the acceptance kernels read.
    HeadBufs hb{sc->cand_beg, sc->cand_cnt, sc->cand_x, sc->node_cand, sc->cand_lx, sc->hp_max, sc->hp_sum, sc->hp_arg, sc->hp_topv, sc->hp_topi,
                sc->row_mx, sc->row_sum, sc->row_arg, sc->cand_rank};
    return run_head_bufs(m, nullptr, h, drafts, nullptr, draft_len, B, K, topk, p, mode, accept_len, out_tokens, nullptr, nullptr, hb, stream);
}

}  // namespace laser

// Retrieval pool: construction of the regrouped pool and its suffix index on the host (few occurrences, or no memory on the
// device; pool_index.hip builds the others), and the per-context lookup + frequency-greedy chain kernel (Sec. 3.2 pool
// construction, Sec. 3.3 Eq. 5).
//
// Index layout (all device resident, immutable after the build):
//   P[N]        int32   tokens, sub-pools laid out by ascending key
//   seq_end[N]  uint32  per position: one past the last position of its sequence
//   sa[Ne]      uint32  every position that has an in-sequence successor, sorted inside its
//                       sub-pool by the text read backwards from it (P[e], P[e-1], ... up to n_max
//                       tokens, "before the sequence start" ordering first), then by position.
//                       All occurrences of any n-gram (n <= n_max) are therefore one contiguous run of
//                       sa. Only the runs of n_max-grams are position-ascending: inside the run of a shorter
//                       n-gram the order is set by the tokens further back first, so the smallest position
//                       of a run has to be searched for (the lookup takes an explicit minimum).
//   table[cap]  16 B    open addressing (linear probing, load <= 0.5): (key, n, n-gram) -> run in sa
// A lookup hashes (key, n, suffix), probes, and confirms a hit by comparing key, n and the actual
// tokens at the run's first occurrence, so hash collisions cannot produce a false match.
#include <algorithm>
#include <cstring>
#include <numeric>
#include <thread>
#include <type_traits>
#include <vector>

#include "pool.h"

namespace laser {

// ------------------------------------------------------------------------------------ kernel
constexpr int kCand = 512;         // occurrences a wave keeps in LDS (more: streamed from the index, re-checked against the chain); see retrieve_kernel
constexpr int kVote = 512;         // vote-table slots (power of two; wider votes are partitioned)
constexpr int kWideVote = 1024;    // ... up to kFourGroupsMax contexts, for votes out of LDS that overflow the smaller table
// Groups of 64 occurrences whose loads a vote over a streamed run has in flight together. A wave alone waits for memory: four.
// Beyond 1024 contexts the waves of a compute unit cover each other's waits and four groups each outgrow its cache: one. A run
// of 10000 occurrences, chains of 16, one group / four, us: 8 contexts 12075 / 9417, 1024 contexts 12278 / 10199, 2048
// contexts 12590 / 19220.
constexpr int kFourGroupsMax = 1024;
constexpr int kEmptyTok = -1;
constexpr int kOwnMax = LASER_MAX_OWN_TEXT;   // tokens of a sequence's own text (temporary branch) a lookup can take

__device__ inline uint32_t fmix32(uint32_t h) {   // bijective 32-bit mixer
    h ^= h >> 16; h *= 0x85EBCA6Bu; h ^= h >> 13; h *= 0xC2B2AE35u; h ^= h >> 16;
    return h;
}

struct RetrieveArgs {
    const int32_t* P; const uint32_t* seq_end; const uint32_t* sa; const IndexEntry* table;
    uint64_t cap_mask;
    const int64_t* keys; const int32_t* ctx_tail;
    int B, n_min, n_max, K, min_tokens;
    int32_t* drafts; int32_t* draft_len; int32_t* match_n; int64_t* pool_index;
    // temporary branch (Sec. 3.2): the sequence's own text, searched as one more sequence of its key's sub-pool,
    // placed after the pool's sequences; NULL = none
    const int32_t* own; const int32_t* own_len; int own_cap;
};

// The chain from its step j0 (1-based; steps before it are done) to its end, over at most 64 Q survivors: pool occurrences
// cand[0 .. m) and own-text occurrences own_cand[0 .. mo), number i with lane i % 64. Returns the chain's length (j0 - 1: no
// survivor has a successor) and this lane's smallest surviving positions. Bound by one memory round trip per kAhead steps;
// with the vote table of retrieve_kernel alone a step was a round trip and four passes over LDS: 4096 lookups of 16 tokens in
// a pool of 750 k 103 -> 37 us (90 us with one survivor per lane only: the hot keys' lookups, a few hundred occurrences
// thinned by a tenth per step, decide when the launch ends).
// A ballot counts one token, in 0.13 us at Q = 4: a vote that is still open after kBallots of them goes through the vote
// table (vote_tok, vote_cnt: kVote slots, more than there are voters). 2048 lookups over 256 occurrences, all with successors of
// their own, K = 1 / 4 / 16: ballots alone 47.8 / 48.8 / 56.4 us, now 14.6 / 14.3 / 27.4; votes by the table alone 14.1 /
// 20.1 / 45.0. Occurrences that agree but for a tenth per step: ballots alone 10.1 / 11.1 / 20.0, now 12.5 / 9.6 / 20.3,
// the table alone 12.0 / 29.4 / 75.2.
template <int Q, int kAhead, bool OWN>
__device__ __forceinline__ int follow_lanes(const RetrieveArgs& a, const uint32_t* cand, const uint32_t* cand_end, uint32_t m, const uint32_t* own_cand,
                                   const int32_t* own, uint32_t own_len, uint32_t mo, int j0, int* chain, int* vote_tok, int* vote_cnt,
                                   uint32_t& lane_min, uint32_t& lane_own) {
    constexpr int kBallots = 8;
    static_assert(64 * Q < kVote, "every voter may bring a token of its own");
    const int lane = threadIdx.x;
    uint32_t e[Q], end[Q];
    const int32_t* text[Q];
    bool live[Q], mine_own[Q];
#pragma unroll
    for (int s = 0; s < Q; ++s) {
        const uint32_t i = (uint32_t)(s * 64 + lane);
        live[s] = i < m + mo;
        mine_own[s] = OWN && live[s] && i >= m;
        e[s] = mine_own[s] ? own_cand[OWN ? i - m : 0] : live[s] ? cand[i] : 0u;
        end[s] = mine_own[s] ? own_len : live[s] ? cand_end[i] : 0u;
        text[s] = mine_own[s] ? own : a.P;
    }
    int len = j0 - 1;
    bool more = true;
    for (int j = j0, next; j <= a.K && more; j = next) {
        next = j + kAhead;
        int open = 0;                                  // step whose vote the ballots left open
        int tok[Q][kAhead];
#pragma unroll
        for (int s = 0; s < Q; ++s)
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
                tok[s][q] = live[s] && j + q <= a.K && e[s] + (uint32_t)(j + q) < end[s] ? text[s][e[s] + (uint32_t)(j + q)] : 0;
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            bool ok[Q];
            uint64_t rest[Q], win[Q];
            int left = 0;                              // voters not counted yet
#pragma unroll
            for (int s = 0; s < Q; ++s) {
                ok[s] = more && live[s] && j + q <= a.K && e[s] + (uint32_t)(j + q) < end[s];
                rest[s] = __ballot(ok[s]);
                win[s] = 0;
                left += __popcll(rest[s]);
            }
            int win_tok = 0, win_cnt = 0, ballots = 0;
#pragma unroll
            for (int s = 0; s < Q; ++s)
                while (rest[s] && left >= win_cnt) {   // larger count, then smaller token id: an equal count can still win
                    if (Q > 1 && ballots++ == kBallots) { left = -1; break; }
                    const int t = __builtin_amdgcn_readlane(tok[s][q], __ffsll((unsigned long long)rest[s]) - 1);
                    uint64_t same[Q];
                    int c = 0;
#pragma unroll
                    for (int u = 0; u < Q; ++u) {
                        same[u] = u < s ? 0ull : __ballot(ok[u] && tok[u][q] == t);
                        c += __popcll(same[u]);
                        rest[u] &= ~same[u];
                    }
                    left -= c;
                    if (c > win_cnt || (c == win_cnt && t < win_tok)) {
                        win_cnt = c; win_tok = t;
#pragma unroll
                        for (int u = 0; u < Q; ++u) win[u] = same[u];
                    }
                }
            if (Q > 1 && left < 0) { open = j + q; win_cnt = 0; }
            if (win_cnt == 0) { more = false; continue; }          // no survivor has a successor left, or K steps are done
            if (lane == 0) chain[j + q - 1] = win_tok;
            len = j + q;
#pragma unroll
            for (int s = 0; s < Q; ++s) live[s] = (win[s] >> lane) & 1ull;
        }
        if (Q > 1 && open) {
            int t[Q];
#pragma unroll
            for (int s = 0; s < Q; ++s) t[s] = live[s] && e[s] + (uint32_t)open < end[s] ? text[s][e[s] + (uint32_t)open] : -1;
            for (int i = lane; i < kVote; i += 64) { vote_tok[i] = kEmptyTok; vote_cnt[i] = 0; }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < Q; ++s)
                if (t[s] >= 0) {
                    uint32_t at = fmix32((uint32_t)t[s]) & (kVote - 1);
                    for (;;) {
                        const int was = atomicCAS(&vote_tok[at], kEmptyTok, t[s]);
                        if (was == kEmptyTok || was == t[s]) break;
                        at = (at + 1) & (kVote - 1);
                    }
                    atomicAdd(&vote_cnt[at], 1);
                }
            __syncthreads();
            int bt = 0, bc = 0;
            for (int i = lane; i < kVote; i += 64) {
                const int c = vote_cnt[i], tk = vote_tok[i];
                if (c > bc || (c == bc && c > 0 && tk < bt)) { bc = c; bt = tk; }
            }
            for (int off = 32; off > 0; off >>= 1) {
                const int oc = __shfl_xor(bc, off), ot = __shfl_xor(bt, off);
                if (oc > bc || (oc == bc && oc > 0 && ot < bt)) { bc = oc; bt = ot; }
            }
            __syncthreads();
            if (lane == 0) chain[open - 1] = bt;
            len = open;
#pragma unroll
            for (int s = 0; s < Q; ++s) live[s] = t[s] == bt;
            next = open + 1;
            more = true;
        }
    }
    lane_min = lane_own = 0xFFFFFFFFu;
#pragma unroll
    for (int s = 0; s < Q; ++s) {
        if (live[s] && !mine_own[s]) lane_min = min(lane_min, e[s]);
        if (live[s] && mine_own[s]) lane_own = min(lane_own, e[s]);
    }
    return len;
}

// One wavefront (= one workgroup of 64 lanes) per context. OWN: with the temporary branch. Occurrences in the own
// text are found by a scan of it (it is at most kOwnMax tokens and the wave has it in L2 anyway), always kept
// in LDS (own_cand, position-ascending) and take part in every vote and filter next to the pool's.
template <bool OWN, int kGroups>
__global__ __launch_bounds__(64) void retrieve_kernel(RetrieveArgs a) {
    // Up to kFourGroupsMax contexts a compute unit has few waves and LDS to spare: twice the occurrences are kept, the vote table is
    // larger, and votes that are likely to agree go by ballot at once (below).
    constexpr bool kWide = kGroups == 4;
    constexpr int kCand = kWide ? 1024 : laser::kCand, kTable = kWide ? kWideVote : kVote;
    __shared__ uint32_t cand[kCand];
    // Beside each occurrence kept in LDS: the end of its sequence, and the successor token the current vote read for
    // it (-1: none). The filter that follows a vote then needs no memory round trip at all, the vote one instead of
    // two -- the lookup is a chain of dependent round trips, and these were three of the four per chain step.
    __shared__ uint32_t cand_end[kCand];
    __shared__ int cand_tok[kCand];
    __shared__ uint32_t own_cand[OWN ? kOwnMax : 1];
    __shared__ int vote_tok[kTable];
    __shared__ int vote_cnt[kTable];
    __shared__ int chain[LASER_MAX_DRAFT + 1];
    __shared__ int best_chain[LASER_MAX_DRAFT + 1];
    __shared__ int sh_distinct;

    const int b = blockIdx.x;
    const int lane = threadIdx.x;
    const int64_t key = a.keys[b];
    const int32_t* tail = a.ctx_tail + (size_t)b * a.n_max;

    int valid = 0;
    while (valid < a.n_max && tail[a.n_max - 1 - valid] >= 0) ++valid;
    const int32_t* own = OWN ? a.own + (size_t)b * a.own_cap : nullptr;
    const uint32_t own_len = OWN ? (uint32_t)min(max(a.own_len[b], 0), a.own_cap) : 0u;

    int best_len = 0, best_n = 0;
    long long best_idx = -1;
    int res_len = 0, res_n = 0;
    long long res_idx = -1;
    bool done = false;

    const int n_hi = valid < a.n_max ? valid : a.n_max;
    for (int n = n_hi; n >= a.n_min && !done && a.K > 0; --n) {
        // ---- index probe (every lane does the same probe; addresses are uniform) ----
        const int32_t* w = tail + (a.n_max - n);
        uint64_t slot = ngram_hash(key, n, w) & a.cap_mask;
        uint32_t start = 0, count = 0;
        for (;;) {
            IndexEntry e = a.table[slot];
            if (e.count_n == 0) break;
            if (e.key == key && (int)(e.count_n >> 28) == n) {
                uint32_t e0 = a.sa[e.start];
                bool same = true;
                for (int i = 0; i < n; ++i) same = same && (a.P[e0 - (n - 1) + i] == w[i]);
                if (same) { start = e.start; count = e.count_n & 0x0FFFFFFFu; break; }
            }
            slot = (slot + 1) & a.cap_mask;
        }
        // ---- occurrences in the own text: positions e with own[e-n+1..e] == w and a successor e+1 < own_len ----
        uint32_t mo = 0;
        if constexpr (OWN) {
            for (uint32_t e0 = (uint32_t)(n - 1); e0 + 1 < own_len; e0 += 64) {
                const uint32_t e = e0 + lane;
                bool hit = e + 1 < own_len;
                for (int i = 0; i < n && hit; ++i) hit = own[e - (n - 1) + i] == w[i];
                const uint64_t mask = __ballot(hit);
                if (hit) own_cand[mo + __popcll(mask & ((1ull << lane) - 1ull))] = e;
                mo += __popcll(mask);
            }
            __syncthreads();
        }
        if (count == 0 && mo == 0) continue;

        // ---- frequency-greedy chain over the occurrences sa[start .. start+count) ----
        // Survivors are either materialised in LDS (m <= kCand) or, while there are too many,
        // re-derived from the run by re-checking the chain so far.
        bool in_lds = count <= (uint32_t)kCand;
        uint32_t m = count;
        if (in_lds)
            for (uint32_t i = lane; i < count; i += 64) {         // (four groups requested together held up lookups of few by 3 %)
                const uint32_t e = a.sa[start + i];
                cand[i] = e;
                cand_end[i] = a.seq_end[e];
            }
        __syncthreads();

        int len = 0;
        bool in_lanes = false;                     // the survivors ended up one to a lane
        uint32_t lane_min = 0xFFFFFFFFu, lane_own = 0xFFFFFFFFu;      // ... their smallest positions, pool and own text
        for (int j = 1; j <= a.K; ++j) {
            // At most 256 survivors: each lane follows one, or up to four, to the end. Their next tokens are requested eight at
            // a time (neighbours in memory; one at a time where four lanes' worth have four steps or fewer to go: a vote may
            // end most of them), a vote is a ballot per distinct token, ended when no other token can win, and the filter
            // is the winner's lane masks: no LDS pass, one memory round trip for eight steps. With one or two steps to go
            // ballots pay off for fewer: 64 occurrences that all differ, 2048 lookups, K = 1 / 2: 12.7 / 12.8 us, by the
            // vote table 9.5 / 10.4.
            const int steps = a.K - j + 1;
            if (in_lds && m + mo <= (steps > 1 ? 256u : 32u)) {
                in_lanes = true;
                auto follow = [&](auto q, auto ahead) {
                    len = follow_lanes<decltype(q)::value, decltype(ahead)::value, OWN>(a, cand, cand_end, m, own_cand, own, own_len, mo, j, chain, vote_tok, vote_cnt, lane_min, lane_own);
                };
                using std::integral_constant;
                if (m + mo <= (steps > 2 ? 64u : 32u)) follow(integral_constant<int, 1>{}, integral_constant<int, 8>{});
                else if (steps <= 4) follow(integral_constant<int, 4>{}, integral_constant<int, 1>{});
                else follow(integral_constant<int, 4>{}, integral_constant<int, 8>{});
                break;
            }
            int win_tok = -1, win_cnt = 0;
            bool open = true;
            // More survivors that agreed at the step before (j > 1) are likely to agree again: a ballot per distinct token, sixteen
            // survivors to a lane; a vote still open after eight of them goes through the table. 1024 contexts, chains of 8, us with the
            // table alone / with 16 survivors to a lane from the first step to the last / so: 512 occurrences that agree 69 / 24 / 39,
            // that split over 20 tokens at once 16.1 / 44 / 16.0; 800 thinned by a tenth per step 115 (streamed) / 26 / 46. The second
            // form paid in ballots and registers whatever the occurrences did, and held up the lookups of few by 3 to 18 %.
            if constexpr (kWide) {
                if (in_lds && j > 1 && m + mo <= (uint32_t)kCand) {
                    constexpr int Q = kCand / 64;
                    int tok[Q];
                    uint32_t rest = 0;                     // bit u: this lane's voter u is not counted yet
                    int left = 0;
#pragma unroll
                    for (int u = 0; u < Q; ++u) {
                        const uint32_t i = u * 64 + lane;
                        const bool is_own = OWN && i >= m && i < m + mo;
                        const uint32_t e = is_own ? own_cand[OWN ? i - m : 0] : i < m ? cand[i] : 0u;
                        const bool ok = e + (uint32_t)j < (is_own ? own_len : i < m ? cand_end[i] : 0u);
                        tok[u] = ok ? (is_own ? own : a.P)[e + j] : -1;
                    }
#pragma unroll
                    for (int u = 0; u < Q; ++u) {
                        if (u * 64 + lane < m) cand_tok[u * 64 + lane] = tok[u];
                        rest |= (tok[u] >= 0 ? 1u : 0u) << u;
                        left += __popcll(__ballot(tok[u] >= 0));
                    }
                    open = false;
                    int ballots = 0;
                    while (left >= win_cnt) {              // larger count, then smaller token id: an equal count can still win
                        const uint64_t voters = __ballot(rest != 0);
                        if (!voters) break;
                        if (ballots++ == 8) { open = true; break; }
                        int mine = 0;
#pragma unroll
                        for (int u = Q - 1; u >= 0; --u) mine = ((rest >> u) & 1u) ? tok[u] : mine;
                        const int t = __builtin_amdgcn_readlane(mine, __ffsll((unsigned long long)voters) - 1);
                        int c = 0;
#pragma unroll
                        for (int u = 0; u < Q; ++u) {
                            const bool is = tok[u] == t;
                            rest &= ~((is ? 1u : 0u) << u);
                            c += __popcll(__ballot(is));
                        }
                        left -= c;
                        if (c > win_cnt || (c == win_cnt && t < win_tok)) { win_cnt = c; win_tok = t; }
                    }
                    __syncthreads();
                }
            }
            // The table is only as large as this vote can need (4 slots per voter, 64..kVote): clearing and scanning
            // 1024 slots with one wave cost more than the votes of the few dozen occurrences a typical lookup has.
            const uint32_t voters = (in_lds ? m : count) + mo;
            int vsz = 64;
            while (vsz < kVote && (uint32_t)vsz < 4u * voters) vsz *= 2;
            // The vote may need several passes when too many distinct successors show up. Splitting ends: the finest part is 512 neighbouring
            // hash values, and no such 512 belong to more than 318 tokens (counted over all; 1024 belong to up to 597, which would
            // not fit: the divisor stays kVote beside the larger table, too).
            for (uint32_t nparts = 1; open;) {
                // distinct tokens beyond which a vote pass is repeated, with the larger table or split; a slot for every voter is enough
                const int vfill = (uint32_t)vsz >= voters ? vsz : vsz / 4 * 3;
                win_tok = -1; win_cnt = 0;
                bool overflow = false;
                for (uint32_t part = 0; part < nparts && !overflow; ++part) {
                    for (int i = lane; i < vsz; i += 64) { vote_tok[i] = kEmptyTok; vote_cnt[i] = 0; }
                    if (lane == 0) sh_distinct = 0;
                    __syncthreads();
                    const uint32_t total_pool = in_lds ? m : count;
                    const uint32_t total = total_pool + mo;
                    // kGroups groups of 64 voters at a time, every kind of load of all of them before the first is used: a run
                    // that is streamed from the index is a chain of round trips per group.
                    for (uint32_t i0 = 0; i0 < total; i0 += 64 * kGroups) {
                        uint32_t e[kGroups], end[kGroups];
                        int tok[kGroups];
                        bool ok[kGroups];
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) {
                            const uint32_t i = i0 + u * 64 + lane;
                            e[u] = i < total_pool ? (in_lds ? cand[i] : a.sa[start + i]) : 0u;
                        }
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) {
                            const uint32_t i = i0 + u * 64 + lane;
                            end[u] = i < total_pool ? (in_lds ? cand_end[i] : a.seq_end[e[u]]) : 0u;
                        }
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) ok[u] = e[u] + (uint32_t)j < end[u];
                        if (!in_lds)
                            for (int c = 1; c < j; ++c) {
                                int t[kGroups];
#pragma unroll
                                for (int u = 0; u < kGroups; ++u) t[u] = ok[u] ? a.P[e[u] + c] : -1;
#pragma unroll
                                for (int u = 0; u < kGroups; ++u) ok[u] = ok[u] && t[u] == chain[c - 1];
                            }
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) tok[u] = ok[u] ? a.P[e[u] + j] : 0;
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) {
                            const uint32_t i = i0 + u * 64 + lane;
                            if (in_lds && i < total_pool) cand_tok[i] = ok[u] ? tok[u] : -1;
                            if (OWN && i >= total_pool && i < total) {
                                const uint32_t eo = own_cand[OWN ? i - total_pool : 0];
                                ok[u] = eo + (uint32_t)j < own_len;
                                if (ok[u]) tok[u] = own[eo + j];
                            }
                            if (ok[u]) {
                                uint32_t hh = fmix32((uint32_t)tok[u]);
                                if (nparts == 1 || (hh / kVote) % nparts == part) {
                                    uint32_t s = hh & (vsz - 1);
                                    for (int probe = 0; probe < vsz; ++probe) {
                                        int cur = vote_tok[s];
                                        if (cur == kEmptyTok) {
                                            int prev = atomicCAS(&vote_tok[s], kEmptyTok, tok[u]);
                                            if (prev == kEmptyTok) { atomicAdd(&sh_distinct, 1); cur = tok[u]; }
                                            else cur = prev;
                                        }
                                        if (cur == tok[u]) { atomicAdd(&vote_cnt[s], 1); break; }
                                        s = (s + 1) & (vsz - 1);
                                    }
                                }
                            }
                        }
                        // stop feeding a table that is getting too full; the pass will be split
                        if ((i0 & 1023u) == 1024u - 64 * kGroups) {
                            __syncthreads();
                            if (sh_distinct > vfill) break;
                        }
                    }
                    __syncthreads();
                    overflow = sh_distinct > vfill;
                    __syncthreads();               // everyone has read the counter before it is reset
                    if (overflow) break;
                    // best of this part: larger count, then smaller token id
                    int bt = -1, bc = 0;
                    for (int i = lane; i < vsz; i += 64) {
                        int c = vote_cnt[i], t = vote_tok[i];
                        if (c > bc || (c == bc && c > 0 && t < bt)) { bc = c; bt = t; }
                    }
                    for (int off = 32; off > 0; off >>= 1) {
                        int oc = __shfl_xor(bc, off), ot = __shfl_xor(bt, off);
                        if (oc > bc || (oc == bc && oc > 0 && ot < bt)) { bc = oc; bt = ot; }
                    }
                    if (bc > win_cnt || (bc == win_cnt && bc > 0 && bt < win_tok)) { win_cnt = bc; win_tok = bt; }
                    __syncthreads();
                }
                if (!overflow) break;
                if (kWide && in_lds && vsz < kTable) vsz = kTable;
                else nparts *= 2;
            }
            if (win_cnt == 0) break;       // no survivor has a successor left
            if (lane == 0) chain[j - 1] = win_tok;
            len = j;
            // ---- keep the occurrences that agree with the winner ----
            if (in_lds) {
                uint32_t out = 0;
                for (uint32_t i0 = 0; i0 < m; i0 += 64) {
                    uint32_t i = i0 + lane;
                    uint32_t e = 0, end = 0; bool keep = false;
                    if (i < m) {
                        e = cand[i];
                        end = cand_end[i];
                        keep = cand_tok[i] == win_tok;     // what the vote just read for this occurrence (tokens are >= 0)
                    }
                    uint64_t mask = __ballot(keep);
                    uint32_t pos = out + __popcll(mask & ((1ull << lane) - 1ull));
                    __syncthreads();               // all reads of this chunk precede the writes
                    if (keep) { cand[pos] = e; cand_end[pos] = end; }   // pos <= i: never overtakes unread entries
                    out += __popcll(mask);
                }
                m = out;
                __syncthreads();
            } else {
                __syncthreads();
                if ((uint32_t)win_cnt <= (uint32_t)kCand) {   // few enough now: materialise
                    uint32_t out = 0;
                    for (uint32_t i0 = 0; i0 < count; i0 += 64 * kGroups) {
                        uint32_t e[kGroups], end[kGroups];
                        bool keep[kGroups];
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) e[u] = i0 + u * 64 + lane < count ? a.sa[start + i0 + u * 64 + lane] : 0u;
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) end[u] = i0 + u * 64 + lane < count ? a.seq_end[e[u]] : 0u;
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) keep[u] = e[u] + (uint32_t)j < end[u];
                        for (int c = 1; c <= j; ++c) {
                            int t[kGroups];
#pragma unroll
                            for (int u = 0; u < kGroups; ++u) t[u] = keep[u] ? a.P[e[u] + c] : -1;
#pragma unroll
                            for (int u = 0; u < kGroups; ++u) keep[u] = keep[u] && t[u] == chain[c - 1];
                        }
#pragma unroll
                        for (int u = 0; u < kGroups; ++u) {
                            const uint64_t mask = __ballot(keep[u]);
                            const uint32_t pos = out + __popcll(mask & ((1ull << lane) - 1ull));
                            if (keep[u]) { cand[pos] = e[u]; cand_end[pos] = end[u]; }
                            out += __popcll(mask);
                        }
                    }
                    m = out;
                    in_lds = true;
                    __syncthreads();
                }
            }
            if constexpr (OWN) {
                uint32_t out = 0;
                for (uint32_t i0 = 0; i0 < mo; i0 += 64) {
                    const uint32_t i = i0 + lane;
                    uint32_t e = 0; bool keep = false;
                    if (i < mo) {
                        e = own_cand[i];
                        keep = e + (uint32_t)j < own_len && own[e + j] == win_tok;
                    }
                    const uint64_t mask = __ballot(keep);
                    const uint32_t pos = out + __popcll(mask & ((1ull << lane) - 1ull));
                    __syncthreads();               // all reads of this chunk precede the writes
                    if (keep) own_cand[pos] = e;   // pos <= i: never overtakes unread entries
                    out += __popcll(mask);
                }
                mo = out;
                __syncthreads();
            }
        }
        // ---- smallest surviving position ----
        uint32_t mn = 0xFFFFFFFFu;
        if (in_lanes) {
            mn = lane_min;
        } else if (in_lds) {
            for (uint32_t i = lane; i < m; i += 64) mn = min(mn, cand[i]);
        } else {
            for (uint32_t i = lane; i < count; i += 64) {
                uint32_t e = a.sa[start + i];
                bool keep = (e + (uint32_t)len) < a.seq_end[e];
                for (int c = 1; c <= len && keep; ++c) keep = (a.P[e + c] == chain[c - 1]);
                if (keep) mn = min(mn, e);
            }
        }
        for (int off = 32; off > 0; off >>= 1) mn = min(mn, (uint32_t)__shfl_xor((int)mn, off));
        __syncthreads();
        // pool positions precede the own text's; a result that survives only there is reported as -2 - position
        // (own_cand stays position-ascending through the filters, so its first entry is the smallest)
        long long idx = (long long)mn;
        if (OWN && mn == 0xFFFFFFFFu) {
            uint32_t first_own = in_lanes ? lane_own : mo > 0 ? own_cand[0] : 0xFFFFFFFFu;
            for (int off = 32; off > 0; off >>= 1) first_own = min(first_own, (uint32_t)__shfl_xor((int)first_own, off));
            idx = first_own != 0xFFFFFFFFu ? -2ll - (long long)first_own : -1ll;
        }

        if (len >= a.min_tokens) {
            res_len = len; res_n = n; res_idx = idx; done = true;
        } else if (len > best_len) {
            best_len = len; best_n = n; best_idx = idx;
            for (int i = lane; i < len; i += 64) best_chain[i] = chain[i];
            __syncthreads();
        }
    }
    const int* src = chain;
    if (!done) { res_len = best_len; res_n = best_n; res_idx = best_idx; src = best_chain; }
    __syncthreads();
    for (int i = lane; i < a.K; i += 64) a.drafts[(size_t)b * a.K + i] = i < res_len ? src[i] : -1;
    if (lane == 0) {
        a.draft_len[b] = res_len;
        a.match_n[b] = res_len > 0 ? res_n : 0;
        a.pool_index[b] = res_len > 0 ? res_idx : -1;
    }
}

// ---------------------------------------------------------------------------------------------- token trees
// Tree-based drafting (Sec. 3.3): the sub-tree of the key's trie below the node the context suffix reaches, cut to
// its K most frequent nodes. A node is a path of successor tokens; its frequency is the number of occurrences of the
// suffix whose continuation starts with that path. Nodes are taken best first: always the best node not yet taken
// whose parent is taken (higher frequency, then smaller depth, then the parent taken earlier, then the smaller token
// id); a child is never more frequent than its parent, so these are the K best nodes of the whole sub-tree.
// One wavefront per context. Taking a node means one vote over the occurrences that continue with its path
// (re-checked against the path, so any number of occurrences works) to find its children and their frequencies;
// the best K - (taken) of them join the frontier. The pseudo-sequence lists the taken nodes depth-first, siblings
// in the order taken.
constexpr int kTreeMax = LASER_MAX_TREE;                       // nodes of one tree
constexpr int kFrontier = kTreeMax * (kTreeMax + 1) / 2 + 16;  // every expansion adds at most K - taken children

struct TreeArgs {
    const int32_t* P; const uint32_t* seq_end; const uint32_t* sa; const IndexEntry* table;
    uint64_t cap_mask;
    const int64_t* keys; const int32_t* ctx_tail;
    int B, n_min, n_max, K, min_tokens;
    int32_t* tree_tokens; int32_t* tree_parent; int32_t* tree_freq; int32_t* tree_len; int32_t* match_n;
};

__global__ __launch_bounds__(64) void retrieve_tree_kernel(TreeArgs a) {
    __shared__ uint32_t cand[kCand];
    __shared__ uint32_t cand_end[kCand];
    __shared__ int vote_tok[kVote];
    __shared__ int vote_cnt[kVote];
    __shared__ int sh_distinct;
    __shared__ int t_tok[kTreeMax], t_par[kTreeMax], t_depth[kTreeMax], t_cnt[kTreeMax];     // taken nodes, in the order taken
    __shared__ int f_tok[kFrontier], f_cnt[kFrontier], f_par[kFrontier], f_depth[kFrontier];
    __shared__ int ch_tok[kTreeMax], ch_cnt[kTreeMax];                                       // best children of one expansion
    __shared__ int path[kTreeMax];
    __shared__ int b_tok[kTreeMax], b_par[kTreeMax], b_cnt[kTreeMax];                        // best tree seen (pseudo-sequence form)
    __shared__ int o_tok[kTreeMax], o_par[kTreeMax], o_cnt[kTreeMax], dfs_pos[kTreeMax], stack[kTreeMax];

    const int b = blockIdx.x, lane = threadIdx.x;
    const int64_t key = a.keys[b];
    const int32_t* tail = a.ctx_tail + (size_t)b * a.n_max;
    int valid = 0;
    while (valid < a.n_max && tail[a.n_max - 1 - valid] >= 0) ++valid;

    int best_len = 0, best_n = 0, res_len = 0, res_n = 0;
    bool done = false;
    const int n_hi = valid < a.n_max ? valid : a.n_max;
    for (int n = n_hi; n >= a.n_min && !done && a.K > 0; --n) {
        // ---- index probe (as in retrieve_kernel) ----
        const int32_t* w = tail + (a.n_max - n);
        uint64_t slot = ngram_hash(key, n, w) & a.cap_mask;
        uint32_t start = 0, count = 0;
        for (;;) {
            IndexEntry e = a.table[slot];
            if (e.count_n == 0) break;
            if (e.key == key && (int)(e.count_n >> 28) == n) {
                uint32_t e0 = a.sa[e.start];
                bool same = true;
                for (int i = 0; i < n; ++i) same = same && (a.P[e0 - (n - 1) + i] == w[i]);
                if (same) { start = e.start; count = e.count_n & 0x0FFFFFFFu; break; }
            }
            slot = (slot + 1) & a.cap_mask;
        }
        if (count == 0) continue;
        const bool in_lds = count <= (uint32_t)kCand;
        if (in_lds)
            for (uint32_t i = lane; i < count; i += 64) {
                const uint32_t e = a.sa[start + i];
                cand[i] = e;
                cand_end[i] = a.seq_end[e];
            }
        __syncthreads();

        int taken = 0, fsize = 0;
        // children of taken node `node` (-1: the root) at depth d: the best K - taken of them go to the frontier
        auto expand = [&](int node, int d) {
            for (int i = node, j = d - 1; j >= 0; --j) {           // every lane walks the same path (LDS broadcast reads)
                if (lane == 0) path[j] = t_tok[i];
                i = t_par[i];
            }
            const int want = a.K - taken;
            int n_ch = 0;                                            // uniform: entries of ch_*
            __syncthreads();
            int vsz = 64;
            while (vsz < kVote && (uint32_t)vsz < 4u * count) vsz *= 2;
            const int vfill = vsz / 4 * 3;
            for (uint32_t nparts = 1;; nparts *= 2) {
                bool overflow = false;
                n_ch = 0;
                for (uint32_t part = 0; part < nparts && !overflow; ++part) {
                    for (int i = lane; i < vsz; i += 64) { vote_tok[i] = kEmptyTok; vote_cnt[i] = 0; }
                    if (lane == 0) sh_distinct = 0;
                    __syncthreads();
                    for (uint32_t i0 = 0; i0 < count; i0 += 64) {
                        const uint32_t i = i0 + lane;
                        if (i < count) {
                            const uint32_t e = in_lds ? cand[i] : a.sa[start + i];
                            bool ok = (e + (uint32_t)d + 1u) < (in_lds ? cand_end[i] : a.seq_end[e]);
                            for (int c = 0; c < d && ok; ++c) ok = a.P[e + 1 + c] == path[c];
                            if (ok) {
                                const int tok = a.P[e + d + 1];
                                const uint32_t hh = fmix32((uint32_t)tok);
                                if (nparts == 1 || (hh / kVote) % nparts == part) {
                                    uint32_t s = hh & (vsz - 1);
                                    for (int probe = 0; probe < vsz; ++probe) {
                                        int cur = vote_tok[s];
                                        if (cur == kEmptyTok) {
                                            const int prev = atomicCAS(&vote_tok[s], kEmptyTok, tok);
                                            if (prev == kEmptyTok) { atomicAdd(&sh_distinct, 1); cur = tok; }
                                            else cur = prev;
                                        }
                                        if (cur == tok) { atomicAdd(&vote_cnt[s], 1); break; }
                                        s = (s + 1) & (vsz - 1);
                                    }
                                }
                            }
                        }
                        if ((i0 & 1023u) == 960u) {
                            __syncthreads();
                            if (sh_distinct > vfill) break;
                        }
                    }
                    __syncthreads();
                    overflow = sh_distinct > vfill;
                    __syncthreads();
                    if (overflow) break;
                    // this part's best `want` (count desc, token asc), merged into the sorted child list
                    for (int round = 0; round < want; ++round) {
                        int bc = 0, bt = 0x7FFFFFFF, bs = -1;
                        for (int i = lane; i < vsz; i += 64) {
                            const int c = vote_cnt[i], t = vote_tok[i];
                            if (c > bc || (c == bc && c > 0 && t < bt)) { bc = c; bt = t; bs = i; }
                        }
                        for (int off = 32; off > 0; off >>= 1) {
                            const int oc = __shfl_xor(bc, off), ot = __shfl_xor(bt, off), os = __shfl_xor(bs, off);
                            if (oc > bc || (oc == bc && oc > 0 && ot < bt)) { bc = oc; bt = ot; bs = os; }
                        }
                        if (bc == 0) break;                          // uniform
                        // insert (bt, bc) into ch_* (sorted, at most `want` entries); lane 0 does the shifting
                        int pos = n_ch;
                        while (pos > 0 && (ch_cnt[pos - 1] < bc || (ch_cnt[pos - 1] == bc && ch_tok[pos - 1] > bt))) --pos;
                        if (pos < want) {
                            if (lane == 0) {
                                const int last = n_ch < want ? n_ch : want - 1;
                                for (int q = last; q > pos; --q) { ch_tok[q] = ch_tok[q - 1]; ch_cnt[q] = ch_cnt[q - 1]; }
                                ch_tok[pos] = bt; ch_cnt[pos] = bc;
                                vote_cnt[bs] = 0;
                            }
                            if (n_ch < want) ++n_ch;
                        } else if (lane == 0) {
                            vote_cnt[bs] = 0;
                        }
                        __syncthreads();
                        if (pos >= want) break;                      // nothing later in this part can enter either
                    }
                    __syncthreads();
                }
                if (!overflow) break;
            }
            for (int i = lane; i < n_ch; i += 64) {
                f_tok[fsize + i] = ch_tok[i]; f_cnt[fsize + i] = ch_cnt[i]; f_par[fsize + i] = node; f_depth[fsize + i] = d + 1;
            }
            fsize += n_ch;
            __syncthreads();
        };
        // The same for at most 256 occurrences, four to a lane: each carries a bit per taken node it continues with, so
        // that a path is not walked again (one token decides the newest bit), and children are counted with a ballot per
        // distinct token instead of through the vote table: 8 trees of 16 nodes 90 -> 49 us.
        constexpr int Q = 4;
        const bool in_lanes = count <= 64u * Q;
        uint32_t le[Q], lend[Q], lbits[Q];
#pragma unroll
        for (int s = 0; s < Q; ++s) {
            const uint32_t i = (uint32_t)(s * 64 + lane);
            const bool have = in_lanes && i < count;
            le[s] = have ? cand[i] : 0u;
            lend[s] = have ? cand_end[i] : 0u;         // an idle lane has no successor
            lbits[s] = 0u;
        }
        auto expand_lanes = [&](int node, int d) {
            const int want = a.K - taken;
            const int par = node >= 0 ? t_par[node] : -1, own_tok = node >= 0 ? t_tok[node] : 0;
            int tok[Q];
            uint64_t rest[Q];
            bool ok[Q];
            int left = 0;                                            // occurrences not counted yet
#pragma unroll
            for (int s = 0; s < Q; ++s) {
                const bool reach = (par < 0 || ((lbits[s] >> par) & 1u)) && le[s] + (uint32_t)d < lend[s];
                const int at = node >= 0 && reach ? a.P[le[s] + (uint32_t)d] : 0;
                const bool more = reach && le[s] + (uint32_t)d + 1u < lend[s];
                tok[s] = more ? a.P[le[s] + (uint32_t)d + 1u] : 0;
                const bool in = node < 0 || (reach && at == own_tok);
                if (node >= 0 && in) lbits[s] |= 1u << node;
                ok[s] = in && more;
            }
#pragma unroll
            for (int s = 0; s < Q; ++s) { rest[s] = __ballot(ok[s]); left += __popcll(rest[s]); }
            int n_ch = 0;
#pragma unroll
            for (int s = 0; s < Q; ++s)
                while (rest[s] && (n_ch < want || left >= ch_cnt[want - 1])) {      // an equal count can still enter
                    const int t = __builtin_amdgcn_readlane(tok[s], __ffsll((unsigned long long)rest[s]) - 1);
                    int c = 0;
#pragma unroll
                    for (int u = s; u < Q; ++u) {
                        const uint64_t same = __ballot(ok[u] && tok[u] == t);
                        c += __popcll(same);
                        rest[u] &= ~same;
                    }
                    left -= c;
                    int pos = n_ch;                                  // as above: count desc, token asc
                    while (pos > 0 && (ch_cnt[pos - 1] < c || (ch_cnt[pos - 1] == c && ch_tok[pos - 1] > t))) --pos;
                    __syncthreads();
                    if (pos < want) {
                        const int last = n_ch < want ? n_ch : want - 1;
                        if (lane == 0) {
                            for (int q = last; q > pos; --q) { ch_tok[q] = ch_tok[q - 1]; ch_cnt[q] = ch_cnt[q - 1]; }
                            ch_tok[pos] = t; ch_cnt[pos] = c;
                        }
                        if (n_ch < want) ++n_ch;
                    }
                    __syncthreads();
                }
            for (int i = lane; i < n_ch; i += 64) {
                f_tok[fsize + i] = ch_tok[i]; f_cnt[fsize + i] = ch_cnt[i]; f_par[fsize + i] = node; f_depth[fsize + i] = d + 1;
            }
            fsize += n_ch;
            __syncthreads();
        };
        if (in_lanes) expand_lanes(-1, 0);
        else expand(-1, 0);
        while (taken < a.K && fsize > 0) {
            // best frontier entry: count desc, depth asc, parent asc, token asc
            int bi = -1, bc = 0, bd = 0, bp = 0, bt = 0;
            auto better = [](int c, int d, int p, int t, int c2, int d2, int p2, int t2) {
                return c != c2 ? c > c2 : (d != d2 ? d < d2 : (p != p2 ? p < p2 : t < t2));
            };
            for (int i = lane; i < fsize; i += 64)
                if (bi < 0 || better(f_cnt[i], f_depth[i], f_par[i], f_tok[i], bc, bd, bp, bt)) {
                    bi = i; bc = f_cnt[i]; bd = f_depth[i]; bp = f_par[i]; bt = f_tok[i];
                }
            for (int off = 32; off > 0; off >>= 1) {
                const int oi = __shfl_xor(bi, off), oc = __shfl_xor(bc, off), od = __shfl_xor(bd, off), op = __shfl_xor(bp, off),
                          ot = __shfl_xor(bt, off);
                if (oi >= 0 && (bi < 0 || better(oc, od, op, ot, bc, bd, bp, bt))) { bi = oi; bc = oc; bd = od; bp = op; bt = ot; }
            }
            __syncthreads();
            if (lane == 0) {
                t_tok[taken] = bt; t_par[taken] = bp; t_depth[taken] = bd; t_cnt[taken] = bc;
                const int last = fsize - 1;
                f_tok[bi] = f_tok[last]; f_cnt[bi] = f_cnt[last]; f_par[bi] = f_par[last]; f_depth[bi] = f_depth[last];
            }
            --fsize;
            ++taken;
            __syncthreads();
            if (taken < a.K) {
                if (in_lanes) expand_lanes(taken - 1, bd);
                else expand(taken - 1, bd);
            }
        }
        // ---- pseudo-sequence: depth-first, siblings in the order taken ----
        if (lane == 0) {
            int sp = 0, n_out = 0;
            for (int i = taken - 1; i >= 0; --i) if (t_par[i] < 0) stack[sp++] = i;
            while (sp > 0) {
                const int i = stack[--sp];
                dfs_pos[i] = n_out;
                o_tok[n_out] = t_tok[i]; o_cnt[n_out] = t_cnt[i];
                o_par[n_out] = t_par[i] < 0 ? -1 : dfs_pos[t_par[i]];
                ++n_out;
                for (int c = taken - 1; c > i; --c) if (t_par[c] == i) stack[sp++] = c;
            }
        }
        __syncthreads();
        if (taken >= a.min_tokens) {
            res_len = taken; res_n = n; done = true;
        } else if (taken > best_len) {
            best_len = taken; best_n = n;
            for (int i = lane; i < taken; i += 64) { b_tok[i] = o_tok[i]; b_par[i] = o_par[i]; b_cnt[i] = o_cnt[i]; }
            __syncthreads();
        }
    }
    const int *s_tok = o_tok, *s_par = o_par, *s_cnt = o_cnt;
    if (!done) { res_len = best_len; res_n = best_n; s_tok = b_tok; s_par = b_par; s_cnt = b_cnt; }
    __syncthreads();
    for (int i = lane; i < a.K; i += 64) {
        a.tree_tokens[(size_t)b * a.K + i] = i < res_len ? s_tok[i] : -1;
        a.tree_parent[(size_t)b * a.K + i] = i < res_len ? s_par[i] : -1;
        if (a.tree_freq) a.tree_freq[(size_t)b * a.K + i] = i < res_len ? s_cnt[i] : 0;
    }
    if (lane == 0) {
        a.tree_len[b] = res_len;
        a.match_n[b] = res_len > 0 ? res_n : 0;
    }
}

// Appends the tokens a step emitted (out_tokens[b][0 .. accept_len[b]]) to row b of the own-text buffer; a full row
// drops its oldest tokens (sliding window of `cap`). One workgroup per sequence.
__global__ __launch_bounds__(256) void own_text_append_kernel(int32_t* own, int32_t* own_len, int cap, const int32_t* out_tokens,
                                                              const int32_t* accept_len, int K) {
    const int b = blockIdx.x, tid = threadIdx.x;
    if (accept_len[b] < 0) return;                     // nothing was emitted for this sequence (it had finished before the step)
    int32_t* row = own + (size_t)b * cap;
    const int32_t* nw = out_tokens + (size_t)b * (K + 1);
    int n_new = min(accept_len[b], K) + 1;
    int len = min(max(own_len[b], 0), cap);
    const int skip = max(n_new - cap, 0);              // more new tokens than the row holds: keep the newest
    n_new -= skip;
    const int shift = max(len + n_new - cap, 0);
    if (shift > 0) {
        const int keep = len - shift;                  // row[shift .. len) moves to row[0 .. keep)
        for (int base = 0; base < keep; base += 256) {
            const int i = base + tid;
            const int32_t v = i < keep ? row[i + shift] : 0;
            __syncthreads();                           // every read of this chunk precedes its writes; later chunks read beyond them
            if (i < keep) row[i] = v;
        }
        len = max(keep, 0);
    }
    for (int i = tid; i < n_new; i += 256) row[len + i] = nw[skip + i];
    if (tid == 0) own_len[b] = len + n_new;
}

// ------------------------------------------------------------------------------------ host build
namespace {

struct SubPool { int64_t key; uint32_t begin, end; };

// Occurrences from which the device builds. It takes three launches per byte of a token and n, whatever the size, the host
// a comparison sort. us, device / host, for n_max 1 / 4 / 8: two bytes, 4096 occurrences 250 / 467 / 750 against 359 / 496
// / 792; three bytes, 4096: 272 / 562 / 937 against 325 / 480 / 846, 8192: 274 / 600 / 1068 against 322 / 763 / 1680;
// four bytes, 4096: 299 / 652 / 1083 against 243 / 416 / 817, 8192: 311 / 709 / 1248 against 385 / 778 / 1614.
constexpr int64_t kDeviceBuildMin = 4096, kDeviceBuildMinWide = 8192;

}  // namespace

static int build_pool(const int32_t* tokens, const int64_t* seq_off, const int64_t* seq_key,
                      int64_t n_seq, int n_max, int builder, int64_t mem_limit, hipStream_t stream, Pool** out) {
    const int64_t n_tok = n_seq > 0 ? seq_off[n_seq] : 0;
    LASER_REQUIRE(n_tok < 0xFFFFFFFFll, LASER_E_LIMIT, "pool of %lld tokens exceeds 2^32-2", (long long)n_tok);
    for (int64_t s = 0; s < n_seq; ++s)
        LASER_REQUIRE(seq_off[s + 1] >= seq_off[s], LASER_E_INVALID_ARG, "seq_off not ascending at %lld", (long long)s);

    // 1. regroup: ascending key, supply order inside a key
    std::vector<int64_t> order(n_seq);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int64_t x, int64_t y) { return seq_key[x] < seq_key[y]; });

    // Many occurrences: the rest happens on the device, unless it cannot hold the working arrays (17 bytes per token
    // besides the pool itself). Few: the host is done before the device's ~40 dependent launches are.
    uint32_t bits = 0;                                // all tokens or-ed together
    const int64_t least = builder == LASER_BUILDER_DEVICE ? 1 : kDeviceBuildMin;
    if (builder != LASER_BUILDER_HOST && n_tok - n_seq >= least)
        for (int64_t i = 0; i < n_tok; ++i) bits |= (uint32_t)tokens[i];
    const bool wide = builder == LASER_BUILDER_AUTO && bits + 1u >= 1u << 16;
    if (builder != LASER_BUILDER_HOST && n_tok - n_seq >= (wide ? kDeviceBuildMinWide : least)) {
        PoolLayout lay;
        uint32_t pos = 0;
        for (int64_t i = 0; i < n_seq; ++i) {
            const int64_t s = order[i];
            const uint32_t len = (uint32_t)(seq_off[s + 1] - seq_off[s]);
            if (lay.sub_key.empty() || lay.sub_key.back() != seq_key[s]) lay.sub_key.push_back(seq_key[s]);
            if (bits >> 31)
                for (uint32_t t = 0; t < len; ++t)
                    LASER_REQUIRE(tokens[seq_off[s] + t] >= 0, LASER_E_INVALID_ARG, "negative token in sequence %lld", (long long)s);
            if (len == 0) continue;
            lay.dst_off.push_back(pos);
            lay.src_off.push_back((uint32_t)seq_off[s]);
            lay.sub.push_back((uint32_t)lay.sub_key.size() - 1);
            pos += len;
        }
        lay.dst_off.push_back(pos);
        lay.token_bits = bits;
        Pool* p = new Pool();
        bool no_memory = false;
        const int rc = build_index_device(tokens, lay, n_max, mem_limit, stream, p, &no_memory);
        if (rc == LASER_OK) { *out = p; return rc; }
        delete p;
        if (!no_memory) return rc;
    }

    std::vector<int32_t> P((size_t)n_tok);
    std::vector<uint32_t> seq_begin((size_t)n_tok), seq_end((size_t)n_tok);
    std::vector<SubPool> subs;
    {
        uint32_t pos = 0;
        for (int64_t i = 0; i < n_seq; ++i) {
            const int64_t s = order[i];
            const uint32_t len = (uint32_t)(seq_off[s + 1] - seq_off[s]);
            if (subs.empty() || subs.back().key != seq_key[s]) subs.push_back({seq_key[s], pos, pos});
            for (uint32_t t = 0; t < len; ++t) {
                const int32_t tok = tokens[seq_off[s] + t];
                LASER_REQUIRE(tok >= 0, LASER_E_INVALID_ARG, "negative token in sequence %lld", (long long)s);
                P[pos + t] = tok;
                seq_begin[pos + t] = pos;
                seq_end[pos + t] = pos + len;
            }
            pos += len;
            subs.back().end = pos;
        }
    }

    // 2. sorted occurrence array: per sub-pool, positions with a successor, by reversed text
    std::vector<uint32_t> sa;
    sa.reserve((size_t)n_tok);
    std::vector<uint32_t> sub_sa_begin(subs.size() + 1);
    for (size_t g = 0; g < subs.size(); ++g) {
        sub_sa_begin[g] = (uint32_t)sa.size();
        for (uint32_t e = subs[g].begin; e < subs[g].end; ++e)
            if (e + 1 < seq_end[e]) sa.push_back(e);
    }
    sub_sa_begin[subs.size()] = (uint32_t)sa.size();

    auto back_tok = [&](uint32_t e, int i) -> int64_t {       // i-th token back from e, or -1 before the sequence
        return (e - seq_begin[e] >= (uint32_t)i) ? (int64_t)P[e - i] : -1;
    };
    auto less = [&](uint32_t x, uint32_t y) {
        for (int i = 0; i < n_max; ++i) {
            const int64_t a = back_tok(x, i), b = back_tok(y, i);
            if (a != b) return a < b;
        }
        return x < y;
    };
    {
        const unsigned hw = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
        const size_t G = subs.size();
        if (G <= 1 || hw == 1) {
            for (size_t g = 0; g < G; ++g)
                std::sort(sa.begin() + sub_sa_begin[g], sa.begin() + sub_sa_begin[g + 1], less);
        } else {
            // split the sub-pools into hw contiguous chunks of roughly equal size
            std::vector<std::thread> th;
            std::vector<size_t> cut(hw + 1, G);
            cut[0] = 0;
            const uint64_t total = sa.size();
            size_t g = 0;
            for (unsigned t = 1; t < hw; ++t) {
                const uint64_t target = total * t / hw;
                while (g < G && sub_sa_begin[g] < target) ++g;
                cut[t] = g;
            }
            for (unsigned t = 0; t < hw; ++t)
                th.emplace_back([&, t] {
                    for (size_t q = cut[t]; q < cut[t + 1]; ++q)
                        std::sort(sa.begin() + sub_sa_begin[q], sa.begin() + sub_sa_begin[q + 1], less);
                });
            for (auto& x : th) x.join();
        }
    }

    // 3. runs of equal n-grams -> table entries
    auto same_ngram = [&](uint32_t x, uint32_t y, int n) {
        for (int i = 0; i < n; ++i) {
            const int64_t a = back_tok(x, i), b = back_tok(y, i);
            if (a < 0 || a != b) return false;
        }
        return true;
    };
    auto has_n = [&](uint32_t e, int n) { return e - seq_begin[e] >= (uint32_t)(n - 1); };

    // two passes over the runs (count, then insert) keep the host footprint at the table itself
    auto for_each_run = [&](auto&& fn) -> bool {
        for (size_t g = 0; g < subs.size(); ++g) {
            const uint32_t lo = sub_sa_begin[g], hi = sub_sa_begin[g + 1];
            for (int n = 1; n <= n_max; ++n) {
                uint32_t i = lo;
                while (i < hi) {
                    if (!has_n(sa[i], n)) { ++i; continue; }
                    uint32_t j = i + 1;
                    while (j < hi && same_ngram(sa[i], sa[j], n)) ++j;
                    if (!fn(g, n, i, j - i)) return false;
                    i = j;
                }
            }
        }
        return true;
    };
    uint64_t n_runs = 0;
    uint32_t longest = 0;
    for_each_run([&](size_t, int, uint32_t, uint32_t c) { ++n_runs; longest = std::max(longest, c); return true; });
    LASER_REQUIRE(longest < (1u << 28), LASER_E_LIMIT, "an n-gram occurs %u times (limit 2^28-1)", longest);
    uint64_t cap = 16;
    while (cap < 2 * n_runs) cap <<= 1;
    std::vector<IndexEntry> table(cap);
    std::memset(table.data(), 0, cap * sizeof(IndexEntry));
    for_each_run([&](size_t g, int n, uint32_t start, uint32_t c) {
        int32_t w[LASER_MAX_NGRAM];
        const uint32_t e0 = sa[start];
        for (int i = 0; i < n; ++i) w[i] = P[e0 - (n - 1) + i];
        uint64_t slot = ngram_hash(subs[g].key, n, w) & (cap - 1);
        while (table[slot].count_n != 0) slot = (slot + 1) & (cap - 1);
        table[slot] = {subs[g].key, start, c | ((uint32_t)n << 28)};
        return true;
    });

    // 4. upload
    Pool* p = new Pool();
    p->n_tokens = n_tok; p->n_keys = (int64_t)subs.size(); p->n_entries = (int64_t)n_runs;
    p->n_sa = (int64_t)sa.size(); p->n_max = n_max; p->cap_mask = cap - 1;
    auto up = [&](void** dst, const void* src, size_t bytes) -> int {
        const size_t alloc = bytes ? bytes : 16;
        LASER_HIP_CHECK(hipMalloc(dst, alloc));
        p->device_bytes += (int64_t)alloc;
        if (bytes) LASER_HIP_CHECK(hipMemcpyAsync(*dst, src, bytes, hipMemcpyHostToDevice, stream));
        return LASER_OK;
    };
    int rc;
    if ((rc = up((void**)&p->P, P.data(), P.size() * 4)) || (rc = up((void**)&p->seq_end, seq_end.data(), seq_end.size() * 4)) ||
        (rc = up((void**)&p->sa, sa.data(), sa.size() * 4)) || (rc = up((void**)&p->table, table.data(), cap * sizeof(IndexEntry)))) {
        (void)hipFree(p->P); (void)hipFree(p->seq_end); (void)hipFree(p->sa); (void)hipFree(p->table);
        delete p;
        return rc;
    }
    LASER_HIP_CHECK(hipStreamSynchronize(stream));
    *out = p;
    return LASER_OK;
}

}  // namespace laser

using namespace laser;

extern "C" int laser_pool_build(const int32_t* tokens, const int64_t* seq_off, const int64_t* seq_key,
                                int64_t n_seq, int n_max, void* stream, laser_pool** out) {
    return laser_pool_build_with(tokens, seq_off, seq_key, n_seq, n_max, LASER_BUILDER_AUTO, -1, stream, out);
}

extern "C" int laser_pool_build_with(const int32_t* tokens, const int64_t* seq_off, const int64_t* seq_key, int64_t n_seq,
                                     int n_max, int builder, int64_t mem_limit, void* stream, laser_pool** out) {
    LASER_REQUIRE(out != nullptr, LASER_E_INVALID_ARG, "out is NULL");
    LASER_REQUIRE(n_seq >= 0, LASER_E_INVALID_ARG, "n_seq < 0");
    LASER_REQUIRE(n_seq == 0 || (tokens && seq_off && seq_key), LASER_E_INVALID_ARG, "NULL input array");
    LASER_REQUIRE(n_max >= 1 && n_max <= LASER_MAX_NGRAM, LASER_E_INVALID_ARG, "n_max %d outside 1..%d", n_max, LASER_MAX_NGRAM);
    LASER_REQUIRE(n_seq == 0 || seq_off[0] == 0, LASER_E_INVALID_ARG, "seq_off[0] != 0");
    LASER_REQUIRE(builder >= LASER_BUILDER_AUTO && builder <= LASER_BUILDER_DEVICE, LASER_E_INVALID_ARG, "unknown builder %d", builder);
    Pool* p = nullptr;
    int rc = build_pool(tokens, seq_off, seq_key, n_seq, n_max, builder, mem_limit, (hipStream_t)stream, &p);
    if (rc == LASER_OK) *out = reinterpret_cast<laser_pool*>(p);
    return rc;
}

extern "C" int laser_pool_destroy(laser_pool* pool) {
    if (!pool) return LASER_OK;
    Pool* p = reinterpret_cast<Pool*>(pool);
    (void)hipFree(p->P); (void)hipFree(p->seq_end); (void)hipFree(p->sa); (void)hipFree(p->table);
    delete p;
    return LASER_OK;
}

extern "C" int laser_pool_info(const laser_pool* pool, int64_t* n_tokens, int64_t* n_keys,
                               int64_t* n_index_entries, int64_t* device_bytes) {
    LASER_REQUIRE(pool != nullptr, LASER_E_INVALID_ARG, "pool is NULL");
    const Pool* p = reinterpret_cast<const Pool*>(pool);
    if (n_tokens) *n_tokens = p->n_tokens;
    if (n_keys) *n_keys = p->n_keys;
    if (n_index_entries) *n_index_entries = p->n_entries;
    if (device_bytes) *device_bytes = p->device_bytes;
    return LASER_OK;
}

extern "C" int laser_pool_read_tokens(const laser_pool* pool, int64_t start, int64_t count, int32_t* out_host) {
    LASER_REQUIRE(pool != nullptr && out_host != nullptr, LASER_E_INVALID_ARG, "NULL argument");
    const Pool* p = reinterpret_cast<const Pool*>(pool);
    LASER_REQUIRE(start >= 0 && count >= 0 && start + count <= p->n_tokens, LASER_E_INVALID_ARG,
                  "range [%lld, +%lld) outside the pool", (long long)start, (long long)count);
    if (count) LASER_HIP_CHECK(hipMemcpy(out_host, p->P + start, (size_t)count * 4, hipMemcpyDeviceToHost));
    return LASER_OK;
}

static int retrieve_impl(const laser_pool* pool, const int64_t* keys, const int32_t* ctx_tail, const int32_t* own,
                         const int32_t* own_len, int own_cap, int B, int n_min, int n_max, int K, int min_tokens,
                         int32_t* drafts, int32_t* draft_len, int32_t* match_n, int64_t* pool_index, void* stream) {
    LASER_REQUIRE(pool != nullptr, LASER_E_INVALID_ARG, "pool is NULL");
    const Pool* p = reinterpret_cast<const Pool*>(pool);
    LASER_REQUIRE(B >= 0, LASER_E_INVALID_ARG, "B < 0");
    LASER_REQUIRE(K >= 0 && K <= LASER_MAX_DRAFT, LASER_E_INVALID_ARG, "K %d outside 0..%d", K, LASER_MAX_DRAFT);
    LASER_REQUIRE(n_max >= 1 && n_max <= p->n_max, LASER_E_INVALID_ARG, "n_max %d outside 1..%d (the pool's)", n_max, p->n_max);
    LASER_REQUIRE(n_min >= 1 && n_min <= n_max, LASER_E_INVALID_ARG, "n_min %d outside 1..n_max", n_min);
    if (B == 0) return LASER_OK;
    LASER_REQUIRE(keys && ctx_tail && draft_len && match_n && pool_index && (drafts || K == 0),
                  LASER_E_INVALID_ARG, "NULL device buffer");
    RetrieveArgs a{p->P, p->seq_end, p->sa, p->table, p->cap_mask, keys, ctx_tail,
                   B, n_min, n_max, K, min_tokens < 1 ? 1 : min_tokens, drafts, draft_len, match_n, pool_index,
                   own, own_len, own_cap};
    const bool four = B <= kFourGroupsMax;
    const auto kernel = own ? (four ? retrieve_kernel<true, 4> : retrieve_kernel<true, 1>) : (four ? retrieve_kernel<false, 4> : retrieve_kernel<false, 1>);
    hipLaunchKernelGGL(kernel, dim3(B), dim3(64), 0, (hipStream_t)stream, a);
    LASER_HIP_CHECK(hipGetLastError());
    return LASER_OK;
}

extern "C" int laser_retrieve_drafts(const laser_pool* pool, const int64_t* keys, const int32_t* ctx_tail,
                                     int B, int n_min, int n_max, int K, int min_tokens,
                                     int32_t* drafts, int32_t* draft_len, int32_t* match_n,
                                     int64_t* pool_index, void* stream) {
    return retrieve_impl(pool, keys, ctx_tail, nullptr, nullptr, 0, B, n_min, n_max, K, min_tokens, drafts, draft_len,
                         match_n, pool_index, stream);
}

extern "C" int laser_retrieve_drafts_temp(const laser_pool* pool, const int64_t* keys, const int32_t* ctx_tail,
                                          const int32_t* own_tokens, const int32_t* own_len, int own_cap,
                                          int B, int n_min, int n_max, int K, int min_tokens,
                                          int32_t* drafts, int32_t* draft_len, int32_t* match_n,
                                          int64_t* pool_index, void* stream) {
    LASER_REQUIRE(own_cap >= 1 && own_cap <= LASER_MAX_OWN_TEXT, LASER_E_INVALID_ARG, "own_cap %d outside 1..%d", own_cap,
                  LASER_MAX_OWN_TEXT);
    LASER_REQUIRE(B <= 0 || (own_tokens && own_len), LASER_E_INVALID_ARG, "NULL own-text buffer");
    return retrieve_impl(pool, keys, ctx_tail, own_tokens, own_len, own_cap, B, n_min, n_max, K, min_tokens, drafts,
                         draft_len, match_n, pool_index, stream);
}

extern "C" int laser_retrieve_tree(const laser_pool* pool, const int64_t* keys, const int32_t* ctx_tail, int B, int n_min, int n_max,
                                   int K, int min_tokens, int32_t* tree_tokens, int32_t* tree_parent, int32_t* tree_freq,
                                   int32_t* tree_len, int32_t* match_n, void* stream) {
    LASER_REQUIRE(pool != nullptr, LASER_E_INVALID_ARG, "pool is NULL");
    const Pool* p = reinterpret_cast<const Pool*>(pool);
    LASER_REQUIRE(B >= 0, LASER_E_INVALID_ARG, "B < 0");
    LASER_REQUIRE(K >= 0 && K <= LASER_MAX_TREE, LASER_E_INVALID_ARG, "K %d outside 0..%d", K, LASER_MAX_TREE);
    LASER_REQUIRE(n_max >= 1 && n_max <= p->n_max, LASER_E_INVALID_ARG, "n_max %d outside 1..%d (the pool's)", n_max, p->n_max);
    LASER_REQUIRE(n_min >= 1 && n_min <= n_max, LASER_E_INVALID_ARG, "n_min %d outside 1..n_max", n_min);
    if (B == 0) return LASER_OK;
    LASER_REQUIRE(keys && ctx_tail && tree_len && match_n && ((tree_tokens && tree_parent) || K == 0), LASER_E_INVALID_ARG,
                  "NULL device buffer");
    TreeArgs a{p->P, p->seq_end, p->sa, p->table, p->cap_mask, keys, ctx_tail, B, n_min, n_max, K, min_tokens < 1 ? 1 : min_tokens,
               tree_tokens, tree_parent, tree_freq, tree_len, match_n};
    hipLaunchKernelGGL(retrieve_tree_kernel, dim3(B), dim3(64), 0, (hipStream_t)stream, a);
    LASER_HIP_CHECK(hipGetLastError());
    return LASER_OK;
}

extern "C" int laser_own_text_append(int32_t* own_tokens, int32_t* own_len, int own_cap, const int32_t* out_tokens,
                                     const int32_t* accept_len, int B, int K, void* stream) {
    LASER_REQUIRE(B >= 0 && K >= 0 && K <= LASER_MAX_DRAFT, LASER_E_INVALID_ARG, "B < 0 or K outside 0..%d", LASER_MAX_DRAFT);
    LASER_REQUIRE(own_cap >= 1 && own_cap <= LASER_MAX_OWN_TEXT, LASER_E_INVALID_ARG, "own_cap %d outside 1..%d", own_cap,
                  LASER_MAX_OWN_TEXT);
    if (B == 0) return LASER_OK;
    LASER_REQUIRE(own_tokens && own_len && out_tokens && accept_len, LASER_E_INVALID_ARG, "NULL device buffer");
    hipLaunchKernelGGL(own_text_append_kernel, dim3(B), dim3(256), 0, (hipStream_t)stream, own_tokens, own_len, own_cap,
                       out_tokens, accept_len, K);
    LASER_HIP_CHECK(hipGetLastError());
    return LASER_OK;
}

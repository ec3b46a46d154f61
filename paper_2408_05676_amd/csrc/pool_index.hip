// Construction of a pool's suffix index on the device (the layout is described in pool.hip): the occurrence array by a
// least-significant-digit radix sort, its runs by one comparison of each occurrence with the one before it, the table by
// parallel insertion.
//
// What bounds it: on the host the comparison sort, the two passes over the runs and the table inserts were chains of
// cache misses; here every step is a pass over at most four bytes per token and digit, and what is left are the
// copies to the device and the allocations.
#include <algorithm>
#include <cstring>
#include <utility>

#include "pool.h"

namespace laser {

namespace {

constexpr int kSortTile = 4096;      // occurrences a workgroup of 256 threads sorts per pass
constexpr int kSortPer = kSortTile / 256;
constexpr int kRunTile = 2048;       // occurrences of a workgroup in the run kernels
constexpr int kRunPer = kRunTile / 256;

struct IndexArgs {
    const int32_t* src;              // tokens as supplied
    const uint32_t *dst_off, *src_off, *sub;      // PoolLayout
    const int64_t* sub_key;
    uint32_t n_seq, n_tok, n_sa;
    int n_max;
    int32_t* P; uint32_t* seq_end;
    uint32_t *seq_begin, *sub_of;    // per position
    uint8_t* lcp;                    // per entry of sa: tokens it shares with the entry before it (low half) and tokens it has (high half), both up to n_max
    uint32_t n_chunks;
    uint32_t* next;                  // [n_max][n_chunks] first run boundary of the chunk, then of all chunks from there on
    unsigned long long* n_runs;
    uint32_t* longest;               // set when a run is too long for an index entry
    IndexEntry* table; uint64_t cap_mask;
};

// The tokens and their sequence's bounds at every position, and the positions that have a successor in ascending order.
__global__ __launch_bounds__(256) void layout_kernel(IndexArgs a, uint32_t* __restrict__ order) {
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < a.n_tok; i += (uint64_t)gridDim.x * 256) {
        const uint32_t e = (uint32_t)i;
        uint32_t s = 0, hi = a.n_seq;                    // the last sequence that begins at or before e
        while (hi - s > 1) {
            const uint32_t mid = s + (hi - s) / 2;
            if (a.dst_off[mid] <= e) s = mid; else hi = mid;
        }
        const uint32_t b = a.dst_off[s], end = a.dst_off[s + 1];
        a.P[e] = a.src[a.src_off[s] + (e - b)];
        a.seq_begin[e] = b;
        a.seq_end[e] = end;
        a.sub_of[e] = a.sub[s];
        if (e + 1 < end) order[e - s] = e;               // one position of every sequence before it is left out
    }
}

// Eight bits of what occurrence e is sorted by: its token `back` places back (none: before everything), or its sub-pool.
struct Digit { int back; int shift; };
__device__ inline uint32_t digit_of(const IndexArgs& a, Digit dg, uint32_t e) {
    uint32_t v;
    if (dg.back < 0) v = a.sub_of[e];
    else v = e - a.seq_begin[e] >= (uint32_t)dg.back ? (uint32_t)a.P[e - dg.back] + 1u : 0u;
    return (v >> dg.shift) & 255u;
}

__global__ __launch_bounds__(256) void sort_count_kernel(IndexArgs a, Digit dg, const uint32_t* __restrict__ in, uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[256];
    const int tid = threadIdx.x;
    h[tid] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kSortTile;
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
        const uint64_t i = base + r * 256 + tid;
        if (i < a.n_sa) atomicAdd(&h[digit_of(a, dg, in[i])], 1u);
    }
    __syncthreads();
    hist[(size_t)tid * gridDim.x + blockIdx.x] = h[tid];
}

// sum over the lanes before this one; *total = over the wave
__device__ inline uint32_t wave_scan(uint32_t v, int lane, uint32_t* total) {
    uint32_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)x, off);
        if (lane >= off) x += o;
    }
    *total = (uint32_t)__shfl((int)x, 63);
    return x - v;
}
__device__ inline uint32_t block_scan(uint32_t v, uint32_t* sm /*[4]*/, uint32_t* total) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t wt;
    uint32_t x = wave_scan(v, lane, &wt);
    __syncthreads();
    if (lane == 0) sm[wave] = wt;
    __syncthreads();
    uint32_t t = 0;
    for (int w = 0; w < 4; ++w) { if (w < wave) x += sm[w]; t += sm[w]; }
    *total = t;
    return x;
}

// One workgroup per digit value: its counts over the tiles become the sum of the tiles before.
__global__ __launch_bounds__(256) void sort_scan_kernel(uint32_t* __restrict__ hist, uint32_t n_blk, uint32_t* __restrict__ total) {
    __shared__ uint32_t sm[4];
    uint32_t* row = hist + (size_t)blockIdx.x * n_blk;
    uint32_t carry = 0;
    for (uint32_t b0 = 0; b0 < n_blk; b0 += 256) {
        const uint32_t b = b0 + threadIdx.x;
        uint32_t t;
        const uint32_t x = block_scan(b < n_blk ? row[b] : 0u, sm, &t);
        if (b < n_blk) row[b] = carry + x;
        carry += t;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// Stable: a wave takes 1024 neighbouring entries, 64 at a time; entries of a digit keep their order by counting the lanes
// before them that hold the same digit.
__global__ __launch_bounds__(256) void sort_scatter_kernel(IndexArgs a, Digit dg, const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                           const uint32_t* __restrict__ hist, const uint32_t* __restrict__ total) {
    __shared__ uint32_t at[4][256];
    __shared__ uint32_t sm[4];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    for (int w = 0; w < 4; ++w) at[w][tid] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kSortTile + wave * (kSortTile / 4) + lane;
    uint32_t e[kSortPer], d[kSortPer];
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) e[r] = base + r * 64 < a.n_sa ? in[base + r * 64] : 0u;
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
        const bool have = base + r * 64 < a.n_sa;
        d[r] = have ? digit_of(a, dg, e[r]) : 0u;
        if (have) atomicAdd(&at[wave][d[r]], 1u);
    }
    uint32_t all;
    uint32_t x = block_scan(total[tid], sm, &all) + hist[(size_t)tid * gridDim.x + blockIdx.x];
    for (int w = 0; w < 4; ++w) { const uint32_t c = at[w][tid]; at[w][tid] = x; x += c; }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
        const bool have = base + r * 64 < a.n_sa;
        unsigned long long same = __ballot(have);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const unsigned long long m = __ballot((d[r] >> b) & 1u);
            same &= ((d[r] >> b) & 1u) ? m : ~m;
        }
        if (have) {
            const int rank = __popcll(same & ((1ull << lane) - 1ull)), first = __ffsll(same) - 1;
            uint32_t p = 0;
            if (rank == 0) p = atomicAdd(&at[wave][d[r]], (uint32_t)__popcll(same));
            p = (uint32_t)__shfl((int)p, first);
            out[p + rank] = e[r];
        }
    }
}

// Where runs begin. Entry j begins a run of n-grams if it has n tokens and shares fewer than n with entry j - 1; the
// run ends at the next entry that shares fewer than n with its predecessor.
__global__ __launch_bounds__(256) void run_bounds_kernel(IndexArgs a, const uint32_t* __restrict__ sa) {
    __shared__ uint32_t first[LASER_MAX_NGRAM];
    __shared__ uint32_t sm[4];
    const int tid = threadIdx.x;
    if (tid < a.n_max) first[tid] = 0xFFFFFFFFu;
    __syncthreads();
    uint32_t heads = 0;
    for (int k = 0; k < kRunPer; ++k) {
        const uint64_t j = (uint64_t)blockIdx.x * kRunTile + k * 256 + tid;
        if (j >= a.n_sa) break;
        const uint32_t e = sa[j], he = e - a.seq_begin[e];
        const int have = he + 1 < (uint32_t)a.n_max ? (int)he + 1 : a.n_max;
        int l = 0;
        if (j > 0) {
            const uint32_t f = sa[j - 1], hf = f - a.seq_begin[f];
            if (a.sub_of[e] == a.sub_of[f])
                while (l < have && (uint32_t)l <= hf && a.P[e - l] == a.P[f - l]) ++l;
        }
        a.lcp[j] = (uint8_t)(l | (have << 4));
        heads += (uint32_t)(have - l);
        for (int n = l + 1; n <= a.n_max; ++n) atomicMin(&first[n - 1], (uint32_t)j);
    }
    uint32_t t;
    block_scan(heads, sm, &t);
    if (tid == 0 && t) atomicAdd(a.n_runs, (unsigned long long)t);
    if (tid < a.n_max) a.next[(size_t)tid * a.n_chunks + blockIdx.x] = first[tid];
}

// smallest value of this thread and the threads after it
__device__ inline uint32_t block_suffix_min(uint32_t v, uint32_t* sm /*[4]*/) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = (uint32_t)__shfl_down((int)v, off);
        if (lane + off < 64) v = min(v, o);
    }
    __syncthreads();
    if (lane == 0) sm[wave] = v;
    __syncthreads();
    for (int w = wave + 1; w < 4; ++w) v = min(v, sm[w]);
    return v;
}

// One workgroup per n: the first boundary at or after each chunk's begin.
__global__ __launch_bounds__(256) void run_next_kernel(IndexArgs a) {
    __shared__ uint32_t sm[4];
    uint32_t* row = a.next + (size_t)blockIdx.x * a.n_chunks;
    uint32_t carry = a.n_sa;
    for (int64_t c0 = ((int64_t)a.n_chunks - 1) / 256 * 256; c0 >= 0; c0 -= 256) {
        const int64_t c = c0 + threadIdx.x;
        const uint32_t x = min(block_suffix_min(c < a.n_chunks ? row[c] : 0xFFFFFFFFu, sm), carry);
        if (c < a.n_chunks) row[c] = x;
        __syncthreads();                                 // the first thread's result is the next round's carry
        if (threadIdx.x == 0) sm[0] = x;
        __syncthreads();
        carry = sm[0];
    }
}

// Every run becomes a table entry. The half of an entry that marks it taken is exchanged atomically, the key follows as an
// ordinary store (nothing reads keys before the kernel ends). The table has at least twice as many slots as there are runs.
__global__ __launch_bounds__(256) void run_insert_kernel(IndexArgs a, const uint32_t* __restrict__ sa) {
    __shared__ uint32_t sm[4];
    const int tid = threadIdx.x;
    const uint64_t j0 = (uint64_t)blockIdx.x * kRunTile + (uint64_t)tid * kRunPer;
    int lc[kRunPer];
#pragma unroll
    for (int k = 0; k < kRunPer; ++k) lc[k] = j0 + k < a.n_sa ? a.lcp[j0 + k] : 0x0F;     // past the end: neither a boundary nor a run
    for (int n = 1; n <= a.n_max; ++n) {
        uint32_t mine = 0xFFFFFFFFu;
#pragma unroll
        for (int k = kRunPer - 1; k >= 0; --k) if ((lc[k] & 15) < n) mine = (uint32_t)(j0 + k);
        // the first boundary after this thread's entries: of the threads after it, or of the chunks after this one
        const uint32_t here = block_suffix_min(mine, sm);
        uint32_t nxt = (uint32_t)__shfl_down((int)here, 1);
        __syncthreads();
        if ((tid & 63) == 0) sm[tid >> 6] = here;
        __syncthreads();
        if ((tid & 63) == 63) nxt = tid < 255 ? sm[(tid >> 6) + 1] : 0xFFFFFFFFu;
        __syncthreads();
        if (nxt == 0xFFFFFFFFu) nxt = blockIdx.x + 1 < a.n_chunks ? a.next[(size_t)(n - 1) * a.n_chunks + blockIdx.x + 1] : a.n_sa;
        for (int k = kRunPer - 1; k >= 0; --k) {
            int l = 0x0F;
#pragma unroll
            for (int q = 0; q < kRunPer; ++q) l = q == k ? lc[q] : l;
            if ((l & 15) >= n) continue;
            const uint32_t j = (uint32_t)(j0 + k);
            if ((l >> 4) >= n) {
                const uint32_t e = sa[j], count = nxt - j;
                if (count >= (1u << 28)) atomicMax(a.longest, count);
                int32_t w[LASER_MAX_NGRAM];
#pragma unroll
                for (int i = 0; i < LASER_MAX_NGRAM; ++i) w[i] = i < n ? a.P[e - (uint32_t)(n - 1) + i] : 0;
                const int64_t key = a.sub_key[a.sub_of[e]];
                uint64_t slot = ngram_hash(key, n, w) & a.cap_mask;
                const unsigned long long mark = (unsigned long long)j | ((unsigned long long)(count | ((uint32_t)n << 28)) << 32);
                while (atomicCAS(reinterpret_cast<unsigned long long*>(&a.table[slot].start), 0ull, mark) != 0ull) slot = (slot + 1) & a.cap_mask;
                a.table[slot].key = key;
            }
            nxt = j;
        }
    }
}

// What the build allocates; freed on every way out unless handed over. The working arrays are the stream's (hipFree waits for
// all streams of the device: a build beside other work would end when that work does). Given back, they leave the device's
// memory pool at once: by itself it keeps them until a later wait.
struct Buffers {
    hipStream_t stream;
    void* work = nullptr;
    void* p[4] = {};
    ~Buffers() {
        if (work) {
            int dev = 0;
            hipMemPool_t pool;
            uint64_t keep = 0;
            (void)hipFreeAsync(work, stream);
            (void)hipStreamSynchronize(stream);
            if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetMemPool(&pool, dev) == hipSuccess &&
                hipMemPoolGetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep) == hipSuccess)
                (void)hipMemPoolTrimTo(pool, keep);
        }
        for (void* q : p) if (q) (void)hipFree(q);
    }
};

}  // namespace

int build_index_device(const int32_t* tokens, const PoolLayout& lay, int n_max, int64_t mem_limit, hipStream_t stream, Pool* p, bool* no_memory) {
    *no_memory = false;
    IndexArgs a{};
    a.n_seq = (uint32_t)lay.sub.size();
    a.n_tok = lay.dst_off.back();
    a.n_sa = a.n_tok - a.n_seq;
    a.n_max = n_max;
    a.n_chunks = (uint32_t)(((uint64_t)a.n_sa + kRunTile - 1) / kRunTile);
    const uint32_t n_blk = (uint32_t)(((uint64_t)a.n_sa + kSortTile - 1) / kSortTile);
    const size_t n_tok = a.n_tok, n_sa = a.n_sa, n_seq = a.n_seq, n_sub = lay.sub_key.size();

    // working arrays, one allocation (every part 256-byte aligned)
    size_t bytes = 0;
    auto part = [&](size_t n) { const size_t at = bytes; bytes += (n + 255) / 256 * 256; return at; };
    const size_t o_src = part(n_tok * 4), o_begin = part(n_tok * 4), o_sub = part(n_tok * 4), o_alt = part(n_sa * 4), o_hist = part((size_t)n_blk * 1024),
                 o_total = part(1024), o_lcp = part(n_sa), o_next = part((size_t)n_max * a.n_chunks * 4), o_cnt = part(16),
                 o_lay = part((3 * n_seq + 1) * 4), o_key = part(n_sub * 8);
    std::vector<uint32_t> pack(3 * n_seq + 1);
    std::memcpy(pack.data(), lay.dst_off.data(), (n_seq + 1) * 4);
    std::memcpy(pack.data() + n_seq + 1, lay.src_off.data(), n_seq * 4);
    std::memcpy(pack.data() + 2 * n_seq + 1, lay.sub.data(), n_seq * 4);
    Buffers buf{stream};             // P, seq_end, sa, table; working arrays
    size_t taken = 0;
    auto take = [&](void** at, size_t n, bool work) {
        taken += n;
        hipError_t e = hipErrorOutOfMemory;
        if (mem_limit < 0 || taken <= (uint64_t)mem_limit) e = work ? hipMallocAsync(at, n, stream) : hipMalloc(at, n);
        if (e == hipErrorOutOfMemory) { *no_memory = true; (void)hipGetLastError(); }
        return e;
    };
    LASER_HIP_CHECK(take(&buf.p[0], n_tok * 4, false));
    LASER_HIP_CHECK(take(&buf.p[1], n_tok * 4, false));
    LASER_HIP_CHECK(take(&buf.p[2], n_sa * 4, false));
    LASER_HIP_CHECK(take(&buf.work, bytes, true));
    char* const ws = (char*)buf.work;
    a.P = (int32_t*)buf.p[0];
    a.seq_end = (uint32_t*)buf.p[1];
    a.src = (const int32_t*)(ws + o_src);
    a.seq_begin = (uint32_t*)(ws + o_begin);
    a.sub_of = (uint32_t*)(ws + o_sub);
    a.lcp = (uint8_t*)(ws + o_lcp);
    a.next = (uint32_t*)(ws + o_next);
    a.n_runs = (unsigned long long*)(ws + o_cnt);
    a.longest = (uint32_t*)(ws + o_cnt + 8);
    a.dst_off = (const uint32_t*)(ws + o_lay);
    a.src_off = a.dst_off + n_seq + 1;
    a.sub = a.src_off + n_seq;
    a.sub_key = (const int64_t*)(ws + o_key);
    uint32_t* const hist = (uint32_t*)(ws + o_hist);
    uint32_t* const total = (uint32_t*)(ws + o_total);

    LASER_HIP_CHECK(hipMemcpyAsync(ws + o_src, tokens, n_tok * 4, hipMemcpyHostToDevice, stream));
    LASER_HIP_CHECK(hipMemcpyAsync(ws + o_lay, pack.data(), pack.size() * 4, hipMemcpyHostToDevice, stream));
    LASER_HIP_CHECK(hipMemcpyAsync(ws + o_key, lay.sub_key.data(), n_sub * 8, hipMemcpyHostToDevice, stream));
    LASER_HIP_CHECK(hipMemsetAsync(ws + o_cnt, 0, 16, stream));

    // digits, the last token back first, the sub-pool last; as many as the values have. The sorted array has to end in sa.
    auto bits = [](uint32_t v) { int b = 0; while (v) { ++b; v >>= 1; } return b; };
    std::vector<Digit> passes;
    const int tok_bits = bits(lay.token_bits + 1u), sub_bits = bits((uint32_t)(n_sub - 1));
    for (int i = n_max - 1; i >= 0; --i)
        for (int s = 0; s < tok_bits; s += 8) passes.push_back({i, s});
    for (int s = 0; s < sub_bits; s += 8) passes.push_back({-1, s});
    uint32_t* in = passes.size() % 2 ? (uint32_t*)(ws + o_alt) : (uint32_t*)buf.p[2];
    uint32_t* alt = passes.size() % 2 ? (uint32_t*)buf.p[2] : (uint32_t*)(ws + o_alt);
    const unsigned lay_blk = (unsigned)std::min<size_t>((n_tok + 255) / 256, 65536);
    hipLaunchKernelGGL(layout_kernel, dim3(lay_blk), dim3(256), 0, stream, a, in);
    for (const Digit dg : passes) {
        hipLaunchKernelGGL(sort_count_kernel, dim3(n_blk), dim3(256), 0, stream, a, dg, in, hist);
        hipLaunchKernelGGL(sort_scan_kernel, dim3(256), dim3(256), 0, stream, hist, n_blk, total);
        hipLaunchKernelGGL(sort_scatter_kernel, dim3(n_blk), dim3(256), 0, stream, a, dg, in, alt, hist, total);
        std::swap(in, alt);
    }
    const uint32_t* const sa = in;
    hipLaunchKernelGGL(run_bounds_kernel, dim3(a.n_chunks), dim3(256), 0, stream, a, sa);
    hipLaunchKernelGGL(run_next_kernel, dim3((unsigned)n_max), dim3(256), 0, stream, a);
    LASER_HIP_CHECK(hipGetLastError());

    // the table's size follows from the number of runs
    unsigned long long n_runs = 0;
    LASER_HIP_CHECK(hipMemcpyAsync(&n_runs, a.n_runs, 8, hipMemcpyDeviceToHost, stream));
    LASER_HIP_CHECK(hipStreamSynchronize(stream));
    uint64_t cap = 16;
    while (cap < 2 * n_runs) cap <<= 1;
    a.cap_mask = cap - 1;
    LASER_HIP_CHECK(take(&buf.p[3], cap * sizeof(IndexEntry), false));
    a.table = (IndexEntry*)buf.p[3];
    LASER_HIP_CHECK(hipMemsetAsync(a.table, 0, cap * sizeof(IndexEntry), stream));
    hipLaunchKernelGGL(run_insert_kernel, dim3(a.n_chunks), dim3(256), 0, stream, a, sa);
    LASER_HIP_CHECK(hipGetLastError());
    uint32_t longest = 0;
    LASER_HIP_CHECK(hipMemcpyAsync(&longest, a.longest, 4, hipMemcpyDeviceToHost, stream));
    LASER_HIP_CHECK(hipStreamSynchronize(stream));
    LASER_REQUIRE(longest < (1u << 28), LASER_E_LIMIT, "an n-gram occurs %u times (limit 2^28-1)", longest);

    p->P = (int32_t*)buf.p[0]; p->seq_end = (uint32_t*)buf.p[1]; p->sa = (uint32_t*)buf.p[2]; p->table = (IndexEntry*)buf.p[3];
    for (int i = 0; i < 4; ++i) buf.p[i] = nullptr;
    p->cap_mask = cap - 1;
    p->n_tokens = (int64_t)n_tok; p->n_keys = (int64_t)n_sub; p->n_entries = (int64_t)n_runs; p->n_sa = (int64_t)n_sa; p->n_max = n_max;
    p->device_bytes = (int64_t)(n_tok * 8 + n_sa * 4 + cap * sizeof(IndexEntry));
    return LASER_OK;
}

}  // namespace laser

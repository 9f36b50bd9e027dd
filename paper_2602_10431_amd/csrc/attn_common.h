// What the attention kernels share: their arguments, the accesses that are coherent across the XCDs, and the combination of
// key ranges by the workgroup that arrives last.
#pragma once
#include "qtale_dev.h"
#include "qtale_kernels.h"

namespace qtale {

constexpr float kNegBig = -1.0e30f;

struct AttnDev {
    const half_t* qkv;
    half_t* out;
    int nh, nkv, width;          // width = (nh + 2 nkv) * d
    const int32_t* count;
    const int32_t* cu_exec;
    const int32_t* row_seq;
    const int4* items;           // prefill work list: (sequence or -1, query tile, first compact row, rows) per item
    int items_max;               // host bound on the number of work items (row stride of the logical grid)
    const int32_t* tiles;        // prefill, split keys: key tiles per range
    half_t* k_cache;
    half_t* v_cache;
    const int32_t* kv_old;
    int cap;
    float scale_log2;            // log2(e) / sqrt(d)
    const float2* cs;            // decode: [row][D / 2] (cos, sin) at the row's position
    int32_t* arrive;             // split keys: ranges done so far, [row][kv head] or (prefill) [item][head]
    const int32_t* chunk;        // decode, split keys: cached keys per range (nullable: n_split ranges of equal length per row)
    float* part;                 // split keys, decode: [row][head][split][D + 2] fp32 (numerators, reference point, denominator)
    int n_split;                 // bound on the key ranges per (row, kv head) or item; 1 = no split
};

// Accesses that are coherent across the XCDs (and with the counter they are used with).
__device__ __forceinline__ void agent_store(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float agent_load(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// A cached key or value of a sequence with one executed row is read once per call: loaded as non-temporal it does not turn over the L2
// on its way.  (One query head per kv head, 64 rows x 32 heads x 2048 keys, 27 GB of caches in rotation so that nothing stays in the
// memory-side cache: layer 449.5 -> 413.6 us, 6.0 -> 6.6 TB/s in this kernel; 128 rows of the 13B shape 536 -> 493; 8 rows x 2000 keys
// 107 -> 100.)  The rows of a longer new part read the same keys again, which the L2 serves: ordinary loads there.  Layers, us, all
// non-temporal / by the sequence's rows / all ordinary: 7B shape 16 x 4 rows on 2000 keys 294 / 239 / 237, 32 x 4 on 4000 1020 / 658 / 651,
// 31 x 1 + 65 on 1000 264 / 233 / 243, one sequence of 64 beside idle ones on 4000 426 / 271 / 271; four query heads per kv head,
// 32 x 4 on 4000 320 / 303 / 302, 31 x 1 on 100 + 65 on 8000 367 / 342 / 349.
template <class T>
__device__ __forceinline__ T stream_load(const __attribute__((address_space(1))) T* p) { return __builtin_nontemporal_load(p); }

// One side of a branch whose other side makes the same loads as ordinary ones: without something of its own on either end the compiler
// makes one of both, and ordinary.
template <class F>
__device__ __forceinline__ void keep_side(F&& f) {
    __builtin_amdgcn_sched_barrier(0);
    f();
    __builtin_amdgcn_sched_barrier(0);
}

// The cached keys of a (row, kv head) that this workgroup streams.  Without a split all of them.
struct KeyRange {
    int lo, hi, ranges;          // ranges: how many there are for this (row, kv head); the grid holds n_split
    bool none;                   // blockIdx.z is past the last range
};
template <bool SPLIT>
__device__ __forceinline__ KeyRange decode_key_range(const AttnDev& p, int n_cached, int gran) {
    if (!SPLIT) return {0, n_cached, 1, false};
    const int per = p.chunk ? *p.chunk : ((n_cached + p.n_split - 1) / p.n_split + gran - 1) / gran * gran;
    const int ranges = max((n_cached + per - 1) / max(per, 1), 1), z = blockIdx.z;
    const int lo = min(z * per, n_cached);
    return {lo, min(lo + per, n_cached), ranges, z >= ranges};
}

// Split keys, after the workgroup has written its ranges' sums to p.part with agent_store: the range that arrives last
// combines all of them, out = sum_s num_s 2^(m_s - m) / sum_s den_s 2^(m_s - m).  Nobody waits: a workgroup counts itself in
// and leaves unless it is the last.  The ranges may have run on different XCDs, whose L2s are not coherent with each other
// for plain accesses: the partial sums are written and read with agent-scope accesses (they go past the L2), and every
// thread's stores have completed (vmcnt 0, then the barrier) before thread 0 counts.  A release fence instead would write
// back a whole L2 per workgroup.
template <int D, int REP>
__device__ __forceinline__ void combine_key_ranges(const AttnDev& p, int i, int hk, int ranges, int tid) {
    __shared__ int s_arrived;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) s_arrived = __hip_atomic_fetch_add(p.arrive + static_cast<size_t>(i) * p.nkv + hk, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_arrived != ranges - 1) return;
    for (int c = tid; c < REP * D; c += 256) {
        const int r = c / D, e = c % D;
        const float* src = p.part + (static_cast<size_t>(i) * p.nh + hk * REP + r) * p.n_split * (D + 2);
        float num_s[kAttnSplitMax], m_s[kAttnSplitMax], den_s[kAttnSplitMax];
        float mn = kNegBig;
#pragma unroll
        for (int s = 0; s < kAttnSplitMax; ++s) {            // all ranges are requested before any is used
            const float* ps = src + min(s, ranges - 1) * (D + 2);
            num_s[s] = agent_load(ps + e);
            m_s[s] = agent_load(ps + D);
            den_s[s] = agent_load(ps + D + 1);
        }
#pragma unroll
        for (int s = 0; s < kAttnSplitMax; ++s) mn = fmaxf(mn, m_s[s]);
        float num = 0.0f, den = 0.0f;
#pragma unroll
        for (int s = 0; s < kAttnSplitMax; ++s) {
            const float a = s < ranges ? exp2f(m_s[s] - mn) : 0.0f;
            num += num_s[s] * a;
            den += den_s[s] * a;
        }
        p.out[static_cast<size_t>(i) * (p.nh * D) + (hk * REP + r) * D + e] = static_cast<half_t>(num / den);
    }
}

// The prefill work list (AttnList), built by 256 threads: one item per (sequence, tile of kAttnBQ executed rows), carrying the
// sequence's first compact row and row count so that the attention workgroups need no further lookups.  The list is sorted by query tile index, highest
// first, across all sequences (the tile index is the item's length in keys up to the cached prefix): a counting
// sort over the tiles-per-sequence histogram.  `levels` is the host bound on tiles per sequence (<= kItemLevels).
constexpr int kItemLevels = 1024;

template <class Rows>
__device__ __forceinline__ int attn_build_sorted(const AttnList& a, int4* __restrict__ items, Rows&& rows_of) {
    __shared__ int cnt[kItemLevels + 1];      // first: sequences with exactly n tiles; then: sequences with more than n
    __shared__ int offs[kItemLevels + 1];     // items of the tile indices above q
    __shared__ int fill[kItemLevels + 1];
    __shared__ int s_total;
    const int tid = threadIdx.x, lane = tid & 63, levels = a.levels;
    for (int i = tid; i <= levels; i += 256) { cnt[i] = 0; fill[i] = 0; }
    __syncthreads();
    for (int b = tid; b < a.B; b += 256) {
        int first;
        const int nt = min((rows_of(b, first) + kAttnBQ - 1) / kAttnBQ, levels);
        atomicAdd(&cnt[nt], 1);
    }
    __syncthreads();
    if (tid < 64) {
        // two suffix sums over the levels, one wave: lane l owns a chunk of consecutive levels
        const int chunk = (levels + 64) / 64;
        const int lo = lane * chunk, hi = min(lo + chunk, levels + 1);
        int own = 0;
        for (int n = lo; n < hi; ++n) own += cnt[n];
        int above = 0;                                           // sum of the chunks of the lanes above
        {
            int incl = own;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_down(incl, o, 64);
                if (lane + o < 64) incl += t;
            }
            above = incl - own;
        }
        int own2 = 0;
        for (int n = hi - 1; n >= lo; --n) {
            const int h = cnt[n];
            cnt[n] = above;                                      // sequences with more than n tiles
            own2 += above;
            above += h;
        }
        int above2 = 0;
        {
            int incl = own2;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_down(incl, o, 64);
                if (lane + o < 64) incl += t;
            }
            above2 = incl - own2;
        }
        for (int n = hi - 1; n >= lo; --n) {
            offs[n] = above2;                                    // items with a tile index above n
            above2 += cnt[n];
        }
        if (lane == 0) s_total = above2;                         // lane 0 ends below level 0: all items
    }
    __syncthreads();
    for (int b = tid; b < a.B; b += 256) {
        int first;
        const int rows = rows_of(b, first);
        const int nt = min((rows + kAttnBQ - 1) / kAttnBQ, levels);
        if (nt == 0) continue;
        const int pos = cnt[nt] + atomicAdd(&fill[nt], 1);        // place among the sequences, most tiles first
        for (int q = 0; q < nt; ++q) items[offs[q] + pos] = make_int4(b, q, first, rows);
    }
    return s_total;
}

// The same list for calls whose sequences could have more than kItemLevels query tiles: sequence by sequence, each
// sequence's tiles longest first.
template <class Rows>
__device__ __forceinline__ int attn_build_by_sequence(const AttnList& a, int4* __restrict__ items, Rows&& rows_of) {
    __shared__ int s_wave[4];
    __shared__ int s_base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_base = 0;
    __syncthreads();
    for (int b0 = 0; b0 < a.B; b0 += 256) {
        const int b = b0 + threadIdx.x;
        int first = 0;
        const int rows = b < a.B ? rows_of(b, first) : 0;
        const int nt = (rows + kAttnBQ - 1) / kAttnBQ;
        int incl = nt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int start = s_base + incl - nt;
        for (int w = 0; w < wave; ++w) start += s_wave[w];
        for (int q = 0; q < nt; ++q) items[start + q] = make_int4(b, nt - 1 - q, first, rows);   // longest tiles first
        __syncthreads();
        if (threadIdx.x == 0) s_base += s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
        __syncthreads();
    }
    return s_base;
}


__device__ __forceinline__ int tiles_per_range(const AttnList& a, int used, int tiles, int longest) {
    const int fill = static_cast<int>((static_cast<long>(tiles) * a.heads + a.target - 1) / a.target);   // the ranges fill the chip once
    const bool cut = 2l * used * a.heads < a.target;
    return cut ? max(max(fill, (longest + a.n_split - 1) / a.n_split), kAttnTileRange) : max(longest, 1);
}

// List, length of the key ranges and cleared counters, by one workgroup of 256 threads.  A launch of its own for this took 4.6 us
// of every prefill call.
__device__ __forceinline__ void attn_build_list(const AttnList& a) {
    __shared__ int s_tiles, s_longest;
    int4* items = reinterpret_cast<int4*>(a.items);
    const int tid = threadIdx.x;
    if (tid == 0) { s_tiles = 0; s_longest = 0; }
    // sequence tid's rows and cache length are loaded once, together (every trip to memory is a third of this workgroup's time)
    int own_first = 0, own_end = 0, own_old = 0;
    if (tid < a.B) {
        own_first = a.cu_exec[tid];
        own_end = a.cu_exec[tid + 1];
        if (a.n_split > 1 && a.kv_old) own_old = a.kv_old[tid];
    }
    auto rows_of = [&](int b, int& first) {
        first = b == tid ? own_first : a.cu_exec[b];
        return (b == tid ? own_end : a.cu_exec[b + 1]) - first;
    };
    if (a.B <= 64 && a.levels <= 64) {
        // One wave, a sequence per lane: the items of query tile q are the sequences with more than q tiles, in sequence order
        if (a.n_split > 1)
            for (int i = tid; i < a.items_max * a.heads; i += 256) a.arrive[i] = 0;
        if (tid >= 64) return;
        const int rows = tid < a.B ? own_end - own_first : 0, nt = min((rows + kAttnBQ - 1) / kAttnBQ, a.levels);
        int used = 0, tiles = 0, longest = 0;
        for (int q = a.levels - 1; q >= 0; --q) {
            const unsigned long long m = __ballot(nt > q);
            if (nt > q) {
                items[used + __popcll(m & ((1ull << tid) - 1ull))] = make_int4(tid, q, own_first, rows);
                const int keys = own_old + min((q + 1) * kAttnBQ, rows);
                const int n = ((a.kv_old ? min(keys, a.cap) : keys) + 63) / 64;
                tiles += n;
                longest = max(longest, n);
            }
            used += __popcll(m);
        }
        for (int i = used + tid; i < a.items_max; i += 64) items[i] = make_int4(-1, 0, 0, 0);
        if (a.n_split <= 1) return;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            tiles += __shfl_xor(tiles, o, 64);
            longest = max(longest, __shfl_xor(longest, o, 64));
        }
        if (tid == 0) *a.tiles = tiles_per_range(a, used, tiles, longest);
        return;
    }
    const int used = a.levels <= kItemLevels ? attn_build_sorted(a, items, rows_of) : attn_build_by_sequence(a, items, rows_of);
    for (int i = used + threadIdx.x; i < a.items_max; i += 256) items[i] = make_int4(-1, 0, 0, 0);   // unused slots
    if (a.n_split <= 1) return;
    for (int i = threadIdx.x; i < a.items_max * a.heads; i += 256) a.arrive[i] = 0;
    __syncthreads();
    // key tiles of all items, and of the longest
    int tiles = 0, longest = 0;
    for (int b = threadIdx.x; b < a.B; b += 256) {
        int first;
        const int rows = rows_of(b, first), old = !a.kv_old ? 0 : b == tid ? own_old : a.kv_old[b];
        for (int q = 0; q < rows; q += kAttnBQ) {
            const int keys = old + min(q + kAttnBQ, rows);
            const int n = ((a.kv_old ? min(keys, a.cap) : keys) + 63) / 64;
            tiles += n;
            longest = max(longest, n);
        }
    }
    atomicAdd(&s_tiles, tiles);
    atomicMax(&s_longest, longest);
    __syncthreads();
    if (threadIdx.x == 0) *a.tiles = tiles_per_range(a, used, s_tiles, s_longest);
}

// The decode form for 2, 4 or 8 query heads per kv head (attention_gqa.hip); for one it is in attention.hip.
hipError_t launch_attn_decode_gqa(const AttnDev& d, int rep, int head_dim, int rows, hipStream_t stream);

}  // namespace qtale

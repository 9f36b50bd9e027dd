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
    const int32_t* n_items;
    int items_max;               // host bound on the number of work items (row stride of the logical grid)
    half_t* k_cache;
    half_t* v_cache;
    const int32_t* kv_old;
    int cap;
    float scale_log2;            // log2(e) / sqrt(d)
    const float2* cs;            // decode: [row][D / 2] (cos, sin) at the row's position
    int32_t* arrive;             // decode, split keys: [row][kv head] ranges done so far
    const int32_t* chunk;        // decode, split keys: cached keys per range (nullable: n_split ranges of equal length per row)
    float* part;                 // decode, split keys: [row][head][split][D + 2] fp32 (numerators, reference point, denominator)
    int n_split;                 // key ranges per (row, kv head); 1 = no split
};

// Accesses that are coherent across the XCDs (and with the counter they are used with).
__device__ __forceinline__ void agent_store(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float agent_load(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// A cached key or value is read once per call: loaded as non-temporal it does not turn over the L2 on its way.  (One query head
// per kv head, 64 rows x 32 heads x 2048 keys, 27 GB of caches in rotation so that nothing stays in the memory-side cache: layer
// 449.5 -> 413.6 us, 6.0 -> 6.6 TB/s in this kernel; 128 rows of the 13B shape 536 -> 493; 8 rows x 2000 keys 107 -> 100.)
template <class T>
__device__ __forceinline__ T stream_load(const __attribute__((address_space(1))) T* p) { return __builtin_nontemporal_load(p); }

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

// The decode form for 2, 4 or 8 query heads per kv head (attention_gqa.hip); for one it is in attention.hip.
hipError_t launch_attn_decode_gqa(const AttnDev& d, int rep, int head_dim, int rows, hipStream_t stream);

}  // namespace qtale

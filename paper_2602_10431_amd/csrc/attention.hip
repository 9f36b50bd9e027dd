// Attention restricted to executed tokens.
//
// A bypassed token produces no query, key or value at a layer (the whole layer is skipped for it, Eq. 3),
// so an executed token attends causally to the executed tokens of its own sequence only, in original
// order, preceded by that layer's cache entries (which also hold executed tokens only).  Rows of the
// compact q|k|v buffer are in ascending token order, so the executed tokens of sequence b are the rows
// cu_exec[b] .. cu_exec[b+1]-1 and "causal" means "row index <= own row index".
//
// Two kernels:
//   * flash_prefill: matrix-core tiles.  A workgroup of 4 waves owns 128 query rows of one (sequence,
//     head); keys/values stream through LDS in tiles of 64.  S^T = K Q^T is computed so that a lane owns
//     one query column (softmax statistics are per lane), and the probabilities, still in the MFMA
//     accumulator layout, are fed straight back as the B operand of O^T = V^T P^T; V is transposed on
//     its way into LDS.
//     The keys of few query tiles are cut into ranges (attention_prefill_plan).
//   * decode (one query head per kv head; grouped queries: attention_gqa.hip): one workgroup per (executed row, head); lanes stream
//     K and V rows with 16-byte loads, 16 (or 8) lanes per key, online softmax per lane group, merged at the end.  Bandwidth-bound.  It also
//     rotates the query and the call's own keys (table of the normalising kernel) and appends the new row, unless a call
//     has a long new part (attention_rotates); with
//     few rows the cached keys are cut into ranges and the workgroup that arrives last combines them.
#include <algorithm>
#include <type_traits>

#include "attn_common.h"

namespace qtale {

constexpr float kLog2e = 1.4426950408889634f;
template <int D, bool SPLIT>
__global__ void __launch_bounds__(256, 2)
flash_prefill_kernel(AttnDev p) {
    constexpr int KS = D / 16;          // k-steps of the QK^T product
    constexpr int DF = D / 32;          // 32-wide fragments of the head dimension
    constexpr int KSTR = D + 8;         // LDS row stride of the K tile (halves)
    // Transposed V tile Vt[column][key]: 64 keys + room for the column skew, row stride 42 dwords (16 lanes that read
    // 8 bytes of consecutive rows hit 16 different bank pairs).  A thread stores 4 keys (8 bytes) of 8 columns; the
    // 16 lanes that hold the same keys and 16 different column chunks dc would land on two bank pairs, so the key
    // group index is XOR-ed with dc >> 2 (uniform per 32-column fragment on the read side) and rows with bit 1 of dc
    // set are shifted by 8 dwords: bits 1-2, 3 and 4 of the bank index then come from dc >> 2, dc bit 1 and dc bit 0.
    constexpr int VSTR = 64 + 16 + 4;   // LDS row stride of the transposed V tile (halves)
    constexpr int CPR = D / 8;          // 16-byte chunks per K/V row
    constexpr int CH = (64 * CPR) / 256;     // K chunks per thread per tile
    constexpr int VG = (16 * CPR + 255) / 256;   // V groups (4 keys x 8 columns) per thread per tile
    constexpr int kSwShift = CPR == 8 ? 1 : 0;   // 8 chunks per row: two key groups share 16 lanes, swizzle bit 1 instead of bit 0
    __shared__ __attribute__((aligned(16))) half_t Ks2[2][64 * KSTR];    // double-buffered tiles
    __shared__ __attribute__((aligned(16))) half_t Vt2[2][D * VSTR];

    // Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  Every XCD gets a contiguous group of
    // heads (all query heads of a few key/value heads) and walks the work items in list order, the heads of the group
    // innermost: the list is sorted by length, longest first, so an XCD's 64 workgroup slots drain evenly (with the
    // heads outermost the long items of the last head started when most of the work was done: about a third of the
    // kernel time at two sequences of 4096 tokens was an idle tail), and the workgroups that run at the same time
    // belong to a few (sequence, head) pairs and similar key ranges, which the L2 serves.
    // With split keys the whole list repeats per range: the ranges that do not exist (most items have fewer than n_split) end
    // the grid and do not hold up the others.
    const int zs = SPLIT ? p.n_split : 1;
    int h, item;
    if ((p.nh & 7) == 0) {
        const int hx = p.nh >> 3;                                // heads per XCD; gridDim.x = 8 * hx * items_max * zs
        const int local = blockIdx.x >> 3;
        item = local / hx;
        h = (blockIdx.x & 7) * hx + (local - item * hx);
    } else {
        const int per_xcd = gridDim.x >> 3;
        const int L = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
        h = L / (p.items_max * zs);
        item = L - h * (p.items_max * zs);
    }
    int z = 0;
    if (SPLIT) {
        z = item / p.items_max;
        item -= z * p.items_max;
    }
    if (h >= p.nh) return;
    const int4 it = p.items[item];           // one load tells the workgroup everything (unused slots hold -1)
    const int b = it.x, qt = it.y;
    if (b < 0) return;
    const int hk = h / (p.nh / p.nkv);
    const int row_begin = it.z;
    const int n_b = it.w;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lhi = lane >> 5;

    // key/value source: the layer cache (new rows were appended before this kernel) or the compact buffer
    const half_t* kbase;
    const half_t* vbase;
    int kv_stride, base_len;
    if (p.k_cache) {
        base_len = p.kv_old[b];
        kv_stride = D;                                           // cache [B][n_kv_heads][cap][D]: a head's entries are contiguous
        kbase = p.k_cache + (static_cast<size_t>(b) * p.nkv + hk) * p.cap * D;
        vbase = p.v_cache + (static_cast<size_t>(b) * p.nkv + hk) * p.cap * D;
    } else {
        base_len = 0;
        kv_stride = p.width;
        kbase = p.qkv + static_cast<size_t>(row_begin) * p.width + (p.nh + hk) * D;
        vbase = kbase + p.nkv * D;
    }
    const int q_lo = qt * kAttnBQ;                               // first local query index of the block
    const int q_cnt = min(kAttnBQ, n_b - q_lo);
    int n_keys = base_len + q_lo + q_cnt;                        // keys visible to the last query
    if (p.k_cache) n_keys = min(n_keys, p.cap);
    const int all_tiles = (n_keys + 63) / 64;
    int t_lo = 0, n_tiles = all_tiles;                           // this workgroup's tiles
    int ranges = 1;
    if (SPLIT) {
        const int per = *p.tiles;
        ranges = (all_tiles + per - 1) / per;
        if (z >= ranges) return;
        t_lo = z * per;
        n_tiles = min(t_lo + per, all_tiles);
    }

    // this lane's query (column of S^T): local index inside the sequence, clamped to a valid row
    const int q_local = q_lo + min(wave * 32 + l32, q_cnt - 1);
    // keys [0, limit) are visible: those up to its own, of which a full cache may have dropped the last
    const int limit = min(base_len + q_local + 1, n_keys);
    const int wave_hi = min(base_len + q_lo + min(wave * 32 + 31, q_cnt - 1) + 1, n_keys);   // largest limit in the wave
    const int wave_lo = min(base_len + q_lo + min(wave * 32, q_cnt - 1) + 1, n_keys);        // smallest limit in the wave
    const half_t* qrow = p.qkv + static_cast<size_t>(row_begin + q_local) * p.width + h * D;
    // The queries stay as stored; the factor log2(e)/sqrt(d) is applied in fp32 inside the exponent's fused
    // multiply-add (folding it into the fp16 queries would round it, and every product, to 11 bits: an error in
    // the logits that grows with their magnitude).
    half8_t qf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const half8_t*>(qrow + 16 * s + 8 * lhi);
    const float sc = p.scale_log2;

    float16_t o[DF];
#pragma unroll
    for (int df = 0; df < DF; ++df)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[df][r] = 0.0f;
    float m_run = kNegBig, l_run = 0.0f;

    // global -> register staging of one tile.  K: chunk c is key c / CPR, 8 halves at (c % CPR)*8.
    // V: a thread owns 4 consecutive keys x 8 columns and transposes them in registers, so that the
    // transposed tile Vt[column][key] is written with 8-byte stores.
    // One register set: tile t+1 waits in it while tile t is computed.
    // Element offsets inside a tile are fixed per thread; a tile adds key0 * kv_stride, and the minimum with the
    // offset of the same column chunk in the last visible key keeps the (partial) last tile inside the sequence.
    u32x4_t kregs[CH], vregs[VG][4];
    uint32_t k_off[CH], k_max[CH], v_off[VG], v_max[VG];            // byte offsets (below 4 GB: 32-bit lane offsets on a uniform base)
    const uint32_t row_bytes = static_cast<uint32_t>(kv_stride) * 2u;
    const uint32_t last_row = static_cast<uint32_t>(n_keys - 1) * row_bytes;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int c = i * 256 + tid;
        k_off[i] = static_cast<uint32_t>(c / CPR) * row_bytes + (c % CPR) * 16;
        k_max[i] = last_row + (c % CPR) * 16;
    }
#pragma unroll
    for (int i = 0; i < VG; ++i) {
        const int g = min(i * 256 + tid, 16 * CPR - 1);
        v_off[i] = static_cast<uint32_t>(4 * (g / CPR)) * row_bytes + (g % CPR) * 16;
        v_max[i] = last_row + (g % CPR) * 16;
    }
    const char* kbytes = reinterpret_cast<const char*>(kbase);
    const char* vbytes = reinterpret_cast<const char*>(vbase);
    auto fetch = [&](int tile, u32x4_t* kreg, u32x4_t (*vreg)[4]) {
        const uint32_t t_off = static_cast<uint32_t>(tile * 64) * row_bytes;
#pragma unroll
        for (int i = 0; i < CH; ++i)
            kreg[i] = *reinterpret_cast<const u32x4_t*>(kbytes + min(k_off[i] + t_off, k_max[i]));
#pragma unroll
        for (int i = 0; i < VG; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                vreg[i][u] = *reinterpret_cast<const u32x4_t*>(vbytes + min(v_off[i] + t_off + static_cast<uint32_t>(u) * row_bytes, v_max[i]));
    };
    auto stage = [&](int buf, const u32x4_t* kreg, const u32x4_t (*vreg)[4]) {
        half_t* Ks = Ks2[buf];
        half_t* Vt = Vt2[buf];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = i * 256 + tid;
            *reinterpret_cast<u32x4_t*>(&Ks[(c / CPR) * KSTR + (c % CPR) * 8]) = kreg[i];
        }
#pragma unroll
        for (int i = 0; i < VG; ++i) {
            const int g = i * 256 + tid;
            if (g >= 16 * CPR) continue;
            const int kg = g / CPR, dc = g % CPR;
            const int vcol = 4 * (kg ^ ((dc >> 2) << kSwShift)) + 16 * ((dc >> 1) & 1);
#pragma unroll
            for (int w = 0; w < 4; ++w) {                        // word w holds columns 2w, 2w+1 of each key
                const uint32_t a0 = vreg[i][0][w], a1 = vreg[i][1][w], a2 = vreg[i][2][w], a3 = vreg[i][3][w];
                uint2 even, odd;
                even.x = (a0 & 0xffffu) | (a1 << 16);
                even.y = (a2 & 0xffffu) | (a3 << 16);
                odd.x = (a0 >> 16) | (a1 & 0xffff0000u);
                odd.y = (a2 >> 16) | (a3 & 0xffff0000u);
                *reinterpret_cast<uint2*>(&Vt[(dc * 8 + 2 * w) * VSTR + vcol]) = even;
                *reinterpret_cast<uint2*>(&Vt[(dc * 8 + 2 * w + 1) * VSTR + vcol]) = odd;
            }
        }
    };

    // Tile t+1 is parked in the other LDS buffer and tile t+2 requested before tile t is computed: one barrier per
    // tile, a whole tile time to cover the latency of a fetch, and the staging of one wave overlaps the MFMAs of the
    // others.
    fetch(t_lo, kregs, vregs);
    stage(t_lo & 1, kregs, vregs);
    if (t_lo + 1 < n_tiles) fetch(t_lo + 1, kregs, vregs);
    __syncthreads();
    // this lane's row of a V^T fragment: row l32, shifted by the row's skew; key group lhi (v_rd0) or 1 - lhi (v_rd1:
    // fragments whose swizzle flips bit 0 of the key group)
    const int v_row = l32 * VSTR + 16 * ((l32 >> 4) & 1);
    const int v_rd0 = v_row + 4 * lhi, v_rd1 = v_row + 4 * (1 - lhi);
    for (int tile = t_lo; tile < n_tiles; ++tile) {
        if (tile + 1 < n_tiles) stage((tile + 1) & 1, kregs, vregs);
        if (tile + 2 < n_tiles) fetch(tile + 2, kregs, vregs);
        const half_t* Ks = Ks2[tile & 1];
        const half_t* Vt = Vt2[tile & 1];
        const int key0 = tile * 64;
        if (key0 < wave_hi) {
            // S^T = K Q^T : rows = keys (two 32-key fragments), column = this lane's query
            // (the fragments of the whole tile are named before the MFMAs so that the compiler may issue their reads as
            // early as registers allow)
            float16_t st[2];
            half8_t ka[2][KS];
#pragma unroll
            for (int kf = 0; kf < 2; ++kf)
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    ka[kf][s] = *reinterpret_cast<const half8_t*>(&Ks[(kf * 32 + l32) * KSTR + 16 * s + 8 * lhi]);
#pragma unroll
            for (int kf = 0; kf < 2; ++kf) {
#pragma unroll
                for (int r = 0; r < 16; ++r) st[kf][r] = 0.0f;
#pragma unroll
                for (int s = 0; s < KS; ++s) st[kf] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ka[kf][s], qf[s], st[kf], 0, 0, 0);
            }
            // online softmax over the 32 scores this lane holds (the lane 32 away holds the other 32);
            // only tiles that reach past the wave's smallest causal limit need the mask
            if (key0 + 64 > wave_lo) {
#pragma unroll
                for (int kf = 0; kf < 2; ++kf)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int key = key0 + kf * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
                        if (key >= limit) st[kf][r] = -INFINITY;   // a range may hold no visible key of this query
                    }
            }
            float mx = -INFINITY;
#pragma unroll
            for (int kf = 0; kf < 2; ++kf)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, st[kf][r]);
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            // Reference point of the exponentials, in units of log2 (sc > 0: same arg-max).  Any value works as long
            // as numerators and denominator share it, so it only follows the running maximum when some lane's maximum
            // has grown by more than kLazy (probabilities then stay below 2^kLazy, far inside fp16): with 64 queries
            // per wave some maximum moves in most tiles, and rescaling the 64 output accumulators every time costs a
            // fifth of the kernel's vector instructions.
            constexpr float kLazy = 4.0f;
            const float m_cand = fmaxf(m_run, mx * sc);
            const float m_new = __any(m_cand > m_run + kLazy) ? m_cand : m_run;
            float psum = 0.0f;
            half8_t pf[4];
#pragma unroll
            for (int kf = 0; kf < 2; ++kf)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    float2_t pv;
                    pv[0] = __builtin_amdgcn_exp2f(fmaf(st[kf][r], sc, -m_new));
                    pv[1] = __builtin_amdgcn_exp2f(fmaf(st[kf][r + 1], sc, -m_new));
                    psum += pv[0] + pv[1];                           // in 32 bits
                    const half2_t ph = __builtin_convertvector(pv, half2_t);   // one packed conversion per pair
                    pf[kf * 2 + (r >> 3)][r & 7] = ph[0];
                    pf[kf * 2 + (r >> 3)][(r & 7) + 1] = ph[1];
                }
            if (__any(m_new != m_run)) {                         // rescale only when the reference point moved
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                l_run *= alpha;
#pragma unroll
                for (int df = 0; df < DF; ++df)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[df][r] *= alpha;
                m_run = m_new;
            }
            l_run += psum;
            // O^T += V^T P^T : k-step s2 covers keys 16 s2 .. 16 s2 + 15 of the tile; operand element e of a
            // lane is key 16 s2 + 8 (e/4) + 4 (lane/32) + e%4, the order the accumulator layout produced
            half8_t va[4][DF];
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2) {
#pragma unroll
                for (int df = 0; df < DF; ++df) {
                    // key groups 4 s2 + lhi and 4 s2 + 2 + lhi of column df * 32 + l32, at their swizzled places
                    const int sw = df << kSwShift;               // (dc >> 2) << kSwShift with dc = (df * 32 + l32) >> 3
                    const half_t* vrow = &Vt[(df * 32) * VSTR] + ((sw & 1) ? v_rd1 : v_rd0);
                    const half4_t v0 = *reinterpret_cast<const half4_t*>(vrow + 4 * ((4 * s2) ^ (sw & ~1)));
                    const half4_t v1 = *reinterpret_cast<const half4_t*>(vrow + 4 * ((4 * s2 + 2) ^ (sw & ~1)));
                    va[s2][df][0] = v0[0]; va[s2][df][1] = v0[1]; va[s2][df][2] = v0[2]; va[s2][df][3] = v0[3];
                    va[s2][df][4] = v1[0]; va[s2][df][5] = v1[1]; va[s2][df][6] = v1[2]; va[s2][df][7] = v1[3];
                }
            }
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2)
#pragma unroll
                for (int df = 0; df < DF; ++df) o[df] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[s2][df], pf[s2], o[df], 0, 0, 0);
        }
        __syncthreads();
    }

    float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    if (SPLIT && ranges > 1) {
        // This range's sums go to memory (rules of access as for the decode kernels' key ranges), two values of a lane at a
        // time; the range that arrives last adds all of them in range order, its own from memory too, and goes on.
        __shared__ int s_arrived;
        constexpr int PAIRS = DF * 8 + 1;                        // pairs per lane; the last one is (reference point, denominator)
        const size_t slot = static_cast<size_t>(item) * p.nh + h;
        uint64_t* mine = reinterpret_cast<uint64_t*>(p.part) + ((slot * zs + z) * 4 + wave) * (PAIRS * 64) + lane;
        auto put = [&](int at, float a, float c) {
            __hip_atomic_store(mine + at * 64, static_cast<uint64_t>(__float_as_uint(a)) | (static_cast<uint64_t>(__float_as_uint(c)) << 32),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
#pragma unroll
        for (int df = 0; df < DF; ++df)
#pragma unroll
            for (int r = 0; r < 16; r += 2) put(df * 8 + (r >> 1), o[df][r], o[df][r + 1]);
        put(PAIRS - 1, m_run, l_tot);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_arrived = __hip_atomic_fetch_add(p.arrive + slot, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_arrived != ranges - 1) return;
        const uint64_t* first = reinterpret_cast<const uint64_t*>(p.part) + (slot * zs * 4 + wave) * (PAIRS * 64) + lane;
        auto get = [&](int s, int at) { return __hip_atomic_load(first + static_cast<size_t>(s) * (4 * PAIRS * 64) + at * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        m_run = kNegBig;
        l_tot = 0.0f;
#pragma unroll
        for (int df = 0; df < DF; ++df)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[df][r] = 0.0f;
        for (int s = 0; s < ranges; ++s) {
            uint64_t v[PAIRS];
#pragma unroll
            for (int at = 0; at < PAIRS; ++at) v[at] = get(s, at);
            const float m_s = __uint_as_float(static_cast<uint32_t>(v[PAIRS - 1])), l_s = __uint_as_float(static_cast<uint32_t>(v[PAIRS - 1] >> 32));
            const float m_new = fmaxf(m_run, m_s);
            const float a = __builtin_amdgcn_exp2f(m_run - m_new), c = __builtin_amdgcn_exp2f(m_s - m_new);
            m_run = m_new;
            l_tot = l_tot * a + l_s * c;
#pragma unroll
            for (int df = 0; df < DF; ++df)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    o[df][r] = o[df][r] * a + __uint_as_float(static_cast<uint32_t>(v[df * 8 + (r >> 1)] >> (32 * (r & 1)))) * c;
        }
    }
    const float inv = 1.0f / l_tot;
    if (wave * 32 + l32 < q_cnt) {
        half_t* orow = p.out + static_cast<size_t>(row_begin + q_local) * (p.nh * D) + h * D;
#pragma unroll
        for (int df = 0; df < DF; ++df)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                half4_t v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = static_cast<half_t>(o[df][4 * g + e] * inv);
                *reinterpret_cast<half4_t*>(orow + df * 32 + 8 * g + 4 * lhi) = v;
            }
    }
}

// Sum over the LPK (8 or 16) adjacent lanes that share a key, left in every one of them.  Data-parallel-primitive
// modifiers on the adds (quad permutes, then mirror within 8 and within 16 lanes: after the quad steps the
// lanes of a quad hold equal values, so a mirror exchanges whole quads / halves) instead of cross-lane moves
// through the LDS crossbar: the dot products of a decode step need 4 such sums per key and query head.
template <int LPK>
__device__ __forceinline__ float key_group_sum(float x) {
    static_assert(LPK == 8 || LPK == 16, "8 or 16 lanes per key");
    auto step = [](float v, auto ctrl) {
        const int moved = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true);
        return v + __builtin_bit_cast(float, moved);
    };
    x = step(x, std::integral_constant<int, 0xB1>{});       // quad_perm [1,0,3,2]
    x = step(x, std::integral_constant<int, 0x4E>{});       // quad_perm [2,3,0,1]
    x = step(x, std::integral_constant<int, 0x141>{});      // row_half_mirror
    if (LPK == 16) x = step(x, std::integral_constant<int, 0x140>{});   // row_mirror
    return x;
}

// Sum of eight products of halves, in fp32 (two per instruction; the softmax scale is applied to the sum).  The instruction
// flushes fp32 denormals, of which there are none here: products of halves are multiples of 2^-48, and so are their rounded
// sums.  The plain exp2 instruction below gives 0 for weights under 2^-126 of the largest, which changes a sum by less than
// 2^-86 of a value of 2^16 and 2^24 keys, far below half a step of the fp16 result.  Attention output against 64 bits
// on the same rotated queries and cache (five head layouts, 3 to 40 rows, scores up to six times the usual): 2.04e-4 to 2.12e-4,
// the rounding of the result alone to all digits shown, as with single products and the library exp2.  This takes the loop from 33 to 25 vector instructions per key and query
// head: four query heads per kv head, 8 rows x 1500 keys, 26 -> 20 us together with the early first request.
__device__ __forceinline__ float dot8(const half8_t& a, const half8_t& b) {
    float acc = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; e += 2) acc = __builtin_amdgcn_fdot2(half2_t{a[e], a[e + 1]}, half2_t{b[e], b[e + 1]}, acc, false);
    return acc;
}

// Decode-style attention, one query head per kv head: workgroup = (executed row, head).  The kernel also
// does what a launch of its own would do before it (rotary embedding and cache append: 5 us per layer for a few KB):
// the queries are rotated as they are read, the call's own keys (rows row_begin .. i of the same sequence) are rotated
// from the compact buffer, and the workgroup appends its own row's key and value.  The cached keys are streamed.
// SPLIT: with few rows there are fewer workgroups than the chip needs to saturate HBM (8 rows x 32 kv heads is
// one workgroup per CU: 4.1 TB/s against 6.0 with eight per CU), so the cached keys of a (row, kv head) are cut into
// n_split contiguous ranges (multiples of the 64- or 128-key step) that separate workgroups stream (range 0 also takes the
// new keys); each writes its unnormalised sums with their maximum and denominator, and the one that arrives last
// combines the ranges in range order, so the result does not depend on who that is.
// FUSED = false: rope_append_kernel has rotated and appended already, the queries are read as they are and all keys from the
// cache (attention_rotates says when).
template <int D, bool SPLIT, bool FUSED>
__global__ void __launch_bounds__(256, SPLIT ? 5 : 8)
attn_decode_kernel(AttnDev p) {
    constexpr int LPK = D / 8;            // lanes per key (each lane owns 8 of the D columns)
    constexpr int KPW = 64 / LPK;         // keys per wave per step
    constexpr int UNR = 4;
    // kv head fastest: the workgroups of one executed row are launched together
    const int i = blockIdx.y;
    if (i >= *p.count) return;
    const int hk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = lane % LPK, slot = lane / LPK;

    // This row's query, key and value and their rotation depend on nothing but i: they are requested first and arrive
    // while the chain row -> sequence -> cache length is followed.  This lane's 8 columns pair with those D / 2 away; the
    // first half subtracts.
    const int psub = sub < LPK / 2 ? sub + LPK / 2 : sub - LPK / 2;
    const float sign = sub < LPK / 2 ? -1.0f : 1.0f;
    const float2* cs0 = FUSED ? p.cs + (sub % (LPK / 2)) * 8 : nullptr;
    auto rotate = [&](const half8_t& mine, const half8_t& other, const float2* cs, half8_t& out) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            out[e] = static_cast<half_t>(fmaf(static_cast<float>(mine[e]), cs[e].x, sign * (static_cast<float>(other[e]) * cs[e].y)));
    };
    const half_t* row_i = p.qkv + static_cast<size_t>(i) * p.width;
    half8_t qa, qb{}, ka{}, kb_{}, v_own{};
    float2 cs_i[8];
    qa = *reinterpret_cast<const half8_t*>(row_i + hk * D + sub * 8);
    if (FUSED) {
        qb = *reinterpret_cast<const half8_t*>(row_i + hk * D + psub * 8);
        ka = *reinterpret_cast<const half8_t*>(row_i + (p.nh + hk) * D + sub * 8);
        kb_ = *reinterpret_cast<const half8_t*>(row_i + (p.nh + hk) * D + psub * 8);
        v_own = *reinterpret_cast<const half8_t*>(row_i + (p.nh + p.nkv + hk) * D + sub * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) cs_i[e] = cs0[static_cast<size_t>(i) * (D / 2) + e];
    }

    if (SPLIT) __builtin_amdgcn_sched_barrier(0);

    const int b = p.row_seq[i];
    const int row_begin = p.cu_exec[b];
    const bool once = p.cu_exec[b + 1] - row_begin == 1;         // no other row reads this sequence's keys
    const size_t head_off = (static_cast<size_t>(b) * p.nkv + hk) * p.cap * D;   // cache [B][n_kv_heads][cap][D]
    const half_t* kbase = p.k_cache + head_off;
    const half_t* vbase = p.v_cache + head_off;
    const int old = p.kv_old[b];
    const int own = i - row_begin;                               // place of this row among the sequence's new rows
    const int n_cached = min(FUSED ? old : old + own + 1, p.cap);
    const int n_new = max(min(own + 1, p.cap - old), 0);         // new keys that fit the cache; later ones are not seen

    const int step = 4 * KPW;             // keys per workgroup step
    const KeyRange range = decode_key_range<SPLIT>(p, n_cached, UNR * step);
    if (SPLIT && range.none) return;
    const int key_lo = range.lo, key_hi = range.hi;
    // Keys past the end of the range are clamped to its last one and masked (so the last step's request for the next one does
    // not read the neighbouring range: half as much again at 128 keys per range).  With split keys the next step is requested
    // before the current one is consumed, so the memory pipe never drains while the lanes do their dot products and
    // exponentials.  Without, eight workgroups per CU run on 64 registers, which do not hold two steps (asked to, the compiler
    // loaded one row after the other, a round trip each: 16 rows x 32 heads x 1000 keys 58 us, 4 x 4 rows 44): the step's loads
    // are issued together at its start and the other workgroups fill the wait.
    // Addresses are a uniform base that walks with the step plus a 32-bit lane offset inside it.
    half8_t kn[UNR], vn[UNR];
    const int last = max(key_hi - 1, 0);                         // an empty cache: slot 0, loaded and not used
    const int lane_key = wave * KPW + slot;
    auto fetch = [&](int kb, auto nt) {
        const int first = min(kb, last);
        // (scalar registers; as ordinary pointers they are folded into a 64-bit sum per load and lane)
        uint64_t ks = reinterpret_cast<uint64_t>(kbase + static_cast<size_t>(first) * D);
        uint64_t vs = reinterpret_cast<uint64_t>(vbase + static_cast<size_t>(first) * D);
        asm("" : "+s"(ks), "+s"(vs));
        using Bytes = const __attribute__((address_space(1))) char*;
        using Piece = const __attribute__((address_space(1))) half8_t*;
        auto load = [&](auto nt) {
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const uint32_t off = static_cast<uint32_t>(min(lane_key + u * step, last - first) * D + sub * 8) * 2u;
                const Piece k = reinterpret_cast<Piece>(reinterpret_cast<Bytes>(ks) + off), v = reinterpret_cast<Piece>(reinterpret_cast<Bytes>(vs) + off);
                kn[u] = nt.value ? stream_load(k) : *k;
                vn[u] = nt.value ? stream_load(v) : *v;
            }
        };
        if (SPLIT && once) keep_side([&] { load(std::true_type{}); });
        else load(nt);
    };
    // Few workgroups (SPLIT): latency counts and registers do not, the stream starts before anything else is computed.  Many
    // workgroups: eight per CU (64 registers) stream at 6.0 TB/s, so the first request waits until the registers are free.
    if (SPLIT) {
        fetch(key_lo, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
    }

    half8_t qh = qa, k_own{};
    if (FUSED) {
        rotate(qa, qb, cs_i, qh);
        rotate(ka, kb_, cs_i, k_own);
    }

    float m_run, l_run, o[8];
    // The row's own key starts the sums of one lane group of range 0 (and goes into the cache); the other groups start
    // empty.
    const bool mine = FUSED && (!SPLIT || blockIdx.z == 0) && wave == 0 && slot == 0 && own < n_new;
    if (mine) {
        const size_t at = head_off + static_cast<size_t>(old + own) * D + sub * 8;
        *reinterpret_cast<half8_t*>(p.k_cache + at) = k_own;
        *reinterpret_cast<half8_t*>(p.v_cache + at) = v_own;
    }
    m_run = mine ? key_group_sum<LPK>(dot8(qh, k_own)) * p.scale_log2 : kNegBig;
    l_run = mine ? 1.0f : 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = mine ? static_cast<float>(v_own[e]) : 0.0f;
    // the sequence's other new keys (none in a decode step of one token per sequence)
    if (FUSED && own > 0 && (!SPLIT || blockIdx.z == 0)) {
        const int n_other = min(own, n_new);
        for (int jb = 0; jb < n_other; jb += step) {             // uniform trip count
            const int j = jb + wave * KPW + slot;
            const bool ok = j < n_other;
            const int rj = row_begin + min(j, own);
            const half_t* row_k = p.qkv + static_cast<size_t>(rj) * p.width + (p.nh + hk) * D;
            const half8_t ja = *reinterpret_cast<const half8_t*>(row_k + sub * 8);
            const half8_t jo = *reinterpret_cast<const half8_t*>(row_k + psub * 8);
            const half8_t vv = *reinterpret_cast<const half8_t*>(row_k + p.nkv * D + sub * 8);
            float2 cs[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) cs[e] = cs0[static_cast<size_t>(rj) * (D / 2) + e];
            if (!SPLIT) __builtin_amdgcn_sched_barrier(0);      // one round trip per step
            half8_t kr;
            rotate(ja, jo, cs, kr);
            const float acc = key_group_sum<LPK>(dot8(qh, kr)) * p.scale_log2;
            const float s = ok ? acc : kNegBig;
            const float mx = fmaxf(m_run, s);
            const float alpha = exp2f(m_run - mx);
            const float pv = ok ? exp2f(s - mx) : 0.0f;
            m_run = mx;
            l_run = l_run * alpha + pv;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = fmaf(pv, static_cast<float>(vv[e]), o[e] * alpha);
        }
    }

    // Without split keys two loops rather than a branch at the loads (32 x 4 rows on 4000 keys 658 and 668 us, in 64 registers either
    // way); with split keys two loops take 126 registers and a branch 94, of which five workgroups fit a CU.
    auto stream = [&](auto nt) {
        for (int kb = key_lo; kb < key_hi; kb += UNR * step) { // trip count is uniform over the workgroup
            const int k0 = kb + wave * KPW + slot;
            half8_t kv[UNR], vv[UNR];
            bool ok[UNR];
            if (!SPLIT) {
                fetch(kb, nt);
                __builtin_amdgcn_sched_barrier(0);                  // all eight loads before the first wait
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                ok[u] = k0 + u * step < key_hi;
                kv[u] = kn[u];
                vv[u] = vn[u];
            }
            if (SPLIT) fetch(kb + UNR * step, nt);                 // past the end: one redundant, unused fetch
            float s[UNR];
            float mx = m_run;
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const float acc = key_group_sum<LPK>(dot8(qh, kv[u])) * p.scale_log2;
                s[u] = ok[u] ? acc : kNegBig;
                mx = fmaxf(mx, s[u]);
            }
            const float alpha = __builtin_amdgcn_exp2f(m_run - mx);
            m_run = mx;
            l_run *= alpha;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] *= alpha;
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const float pv = ok[u] ? __builtin_amdgcn_exp2f(s[u] - mx) : 0.0f;
                l_run += pv;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = fmaf(pv, static_cast<float>(vv[u][e]), o[e]);
            }
        }
    };
    if (!SPLIT && once) stream(std::true_type{});
    else stream(std::false_type{});

    // merge the key slots of a wave (lanes that own the same columns), then the four waves through LDS
    __shared__ float sm[4][D + 2];
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
        const float m2 = __shfl_xor(m_run, off, 64);
        const float l2 = __shfl_xor(l_run, off, 64);
        const float mn = fmaxf(m_run, m2);
        const float a1 = exp2f(m_run - mn), a2 = exp2f(m2 - mn);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float o2 = __shfl_xor(o[e], off, 64);
            o[e] = o[e] * a1 + o2 * a2;
        }
        l_run = l_run * a1 + l2 * a2;
        m_run = mn;
    }
    if (slot == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sm[wave][sub * 8 + e] = o[e];
        if (sub == 0) { sm[wave][D] = m_run; sm[wave][D + 1] = l_run; }
    }
    __syncthreads();
    if (tid < D) {
        float mn = kNegBig;
#pragma unroll
        for (int w = 0; w < 4; ++w) mn = fmaxf(mn, sm[w][D]);
        float num = 0.0f, den = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float a = exp2f(sm[w][D] - mn);
            num += sm[w][tid] * a;
            den += sm[w][D + 1] * a;
        }
        if (SPLIT) {
            // an empty range leaves num = 0, den = 0 and the maximum at its initial value: it drops out of the merge
            float* dst = p.part + ((static_cast<size_t>(i) * p.nh + hk) * p.n_split + blockIdx.z) * (D + 2);
            agent_store(dst + tid, num);
            if (tid == 0) { agent_store(dst + D, mn); agent_store(dst + D + 1, den); }
        } else {
            p.out[static_cast<size_t>(i) * (p.nh * D) + hk * D + tid] = static_cast<half_t>(num / den);
        }
    }
    if (SPLIT) combine_key_ranges<D, 1>(p, i, hk, range.ranges, tid);
}

// CUs of the current device (queried once per device).
static int attn_cus() {
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cus[dev] = n;
    }
    return cus[dev];
}

template <int D, bool FUSED>
static hipError_t launch_decode_d(const AttnDev& d, int rows, hipStream_t stream) {
    const bool split = d.n_split > 1;
    const dim3 grid(d.nkv, rows, split ? d.n_split : 1), block(256);
    if (split) hipLaunchKernelGGL((attn_decode_kernel<D, true, FUSED>), grid, block, 0, stream, d);
    else hipLaunchKernelGGL((attn_decode_kernel<D, false, FUSED>), grid, block, 0, stream, d);
    return hipGetLastError();
}

bool attention_is_decode(bool cache, int T, int B, int nh, int nkv) {
    const int rep = nh / nkv;
    return cache && T <= 4 * B && (rep == 1 || rep == 2 || rep == 4 || rep == 8);
}

bool attention_rotates(int T, int B, int rep, int hidden, int head_dim) {
    return hidden >= head_dim && T - B <= kAttnFuseNew && (rep > 1 || T <= kAttnFuseTokens);
}

// Few rows: cut the cached keys.  With the ranges' length set on the device they are equally long over all rows and fill the chip
// once; sequences of different lengths cut into equally many ranges left the longest ones running alone (20 rows x 8 kv heads x 1500
// to 4500 keys: 66 -> 59 us).  `target`: workgroups that the ranges are to be, per CU about what its registers hold with one query
// head; grouped queries by their number, layers of 32 heads, us, two / three / four per CU, 20 rows x 3000 keys and 28 x 2000: 2
// heads per kv head 143 / 137 / 133, 124 / 127 / 130 (64-wide 95 / 90 / 87, 83 / 84 / 86), 4 92 / 94 / 91, 8 70.1 / 71.0 / 71.6,
// 70.8 / 73.0 / 72.2 (64-wide 54.7 / 55.8 / 55.8, 55.0 / 56.9 / 56.1); one to eight rows within 2 %.  Without it (calls of more
// than 256 tokens) every row is cut so that about four workgroups per CU stream.
int attention_splits(int max_rows, int nh, int nkv, int cap, bool device_chunk, int* target) {
    const int wgs = max_rows * nkv, rep = nh / nkv;
    if (target) *target = attn_cus() * (rep == 1 ? 5 : rep == 2 ? 4 : rep == 4 ? 3 : 2);
    if (max_rows <= 0 || max_rows > kAttnSplitRows || wgs >= 2 * attn_cus()) return 1;
    const int most = std::min(kAttnSplitMax, cap / 128);              // a range is worth its partial sums from about 128 keys on
    return std::max(1, device_chunk ? most : std::min(most, (4 * attn_cus() + wgs - 1) / wgs));
}

size_t attention_prefill_floats(int items_max, int nh, int d) {
    return static_cast<size_t>(items_max) * nh * (4 * 64 * (d / 2 + 2));
}

AttnList attention_prefill_plan(int max_rows, int B, int nh, int d, int max_keys, size_t floats) {
    AttnList l{};
    l.B = B;
    l.items_max = static_cast<int>((static_cast<long>(max_rows) + static_cast<long>(kAttnBQ - 1) * B) / kAttnBQ);   // sum of the sequences' tiles, each rounded up
    l.levels = (max_rows + kAttnBQ - 1) / kAttnBQ;
    l.heads = nh;
    l.target = attn_cus() * (d == 64 ? 3 : 2);
    // no more ranges than the scratch holds, than the longest sequence has tiles for, or than fill the chip (a workgroup whose
    // range does not exist costs its launch: 8 x 84 rows on 300 keys with 16 ranges in the grid 173 -> 179 us)
    const long pairs = static_cast<long>(l.items_max) * nh;
    const size_t room = floats / std::max<size_t>(attention_prefill_floats(l.items_max, nh, d), 1);
    const long wanted = std::min<long>({kAttnTileSplitMax, (static_cast<long>(max_keys) + 64 * kAttnTileRange - 1) / (64 * kAttnTileRange), l.target / std::max(pairs, 1l) + 1});
    l.n_split = 2l * l.levels * nh >= l.target ? 1 : static_cast<int>(std::max<size_t>(std::min<size_t>(wanted, room), 1));
    return l;
}

hipError_t launch_attention(const AttnArgs& a, hipStream_t stream) {
    if (a.max_rows == 0) return hipSuccess;
    AttnDev d{};
    d.qkv = reinterpret_cast<const half_t*>(a.qkv);
    d.out = reinterpret_cast<half_t*>(a.out);
    d.nh = a.nh;
    d.nkv = a.nkv;
    d.width = (a.nh + 2 * a.nkv) * a.d;
    d.count = a.count;
    d.cu_exec = a.cu_exec;
    d.row_seq = a.row_seq;
    d.k_cache = reinterpret_cast<half_t*>(a.k_cache);
    d.v_cache = reinterpret_cast<half_t*>(a.v_cache);
    d.kv_old = a.kv_old;
    d.cap = a.cap;
    d.scale_log2 = kLog2e / sqrtf(static_cast<float>(a.d));
    if (a.decode) {
        d.cs = a.cs;
        d.arrive = a.arrive;
        d.chunk = a.chunk;
        d.part = a.partials;
        d.n_split = a.partials && a.arrive ? attention_splits(a.max_rows, a.nh, a.nkv, a.cap, a.chunk != nullptr, nullptr) : 1;
        const int rep = a.nh / a.nkv;
        if (rep > 1) return launch_attn_decode_gqa(d, rep, a.d, a.max_rows, stream);
        if (a.d == 128) return d.cs ? launch_decode_d<128, true>(d, a.max_rows, stream) : launch_decode_d<128, false>(d, a.max_rows, stream);
        return d.cs ? launch_decode_d<64, true>(d, a.max_rows, stream) : launch_decode_d<64, false>(d, a.max_rows, stream);
    }
    d.items = reinterpret_cast<const int4*>(a.list->items);
    d.items_max = a.list->items_max;
    d.n_split = a.list->n_split;
    d.tiles = a.list->tiles;
    d.arrive = a.list->arrive;
    d.part = a.partials;
    const dim3 grid(8 * ((d.items_max * d.n_split * a.nh + 7) / 8)), block(256);
    if (a.d == 128) {
        if (d.n_split > 1) hipLaunchKernelGGL((flash_prefill_kernel<128, true>), grid, block, 0, stream, d);
        else hipLaunchKernelGGL((flash_prefill_kernel<128, false>), grid, block, 0, stream, d);
    } else {
        if (d.n_split > 1) hipLaunchKernelGGL((flash_prefill_kernel<64, true>), grid, block, 0, stream, d);
        else hipLaunchKernelGGL((flash_prefill_kernel<64, false>), grid, block, 0, stream, d);
    }
    return hipGetLastError();
}

}  // namespace qtale

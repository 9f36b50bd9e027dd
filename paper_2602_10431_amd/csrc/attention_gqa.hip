// Decode-style attention of grouped queries: 2, 4 or 8 query heads share a key/value head, one workgroup per (executed row,
// kv head[, key range]).  It does what attn_decode_kernel does for one query head (rotary embedding, cache append, split keys,
// see there); what differs is the arithmetic.
//
// On the vector ALUs a key costs 25 instructions per query head (dot product, sums over the lanes that share the key,
// exponential, eight multiply-adds), so with four heads the stream of keys and values waited for them: 4.0 to 4.6 TB/s where
// one head streams at 6.0.  Here the two products run on the matrix cores, with the query heads as columns:
//   * a wave's step is 32 keys.  Scores S[key][head] = K Q^T are two 16 x 16 fragments; lane (c, g) = (lane % 16, lane / 16)
//     holds row c of K, columns 32 s + 8 g .. + 7, so its loads are operands as they arrive (64 bytes of each of 16 rows per
//     instruction, the four instructions of a tile cover whole rows);
//   * the result leaves lane (c, g) the scores of keys 4 g + r of both fragments for head c, which is operand order for
//     O^T = V^T P^T if the product's key index 8 g + e is read as key 4 g + e (e < 4) or 16 + 4 g + e - 4: no data moves
//     between lanes;
//   * V^T needs eight keys of one column per lane.  Lane (c, g) loads columns F c .. F c + F - 1 (F = D / 16: whole rows, 4 per
//     instruction) of those eight keys, and fragment f takes column F c + f of each lane: 4 F byte permutes per step, no LDS;
//   * as an fp16 operand a probability (at most 2^4) is split into its rounded value and 2048 times the rest, which go to two of
//     the 16 columns (heads fill 2, 4 or 8), so both products come from the same instruction.  The rest is rounded too: what is
//     lost is at most 2^-23 of the probability, or 2^-36.  The reference point of the exponentials follows the largest score
//     lazily.  Error of the sums before they are rounded to fp16, against 64 bits (2-norm, 700 to 12000 normal keys and values), on
//     the vector ALUs, where probabilities were 32-bit operands / here: 128-wide heads, 2, 4, 8 per kv head 1.83e-7 / 1.64e-7,
//     1.82 / 1.71, 1.84 / 1.68, 64-wide 1.70 / 1.68, 1.78 / 1.75, 1.73 / 1.77; scores four times as large 4.2 to 4.5 / 3.6 to 4.0,
//     3.8 to 4.0 / 3.5; values of one sign 0.25 / 0.3 (the matrix instruction's additions).  The outputs' own rounding is 2.4e-4.
//     (Reference 8 to 12 log2 units below the largest score, the rest not scaled, one chain per score: 2.2 to 2.4, large scores up
//     to 5.2.)
//   * a step's keys are requested again as soon as the scores are formed, its values as soon as they are consumed: 16 KB per
//     wave in flight with one register set, three waves per SIMD (four with 64-wide heads).  A wave's last step requests nothing
//     and a wave without cached keys makes no step: short caches are bound by the launch of many workgroups.
// Kernel time, us, vector ALUs / matrix cores (plain loads) and the layer's time / with non-temporal loads: 128-wide heads, 4 per
// kv head: 16 rows x 1000 keys 22.9 / 19.7, 64 x 2048 99 / 95, layer 194 / 183, 64 x 1024..3072 122 / 109, 128 x 500..1500 118 / 102;
// 64-wide: 8 x 750..2250 15 / 11, 20 x 3000 30.6 / 26, 64 x 2048 54 / 50, layer 109 / 98.  What bounds it now is the stream, and
// with few rows the chain row -> sequence -> length in front of it and the combination of the ranges behind it.  Short caches,
// layers of hidden size 1024 with 32 heads, us, vector ALUs / every wave stepping and requesting past the end / now: 128-wide, 2 per
// kv head 128 rows x 50 keys 69.8 / 73.0 / 67.8, 256 x 50 88.4 / 99.3 / 88.9, 256 x 200 151 / 147 / 139; 4 per kv head 256 x 50 81.9 /
// 82.0 / 76.3; 64-wide, 2 per kv head 256 x 50 80.2 / 80.3 / 72.8, 256 x 200 101.6 / 102.6 / 96.2, 20 x 3000 95 / 87 / 87.
#include <algorithm>
#include <type_traits>

#include "attn_common.h"

namespace qtale {

constexpr int kGqaKeys = 32;                     // keys per wave and step
constexpr int kGqaStep = 4 * kGqaKeys;           // per workgroup
static_assert(kGqaStep == kAttnGqaStep, "the granularity of the key ranges");

template <int D, int REP, bool SPLIT, bool FUSED>
__global__ void __launch_bounds__(256, D == 64 ? 4 : 3)
attn_decode_gqa_kernel(AttnDev p) {
    constexpr int S = D / 32;                    // k-steps of the scores
    constexpr int F = D / 16;                    // output fragments, and columns of V per lane
    typedef half_t VPiece __attribute__((ext_vector_type(F)));
    typedef uint32_t VWords __attribute__((ext_vector_type(F / 2)));
    const int i = blockIdx.y;                    // kv head fastest: the workgroups of one executed row are launched together
    if (i >= *p.count) return;
    const int hk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;

    // This row's query, key and value and their rotation depend on nothing but i: requested first, they arrive while the chain
    // row -> sequence -> cache length is followed.
    const half_t* row_i = p.qkv + static_cast<size_t>(i) * p.width;
    half8_t q[S], k_own[S];
    VPiece v_own{};
    auto load_cs = [&](int row, float2 (*cs)[8]) {               // (cos, sin) of the pairs whose first half this lane holds
        const float2* src = p.cs + static_cast<size_t>(row) * (D / 2) + 8 * g;
#pragma unroll
        for (int s = 0; s < S / 2; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) cs[s][e] = src[32 * s + e];
    };
    auto rotate = [&](half8_t* t, const float2 (*cs)[8]) {       // columns j and j + D / 2 are in the same lane
#pragma unroll
        for (int s = 0; s < S / 2; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float lo = static_cast<float>(t[s][e]), hi = static_cast<float>(t[s + S / 2][e]);
                t[s][e] = static_cast<half_t>(fmaf(lo, cs[s][e].x, -(hi * cs[s][e].y)));
                t[s + S / 2][e] = static_cast<half_t>(fmaf(hi, cs[s][e].x, lo * cs[s][e].y));
            }
    };
    auto scores = [&](const half8_t* k) {                        // 64 columns per chain: one of 128 rounds twice as large sums as often
        float4_t sum[S / 2];
#pragma unroll
        for (int s = 0; s < S; s += 2) {
            sum[s / 2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k[s], q[s], float4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            sum[s / 2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k[s + 1], q[s + 1], sum[s / 2], 0, 0, 0);
        }
        return S == 2 ? sum[0] : sum[0] + sum[S / 2 - 1];
    };
#pragma unroll
    for (int s = 0; s < S; ++s) q[s] = *reinterpret_cast<const half8_t*>(row_i + (hk * REP + (c & (REP - 1))) * D + 32 * s + 8 * g);
    float s_own = 0.0f;
    const bool new_keys = FUSED && (!SPLIT || blockIdx.z == 0);   // this workgroup also takes the call's own keys
    if (FUSED) {
        float2 cs[S / 2][8];
        load_cs(i, cs);
        if (new_keys && wave == 0) {
#pragma unroll
            for (int s = 0; s < S; ++s) k_own[s] = *reinterpret_cast<const half8_t*>(row_i + (p.nh + hk) * D + 32 * s + 8 * g);
            v_own = *reinterpret_cast<const VPiece*>(row_i + (p.nh + p.nkv + hk) * D + F * c);
        }
        rotate(q, cs);
        if (new_keys && wave == 0) {
            rotate(k_own, cs);
            s_own = scores(k_own)[0];                            // every row of K is this key
        }
    }
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
    const KeyRange range = decode_key_range<SPLIT>(p, n_cached, kGqaStep);
    if (SPLIT && range.none) return;

    // kb: first key of a wave's step, inside the range.  Keys past the range's end are clamped to its last one and masked.  Addresses are
    // a uniform base that walks with the step plus a 32-bit lane offset inside it.
    half8_t kn[2][S];
    VPiece vn[8];
    const int last = range.hi - 1;
    using Bytes = const __attribute__((address_space(1))) char*;
    auto base_of = [&](const half_t* base, int kb) {
        uint64_t a = reinterpret_cast<uint64_t>(base + static_cast<size_t>(kb) * D);
        asm("" : "+s"(a));
        return a;
    };
    // (Values, and the keys of 64-wide heads, as non-temporal loads where nt says so.  The keys of 128-wide heads arrive a quarter of a row per
    // instruction and gain nothing or lose: 20 rows x 1500 to 4500 keys, layer 132 us with plain key loads, 135 without;
    // 64-wide heads 64 x 2048 104 and 98.)
    auto fetch_k = [&](int kb, auto nt) {
        const uint64_t a = base_of(kbase, kb);
        const int room = last - kb;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t off = static_cast<uint32_t>(min(16 * u + c, room) * (2 * D) + 16 * g);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const auto* src = reinterpret_cast<const __attribute__((address_space(1))) half8_t*>(reinterpret_cast<Bytes>(a) + off + 64 * s);
                kn[u][s] = D == 64 && nt.value ? stream_load(src) : *src;
            }
        }
    };
    auto fetch_v = [&](int kb, auto nt) {
        const uint64_t a = base_of(vbase, kb);
        const int room = last - kb;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t off = static_cast<uint32_t>(min(4 * g + (e < 4 ? e : 12 + e), room) * (2 * D) + 2 * F * c);
            const auto* src = reinterpret_cast<const __attribute__((address_space(1))) VPiece*>(reinterpret_cast<Bytes>(a) + off);
            vn[e] = nt.value ? stream_load(src) : *src;
        }
    };
    if (new_keys && wave == 0 && own < n_new) {
        const size_t at = head_off + static_cast<size_t>(old + own) * D;
        if (c == 0) {
#pragma unroll
            for (int s = 0; s < S; ++s) *reinterpret_cast<half8_t*>(p.k_cache + at + 32 * s + 8 * g) = k_own[s];
        }
        if (g == 0) *reinterpret_cast<VPiece*>(p.v_cache + at + F * c) = v_own;
    }
    // Running sums of column c (head c % REP; rounded probabilities for c / REP even, the rest for odd): l_run of this lane's
    // keys, o[f] of rows (columns of V) F (4 g + r) + f.  Probabilities are 2^(score - m_run), at most 2^kTop.
    constexpr float kTop = 4.0f, kScale = 2048.0f;
    const float sc = p.scale_log2;
    const float rest = (c / REP) & 1 ? -1.0f : 0.0f, scale = (c / REP) & 1 ? kScale : 1.0f;
    float m_run = kNegBig, l_run = 0.0f;
    float4_t o[F];
#pragma unroll
    for (int f = 0; f < F; ++f) o[f] = float4_t{0.f, 0.f, 0.f, 0.f};
    // adds 32 keys; st: masked scores are -inf
    auto absorb = [&](const float4_t& st0, const float4_t& st1, const VPiece* v) {
        float mx = fmaxf(fmaxf(fmaxf(st0[0], st0[1]), fmaxf(st0[2], st0[3])), fmaxf(fmaxf(st1[0], st1[1]), fmaxf(st1[2], st1[3]))) * sc;
        if (__any(mx > m_run + kTop)) {
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));              // the column's largest score: all its lanes move together
            const float m_new = mx > m_run + kTop ? mx : m_run;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            l_run *= alpha;
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[f][r] *= alpha;
            m_run = m_new;
        }
        half8_t pb;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            float2_t pv;
            pv[0] = __builtin_amdgcn_exp2f(fmaf(e < 4 ? st0[e] : st1[e - 4], sc, -m_run));
            pv[1] = __builtin_amdgcn_exp2f(fmaf(e < 4 ? st0[e + 1] : st1[e - 3], sc, -m_run));
            l_run += pv[0] + pv[1];
            const half2_t hi = __builtin_convertvector(pv, half2_t);
            pv[0] = fmaf(rest, static_cast<float>(hi[0]), pv[0]) * scale;   // exact
            pv[1] = fmaf(rest, static_cast<float>(hi[1]), pv[1]) * scale;
            const half2_t h = __builtin_convertvector(pv, half2_t);
            pb[e] = h[0];
            pb[e + 1] = h[1];
        }
        VWords w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = __builtin_bit_cast(VWords, v[e]);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            u32x4_t va;
#pragma unroll
            for (int e = 0; e < 8; e += 2) va[e >> 1] = __builtin_amdgcn_perm(w[e + 1][f >> 1], w[e][f >> 1], f & 1 ? 0x07060302u : 0x05040100u);
            o[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, va), pb, o[f], 0, 0, 0);
        }
    };
    const float none = -INFINITY;

    // The stream, twice: a branch at the loads of every step leaves the compiler unsure of how many are in flight, so it waits for all
    // of them (layers of 32 64-wide heads, 16 kv heads, 256 rows x 200 keys 103 us, now 96).
    const int k_first = range.lo + wave * kGqaKeys;              // this wave's first cached keys, if there are that many
    auto stream = [&](auto nt) {
        if (nt.value) asm volatile("; one row");                 // (the two would be made one, with ordinary loads)
        else asm volatile("; several rows");
        auto fetch_first = [&] {
            if (k_first < range.hi) {
                fetch_k(k_first, nt);
                fetch_v(k_first, nt);
            }
        };
        const int n_other = nt.value || !new_keys ? 0 : min(own, n_new);   // the sequence's earlier new keys that this workgroup takes
        if (n_other == 0) fetch_first();
        __builtin_amdgcn_sched_barrier(0);
        if (new_keys) {
            if (wave == 0) {                                     // the row's own key: a step of one
                VPiece vv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) vv[e] = v_own;
                absorb(float4_t{g == 0 && own < n_new ? s_own : none, none, none, none}, float4_t{none, none, none, none}, vv);
            }
            // the sequence's earlier new keys (none in a decode step of one token per sequence) in the registers of the first cached
            // step, which is requested afterwards (requested before and again, layers with 2 heads per kv head and sequences of 1 to 6
            // rows, 64 heads of 64, 46 tokens on 100 to 1656 keys 160 -> 154 us, 2 of 128, 8 on 100 to 1494 35.1 -> 34.0)
            if (n_other > 0) {
                for (int jb = wave * kGqaKeys; jb < n_other; jb += kGqaStep) {
                    float4_t st[2];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int rj = row_begin + min(jb + 4 * g + (e < 4 ? e : 12 + e), n_other - 1);
                        vn[e] = *reinterpret_cast<const VPiece*>(p.qkv + static_cast<size_t>(rj) * p.width + (p.nh + p.nkv + hk) * D + F * c);
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int rj = row_begin + min(jb + 16 * u + c, n_other - 1);
                        float2 cs[S / 2][8];
#pragma unroll
                        for (int s = 0; s < S; ++s) kn[u][s] = *reinterpret_cast<const half8_t*>(p.qkv + static_cast<size_t>(rj) * p.width + (p.nh + hk) * D + 32 * s + 8 * g);
                        load_cs(rj, cs);
                        rotate(kn[u], cs);
                        st[u] = scores(kn[u]);
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (jb + 16 * u + 4 * g + r >= n_other) st[u][r] = none;
                    }
                    absorb(st[0], st[1], vn);
                }
                fetch_first();
            }
        }
        auto step = [&](int kb, auto more) {
            float4_t st[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) st[u] = scores(kn[u]);
            if (more.value) {
                fetch_k(kb + kGqaStep, nt);
                __builtin_amdgcn_sched_barrier(0);
            } else {                                             // the last step may hold fewer keys
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (kb + 16 * u + 4 * g + r >= range.hi) st[u][r] = none;
            }
            absorb(st[0], st[1], vn);
            if (more.value) {
                __builtin_amdgcn_sched_barrier(0);
                fetch_v(kb + kGqaStep, nt);
            }
        };
        int kb = k_first;                                        // uniform over the wave
        for (; kb + kGqaStep < range.hi; kb += kGqaStep) step(kb, std::true_type{});
        if (kb < range.hi) step(kb, std::false_type{});
    };
    if (once) stream(std::true_type{});
    else stream(std::false_type{});

    // the four waves meet in LDS; a head's two columns are added there
    __shared__ float sm[4][2 * REP][D + 2];
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (c < 2 * REP) {
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) sm[wave][c][F * (4 * g + r) + f] = o[f][r];
        if (g == 0) { sm[wave][c][D] = m_run; sm[wave][c][D + 1] = l_run; }
    }
    __syncthreads();
    for (int t = tid; t < REP * D; t += 256) {
        const int r = t / D, e = t % D;
        float mn = kNegBig;
#pragma unroll
        for (int w = 0; w < 4; ++w) mn = fmaxf(mn, sm[w][r][D]);
        float num = 0.0f, den = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float a = exp2f(sm[w][r][D] - mn);
            num += fmaf(sm[w][r + REP][e], 1.0f / kScale, sm[w][r][e]) * a;
            den += sm[w][r][D + 1] * a;
        }
        if (SPLIT) {
            // an empty range leaves num = 0, den = 0 and the reference at its initial value: it drops out of the combination
            float* dst = p.part + ((static_cast<size_t>(i) * p.nh + hk * REP + r) * p.n_split + blockIdx.z) * (D + 2);
            agent_store(dst + e, num);
            if (e == 0) { agent_store(dst + D, mn); agent_store(dst + D + 1, den); }
        } else {
            p.out[static_cast<size_t>(i) * (p.nh * D) + (hk * REP + r) * D + e] = static_cast<half_t>(num / den);
        }
    }
    if (SPLIT) combine_key_ranges<D, REP>(p, i, hk, range.ranges, tid);
}

template <int D, int REP>
static hipError_t launch_form(const AttnDev& d, int rows, hipStream_t stream) {
    const bool split = d.n_split > 1;
    const dim3 grid(d.nkv, rows, split ? d.n_split : 1), block(256);
    if (d.cs) {
        if (split) hipLaunchKernelGGL((attn_decode_gqa_kernel<D, REP, true, true>), grid, block, 0, stream, d);
        else hipLaunchKernelGGL((attn_decode_gqa_kernel<D, REP, false, true>), grid, block, 0, stream, d);
    } else {
        if (split) hipLaunchKernelGGL((attn_decode_gqa_kernel<D, REP, true, false>), grid, block, 0, stream, d);
        else hipLaunchKernelGGL((attn_decode_gqa_kernel<D, REP, false, false>), grid, block, 0, stream, d);
    }
    return hipGetLastError();
}

template <int D>
static hipError_t launch_rep(const AttnDev& d, int rep, int rows, hipStream_t stream) {
    switch (rep) {
        case 2: return launch_form<D, 2>(d, rows, stream);
        case 4: return launch_form<D, 4>(d, rows, stream);
        case 8: return launch_form<D, 8>(d, rows, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_attn_decode_gqa(const AttnDev& d, int rep, int head_dim, int rows, hipStream_t stream) {
    return head_dim == 128 ? launch_rep<128>(d, rep, rows, stream) : launch_rep<64>(d, rep, rows, stream);
}

}  // namespace qtale

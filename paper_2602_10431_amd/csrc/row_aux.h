// Device pieces shared by the kernels that begin a layer (router score, decision, first normalisation): the score of a
// row by one wave, the order keys of the decision, the decision of a small call, and what the same kernels prepare for
// the attention kernel (rotary table of the executed rows, cleared arrival counters).
#pragma once
#include "qtale_dev.h"
#include "qtale_kernels.h"

namespace qtale {

// z = fp32( sum_h fp64(x[h]) * fp64(w[h]) + fp64(b) ) of one row, by one wave; the result is in every lane.
template <bool BF16>
__device__ __forceinline__ float router_row_score(const uint16_t* __restrict__ x, int H, const float* __restrict__ w, float b, int lane) {
    const U4* xr = reinterpret_cast<const U4*>(x);
    const float4* wr = reinterpret_cast<const float4*>(w);
    double acc0 = 0.0, acc1 = 0.0;
    const int chunks = H >> 3;
    // (four chunks' loads in flight: the router kernel at 33 tokens 5.8 -> 4.1 us; the order of the sums is unchanged)
#pragma unroll 4
    for (int c = lane; c < chunks; c += 64) {
        const U4 xv = xr[c];
        const float4 w0 = wr[2 * c], w1 = wr[2 * c + 1];
        const uint32_t xs[4] = {xv.x, xv.y, xv.z, xv.w};
        const float ws[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double a0 = static_cast<double>(act_to_float<BF16>(static_cast<uint16_t>(xs[i] & 0xffffu)));
            const double a1 = static_cast<double>(act_to_float<BF16>(static_cast<uint16_t>(xs[i] >> 16)));
            acc0 = fma(a0, static_cast<double>(ws[2 * i]), acc0);
            acc1 = fma(a1, static_cast<double>(ws[2 * i + 1]), acc1);
        }
    }
    return static_cast<float>(wave_sum(acc0 + acc1) + static_cast<double>(b));
}

// fp32 -> uint32 key whose unsigned order is the float order (-0 is first folded onto +0).  A NaN score gets the
// smallest key: it ranks below every number, also below -inf, so it never meets a threshold (as in
// threshold_bins_kernel) and is taken by the ratio rule only after every other token.
__device__ __forceinline__ uint32_t order_key(float f) {
    f += 0.0f;
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The decision of a call of at most 64 tokens, taken by one wave: bit t of the result = token t executes.
__device__ __forceinline__ unsigned long long wave_decide(const SelectArgs& s, const float* score, int lane) {
    const uint32_t key = lane < s.T ? order_key(score[lane]) : 0u;
    bool exec;
    if (s.mode == 0) {
        int rank = 0;
        for (int u = 0; u < s.T; ++u) {
            const uint32_t other = __shfl(key, u, 64);
            rank += (other > key || (other == key && u < lane)) ? 1 : 0;
        }
        exec = rank < s.k;
    } else {
        exec = key >= order_key(s.z_thr);
    }
    return __ballot(exec && lane < s.T);
}

// RowAux::chunk from the number of (executed row, cached key) pairs of the call and the longest cached prefix.
__device__ __forceinline__ void aux_write_chunk(const RowAux& a, int pairs, int longest, int rows) {
    const int want = a.target - rows * a.nkv / 2;              // half a range per row is lost to rounding
    // (fp32: a range more or less does not matter, a 64-bit division would be the longest chain of the kernel)
    float c = want > 0 ? static_cast<float>(pairs) * static_cast<float>(a.nkv) / static_cast<float>(want) : static_cast<float>(longest);
    const int least = (longest + a.max_ranges - 1) / a.max_ranges;
    const int keys = max(max(static_cast<int>(c), least), 1);
    *a.chunk = (keys + a.gran - 1) & ~(a.gran - 1);            // gran is a power of two
}
// (row, key) pairs and longest prefix of one sequence, added to a running pair
__device__ __forceinline__ void aux_count_keys(int rows, int old, int cap, int& pairs, int& longest) {
    const int keys = cap > 0 ? min(old, cap) : old;
    pairs += rows * keys;
    if (rows > 0) longest = max(longest, keys);
}

// Call-wide results of such a decision, by one wave of one workgroup.
__device__ __forceinline__ void wave_write_selection(const SelectArgs& s, const RowAux& aux, unsigned long long mask, const float* score,
                                                     float* z_out, int lane) {
    const int count = __popcll(mask);
    auto before = [&](int t) { return t >= s.T ? count : __popcll(mask & ((1ull << t) - 1ull)); };   // executed tokens below t
    if (lane == 0) {
        *s.count = count;
        if (s.count_copy) *s.count_copy = count;
    }
    if (lane < s.T) {
        const bool exec = (mask >> lane) & 1ull;
        const int pos = before(lane);
        if (z_out) z_out[lane] = score[lane];
        if (s.inv) s.inv[lane] = exec ? pos : -1;
        if (exec) {
            s.idx[pos] = lane;
            if (s.idx_copy) s.idx_copy[pos] = lane;
            if (s.row_seq) {
                int lo = 0, hi = s.B;                               // last b with seq_offsets[b] <= t
                while (lo + 1 < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (s.seq_offsets[mid] <= lane) lo = mid; else hi = mid;
                }
                s.row_seq[pos] = lo;
            }
        }
    }
    for (int b = lane; b <= s.B; b += 64)
        if (s.cu_exec) s.cu_exec[b] = before(s.seq_offsets[b]);
    if (s.kv_len) {
        int pairs = 0, longest = 0;
        for (int b = lane; b < s.B; b += 64) {
            const int n = before(s.seq_offsets[b + 1]) - before(s.seq_offsets[b]);
            const int old = s.kv_len[b];
            s.kv_old[b] = old;
            s.kv_len[b] = s.kv_cap > 0 ? min(old + n, max(old, s.kv_cap)) : old + n;
            aux_count_keys(n, old, s.kv_cap, pairs, longest);
        }
        if (aux.chunk) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                pairs += __shfl_xor(pairs, o, 64);
                longest = max(longest, __shfl_xor(longest, o, 64));
            }
            if (lane == 0) aux_write_chunk(aux, pairs, longest, count);
        }
    }
}

// (cos, sin) of pair p of compact row `row` (token t) at the token's original position, in fp64, rounded once: the
// decode attention kernel rotates its query and its new keys with these.  Thread p < head_dim / 2 of whoever calls.
__device__ __forceinline__ void aux_rope_row(const RowAux& a, int row, int t, int p) {
    if (!a.cs || p >= a.half) return;
    const double inv_freq = pow(static_cast<double>(a.base), -static_cast<double>(p) / static_cast<double>(a.half));
    double s, c;
    sincos(static_cast<double>(a.positions[t]) * inv_freq, &s, &c);
    a.cs[static_cast<size_t>(row) * a.half + p] = make_float2(static_cast<float>(c), static_cast<float>(s));
}

__device__ __forceinline__ void aux_clear(const RowAux& a, int i0, int stride) {
    for (int i = i0; i < a.n_arrive; i += stride) a.arrive[i] = 0;
}

}  // namespace qtale

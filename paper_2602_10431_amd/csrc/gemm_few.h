// Quantized linears for a handful of executed rows (at most kFewRows, the decode steps of a few users): C[M][N] =
// A[M][K] x W'[N][K]^T with the weights streamed once (Sec. 4.1 weights; rows gathered per App. B.2).
//
// What bounds this size is latency: a linear's weights are 2 to 10 us of HBM time, every launch starts with a chain of
// dependent loads on cold caches, and 32-column fragments leave most CUs without work unless K is cut across workgroups,
// which costs one more launch to add the parts.  So here
//   * a fragment is 16 columns wide (v_mfma_f32_16x16x32_f16, four accumulator registers): a hidden-size-wide output is
//     256 fragments, one per CU, and no workgroup needs another one's partial sums;
//   * one round of workgroups, about one per CU: a workgroup is NP column groups of NF fragments x NK k-slices of waves
//     (few_shape below).  (Many small workgroups in several rounds repeat the latency chain: gate/up of the 7B shape at one
//     row took 30 us that way with the activations made in the kernel; 16 waves per workgroup are slower than 8.)
//   * a wave's step is two k-tiles of its fragments: lane (n, q) takes row n, half q & 1 of k-tile q >> 1, 16 bytes per lane
//     straight from the prepacked layout, four MFMAs per fragment.  The weights and activations of kSteps steps are in
//     flight per wave (deeper rings were slower: their registers cost waves);
//   * activations are fetched row-contiguously and re-laid out through a wave-private LDS region;
//   * the k-slices meet once in LDS, in slice order, and the epilogues are the tiled kernels' (residual and scatter
//     included, so the caller needs no kernel to add K parts);
//   * with at most kFewFuseT tokens the kernel also makes its own A: it scores, selects and normalises the tokens (q|k|v),
//     or normalises the fp32 residual (gate/up), into LDS.  Every workgroup repeats this (a few rows from L2, each thread
//     one 16-byte piece of every row, requested BEFORE the weights: a wave's loads return in order), so it runs while the
//     weights are in flight and replaces two launches and one launch.  One more workgroup writes the call-wide results.
// Measured per launch in a stream, 4 bit, group 128, cold weights (before: gemm_decode / gemm_skinny without K parts), us:
//     4096 x 4096    1 row 5.1 (11.6)   8 rows 5.7 (11.6)   16 rows 6.7 (11.7)
//     4096 x 11008   1 row 8.1 (23.4)   8 rows 9.3 (23.5)   16 rows 12.0 (23.6)
//     12288 x 4096   1 row 8.6 (12.2)   8 rows 9.7 (12.2)   16 rows 11.8 (12.3)
//     2 x 11008 x 4096 (SwiGLU)  1 row 12.9 (18.6)   8 rows 13.8 (18.5)   16 rows 16.0 (18.7)
#pragma once
#include <algorithm>

#include "gemm_common.h"
#include "row_aux.h"

namespace qtale {

enum { PRO_NONE = 0, PRO_SELECT = 1, PRO_NORM = 2 };

struct FewDev {
    GemmDev g;
    FewPrologue pro;
};

template <int BITS, int GPT, bool SWIGLU, int NF, int NP, int NK, int MR, int PRO, bool ACT_BF16, bool NT_LOADS>
__global__ void __launch_bounds__(NP * NK * 64)
gemm_few_kernel(FewDev a) {
    using WB = WBits<BITS>;
    // NF fragments per wave: neighbours, or (gate/up) 16 gate columns and the same 16 up columns
    constexpr int GF = SWIGLU ? 1 : NF;            // column fragments of a column group
    static_assert(!SWIGLU || NF == 2, "a gate and an up fragment");
    constexpr int NW = NP * NK;
    constexpr int NT = NW * 64;
    // steps in flight per wave; deeper rings were slower (one token, 7B shape: 53.8 us per layer at 3 / 2 steps, 55.8 at 6 / 4,
    // 57.7 at 8 / 6): the loads that the prologue waits for queue behind more weights, and the registers cost waves
    constexpr int kSteps = NF == 2 ? 2 : 3;
    constexpr int AL = MR / 4;                                    // 16-byte pieces of a step's activations per lane
    constexpr int ASTR = 136;                                     // halves per staged row (128 + 8: conflict-free 16-byte reads)
    const GemmDev& p = a.g;
    const int epi = SWIGLU ? static_cast<int>(EPI_SWIGLU_F16) : PRO == PRO_SELECT ? static_cast<int>(EPI_STORE_F16) : p.epi_rt;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float* red = reinterpret_cast<float*>(smem);                                   // [NW][NF][16 rows][16 columns]
    half_t* As = reinterpret_cast<half_t*>(smem);                                  // PRO: [rows][K + 8], before the sums
    __shared__ double s_dot[PRO == PRO_SELECT ? NW : 1][kFewFuseT];
    __shared__ float s_ss[PRO != PRO_NONE ? NW : 1][kFewFuseT];
    __shared__ float s_score[kFewFuseT];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = wave % NP, wk = wave / NP;
    const int n16 = lane & 15, q = lane >> 4;
    const int a_stride = p.K + 8;

    // ---- the rows this thread helps to make: one piece of 8 columns per row and pass (requested first) --------------------
    constexpr int PASSES = (kFewPasses * 512 + NT - 1) / NT;       // few_prologue_fits: K <= 8 * 512 * kFewPasses
    const int pieces = p.K >> 3;
    u32x4_t xr[PRO == PRO_SELECT ? kFewFuseT : 1][PASSES];
    float4_t hr[PRO == PRO_NORM ? kFewFuseT : 1][PASSES][2];
    u32x4_t gr[PASSES];
    float4_t wr[PASSES][2];
    const bool score_here = PRO == PRO_SELECT && a.pro.router_w != nullptr;
    const int rows_in = PRO == PRO_SELECT ? a.pro.s.T : p.M_max;   // rows past the executed count hold nothing: nobody reads their sums
    if (PRO != PRO_NONE) {
#pragma unroll
        for (int s = 0; s < PASSES; ++s) {
            const int c = min(tid + s * NT, pieces - 1);          // past the row: its last piece again, not used
            if (s > 0 && pieces <= NT) break;
            if (PRO == PRO_SELECT) {
#pragma unroll
                for (int t = 0; t < kFewFuseT; ++t)
                    if (t < rows_in) xr[t][s] = reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.pro.x) + static_cast<size_t>(t) * p.K)[c];
                if (score_here) {
                    wr[s][0] = reinterpret_cast<const float4_t*>(a.pro.router_w)[2 * c];
                    wr[s][1] = reinterpret_cast<const float4_t*>(a.pro.router_w)[2 * c + 1];
                }
            } else {
#pragma unroll
                for (int t = 0; t < kFewFuseT; ++t)
                    if (t < rows_in) {
                        hr[t][s][0] = reinterpret_cast<const float4_t*>(a.pro.h + static_cast<size_t>(t) * p.K)[2 * c];
                        hr[t][s][1] = reinterpret_cast<const float4_t*>(a.pro.h + static_cast<size_t>(t) * p.K)[2 * c + 1];
                    }
            }
            gr[s] = reinterpret_cast<const u32x4_t*>(a.pro.gain)[c];
        }
    }

    // ---- this wave's fragments: one row of 16 per lane ---------------------------------------------------------------
    const uint32_t magic = dequant_magic();
    const int lhi = q & 1, th = q >> 1;
    const char* bptr[NF];
    const uint32_t* sptr[NF];
    int npad[NF];
#pragma unroll
    for (int fn = 0; fn < NF; ++fn) {
        int m = 0, f = (blockIdx.x * NP + wp) * GF;
        if (SWIGLU) {
            m = fn;
        } else {
            f += fn;
            if (p.n_w > 1 && f >= 2 * p.NF[0]) { f -= 2 * p.NF[0]; m = 1; }
            if (p.n_w > 2 && m == 1 && f >= 2 * p.NF[1]) { f -= 2 * p.NF[1]; m = 2; }
        }
        f = min(f, 2 * p.NF[m] - 1);                              // past the last fragment: that one again, never stored
        const int r32 = ((f & 1) << 4) | n16;
        bptr[fn] = reinterpret_cast<const char*>(p.codes[m]) + (static_cast<size_t>(f >> 1) * p.KT * 64 + lhi * 32 + r32) * WB::kLaneBytes;
        sptr[fn] = p.sz[m] + (f >> 1) * 32 + r32;
        npad[fn] = p.npad[m];
    }
    // Steps of this wave: wk, wk + NK, ...; steps past the last one are clamped to it (loaded, not used).
    const int n_steps = (p.KT + 1) >> 1;
    const int n_mine = wk < n_steps ? (n_steps - wk + NK - 1) / NK : 0;
    const int last = wk + (n_mine - 1) * NK;
    typename WB::Tile bq[kSteps][NF];
    uint32_t bsz[kSteps][NF][GPT];
    auto fetch_b = [&](int step, typename WB::Tile* w, uint32_t (*sz)[GPT]) {
        const int kt = min(2 * min(step, last) + th, p.KT - 1);
#pragma unroll
        for (int fn = 0; fn < NF; ++fn) {
            const char* wp = bptr[fn] + static_cast<size_t>(kt) * (64 * WB::kLaneBytes);
            if constexpr (NT_LOADS) w[fn] = WB::template load_lane<true>(wp);
            else w[fn] = WB::load_lane(wp);
#pragma unroll
            for (int g = 0; g < GPT; ++g) sz[fn][g] = sptr[fn][static_cast<size_t>((kt * 64 + g * 32) >> p.gshift) * npad[fn]];
        }
    };
    // Activations of a step (MR rows x 128 columns): fetched row-contiguously (16 lanes per row), parked in a wave-private
    // LDS region and read back in operand order, lane (m, q) row m, columns 64 kt + 16 j + 8 (q & 1) of k-tile kt.  Reading the
    // operand order from memory touches 32 cache lines per instruction and uses 32 bytes of each: at 8 rows the o-proj
    // shape took 7.5 us that way and the down-proj shape 12.4.  Rows past M repeat the last one (their sums are not
    // stored); columns past K the row's last valid piece (the weights there dequantize to 0).
    const int M = PRO != PRO_SELECT && p.count ? min(*p.count, p.M_max) : p.M_max;
    half_t* stage = reinterpret_cast<half_t*>(smem) + wave * (MR * ASTR);
    const half_t* arow[AL];
#pragma unroll
    for (int i = 0; i < AL; ++i) arow[i] = p.A + static_cast<size_t>(min(i * 4 + (lane >> 4), max(M, 1) - 1)) * p.K;
    auto load_a = [&](int step, u32x4_t* ar) {
        const int col = min(min(step, last) * 128 + (lane & 15) * 8, p.K - 8);
#pragma unroll
        for (int i = 0; i < AL; ++i) ar[i] = *reinterpret_cast<const u32x4_t*>(arow[i] + col);
    };
    const int op_row = min(n16, PRO == PRO_NONE ? MR - 1 : max(p.M_max, 1) - 1);
    auto read_a = [&](int step, half8_t* ac) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (PRO == PRO_NONE) ac[j] = *reinterpret_cast<const half8_t*>(stage + op_row * ASTR + th * 64 + 16 * j + 8 * lhi);
            else ac[j] = *reinterpret_cast<const half8_t*>(As + op_row * a_stride + min(min(2 * step + th, p.KT - 1) * 64 + 16 * j + 8 * lhi, p.K - 8));
        }
    };
    u32x4_t areg[PRO == PRO_NONE ? kSteps : 1][AL];
    if (n_mine > 0 && (PRO != PRO_SELECT || static_cast<int>(blockIdx.x) < p.tiles_n)) {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            fetch_b(wk + u * NK, bq[u], bsz[u]);
            if (PRO == PRO_NONE) load_a(wk + u * NK, areg[PRO == PRO_NONE ? u : 0]);    // in step order: a wave's loads return in order
        }
    }

    // ---- A, where the kernel makes it ------------------------------------------------------------------------------------
    if (PRO != PRO_NONE) {
        // sums over the row: this thread's pieces, the wave, then all waves in order through LDS
#pragma unroll
        for (int t = 0; t < kFewFuseT; ++t) {
            if (t >= rows_in) break;
            double acc0 = 0.0, acc1 = 0.0;
            float ss = 0.0f;
#pragma unroll
            for (int s = 0; s < PASSES; ++s) {
                if (tid + s * NT >= pieces) break;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float e0, e1;
                    if (PRO == PRO_SELECT) {
                        e0 = act_to_float<ACT_BF16>(static_cast<uint16_t>(xr[t][s][i] & 0xffffu));
                        e1 = act_to_float<ACT_BF16>(static_cast<uint16_t>(xr[t][s][i] >> 16));
                    } else {
                        e0 = hr[t][s][i >> 1][2 * (i & 1)];
                        e1 = hr[t][s][i >> 1][2 * (i & 1) + 1];
                    }
                    ss = fmaf(e0, e0, ss);
                    ss = fmaf(e1, e1, ss);
                    if (score_here) {
                        acc0 = fma(static_cast<double>(e0), static_cast<double>(wr[s][i >> 1][2 * (i & 1)]), acc0);
                        acc1 = fma(static_cast<double>(e1), static_cast<double>(wr[s][i >> 1][2 * (i & 1) + 1]), acc1);
                    }
                }
            }
            ss = wave_sum(ss);
            if (lane == 0) s_ss[wave][t] = ss;
            if (score_here) {
                const double dot = wave_sum(acc0 + acc1);
                if (lane == 0) s_dot[wave][t] = dot;
            }
        }
        __syncthreads();
        unsigned long long mask = ~0ull;
        if (PRO == PRO_SELECT) {
            const SelectArgs& s = a.pro.s;
            if (tid < s.T) {
                float z;
                if (score_here) {
                    double dot = 0.0;
                    for (int w = 0; w < NW; ++w) dot += s_dot[w][tid];
                    z = static_cast<float>(dot + static_cast<double>(a.pro.router_b));
                } else {
                    z = s.z[tid];
                }
                s_score[tid] = z;
            }
            __syncthreads();
            mask = wave_decide(s, s_score, lane);
            if (static_cast<int>(blockIdx.x) == p.tiles_n) {      // the extra workgroup: everything else the call leaves behind
                if (wave == 0) wave_write_selection(s, a.pro.aux, mask, s_score, score_here ? a.pro.z_out : nullptr, lane);
                aux_clear(a.pro.aux, tid, NT);
                for (int t = wave; t < s.T; t += NW)
                    if ((mask >> t) & 1ull) aux_rope_row(a.pro.aux, __popcll(mask & ((1ull << t) - 1ull)), t, lane);
                return;
            }
        }
#pragma unroll
        for (int t = 0; t < kFewFuseT; ++t) {
            if (t >= rows_in) break;
            if (!((mask >> t) & 1ull)) continue;
            const int row = PRO == PRO_SELECT ? __popcll(mask & ((1ull << t) - 1ull)) : t;
            float ss = 0.0f;
            for (int w = 0; w < NW; ++w) ss += s_ss[w][t];
            const float inv = 1.0f / sqrtf(ss / static_cast<float>(p.K) + a.pro.eps);
#pragma unroll
            for (int s = 0; s < PASSES; ++s) {
                if (tid + s * NT >= pieces) break;
                u32x4_t o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float e0, e1;
                    if (PRO == PRO_SELECT) {
                        e0 = act_to_float<ACT_BF16>(static_cast<uint16_t>(xr[t][s][i] & 0xffffu));
                        e1 = act_to_float<ACT_BF16>(static_cast<uint16_t>(xr[t][s][i] >> 16));
                    } else {
                        e0 = hr[t][s][i >> 1][2 * (i & 1)];
                        e1 = hr[t][s][i >> 1][2 * (i & 1) + 1];
                    }
                    e0 = e0 * inv * act_to_float<ACT_BF16>(static_cast<uint16_t>(gr[s][i] & 0xffffu));
                    e1 = e1 * inv * act_to_float<ACT_BF16>(static_cast<uint16_t>(gr[s][i] >> 16));
                    o[i] = static_cast<uint32_t>(float_to_half_bits(e0)) | (static_cast<uint32_t>(float_to_half_bits(e1)) << 16);
                }
                *reinterpret_cast<u32x4_t*>(As + row * a_stride + (tid + s * NT) * 8) = o;
            }
        }
    }

    // ---- residual rows of the epilogue, requested before the sums are there ----------------------------------------------
    // thread t owns output (row (t % 256) / 16, column t % 16) of column fragments t / 256, t / 256 + NW / 4, ... of the workgroup
    constexpr int EF = (NP * GF * 256 + NT - 1) / NT;             // outputs per thread
    const int er = (tid >> 4) & 15, ec = tid & 15;
    int e_mat[EF], e_n[EF];
    bool e_ok[EF];
    int trow = 0;
    float resid[EF];
    if ((epi == EPI_RESID_F32 || epi == EPI_RESID_SCATTER) && er < M) trow = p.idx[er];
#pragma unroll
    for (int i = 0; i < EF; ++i) {
        const int eg = (tid >> 8) + i * (NT >> 8);                // column fragment inside the workgroup
        int m = 0, f = blockIdx.x * NP * GF + eg;
        if (!SWIGLU) {
            if (p.n_w > 1 && f >= 2 * p.NF[0]) { f -= 2 * p.NF[0]; m = 1; }
            if (p.n_w > 2 && m == 1 && f >= 2 * p.NF[1]) { f -= 2 * p.NF[1]; m = 2; }
        }
        e_mat[i] = m;
        e_n[i] = f * 16 + ec;
        e_ok[i] = eg < NP * GF && er < M && e_n[i] < p.N[m];
        resid[i] = 0.0f;
        if (epi == EPI_RESID_F32 && e_ok[i]) resid[i] = act_to_float(reinterpret_cast<const uint16_t*>(p.resid)[static_cast<size_t>(trow) * p.ldo + e_n[i]], p.bf16);
        if (epi == EPI_RESID_SCATTER && e_ok[i]) resid[i] = reinterpret_cast<const float*>(p.resid)[static_cast<size_t>(er) * p.ldo + e_n[i]];
    }

    float4_t acc[NF];
#pragma unroll
    for (int fn = 0; fn < NF; ++fn) acc[fn] = float4_t{0.f, 0.f, 0.f, 0.f};
    if (PRO != PRO_NONE) __syncthreads();                         // A is in LDS
    for (int i0 = 0; i0 < n_mine; i0 += kSteps) {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            if (i0 + u >= n_mine) break;
            const int step = wk + (i0 + u) * NK;
            half8_t ac[4];
            if (PRO == PRO_NONE) {                                // LDS operations of a wave complete in order: no barrier
#pragma unroll
                for (int i = 0; i < AL; ++i) *reinterpret_cast<u32x4_t*>(stage + (i * 4 + (lane >> 4)) * ASTR + (lane & 15) * 8) = areg[PRO == PRO_NONE ? u : 0][i];
            }
            read_a(step, ac);
            const bool live = 2 * step + th < p.KT;               // a scale|zero word of 0 makes the weights exactly 0
#pragma unroll
            for (int fn = 0; fn < NF; ++fn) {
                typename WB::SZ sz[GPT];
#pragma unroll
                for (int g = 0; g < GPT; ++g) sz[g] = WB::expand(live ? bsz[u][fn][g] : 0u);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const half8_t b = WB::dequant(bq[u][fn], j, sz[GPT == 2 ? (j >> 1) : 0], magic);
                    acc[fn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ac[j], b, acc[fn], 0, 0, 0);
                }
            }
            fetch_b(step + kSteps * NK, bq[u], bsz[u]);
            if (PRO == PRO_NONE) load_a(step + kSteps * NK, areg[PRO == PRO_NONE ? u : 0]);
        }
    }

    // ---- meet: the k-slices' sums in slice order, then the epilogue -----------------------------------------------------------
    __syncthreads();                                              // nobody reads A any more
#pragma unroll
    for (int fn = 0; fn < NF; ++fn)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((wave * NF + fn) << 8) + ((4 * q + r) << 4) + n16] = acc[fn][r];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EF; ++i) {
        if (!e_ok[i]) continue;
        const int eg = (tid >> 8) + i * (NT >> 8);
        float v[2] = {0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            if (SWIGLU) {
                v[0] += red[(((k * NP + eg) * 2) << 8) + (tid & 255)];
                v[1] += red[(((k * NP + eg) * 2 + 1) << 8) + (tid & 255)];
            } else {
                v[0] += red[(((k * NP + eg / GF) * NF + eg % GF) << 8) + (tid & 255)];
            }
        }
        const size_t col = static_cast<size_t>((SWIGLU ? 0 : p.colbase[e_mat[i]]) + e_n[i]);
        if (SWIGLU) reinterpret_cast<uint16_t*>(p.out)[static_cast<size_t>(er) * p.ldo + col] = float_to_half_bits(silu_f(v[0]) * v[1]);
        else if (epi == EPI_STORE_F16) reinterpret_cast<uint16_t*>(p.out)[static_cast<size_t>(er) * p.ldo + col] = float_to_half_bits(v[0]);
        else if (epi == EPI_RESID_F32) reinterpret_cast<float*>(p.out)[static_cast<size_t>(er) * p.ldo + col] = resid[i] + v[0];
        else reinterpret_cast<uint16_t*>(p.out)[static_cast<size_t>(trow) * p.ldo + col] = float_to_act(resid[i] + v[0], p.bf16);
    }
}

// Layer calls of at most eight rows, 4-bit weights of at least 6 MB: non-temporal loads.  They are read once per call, and where the
// layers that take turns do not fit the memory-side cache (256 MB) together, ordinary loads push each other's out of it before any is
// used again.  Whole layers, us, ordinary / non-temporal, 1 and 8 tokens: 7B shape, 322 MB of weights in turn 54.4 / 53.0, 75.4 / 73.9,
// 2 GB 54.7 / 53.0, 74.5 / 72.4; 8B-GQA 347 MB 53.1 / 52.0, 67.9 / 66.2, 2 GB 53.2 / 52.0, 67.9 / 67.3; 13B 2 GB 65.7 / 64.1, 95.8 / 93.8; hidden
// 2560 1.5 GB 38.6 / 38.1, 55.1 / 53.2 (without the linears of 9 MB 39.1, 55.7); 2048, SwiGLU 8192 854 MB 37.3 / 36.1, 51.0 / 48.9; 5632 382 MB
// 34.7 / 32.9, 44.3 / 41.1, 860 MB 34.9 / 34.9, 44.3 / 44.0; 1536 420 MB 32.2 / 31.4, 45.3 / 44.3.
// What fits the cache together is better left there.  A stack knows that (fits_cache, qtale_api.hip): 7B 215 MB 50.8 / 52.3, 71.6 / 74.4,
// 8B-GQA 231 MB 50.3 / 51.9, 64.0 / 65.4, 13B 168 MB 60.4 / 62.0, 91.0 / 100.  Of a call of a single layer it is taken that others follow;
// models whose largest linear is below 6 MB fit whole (24 layers of hidden 1024 163 MB, from 1 MB on 38.1 / 39.3 with 8 tokens, of 1280 252 MB 41.0 /
// 41.8).  Linears called by themselves keep ordinary loads (4096 x 14336, 3 rows 8.2 / 9.8), as do more rows (8B-GQA, 16 rows, 20
// layers 79.1 / 80.5) and 2-bit weights (7B 47.0 / 47.9, 51.9 / 51.6).
static bool few_streams(const GemmDev& d) {
    if (!d.streams || d.bits != 4 || d.M_max > 8) return false;
    size_t bytes = 0;
    for (int i = 0; i < d.n_w; ++i) bytes += static_cast<size_t>(d.NF[i]) * d.KT * 64 * (4 * d.bits);
    return bytes >= (6u << 20);
}

template <int BITS, int GPT, bool SWIGLU, int NF, int NP, int NK, int MR, int PRO, bool NT_LOADS = false>
static hipError_t few_launch(FewDev& a, int frags, hipStream_t stream) {
    constexpr int NW = NP * NK, GROUP = NP * (SWIGLU ? 1 : NF);
    a.g.tiles_n = (frags + GROUP - 1) / GROUP;
    const dim3 grid(a.g.tiles_n + (PRO == PRO_SELECT ? 1 : 0)), block(NW * 64);
    const size_t rows = PRO != PRO_NONE ? static_cast<size_t>(a.g.M_max) * (a.g.K + 8) * 2 : static_cast<size_t>(NW) * MR * 136 * 2;
    const size_t lds = std::max<size_t>(NW * NF * 1024, rows);
    if (PRO != PRO_NONE && a.pro.bf16) {
        auto k = gemm_few_kernel<BITS, GPT, SWIGLU, NF, NP, NK, MR, PRO, PRO != PRO_NONE, NT_LOADS>;
        hipLaunchKernelGGL(k, grid, block, lds, stream, a);
    } else {
        auto k = gemm_few_kernel<BITS, GPT, SWIGLU, NF, NP, NK, MR, PRO, false, NT_LOADS>;
        hipLaunchKernelGGL(k, grid, block, lds, stream, a);
    }
    return hipGetLastError();
}

template <int BITS, int GPT, bool SWIGLU, int NF, int NP, int NK>
static hipError_t few_rows(FewDev& a, int frags, hipStream_t stream) {
    constexpr int PRO = SWIGLU ? PRO_NORM : PRO_SELECT;           // gate/up follows RMSNorm 2, q|k|v the selection
    const bool nt = few_streams(a.g);
    if (a.pro.h || a.pro.x) return nt ? few_launch<BITS, GPT, SWIGLU, NF, NP, NK, 4, PRO, BITS == 4>(a, frags, stream)
                                      : few_launch<BITS, GPT, SWIGLU, NF, NP, NK, 4, PRO>(a, frags, stream);
    if (nt && a.g.M_max <= 4) return few_launch<BITS, GPT, SWIGLU, NF, NP, NK, 4, PRO_NONE, BITS == 4>(a, frags, stream);
    if (nt) return few_launch<BITS, GPT, SWIGLU, NF, NP, NK, 8, PRO_NONE, BITS == 4>(a, frags, stream);
    if (a.g.M_max <= 4) return few_launch<BITS, GPT, SWIGLU, NF, NP, NK, 4, PRO_NONE>(a, frags, stream);
    if (a.g.M_max <= 8) return few_launch<BITS, GPT, SWIGLU, NF, NP, NK, 8, PRO_NONE>(a, frags, stream);
    return few_launch<BITS, GPT, SWIGLU, NF, NP, NK, 16, PRO_NONE>(a, frags, stream);
}

// Columns per workgroup: the narrowest of the measured shapes whose workgroups do not outnumber the CUs, so that one round
// covers the output (us at 8 rows, 256 CUs: 256 fragments 1x1x8 5.7, 2x1x8 6.6; 384: 2x1x8 6.8, 1x1x8 8.2; 768: 1x3x4 9.7,
// 1x1x8 13.2; gate/up, 688 pairs: x3x4 13.8, x2x4 16.1, x1x8 14.9; 896 pairs do not fit any: x2x4 16.8, x3x4 23.3).
template <int BITS, int GPT>
static hipError_t few_shape(FewDev& a, int epi, int cus, hipStream_t stream) {
    a.g.epi_rt = epi;
    if (epi == EPI_SWIGLU_F16) {
        const int pairs = 2 * a.g.NF[0];
        if (pairs <= cus) return few_rows<BITS, GPT, true, 2, 1, 8>(a, pairs, stream);
        if (pairs <= 2 * cus || pairs > 3 * cus) return few_rows<BITS, GPT, true, 2, 2, 4>(a, pairs, stream);
        return few_rows<BITS, GPT, true, 2, 3, 4>(a, pairs, stream);
    }
    int frags = 0;
    for (int i = 0; i < a.g.n_w; ++i) frags += 2 * a.g.NF[i];
    if (frags <= cus) return few_rows<BITS, GPT, false, 1, 1, 8>(a, frags, stream);
    if (frags <= 2 * cus) return few_rows<BITS, GPT, false, 2, 1, 8>(a, frags, stream);
    if (frags <= 3 * cus) return few_rows<BITS, GPT, false, 1, 3, 4>(a, frags, stream);
    return few_rows<BITS, GPT, false, 2, 2, 4>(a, frags, stream);
}

}  // namespace qtale

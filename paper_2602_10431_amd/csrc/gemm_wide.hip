// W4A16 / W3A16 / W2A16 GEMM for the wide outputs at 65 to 256 executed rows (large decode batches, short prompts), and for
// more rows where its workgroups fill the chip once (the rules are in gemm_w4a16.hip): C[M][N] = A[M][K] x W'[N][K]^T
// with the weights dequantized once per 128-row chunk (Sec. 4.1 weights; rows gathered per App. B.2).
//
// At these sizes a linear is a few dozen 128 x 256 tiles, so the prefill kernel leaves most CUs idle, while 64-row chunks of
// 64 columns (gemm_skinny) dequantize every weight once per 64 rows and pull the activations through each CU once per 64
// columns.  Every CU has to read its part of A whatever the split (M x K x 2 bytes per column block), an LDS fragment read
// costs 8 cycles against 8 per MFMA of the CU's four SIMDs, and dequantisation is 13 vector instructions per fragment and
// k-step.  So here
//   * a wave owns up to 128 rows x 64 columns (8 accumulator fragments): a dequantized weight fragment feeds four MFMAs and
//     an activation fragment two, half the LDS reads of a 32-column wave;
//   * a workgroup is 2 column groups x 4 k-slices of such waves, one workgroup and two waves per SIMD per CU: 128 columns
//     per workgroup fill most of the chip for the wide outputs, and the k-slices give each SIMD a second wave to overlap
//     dequantisation with MFMAs;
//   * the two waves of a k-slice share its activation tile through LDS (two buffers per slice, 144 KB), weights go straight to
//     registers two rounds ahead (ring of three slots, the loop is unrolled by three); one barrier per round of four k-tiles;
//   * narrow outputs (o-proj, down-proj) also cut K across workgroups and write fp32 partial tiles that the consumer kernel
//     adds in order (no atomics, no fences);
//   * row fragments past the executed rows are left out (the count may be known on the device only);
//   * the k-slices meet in LDS, 32 columns of every wave at a time; a slice adds and stores its share of the row fragments;
//   * outputs whose workgroups are one to two per CU take two k-slices instead of four: half the waves and LDS, so two workgroups
//     share a CU, each with barriers of its own, and a CU that has two does not run them one after the other (gate/up of 11008
//     columns at 150 rows, 344 workgroups: 48 -> 43 us; one alone takes 37 where four slices take 34).
#include <algorithm>
#include <type_traits>

#include "gemm_common.h"

namespace qtale {

constexpr int kWideNC = 2, kWideFM = kWideRows / 32;

template <int BITS, int GPT, bool SWIGLU, int NK>
__global__ void __launch_bounds__(kWideNC * NK * 64, 2)
gemm_wide_kernel(GemmDev p) {
    using WB = WBits<BITS>;
    constexpr int NC = kWideNC, FM = kWideFM, FN = kWideFrags / kWideNC, NW = NC * NK;
    constexpr int MS = FM / NK;                                  // row fragments that a slice meets
    static_assert(FN == 2 && FM == 4 && FM % NK == 0, "gate and up, or two columns");
    constexpr int TEAM = NC * 64;
    constexpr int kTileHalves = kWideRows * kLdsStride;
    constexpr int SSTR = 36;                                     // slab row stride (floats)
    constexpr int kABytes = 2 * NK * kTileHalves * 2, kSlabBytes = NW * kWideRows * SSTR * 4;
    __shared__ __attribute__((aligned(16))) char smem[kABytes > kSlabBytes ? kABytes : kSlabBytes];
    half_t* As = reinterpret_cast<half_t*>(smem);

    // workgroup -> (column block, row chunk, k-part): all column blocks (padded to a multiple of 8, so that the chunks of one
    // are served by the same XCD's L2) of the first chunk, then of the next.
    const int tiles_pad = (p.tiles_n + 7) & ~7;
    const int chunk = blockIdx.x / tiles_pad, tile_n = blockIdx.x - chunk * tiles_pad;
    const int ks = blockIdx.y;
    if (tile_n >= p.tiles_n) return;
    const int row0 = chunk * p.chunk_rows;
    const int M = min((p.count ? min(*p.count, p.M_max) : p.M_max) - row0, p.chunk_rows);
    if (M <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = wave % NC, wk = wave / NC;
    const int l32 = lane & 31, lhi = lane >> 5;
    const uint32_t magic = dequant_magic();

    const int kt_lo = static_cast<int>(static_cast<long>(p.KT) * ks / p.ksplit);
    const int kt_hi = static_cast<int>(static_cast<long>(p.KT) * (ks + 1) / p.ksplit);
    const int n_rounds = (kt_hi - kt_lo + NK - 1) / NK;
    const int kt_last = kt_hi - 1;
    auto tile_of = [&](int r) { return min(kt_lo + r * NK + wk, kt_last); };

    const char* bbase[FN];
    const uint32_t* sbase[FN];
    int npad[FN];
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        const int vf = min((tile_n * NC + wc) * FN + fn, p.vf_total - 1);   // edge block: the last fragment again, never stored
        int mat, f;
        map_fragment<SWIGLU ? EPI_SWIGLU_F16 : EPI_STORE_F16>(p, vf, mat, f);
        bbase[fn] = reinterpret_cast<const char*>(p.codes[mat]) + static_cast<size_t>(f) * p.KT * (64 * WB::kLaneBytes);
        sbase[fn] = p.sz[mat] + f * 32;
        npad[fn] = p.npad[mat];
    }
    typename WB::Tile bq[3][FN];
    uint32_t bsz[3][FN][GPT];
    auto load_b = [&](int r, typename WB::Tile* q, uint32_t (*sz)[GPT]) {
        const int kt = tile_of(r);
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
            q[fn] = WB::load(bbase[fn], kt, lane);
#pragma unroll
            for (int g = 0; g < GPT; ++g) sz[fn][g] = (sbase[fn] + static_cast<size_t>((kt * 64 + g * 32) >> p.gshift) * npad[fn])[l32];
        }
    };

    float16_t acc[FM][FN];
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[fm][fn][r] = 0.0f;

    const int tl = wc * 64 + lane;                               // lane inside the k-slice's team
    const int n_live = (M + 31) >> 5;                            // row fragments that hold executed rows

    auto run = [&](auto fml_c) {
        constexpr int FML = decltype(fml_c)::value;
        constexpr int A_LD = FML * 32 * 8 / TEAM;                // 16-byte chunks of the slice's tile per lane
        u32x4_t areg[A_LD];
        uint32_t a_off[A_LD];
#pragma unroll
        for (int it = 0; it < A_LD; ++it)
            a_off[it] = static_cast<uint32_t>(row0 + min(it * (TEAM / 8) + (tl >> 3), M - 1)) * static_cast<uint32_t>(p.K) + (tl & 7) * 8;
        auto load_a = [&](int r) {
            const int kt = tile_of(r);
            // chunks at or beyond K (K not a multiple of 64) read the row's last valid one: the weights there are 0
            const int col = kt * 64 + (tl & 7) * 8;
            const uint32_t shift = col >= p.K ? static_cast<uint32_t>(col - (p.K - 8)) : 0u;
            const half_t* base = p.A + kt * 64;
#pragma unroll
            for (int it = 0; it < A_LD; ++it) areg[it] = *reinterpret_cast<const u32x4_t*>(base + (a_off[it] - shift));
        };
        const int a_dst = wk * kTileHalves + (tl >> 3) * kLdsStride + (tl & 7) * 8;
        auto store_a = [&](int buf) {
#pragma unroll
            for (int it = 0; it < A_LD; ++it)
                *reinterpret_cast<u32x4_t*>(As + buf * (NK * kTileHalves) + a_dst + it * (TEAM / 8) * kLdsStride) = areg[it];
        };
        const int a_rd = wk * kTileHalves + l32 * kLdsStride + lhi * 8;

        load_a(0);
        load_b(0, bq[0], bsz[0]);
        load_b(1, bq[1], bsz[1]);
        store_a(0);
        load_a(1);
        __syncthreads();
        // Round r: weights from ring slot S, activations from buffer r & 1.  The activations of round r + 1 (requested a round
        // ago) are parked in the other buffer after the first k-step, whose last reader left it at the previous barrier; the
        // activations and weights of round r + 2 are requested.
        auto round = [&](int r, auto s_c, auto p_c) {
            constexpr int S = decltype(s_c)::value, P = decltype(p_c)::value;
            const int buf = r & 1;
            load_b(r + 2, bq[P], bsz[P]);
            const bool live = kt_lo + r * NK + wk <= kt_last;    // past the part: a scale|zero word of 0 makes the weights 0
            typename WB::SZ sz[FN][GPT];
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
#pragma unroll
                for (int g = 0; g < GPT; ++g) sz[fn][g] = WB::expand(live ? bsz[S][fn][g] : 0u);
            const half_t* src = As + buf * (NK * kTileHalves) + a_rd;
            half8_t a[2][FML];
#pragma unroll
            for (int fm = 0; fm < FML; ++fm) a[0][fm] = *reinterpret_cast<const half8_t*>(src + fm * 32 * kLdsStride);
            half8_t bcur = WB::dequant(bq[S][0], 0, sz[0][0], magic);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j == 1) {
                    store_a(buf ^ 1);
                    load_a(r + 2);
                }
                if (j < 3) {
#pragma unroll
                    for (int fm = 0; fm < FML; ++fm) a[(j + 1) & 1][fm] = *reinterpret_cast<const half8_t*>(src + fm * 32 * kLdsStride + (j + 1) * 16);
                }
#pragma unroll
                for (int fn = 0; fn < FN; ++fn) {
                    const int fnn = fn + 1 < FN ? fn + 1 : 0, jn = fn + 1 < FN ? j : j + 1;
                    half8_t bnext = bcur;
                    if (jn < 4) bnext = WB::dequant(bq[S][fnn], jn, sz[fnn][GPT == 2 ? (jn >> 1) : 0], magic);
#pragma unroll
                    for (int fm = 0; fm < FML; ++fm) acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[j & 1][fm], bcur, acc[fm][fn], 0, 0, 0);
                    bcur = bnext;
                }
            }
            __syncthreads();
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        int r = 0;
        for (; r + 3 <= n_rounds; r += 3) {
            round(r, I0{}, I2{});
            round(r + 1, I1{}, I0{});
            round(r + 2, I2{}, I1{});
        }
        if (r < n_rounds) {
            round(r, I0{}, I2{});
            if (r + 1 < n_rounds) round(r + 1, I1{}, I0{});
        }
    };
    if (n_live <= 2) run(std::integral_constant<int, 2>{});
    else if (n_live == 3) run(std::integral_constant<int, 3>{});
    else run(std::integral_constant<int, 4>{});

    // ---- meet: wave (wc, s) adds and stores row fragment s of its column group, 32 columns of each wave at a time -----------
    float* slab = reinterpret_cast<float*>(smem);                // [wave][128 rows][36]; the last round's barrier has passed
    const int c4 = (lane & 7) * 4, rr = lane >> 3;               // this lane's 4 columns, and row inside a pass of 8
    float4 v[MS][FN][4];
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        if (fn > 0) __syncthreads();
        float* mine = slab + wave * (kWideRows * SSTR);
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
            if (fm < n_live) {
#pragma unroll
                for (int r = 0; r < 16; ++r) mine[(fm * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3)) * SSTR + l32] = acc[fm][fn][r];
            }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < MS; ++m) {
            const int fm = wk * MS + m;
            if (fm >= n_live) continue;
#pragma unroll
            for (int ps = 0; ps < 4; ++ps) {
                v[m][fn][ps] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int s = 0; s < NK; ++s) {
                    const float4 t = *reinterpret_cast<const float4*>(slab + (s * NC + wc) * (kWideRows * SSTR) + (fm * 32 + ps * 8 + rr) * SSTR + c4);
                    v[m][fn][ps].x += t.x; v[m][fn][ps].y += t.y; v[m][fn][ps].z += t.z; v[m][fn][ps].w += t.w;
                }
            }
        }
    }
#pragma unroll
    for (int mf = 0; mf < MS * (SWIGLU ? 1 : FN); ++mf) {
        const int m = mf % MS, fo = mf / MS;
        if (wk * MS + m >= n_live) continue;
        const int vf = (tile_n * NC + wc) * FN + fo;
        if (vf >= p.vf_total) continue;
        int mat, f;
        map_fragment<SWIGLU ? EPI_SWIGLU_F16 : EPI_STORE_F16>(p, vf, mat, f);
        const int ncol = f * 32 + c4;
        if (ncol >= p.N[mat]) continue;                          // N % 4 == 0: the 4 columns are all in or all out
        const int col = (SWIGLU ? 0 : p.colbase[mat]) + ncol;
#pragma unroll
        for (int ps = 0; ps < 4; ++ps) {
            const int lrow = (wk * MS + m) * 32 + ps * 8 + rr;
            if (lrow >= M) continue;
            const size_t row = row0 + lrow;
            float4 o = v[m][fo][ps];
            if (SWIGLU) {
                const float4 u = v[m][FN - 1][ps];
                o.x = silu_f(o.x) * u.x; o.y = silu_f(o.y) * u.y; o.z = silu_f(o.z) * u.z; o.w = silu_f(o.w) * u.w;
            }
            if (!SWIGLU && p.epi_rt == EPI_PARTIAL_F32) {
                *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.out) + (static_cast<size_t>(ks) * p.M_max + row) * p.ldo + col) = o;
            } else {
                uint2 h;
                h.x = static_cast<uint32_t>(float_to_half_bits(o.x)) | (static_cast<uint32_t>(float_to_half_bits(o.y)) << 16);
                h.y = static_cast<uint32_t>(float_to_half_bits(o.z)) | (static_cast<uint32_t>(float_to_half_bits(o.w)) << 16);
                *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(p.out) + row * p.ldo + col) = h;
            }
        }
    }
}

template <int BITS, int GPT>
static hipError_t launch_kind(const GemmDev& d, int epilogue, int slices, hipStream_t stream) {
    const dim3 grid(((d.tiles_n + 7) / 8) * 8 * d.row_chunks, d.ksplit), block(kWideNC * slices * 64);
    if (epilogue == EPI_SWIGLU_F16) {
        if (slices == 2) hipLaunchKernelGGL((gemm_wide_kernel<BITS, GPT, true, 2>), grid, block, 0, stream, d);
        else hipLaunchKernelGGL((gemm_wide_kernel<BITS, GPT, true, 4>), grid, block, 0, stream, d);
    } else {
        if (slices == 2) hipLaunchKernelGGL((gemm_wide_kernel<BITS, GPT, false, 2>), grid, block, 0, stream, d);
        else hipLaunchKernelGGL((gemm_wide_kernel<BITS, GPT, false, 4>), grid, block, 0, stream, d);
    }
    return hipGetLastError();
}

hipError_t launch_gemm_wide(GemmDev& d, int epilogue, int ksplit, int slices, hipStream_t stream) {
    d.tiles_n = gemm_wide_cols(d);
    if (d.tiles_n == 0) return hipSuccess;
    // the chunks share the row fragments evenly: 150 rows are 96 + 54, five fragments and not six
    d.row_chunks = gemm_wide_chunks(d);
    d.chunk_rows = (((d.M_max + 31) / 32 + d.row_chunks - 1) / d.row_chunks) * 32;
    d.ksplit = ksplit;
    d.epi_rt = epilogue;
    if (d.bits == 3) return d.gshift == 5 ? launch_kind<3, 2>(d, epilogue, slices, stream) : launch_kind<3, 1>(d, epilogue, slices, stream);
    if (d.bits == 2) return d.gshift == 5 ? launch_kind<2, 2>(d, epilogue, slices, stream) : launch_kind<2, 1>(d, epilogue, slices, stream);
    return d.gshift == 5 ? launch_kind<4, 2>(d, epilogue, slices, stream) : launch_kind<4, 1>(d, epilogue, slices, stream);
}

}  // namespace qtale

// Host-side launchers of the gfx950 kernels (internal; the public boundary is include/qtale.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace qtale {

struct PrepackDims {
    int NF, KT, NGP;
    size_t code_bytes, sz_bytes;
};
PrepackDims prepack_dims(int N, int K, int group, int bits);

hipError_t launch_quantize(const float* W, int N, int K, int bits, int group, uint32_t* codes,
                           uint16_t* scales, uint16_t* zeros, void* prepacked /*nullable*/, hipStream_t stream);
hipError_t launch_prepack(const uint32_t* codes, const uint16_t* scales, const uint16_t* zeros, int N,
                          int K, int bits, int group, void* prepacked, hipStream_t stream);

// What the kernel that normalises the executed rows also prepares for the decode attention kernel.
struct RowAux {
    float2* cs;                // nullable: [rows][half] (cos, sin) of every executed row's position
    const int32_t* positions;  // [T]
    int half;                  // head_dim / 2
    float base;
    int32_t* arrive;           // [n_arrive] counters to clear
    int n_arrive;
    // split keys: *chunk = cached keys per range such that the executed rows' ranges are equally long and about `target` of
    // them cover the call (a multiple of `gran`, at most `max_ranges` ranges per row)
    int32_t* chunk;            // nullable
    int nkv, target, gran, max_ranges;
};

// ---- router + selection --------------------------------------------------------------------
hipError_t launch_router_score(const void* x, int bf16, int T, int H, const float* w, float b,
                               float* z, hipStream_t stream);

// Two-output MLP router: z_t = (W2 relu(W1 x_t + b1) + b2)[0] - (...)[1]; W1 [R][H], b1 [R], W2 [2][R], b2 [2] fp32.
hipError_t launch_router_mlp(const void* x, int bf16, int T, int H, const float* W1, const float* b1, const float* W2,
                             const float* b2, int R, float* z, hipStream_t stream);

struct SelectArgs {
    const float* z;            // [T]
    int T;
    int mode;                  // 0 ratio, 1 threshold
    int k;                     // ratio mode: number of tokens to execute
    float z_thr;               // threshold mode
    const int32_t* seq_offsets;  // [B+1]
    int B;
    int32_t* idx;              // [T] out
    int32_t* count;            // [1] out
    int32_t* cu_exec;          // [B+1] out (nullable)
    int32_t* row_seq;          // [T] out: sequence of each executed row (nullable)
    int32_t* kv_len;           // [B] in/out (nullable): advanced by the executed count of each sequence
    int32_t* kv_old;           // [B] out (nullable unless kv_len given): kv_len before the call
    int kv_cap;                // capacity of the cache behind kv_len (0 = unknown): kv_len is not advanced beyond it
    int32_t* idx_copy;         // nullable: second destination for idx (caller-visible output)
    int32_t* inv;              // nullable (small-call kernel only): [T] compact row of token t, -1 when bypassed
    int32_t* count_copy;       // nullable
};
hipError_t launch_select(const SelectArgs& a, hipStream_t stream);

// Decode-sized calls: selection / compaction and gather + RMSNorm 1 in one launch, reading the scores z [T] a router
// kernel has written; same outputs as launch_select + launch_gather_rmsnorm.  Only valid when
// fused_select_norm_fits(T, max_rows); max_rows > 0 is the host bound on executed rows.
bool fused_select_norm_fits(int T, int max_rows);
hipError_t launch_select_norm(const void* x, int bf16, int H, const float* z, const void* gain, float eps, void* out_f16,
                              const SelectArgs& s, const RowAux& aux, int max_rows, hipStream_t stream);

// Decode-sized stacks: the last kernel of layer l (sum of the down-proj's K parts + residual + scatter, Eq. 1 and 3) also
// scores every token for layer l + 1 (Eq. 2, linear router; the same fp64 summation order as launch_router_score, on the
// values just stored).  inv [T] is the token -> compact row map of select_norm (-1 = bypassed: the row is only scored).
hipError_t launch_reduce_scatter_score(const float* part, int n_parts, int part_rows, const float* h, int H, const int32_t* inv,
                                       int T, void* x, int bf16, const float* w_next, float b_next, float* z_next,
                                       hipStream_t stream);

// Threshold calibration: bins[b] (kThetaGrid + 1 counters, cleared here) = number of scores that reach exactly
// b of the kThetaGrid ascending thresholds zthr_dev (device array).
constexpr int kThetaGrid = 50;
hipError_t launch_threshold_bins(const float* scores, long n, const float* zthr_dev, unsigned long long* bins,
                                 hipStream_t stream);

// ---- row operations ---------------------------------------------------------------------------
// n1[i] = fp16(rmsnorm(x[idx[i]]) * gain) for i < *count
hipError_t launch_gather_rmsnorm(const void* x, int bf16, int H, const int32_t* idx, const int32_t* count,
                                 int max_rows, const void* gain, float eps, void* out_f16, const RowAux& aux,
                                 hipStream_t stream);
// n2[i] = fp16(rmsnorm(h[i]) * gain), h fp32
hipError_t launch_rmsnorm_f32(const float* h, int H, const int32_t* count, int max_rows, const void* gain,
                              int gain_bf16, float eps, void* out_f16, hipStream_t stream);

// Work list of the prefill attention kernel, built by one workgroup of the launch before it (launch_rope_append): one item per
// (sequence, tile of kAttnBQ executed rows), {sequence or -1, query tile, first compact row, rows}, longest first.  The keys of
// an item may be cut into ranges (attention_prefill_plan).
struct AttnList {
    const int32_t* cu_exec;    // [B+1]; null: no list is wanted
    int B;
    void* items;               // [items_max] x int4, 16-byte aligned
    int items_max;             // host bound on the number of items
    int levels;                // host bound on the query tiles of a sequence
    const int32_t* kv_old;     // [B] cached keys of each sequence (null without a cache)
    int cap;
    int heads, target;         // query heads, workgroups that run at once
    int n_split;               // bound on the key ranges of an item; 1: not cut, the rest is unused
    int32_t* tiles;            // out: key tiles per range
    int32_t* arrive;           // [items_max x heads] counters to clear
};

struct RopeArgs {
    void* qkv;                 // [rows][(nh+2nkv)*d] fp16, q and k rotated in place
    int nh, nkv, d;
    float base;
    const int32_t* idx;        // compact row -> token
    const int32_t* positions;  // [T]
    const int32_t* count;
    int max_rows;
    // optional cache append
    void* k_cache; void* v_cache; int cap;
    const int32_t* row_seq; const int32_t* cu_exec; const int32_t* kv_old;
    AttnList list;             // cu_exec null: attention needs no list
};
hipError_t launch_rope_append(const RopeArgs& a, hipStream_t stream);

// Consumers of the decode GEMM's partial tiles (part = fp32 [n_parts][max_rows][H], added in part order):
//   h[i] = x[idx[i]] + sum(part[.][i]);  n2[i] = fp16(rmsnorm(h[i]) * gain)          (after the o-proj)
hipError_t launch_reduce_rmsnorm(const float* part, int n_parts, const void* x, int bf16, const int32_t* idx, int H,
                                 const int32_t* count, int max_rows, const void* gain, float eps, float* h,
                                 void* out_f16, hipStream_t stream);
//   x[idx[i]] = act(h[i] + sum(part[.][i]))                                           (after the down-proj)
hipError_t launch_reduce_scatter(const float* part, int n_parts, const float* h, int H, const int32_t* idx,
                                 const int32_t* count, int max_rows, void* x, int bf16, hipStream_t stream);

// ---- W4A16 / W3A16 GEMM ---------------------------------------------------------------------------------
enum GemmEpilogue { EPI_STORE_F16 = 0, EPI_RESID_F32 = 1, EPI_SWIGLU_F16 = 2, EPI_RESID_SCATTER = 3,
                    EPI_PARTIAL_F32 = 4 };   // fp32 partial tiles [parts][M_max][ldo]: decode and wide kernels

struct GemmWeights {
    const void* prepacked;
    int N, K;
};

struct GemmArgs {
    const void* A;             // [M][K] fp16
    const int32_t* count;      // device row count (nullable: use M_max)
    int M_max;                 // host upper bound of rows
    int rows_exact;            // nonzero: the row count equals M_max (ratio mode); zero: M_max is a bound, the count is read on the device
    int K;
    int group;
    int bits;                  // 4, 3 or 2
    int streams;               // nonzero: more weights than the memory-side cache holds are read before these are again
    int n_w;                   // number of weight matrices: 1, 2 (gate/up interleaved), 3 (q|k|v concatenated)
    GemmWeights w[3];
    int epilogue;
    void* out;                 // STORE/SWIGLU: fp16 [M][ldo]; RESID_F32: fp32 [M][ldo]; RESID_SCATTER: act dtype x [T][ldo]
    int ldo;
    const void* resid;         // RESID_F32: x (act dtype, rows via idx); RESID_SCATTER: h fp32 [M][ldo]
    const int32_t* idx;        // compact row -> token row (RESID_F32 reads, RESID_SCATTER writes)
    int bf16;                  // act dtype of x
    // Calls below the tiled kernel's range with a RESID_* epilogue: when `part` is given the GEMM may cut K across
    // workgroups and write fp32 partial tiles [*n_parts][M_max][ldo] there INSTEAD of applying its epilogue; the
    // caller then runs the consumer that adds the parts (launch_reduce_rmsnorm / launch_reduce_scatter).
    float* part;               // nullable
    size_t part_floats;        // its size: at most part_floats / (M_max x ldo) parts are written
    int* n_parts;              // host out, required with `part`: 0 = epilogue applied as usual, else parts written
    const struct FewPrologue* pro;   // nullable: A is made by the kernel itself (only where few_prologue_fits)
};
constexpr int kGemmPartRows = 64;      // rows of the small-row kernels, and of the workspace's own part buffer
constexpr int kGemmWideRows = 256;
constexpr int kGemmPartMax = 4;

// A handful of rows: the GEMM can make its own activations (launch_gemm_w4a16 with `pro`).
constexpr int kFewRows = 16;           // rows up to which gemm_few_kernel is used
constexpr int kFewFuseT = 4;           // tokens of a call up to which it selects and normalises them itself
constexpr int kFewPasses = 2;          // 8-column pieces of a row per thread of a 512-thread workgroup
struct FewPrologue {
    // h != null: A = RMSNorm(h rows) * gain (launch_rmsnorm_f32).  Else: router score, decision, gather and RMSNorm of x
    // (launch_router_score + launch_select_norm), with everything those write.
    const float* h;
    const void* x;
    const float* router_w;     // null: the scores are in s.z already
    float router_b;
    float* z_out;              // scores go here when router_w is given
    const void* gain;
    float eps;
    int bf16;                  // dtype of x and gain
    SelectArgs s;
    RowAux aux;
};
bool few_prologue_fits(int T, int max_rows, int hidden);
hipError_t launch_gemm_w4a16(const GemmArgs& a, hipStream_t stream);

// ---- attention over executed tokens ---------------------------------------------------------------
struct AttnArgs {
    const void* qkv;           // [rows][(nh+2nkv)*d] fp16 (q rotated, k rotated, v)
    void* out;                 // [rows][nh*d] fp16
    int nh, nkv, d;
    const int32_t* count;
    int max_rows;              // host bound on executed rows
    int B;
    const int32_t* cu_exec;    // [B+1]
    const int32_t* row_seq;    // [rows]
    // cache (nullable): when given, keys/values are read from the cache only (launch_rope_append has appended the new
    // rows; calls with `cs` append them here)
    void* k_cache; void* v_cache; int cap;
    const int32_t* kv_old;     // [B]
    int T;                     // tokens in the call
    const AttnList* list;      // prefill: what launch_rope_append has built
    bool decode;               // attention_is_decode: one workgroup per (row, kv head)
    // of those, the calls that attention_rotates names: q and k of the new rows arrive unrotated, the kernel rotates them
    // with this table (RowAux) and appends the new keys and values to the cache.  Else null, launch_rope_append came before.
    const float2* cs;
    const int32_t* chunk;      // decode, nullable: keys per range (RowAux, only with cs); else every row is cut into equally many ranges
    int32_t* arrive;           // decode, nullable: max_rows x nkv zeroed counters (RowAux); without them keys are not split
    float* partials;           // scratch (nullable) of the key ranges.  Decode: min(max_rows, kAttnSplitRows) x nh x kAttnSplitMax x
                               // (d + 2) fp32; prefill: attention_prefill_floats() per range
};
constexpr int kAttnBQ = 128;   // executed rows per prefill-attention workgroup
// Prefill: items_max, levels, heads, target and n_split of the list for a call of at most max_rows executed rows in B sequences
// whose longest has at most max_keys keys; `floats` is the scratch that the partial sums may take (attention_prefill_floats per
// range).  Keys are cut where the (query tile, head) pairs are fewer than half of the workgroups that run at once, into ranges of
// at least kAttnTileRange tiles of 64 keys: a range's sums are 34 or 68 KB that go past the L2 and back.  Layers, us, not cut / cut
// into ranges that fill the chip: 100 rows on 2000 keys, 32 heads of 128 197 / 155, of 64 109 / 84; 300 rows on 3000 keys 322 /
// 263; 2 x 560 rows on 1400 keys, heads of 64 (320 pairs for 768 slots) 280 / 258; but 1200 rows on 1000 keys, heads of 128 (320
// for 512) 722 / 732, heads of 64 (512 for 768) 307 / 311; ranges of at least 4, 8 and 12 tiles: 1000 rows of the 7B shape (8
// tiles at most) 317, 315, 316, 100 rows on 2000 keys 155, 157, 162, without a bound the former loses 14.
AttnList attention_prefill_plan(int max_rows, int B, int nh, int d, int max_keys, size_t floats);
size_t attention_prefill_floats(int items_max, int nh, int d);
constexpr int kAttnTileRange = 8;
constexpr int kAttnTileSplitMax = 16;   // key ranges per item
constexpr int kAttnSplitRows = 128;   // decode attention splits the keys only up to this many rows
constexpr int kAttnSplitMax = 8;      // and into at most this many ranges
constexpr int kAttnGqaStep = 128;     // grouped queries: keys per step of a workgroup, its ranges are multiples of it
bool attention_is_decode(bool cache, int T, int B, int nh, int nkv);
// Decode-style calls whose attention kernel also rotates and appends.  (The rows' table lies in the buffer of the residual: head_dim
// must not exceed hidden.)  The kernel rotates a sequence's new keys again for each of its rows, so a long new part beside many
// single tokens costs more than the launch that it saves.  T - B bounds the longest new part if no sequence is empty, T if most
// are (idle slots of a fixed batch).  Layers on 1000 cached
// keys, us, rotating inside / before: 7B shape 4 x 4 tokens 85.6 / 88.8, 31 x 1 + 65 242.4 / 242.5, 31 x 1 + 97 278 / 273,
// 63 x 1 + 190 536 / 502, 127 x 1 + 385 1056 / 920; 8B-GQA 32 x 2 141 / 145, 31 x 1 + 97 204 / 206, 63 x 1 + 190 346 / 340.
// One sequence of 140 / 200 / 256 / 350 tokens beside empty ones, 300 cached keys: 32 heads of 64 (rep 1) 98.6 / 87.2, 122.5 / 97.8, 149 /
// 110, 227 / 157 (before the fusion 99.8, 113, 128, 177); grouped heads (rep 2 to 8) lose at most 4 to 13 % to the separate launch and
// were slower before the fusion, so there the pure decode calls decide, which gain 1 to 5 % from it (rep 1, 200 tokens: 2 %).
constexpr int kAttnFuseNew = 96;
constexpr int kAttnFuseTokens = 160;   // one query head per kv head
bool attention_rotates(int T, int B, int rep, int hidden, int head_dim);
// Key ranges per (row, kv head) of a decode-style call (1 = not split).  device_chunk: the ranges' length is set on the device
// (RowAux::chunk) and the result is the bound on their number; target (nullable): workgroups that run at once.
int attention_splits(int max_rows, int nh, int nkv, int cap, bool device_chunk, int* target);
hipError_t launch_attention(const AttnArgs& a, hipStream_t stream);

}  // namespace qtale

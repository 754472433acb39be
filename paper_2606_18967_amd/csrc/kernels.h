// kernels.h -- launcher prototypes shared by the engine and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// Activation element types fed to the GEMMs.
enum act_t : int { ACT_F32 = 0, ACT_BF16 = 1, ACT_F16 = 2 };

inline size_t act_bytes(act_t a) { return a == ACT_F32 ? 4 : 2; }

// Row geometry of one forward call: B sequences with n new tokens each; row
// r = b*n + i sits at absolute position kv_len[slots[b]] + off + i.  A ragged
// prefill packs the rows of its sequences instead: sequence b has lim[b] <= n
// rows, from row0[b] on, and *live rows in all; its launches are sized for B*n
// rows, and what lies past *live is skipped.
struct rows_t {
    int B, n, off;
    const int32_t* slots;   // device [B]
    const int32_t* kv_len;  // device [max_slots]
    int max_slots, max_ctx;
    uint32_t* err;          // device error words
    const int32_t* lim = nullptr;   // device [B], row0 [B] and live [1], or NULL (no packing)
    const int32_t* row0 = nullptr;
    const int32_t* live = nullptr;
};

// KV cache geometry.  The element offset of (slot, layer, KV head h,
// position p) is page * PS + layer * LS + h * HS + (p % P) * head_dim, with
//   dense cache [L][max_slots][n_kv][max_ctx][head_dim]: P = max_ctx and
//     page = slot;
//   paged cache, pages [n_pages][L][n_kv][P][head_dim]: page =
//     bt[slot * mpp + p / P] from the caller's block table (an entry outside
//     [0, n_pages) is reported as ERR_PAGE and its positions are skipped).
struct kv_geom {
    int P;                     // positions per page
    long long PS, LS, HS;      // element strides of a page, a layer and a KV head
    const int32_t* bt;         // device int32 [max_slots][mpp], or NULL for the dense cache
    int mpp, n_pages;
};

struct cache_t {
    void* k;
    void* v;
    int kv_f32;             // 1: fp32 cache, 0: bf16 cache
    int n_kv, head_dim;
    kv_geom g;
};

// How one forward's attention divides the cached context among work-groups,
// made on the device from the sequences' actual lengths by the forward's first
// kernel (launch_embed_rmsnorm) and read by every layer's attention: items of
// about equal length, whole sequences that do not all fit at once longest first.
// An item is a chunk [p0, p1) of one sequence's positions [0, ctx), ctx = basepos
// + nlive clipped to max_ctx; nch is the sequence's number of chunks (they are
// consecutive items), 0 in items past the last.  A sequence without a usable slot
// or position is one empty item.  Its rows are row0 .. row0 + nlive - 1.
struct att_item { int row0, slot, basepos, ctx, p0, p1, nch, nlive; };
struct att_plan {
    int2* seq;             // device [B]: first item and number of items of each sequence (unless whole)
    att_item* item;        // device [max_items]
    int target, min_chunk; // items wanted (where there are fewer sequences), shortest chunk (a multiple of 32)
    int max_items;         // grid size: max(target, B), fewer where max_ctx allows no more
    bool whole;            // every sequence is one item: no combine
    bool in_order;         // and the items are in the sequences' order
    bool kv_first;         // the new K/V rows are stored by a launch before the attention (bf16 cache)
    int mq, zs;            // 16-row query tiles per work-group, query-row slices
};
// the launch geometry of B sequences x n rows (no device pointers)
att_plan attention_plan(int B, int n, int n_q, int n_kv, int max_ctx, int kv_f32);
size_t attention_plan_bytes(int max_slots, int n_kv);
void attention_plan_bind(att_plan& p, void* buf, int max_slots);

// ---- model kernels (kernels_model.hip)
// A kernel input produced by a split-K projection is given as partials P with
// S > 1 splits ([S][rows][cols], summed on read); S <= 1 means the producer
// wrote its output directly.
void launch_embed_rmsnorm(const rows_t& r, const int32_t* tokA, int sA, const int32_t* tokB, int sB,
                          const void* E, int w_f32, int H, int V, float* h, const void* gain, float eps,
                          void* out, act_t out_t, const att_plan& plan, hipStream_t s);
// (live as rows_t::live)
void launch_add_rmsnorm(float* h, const float* P, int S, int R, int H, const void* gain, int g_f32,
                        float eps, void* out, act_t out_t, const int32_t* live, hipStream_t s);
// q_out NULL: the K/V rows alone
void launch_rope_kv(const rows_t& r, const float* qkv, const float* P, int S, const float2* rope, int n_q,
                    const cache_t& c, int layer, float* q_out, hipStream_t s);
// Attention in two launches: each item's softmax-weighted sums (the output
// itself where a sequence is one item), then the combine over the items of a
// sequence, which a plan with whole set does without.
// The QKV projection's output as k_rope_kv reads it (qkv, or S > 1 split-K
// partials P) with the RoPE table.  The attention applies RoPE and writes the
// new rows: with a bf16 cache the attention kernel itself rotates its query
// rows and writes its KV head's new K (rotated) and V rows of its context
// range before reading them, unless k_rope_kv has stored them (att_plan::kv_first);
// with an fp32 cache k_rope_kv runs first, writing the rotated queries into q
// (scratch, [rows][n_q][head_dim] fp32).
struct qkv_src {
    const float* qkv;
    const float* P;
    int S;
    const float2* rope;
};
// ev0/ev1, when given, are bound to the attention kernel's own dispatch
// (hipExtLaunchKernelGGL): their elapsed time is the kernel's run time.
void launch_attention(const rows_t& r, const att_plan& plan, qkv_src qs, float* q, int n_q, const cache_t& c, int layer,
                      float* part, void* out, act_t out_t, hipStream_t s, hipEvent_t ev0 = nullptr,
                      hipEvent_t ev1 = nullptr);
void launch_attention_combine(const rows_t& r, const att_plan& plan, int n_q, int n_kv, int head_dim, const float* part,
                              void* out, act_t out_t, hipStream_t s);
// partial-result floats for any forward of up to R rows
size_t attention_part_floats(int R, int n_q, int n_kv, int head_dim, int kv_f32);
void launch_silu_mul(const float* gu, const float* P, int S, int R, int F, void* out, act_t out_t, const int32_t* live,
                     hipStream_t s);
void launch_kv_advance(int B, const int32_t* slots, const int32_t* inc, int inc_const,
                       int32_t* kv_len, int max_slots, uint32_t* err, hipStream_t s);
// One round of a ragged prefill: lim[b] = clamp(len[b] - t0, 0, nc), row0 their
// prefix sums, live their sum; a length outside [0, ld] sets ERR_LEN and counts
// as 0
void launch_prefill_lim(int B, const int32_t* len, int t0, int nc, int ld, int32_t* lim, int32_t* row0, int32_t* live,
                        uint32_t* err, hipStream_t s);
void launch_kv_poison(int B, const int32_t* slots, const int32_t* kv_len, int span,
                      const cache_t& c, int n_layers, int max_slots, int max_ctx, hipStream_t s);

// ---- GEMMs (kernels_gemm.hip): C[M][N] (fp32, row stride ldc) = or += A[M][K] W^T
enum gemm_mode : int { GEMM_STORE = 0, GEMM_ADD = 1 };
// bf16 MFMA GEMM: DMA-fed tiles where N is a multiple of 128, a weight-streaming
// kernel at other multiples of 64.  part is split-K scratch of part_cap floats
// (no split when too small).  Returns the number of K splits S used.  With
// defer_reduce and S > 1 the partials are left in part ([S][M][N]) for the
// consumer to sum; otherwise C holds the result.  lds_dma = false puts the
// register-staged kernel in the place of the 320-row tiles (same sums).  live (device): row tiles past *live are
// skipped (rows_t).
int launch_gemm_bf16(const uint16_t* A, const uint16_t* W, float* C, float* part, size_t part_cap, int M, int N, int K,
                     int ldc, gemm_mode mode, bool defer_reduce, hipStream_t s, bool lds_dma = true,
                     const int32_t* live = nullptr);
// The gate/up projection with SwiGLU in its epilogue: out[M][F] (type out_t)
// = SiLU(g) * u, [g | u] = A W^T with W [2F][K] (gate rows, then up rows).
// Returns 1 when launched, 0 when the shape has no fused kernel (the caller
// then runs the plain GEMM and launch_silu_mul).  part_cap: the scratch that
// the plain GEMM would have, by which it splits or not.  The int4 form takes the
// packed drafter layout of kernels_q4.hip.
int launch_gemm_bf16_swiglu(const uint16_t* A, const uint16_t* W, void* out, act_t out_t, int M, int F, int K,
                            size_t part_cap, hipStream_t s, bool lds_dma = true, const int32_t* live = nullptr);
int launch_gemm_q4_swiglu(const uint16_t* A, const uint32_t* Wq, const uint16_t* Sc, const uint8_t* Z, int fmt,
                          void* out, act_t out_t, int M, int F, int K, hipStream_t s);
size_t gemm_part_floats(int M, int N, int K);
// ---- drafter weight formats: RTN over groups of 128 weights along K, one
// fp16 scale per (column, group); int4 symmetric (codes stored as q + 8),
// int4 asymmetric (codes q in 0..15 plus a zero point z per (column,
// group), w = s (q - z)) and int8 symmetric (codes stored as q + 128).
enum qfmt : int { QF_W4 = 0, QF_W4A = 1, QF_W8 = 2 };
// bytes of the packed codes of an [N][K] matrix
inline size_t qfmt_code_bytes(int fmt, int N, int K) { return (size_t)N * K / (fmt == QF_W8 ? 1 : 2); }

// ---- quantized drafter GEMM (kernels_q4.hip): C[M][N] (+)= A[M][K] Wq^T,
// A fp16, Wq in the packed 32-column tile layout of format fmt, Z the zero
// points (QF_W4A only), N % 32 == 0.  Returns the number of K splits S
// (partials left in part as [S][M][N] when S > 1, for the consumer to sum),
// or -1 for an unsupported shape or a too small part.
int launch_gemm_q4(const uint16_t* A, const uint32_t* Wq, const uint16_t* Sc, const uint8_t* Z, int fmt, float* C,
                   float* part, size_t part_cap, int M, int N, int K, int ldc, gemm_mode mode, hipStream_t s);
size_t gemm_q4_part_floats(int M, int N, int K);
// 1 if the quantized GEMM supports reduction length K.
int gemm_q4_k_ok(int K);
void launch_gemm_f32(const float* A, const float* W, float* C, int M, int N, int K, int ldc,
                     gemm_mode mode, hipStream_t s);
void launch_gemm_q4_f32(const float* A, const uint32_t* Wq, const uint16_t* Sc, const uint8_t* Z, int fmt, float* C,
                        int M, int N, int K, int ldc, gemm_mode mode, hipStream_t s);

// ---- RTN quantizer (kernels_quant.hip): W [N][K] (fp32 or bf16) into the
// packed layout of format fmt, scales Sc and (QF_W4A) zero points Z
void launch_quant(int fmt, const void* W, int w_f32, int N, int K, uint32_t* Wq, uint16_t* Sc, uint8_t* Z,
                  hipStream_t s);

// ---- sampling and acceptance (kernels_sample.hip)
struct rng_t { uint64_t seed, step; };
enum { STREAM_TOKEN = 0, STREAM_ACCEPT = 1, STREAM_RESIDUAL = 2 };
int sample_chunks(int V);
size_t sample_part_floats(int rows, int V);
// Draws one token per row b of logits (row stride ld) with the TOKEN stream at
// position kv_len[slots[b]] + pos_off.  Writes tok[b*tok_stride] and, if
// stats != null, stats[b*stats_stride + {0,1}] = (max, lse) of logits/T.
void launch_sample(const rows_t& r, const float* logits, long ld, int V, float T, rng_t rng,
                   int pos_off, int32_t* tok, int tok_stride, float* stats, int stats_stride,
                   float* part, hipStream_t s);
void launch_accept(const rows_t& r, int gamma, int V, float T, rng_t rng, const int32_t* draft,
                   const float* q_logits, const float* q_stats, const float* p_logits,
                   int32_t* out_tok, int32_t* n_emit, int32_t* next_tok, float* part,
                   float* work, hipStream_t s);
size_t accept_work_floats(int B, int gamma);
size_t accept_part_floats(int B, int gamma, int V);

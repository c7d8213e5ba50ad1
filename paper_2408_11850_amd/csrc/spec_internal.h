// Internal declarations shared by the kernel files and the host runtime (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/spec.h"

typedef __hip_bfloat16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
// four bf16 of a borrowed tensor (embedding, norm gains), which may start at any element; one 8-byte load all the same
typedef __attribute__((ext_vector_type(4), aligned(2))) unsigned short bf16x4u;
__device__ __forceinline__ float bf16x4_at(bf16x4u v, int i) { return __uint_as_float((unsigned)v[i] << 16); }

// over the lanes c, c + 16, c + 32, c + 48: swaps of 16 and 32 lanes between registers, no trip through LDS
__device__ __forceinline__ float groups_max(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float groups_sum(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

#define SPEC_PAGE_TOKENS 64      // tokens per KV page
#define SPEC_RING_MAX 64         // most slots of the draft-token / q-row ring
// Compute units of the device the library runs on: 256 (MI355X) until spec_init has asked the device.
int spec_num_cu();
void spec_set_num_cu(int n);
#define SPEC_PEARL_WGS_PER_CU 1   // projection workgroups per CU and stream while draft and target overlap

// ---------------------------------------------------------------------------------------
// Projection (skinny GEMM) plan: y[M][N] = x[M][K] W^T, W panel-packed.
// The K axis is cut into S slices (one per group of workgroups) and each slice into 8
// wave-slices of `spw` 32-wide steps; partial sums of slice s go to P[s][M][N] (fp32).
// ---------------------------------------------------------------------------------------
struct GemmPlan {
  int M, N, K;
  int steps;   // K rounded up to 32, divided by 32
  int NT;      // N / 16 panels
  int MT;      // 16-row tiles of x (1 or 2)
  int S;       // K slices
  int spw;     // steps per wave
  int Gs;      // workgroups per slice
  size_t partial_bytes() const { return (size_t)S * M * N * sizeof(float); }
  size_t weight_bytes() const { return (size_t)NT * steps * 1024; }
};
// wgs_per_cu: 2 = fill both workgroup slots of every CU (a stream running alone), 1 = leave one slot to
// the other stream's kernels.  The K split (S, spw) does not depend on it.
GemmPlan gemm_plan(int M, int N, int K, int wgs_per_cu = 2);
// stamp: optional device words that receive the launch's time stamps (see STAMP_WAYS)
hipError_t launch_gemm_partials(const GemmPlan& p, const bf16* x, const void* wp, float* partials, hipStream_t st,
                                int tag, unsigned long long* stamp = nullptr);

// The RMSNorm of the decode path is split in three: whoever updates the residual stream h stores x' = bf16(h * gain)
// and pieces of the rows' sums of squares; the projection runs on x' unchanged; its epilogue multiplies the sums by
// inv_m = 1 / sqrt(sum_w ssq[m][w] / d + eps) (the projection is linear in its rows and bf16 keeps the same relative
// precision at any scale).
#define SSQ_STRIDE 1024                    // floats per row of sums of squares: at most one piece per 16 columns
#define SPEC_D_MODEL_MAX (16 * SSQ_STRIDE)

// Optional time stamps of a projection launch: STAMP_WAYS pairs (workgroup b uses pair b % STAMP_WAYS, so that the
// atomics of a launch do not queue on one address: one pair cost 3.5 us per launch), stamp[2 i] = max over its workgroups
// of ~(start), stamp[2 i + 1] = max of their end, in ticks of the constant-rate wall clock; all start at 0.  The kernel's
// own duration, first workgroup in to last workgroup out, without the dispatch overhead that events around a launch
// include.
#define STAMP_WAYS 16

// ---------------------------------------------------------------------------------------
// Whole-K projection (proj.hip): the K axis inside one workgroup, the element-wise work behind it in the epilogue.
// ---------------------------------------------------------------------------------------
enum { PROJ_STORE = 0, PROJ_RESID = 1, PROJ_SWIGLU = 2 };
struct ProjPlan {
  int M, N, K;
  int steps;   // K rounded up to 32, divided by 32
  int NT;      // N / 16 panels
  int mode;    // how tokens and outputs fill the MFMA operands (see proj.hip)
  int units;   // pieces of work: panel pairs (SWIGLU), panels or half panels
  int RP;      // panels a wave streams at a time
  int G;       // workgroups
  int epi;     // PROJ_* epilogue the plan is for
  int pieces() const { return units; }   // RESID: sums of squares per row
  size_t weight_bytes() const { return (size_t)NT * steps * 1024; }
};
ProjPlan proj_plan(int M, int N, int K, int epi, int wgs_per_cu);
bool proj_whole_k(int M, int N, int K);   // whether this kernel is the faster one (else K slices, gemm.hip)
struct ProjArgs {
  const bf16* x;               // [M][K]
  const void* w;               // packed panels
  unsigned long long* stamp;   // see STAMP_WAYS
  const float* ssq;            // STORE, SWIGLU: sums of squares of the rows behind x (null: no scaling) ...
  int ssq_w;                   // ... pieces per row
  float eps;
  float* y;                    // STORE: [M][N]
  float* h;                    // RESID: residual stream [M][N], updated in place
  const bf16* gain;            // RESID: gain of the following norm [N]
  bf16* xo;                    // RESID: bf16(h * gain) [M][N];  SWIGLU: z [M][N / 2]
  float* ssq_out;              // RESID: sums of squares of h, one piece per 16 columns
  int M, N, K, steps;          // set by launch_proj ...
  int per, rem;                // ... units per workgroup; the first `rem` take one more
};
bool proj_plan_ok(const ProjPlan& p);     // whether a kernel is built for it
// prio: 0 = as any kernel, 1 = its waves issue ahead of others' on a CU, 2 = a stand-alone call (STORE only), as 0
hipError_t launch_proj(const ProjPlan& p, ProjArgs a, hipStream_t st, int prio);

// What a whole-K projection's STORE / SWIGLU epilogue does, from K slices: y = sum of the S slices * 1 / rms(row) with the
// scaling of ProjArgs (ssq, ssq_w, eps; K columns), to a.y, or bf16(silu(gate) * up) to a.xo
hipError_t launch_slices_epilogue(const float* partials, int S, int epi, const ProjArgs& a, int M, int N, int K, hipStream_t st);
// y = the sum of the K slices, n = M * N elements
hipError_t launch_reduce_partials(float* y, const float* partials, int S, size_t n, hipStream_t st);
hipError_t launch_pack_weight(void* dst, const void* src, int N, int K, int panel_start, int panel_step, hipStream_t st);
hipError_t launch_read_probe(const void* src, size_t bytes, void* out, hipStream_t st);

// ---------------------------------------------------------------------------------------
// KV cache geometry.  Pool element order: [page][layer][k|v][kv_head][page block], where a K
// block is [P/16 tiles][dh/32 steps][64 lanes][8] and a V block is [P/32 chunks][dh][32 slots]
// (both already in the operand order of the 16x16x32 MFMA).
// ---------------------------------------------------------------------------------------
struct KvGeom {
  int n_layers, n_kv_heads, head_dim;
  __host__ __device__ size_t head_block() const { return (size_t)SPEC_PAGE_TOKENS * head_dim; }
  __host__ __device__ size_t page_elems() const { return (size_t)n_layers * 2 * n_kv_heads * head_block(); }
  __host__ __device__ size_t offset(int page, int layer, int kv, int head) const {
    return (((size_t)page * n_layers + layer) * 2 + kv) * n_kv_heads * head_block() + (size_t)head * head_block();
  }
};

struct TokenSrc {           // by-value kernel argument: where each input token of a forward comes from
  int n;
  int imm[SPEC_MAX_TOKENS];   // token id, or -1 to read ring[slot]
  int slot[SPEC_MAX_TOKENS];
};
struct PageUpdate {         // by-value kernel argument: new block-table entries
  int first, count;
  int page[8];
};

// the first launch of a forward (see begin_kernel); *W_out = pieces of sums of squares per row
struct BeginArgs {
  const bf16 *embed, *gain;   // embedding matrix, gain of the first norm
  const int* ring;            // draft tokens
  float* h;                   // residual stream
  bf16* xo;
  float* ssq;
  float2* tab;
  int *len_dev, *block_table;
  int d, vocab, dh, len;
  float theta;
};
hipError_t launch_begin(const BeginArgs& a, const TokenSrc& src, const PageUpdate& pages, int* W_out, hipStream_t st);
hipError_t launch_set_int(int* dst, int value, hipStream_t st);
hipError_t launch_set_pages(int* block_table, PageUpdate u, hipStream_t st);
hipError_t launch_embed(float* h, const bf16* embed, const int* tok, int M, int d, int vocab, hipStream_t st);
// a = rmsnorm(h) * gain; S > 1: after h += the sum of the S slices P[s][M][d]
hipError_t launch_norm(float* h, const bf16* gain, bf16* a, int M, int d, float eps, hipStream_t st, const float* P = nullptr,
                       int S = 1);
// h += sum_s partials[s], a = bf16(h * gain) (not normalised), ssq[m][w] = sum of h^2 over the w-th
// piece of 1024 columns of row m (row stride SSQ_STRIDE; pieces beyond W
// are never written); returns the number of pieces W through *W_out
hipError_t launch_add_sumsq(float* h, const float* partials, int S, const bf16* gain, bf16* a, float* ssq, int M,
                            int d, int* W_out, hipStream_t st);
hipError_t launch_rope_table(float2* tab, const int* len_ptr, int M, int dh, float theta, hipStream_t st);
// y: the fused QKV projection [M][(Hq + 2 Hkv) dh] of M new tokens; tab: their [M][dh/2] (cos, sin) from launch_begin.
// Rotates q and k, appends k and v to the pages and attends over the cache and the new tokens.
hipError_t launch_attention(const float* y, const float2* tab, bf16* pool, const int* block_table, const int* len_ptr,
                            KvGeom g, int layer, int M, int Hq, int split_tokens, float* opart, float* mlpart, bf16* out,
                            hipStream_t st);
int attention_one_launch_room(int Hkv);   // most positions of room for which a decode attention is one launch
size_t attention_workspace_floats(int Hq, int Hkv, int dh, int max_seq);
// prompt-sized (matrix-core bound) kernels: epilogue 0 = store fp32, 1 = add into fp32, 2 = silu(gate)*up -> bf16
#define SPEC_PREFILL_BLOCK_MAX 4096   // most prompt tokens one dense pass takes
hipError_t launch_dense_gemm(const bf16* x, const void* wp, int M, int N, int K, int epi, float* y, bf16* z,
                             hipStream_t st, int ldz = 0);   // ldz: row stride of z, 0 = N / 2
// the tile that launch_dense_gemm takes for a shape, and with the results of an epilogue
enum { DENSE_LARGE = 0 /* 256 x 256 */, DENSE_SMALL = 1 /* 128 x 128 */, DENSE_WIDE = 2 /* 256 x 192 */, DENSE_NARROW = 3 /* 128 x 96 */ };
int dense_tile(int M, int NT, int steps);
int dense_epi_tile(int M, int NT, int steps, int epi);
// K slices of a prompt projection for launch_norm to add: how many (1: none, call launch_dense_gemm), P[S][M][N], and the floats
// that hold P for every shape
int dense_slices(int M, int N, int K);
hipError_t launch_dense_slices(const bf16* x, const void* wp, int M, int N, int K, int S, float* P, hipStream_t st);
size_t dense_slices_floats();
// fused QKV projection of a prompt block with RoPE and the paged K / V append in its epilogue
hipError_t launch_dense_qkv_rope(const bf16* x, const void* wp, int M, int K, bf16* q, bf16* pool, const int* block_table,
                                 const int* len_ptr, const float2* tab, KvGeom g, int layer, int Hq, hipStream_t st);
hipError_t launch_prefill_attention(const bf16* q, const bf16* pool, const int* block_table, const int* len_ptr,
                                    KvGeom g, int layer, int M, int Hq, bf16* out, hipStream_t st);

// sampling / acceptance
struct AcceptArgs {
  int kind;                 // SPEC_ACCEPT_*
  int n_rows;               // rows of target logits available
  int n_test;               // draft tokens to test
  int slot[SPEC_MAX_TOKENS];// ring slot of the token / q row tested against logits row i
  float r[SPEC_MAX_TOKENS];
  float u_resample;
  long long force_mask;     // < 0: none
  int guided;               // 1: row i >= 1 exists only if the drafts tested by rows 0..i-1 equal guess[0..i-1]; no bonus row
  int guess[SPEC_MAX_TOKENS];
};
struct AcceptResult {       // device -> pinned host
  int n_accepted;
  int token;                // corrected / bonus / autoregressive token, -1 if none
  int rejected;             // 1 if a rejection happened
  int off_path;             // 1 if a guided test ended at a draft that left the guessed path (no rejection)
  int ring[SPEC_RING_MAX];  // snapshot of the draft-token ring
};
hipError_t launch_sample_row(const float* logits, int V, float mult, int greedy, float u, float* q_out, int* tok_out,
                             hipStream_t st);
size_t accept_scratch_floats(int V);   // scratch of one acceptance (rows <= SPEC_MAX_TOKENS)
hipError_t launch_accept(const float* logits, int V, float mult, int greedy, const float* qcache, const int* ring,
                         const int* x_direct, AcceptArgs a, float* scratch, AcceptResult* result_dev,
                         hipStream_t st, int* out2 = nullptr);

// Which of two overlapped chains issues first for windows of gamma, SPEC_TARGET, SPEC_DRAFT or -1 (neither): the rule, and what
// the next forwards of a context launch with
int favoured_chain(const spec_model_desc& target, const spec_model_desc& draft, int gamma);
int favoured_now(const spec_ctx* c);

void spec_set_error(const char* fmt, ...);

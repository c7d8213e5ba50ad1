// Small per-token kernels around the projections (gfx950): the first launch of a forward (begin_kernel), what follows a
// projection in K slices (residual add, scaling, SiLU * mul), and embedding, RMSNorm and rotation table of a prompt block.
#include "spec_internal.h"

__global__ void set_int_kernel(int* dst, int v) { dst[0] = v; }
hipError_t launch_set_int(int* dst, int value, hipStream_t st) {
  set_int_kernel<<<1, 1, 0, st>>>(dst, value);
  return hipGetLastError();
}
__global__ void set_pages_kernel(int* bt, PageUpdate u) {
  int i = threadIdx.x;
  if (i < u.count) bt[u.first + i] = u.page[i];
}
hipError_t launch_set_pages(int* block_table, PageUpdate u, hipStream_t st) {
  set_pages_kernel<<<1, 64, 0, st>>>(block_table, u);
  return hipGetLastError();
}

// h[m][:] = float(E[tok[m]][:]); an id outside the vocabulary reads row 0 (ids are validated on the host); d % 4 == 0
__global__ void embed_kernel(float* __restrict__ h, const bf16* __restrict__ E, const int* __restrict__ tok, int d,
                             int vocab) {
  const int m = blockIdx.x;
  int t = tok[m];
  if (t < 0 || t >= vocab) t = 0;
  const bf16x4u* row = reinterpret_cast<const bf16x4u*>(E + (size_t)t * d);
  for (int i = threadIdx.x; i < d >> 2; i += blockDim.x) {
    const bf16x4u e = row[i];
    reinterpret_cast<f32x4*>(h + (size_t)m * d)[i] = f32x4{bf16x4_at(e, 0), bf16x4_at(e, 1), bf16x4_at(e, 2), bf16x4_at(e, 3)};
  }
}
hipError_t launch_embed(float* h, const bf16* embed, const int* tok, int M, int d, int vocab, hipStream_t st) {
  embed_kernel<<<M, 256, 0, st>>>(h, embed, tok, d, vocab);
  return hipGetLastError();
}

// a[m] = h[m] * rsqrt(mean(h[m]^2) + eps) * gain, for a prompt block.  One workgroup of 1024 threads per row; a thread keeps
// its (at most 4) float4 pieces of the row in registers.  Bound by HBM: the row once in, half of it out.  SLICES: first adds
// the S slices P[s][m] of a projection to the row (their sum in ascending order, then to h), which costs no launch of its own.
#define NORM_THREADS 1024
#define NORM_PIECES 4      // d_model <= 4 * 4 * 1024
static_assert(SPEC_D_MODEL_MAX <= 4 * NORM_PIECES * NORM_THREADS, "a row fits the registers of a workgroup");
template <bool SLICES>
__global__ __launch_bounds__(NORM_THREADS) void norm_kernel(float* __restrict__ h, const float* __restrict__ P, int S, int M,
                                                            const bf16* __restrict__ gain, bf16* __restrict__ a, int d, float eps) {
  __shared__ float sh[NORM_THREADS / 64];
  const int m = blockIdx.x;
  const int d4 = d >> 2;
  f32x4* hr = reinterpret_cast<f32x4*>(h + (size_t)m * d);
  f32x4 v[NORM_PIECES];
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < NORM_PIECES; ++it) {
    const int i = threadIdx.x + it * NORM_THREADS;
    v[it] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (i < d4) {
      v[it] = hr[i];
      if (SLICES) {
        const f32x4* p = reinterpret_cast<const f32x4*>(P) + (size_t)m * d4 + i;
        const size_t next = (size_t)M * d4;
        f32x4 t = p[0];
#pragma unroll 4
        for (int s = 1; s < S; ++s) t += p[s * next];
        v[it] += t;
        hr[i] = v[it];
      }
    }
    ss += v[it].x * v[it].x + v[it].y * v[it].y + v[it].z * v[it].z + v[it].w * v[it].w;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int i = 0; i < NORM_THREADS / 64; ++i) tot += sh[i];
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
  for (int it = 0; it < NORM_PIECES; ++it) {
    const int i = threadIdx.x + it * NORM_THREADS;
    if (i < d4) {
      const bf16x4u g = reinterpret_cast<const bf16x4u*>(gain)[i];
      bf16 o[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = __float2bfloat16(v[it][r] * inv * bf16x4_at(g, r));
      reinterpret_cast<uint2*>(a + (size_t)m * d)[i] = *reinterpret_cast<const uint2*>(o);
    }
  }
}
hipError_t launch_norm(float* h, const bf16* gain, bf16* a, int M, int d, float eps, hipStream_t st, const float* P, int S) {
  if ((d & 3) || d > SPEC_D_MODEL_MAX) return hipErrorInvalidValue;
  if (S > 1) norm_kernel<true><<<M, NORM_THREADS, 0, st>>>(h, P, S, M, gain, a, d, eps);
  else norm_kernel<false><<<M, NORM_THREADS, 0, st>>>(h, nullptr, 0, M, gain, a, d, eps);
  return hipGetLastError();
}

// The residual add alone, spread over d/1024 workgroups per row (one compute unit cannot pull the S slices of a
// long row fast enough): h += sum_s P[s] in ascending order, and the sum of squares of each
// 1024-column piece, plus x' = bf16(h * gain) for the next projection (whose consumers apply 1/rms).
#define ADDSQ_THREADS 256
__global__ __launch_bounds__(ADDSQ_THREADS) void add_sumsq_kernel(float* __restrict__ h, const float* __restrict__ P,
                                                                  int S, const bf16* __restrict__ gain,
                                                                  bf16* __restrict__ a, float* __restrict__ ssq, int M,
                                                                  int d, int W) {
  __shared__ float sh[ADDSQ_THREADS / 64];
  const int m = blockIdx.y, w = blockIdx.x;
  const int d4 = d >> 2;
  const int i = w * ADDSQ_THREADS + threadIdx.x;
  float ss = 0.f;
  if (i < d4) {
    f32x4* hr = reinterpret_cast<f32x4*>(h + (size_t)m * d);
    const f32x4* P4 = reinterpret_cast<const f32x4*>(P);
    f32x4 t = hr[i];
    int s = 0;
    for (; s + 4 <= S; s += 4) {
      const f32x4 p0 = P4[((size_t)(s + 0) * M + m) * d4 + i], p1 = P4[((size_t)(s + 1) * M + m) * d4 + i];
      const f32x4 p2 = P4[((size_t)(s + 2) * M + m) * d4 + i], p3 = P4[((size_t)(s + 3) * M + m) * d4 + i];
      t += p0; t += p1; t += p2; t += p3;
    }
    for (; s < S; ++s) t += P4[((size_t)s * M + m) * d4 + i];
    hr[i] = t;
    ss = t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w;
    const bf16* g = gain + (size_t)i * 4;
    bf16* dst = a + (size_t)m * d + (size_t)i * 4;
    dst[0] = __float2bfloat16(t.x * __bfloat162float(g[0]));
    dst[1] = __float2bfloat16(t.y * __bfloat162float(g[1]));
    dst[2] = __float2bfloat16(t.z * __bfloat162float(g[2]));
    dst[3] = __float2bfloat16(t.w * __bfloat162float(g[3]));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) {
    float tot = 0.f;
#pragma unroll
    for (int k = 0; k < ADDSQ_THREADS / 64; ++k) tot += sh[k];
    ssq[m * SSQ_STRIDE + w] = tot;
  }
}
hipError_t launch_add_sumsq(float* h, const float* partials, int S, const bf16* gain, bf16* a, float* ssq, int M,
                            int d, int* W_out, hipStream_t st) {
  const int W = ((d >> 2) + ADDSQ_THREADS - 1) / ADDSQ_THREADS;
  if (!partials || (d & 3) || d > SPEC_D_MODEL_MAX) return hipErrorInvalidValue;
  add_sumsq_kernel<<<dim3(W, M), ADDSQ_THREADS, 0, st>>>(h, partials, S, gain, a, ssq, M, d, W);
  *W_out = W;
  return hipGetLastError();
}

// A row's K slices added in ascending order and scaled by its 1 / rms, which every wave works out from the row's pieces: the
// epilogues of a whole-K projection for the narrow, deep matrices that run in slices.  Latency: 1024 columns per workgroup.
__global__ __launch_bounds__(256) void slices_epilogue_kernel(const float* __restrict__ P, int S, ProjArgs a, int swiglu) {
  const int m = blockIdx.y, lane = threadIdx.x & 63;
  const int i = (blockIdx.x * 256 + threadIdx.x) * 4;      // output column
  const int n = swiglu ? a.N / 2 : a.N;
  const f32x4* row = reinterpret_cast<const f32x4*>(a.ssq + (size_t)m * SSQ_STRIDE);
  float ss = 0.f;
  for (int k = lane; k * 4 < a.ssq_w; k += 64) {
    const f32x4 t = row[k];
#pragma unroll
    for (int r = 0; r < 4; ++r) ss += k * 4 + r < a.ssq_w ? t[r] : 0.f;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  const float inv = 1.0f / sqrtf(ss / (float)a.K + a.eps);
  if (i >= n) return;
  // gate and up panels of 16 columns take turns
  const int c0 = swiglu ? (i >> 4) * 32 + (i & 15) : i;
  const float* src = P + (size_t)m * a.N + c0;
  const size_t slice = (size_t)gridDim.y * a.N;
  f32x4 t = {0.f, 0.f, 0.f, 0.f}, u = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = 0; s < S; ++s) {
    t += *reinterpret_cast<const f32x4*>(src + s * slice);
    if (swiglu) u += *reinterpret_cast<const f32x4*>(src + s * slice + 16);
  }
  t *= inv;
  if (!swiglu) {
    *reinterpret_cast<f32x4*>(a.y + (size_t)m * n + i) = t;
    return;
  }
  bf16 o[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) o[r] = __float2bfloat16(t[r] / (1.0f + __expf(-t[r])) * (u[r] * inv));
  *reinterpret_cast<uint2*>(a.xo + (size_t)m * n + i) = *reinterpret_cast<const uint2*>(o);
}
hipError_t launch_slices_epilogue(const float* partials, int S, int epi, const ProjArgs& args, int M, int N, int K, hipStream_t st) {
  const bool swiglu = epi == PROJ_SWIGLU;
  if (!args.ssq || (epi != PROJ_STORE && !swiglu) || (N & (swiglu ? 31 : 15)) || args.ssq_w > SSQ_STRIDE) return hipErrorInvalidValue;
  ProjArgs a = args;
  a.M = M; a.N = N; a.K = K;
  const int n = swiglu ? N / 2 : N;
  slices_epilogue_kernel<<<dim3((n + 1023) / 1024, M), 256, 0, st>>>(partials, S, a, swiglu);
  return hipGetLastError();
}

// (cos, sin) of the rotation angle pos * theta^(-2e/dh) of pair e, in fp64, once per forward or prompt block instead of
// once per layer and head.
__device__ __forceinline__ float2 rope_angle(int pos, int e, int dh, float theta) {
  const double ang = (double)pos * pow((double)theta, -2.0 * (double)e / (double)dh);
  return make_float2((float)cos(ang), (float)sin(ang));
}
__global__ void rope_table_kernel(float2* __restrict__ tab, const int* __restrict__ len_ptr, int dh, float theta) {
  const int i = blockIdx.x, e = threadIdx.x, half = dh >> 1;
  if (e < half) tab[(size_t)i * half + e] = rope_angle(len_ptr[0] + i, e, dh, theta);
}
hipError_t launch_rope_table(float2* tab, const int* len_ptr, int M, int dh, float theta, hipStream_t st) {
  rope_table_kernel<<<M, 64, 0, st>>>(tab, len_ptr, dh, theta);
  return hipGetLastError();
}

// First launch of a forward, outside its captured part: everything the chain reads that changes from call to call comes in
// as arguments.  Workgroup (x, i): 1024 columns of token i's embedding as residual stream, x' = bf16(h * gain) of the first
// norm and the piece's sum of squares (a token outside the vocabulary reads row 0; ids are validated on the host).  The last
// x: the rotation angles of position len + i; for i = 0 also the length and the new entries of the page table.
#define BEGIN_THREADS 256
__global__ __launch_bounds__(BEGIN_THREADS) void begin_kernel(BeginArgs a, TokenSrc src, PageUpdate pages) {
  __shared__ float sh[BEGIN_THREADS / 64];
  const int i = blockIdx.y, t = threadIdx.x;
  if (blockIdx.x == gridDim.x - 1) {
    const int half = a.dh >> 1;
    if (t < half) a.tab[(size_t)i * half + t] = rope_angle(a.len + i, t, a.dh, a.theta);
    if (i == 0) {
      if (t == 0) a.len_dev[0] = a.len;
      if (t < pages.count) a.block_table[pages.first + t] = pages.page[t];
    }
    return;
  }
  int tok = src.imm[i] >= 0 ? src.imm[i] : a.ring[src.slot[i]];
  if (tok < 0 || tok >= a.vocab) tok = 0;
  const int col = (blockIdx.x * BEGIN_THREADS + t) * 4;
  float ss = 0.f;
  if (col < a.d) {
    const bf16x4u e = *reinterpret_cast<const bf16x4u*>(a.embed + (size_t)tok * a.d + col);
    const bf16x4u g = *reinterpret_cast<const bf16x4u*>(a.gain + col);
    f32x4 h;
    bf16 o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      h[r] = bf16x4_at(e, r);
      o[r] = __float2bfloat16(h[r] * bf16x4_at(g, r));
      ss += h[r] * h[r];
    }
    *reinterpret_cast<f32x4*>(a.h + (size_t)i * a.d + col) = h;
    *reinterpret_cast<uint2*>(a.xo + (size_t)i * a.d + col) = *reinterpret_cast<const uint2*>(o);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((t & 63) == 0) sh[t >> 6] = ss;
  __syncthreads();
  if (t == 0) a.ssq[(size_t)i * SSQ_STRIDE + blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}
hipError_t launch_begin(const BeginArgs& a, const TokenSrc& src, const PageUpdate& pages, int* W_out, hipStream_t st) {
  *W_out = (a.d + 4 * BEGIN_THREADS - 1) / (4 * BEGIN_THREADS);
  if (src.n < 1 || src.n > SPEC_MAX_TOKENS || (a.d & 3) || (a.dh >> 1) > BEGIN_THREADS || pages.count > 8) return hipErrorInvalidValue;
  begin_kernel<<<dim3(*W_out + 1, src.n), BEGIN_THREADS, 0, st>>>(a, src, pages);
  return hipGetLastError();
}

// Multi-token decode attention over the paged KV cache (gfx950), grouped-query, causal inside
// the block of M new tokens; rotates q and k and appends k and v to the pages on the way.
//
// The M*G query rows that share one KV head (G = query heads per KV head) form the column
// dimension of 16x16x32 MFMAs: S^T = K Q^T per 16 positions, then O^T += V^T P^T per 32
// positions.  K and V pages are stored in MFMA operand order (see KvGeom), so a wave streams a
// page with consecutive fully-coalesced 1 KiB loads and nothing is staged through LDS.  One wave
// owns one 16-row tile of queries and a set of 32-position chunks (split-KV); a second kernel
// merges the splits with their running max / sum.
//
// The new tokens never go through memory: q fragments are rotated as they are loaded from the fp32 QKV projection, and
// one wave per KV head and row tile takes the new positions as a chunk of its own, whose K / V fragments it makes from
// the projection in registers (the one of row tile 0 also stores them to the pages, last).  So the cache's chunks need no
// causal mask, nobody waits for an append, and a rotation kernel (4.4 us per layer) is gone.
//
// What bounds it is a chain of latencies: kernel start, page id, K / V, softmax, result (traced; 7B shape, M = 1, 4096
// positions: 16.0 us for 67 MB, 4.6 the merge; 70B, M = 7: 13.2 + 5.5; with a rotation kernel in front 4.9 + 14.2 + 4.6 and
// 4.9 + 11.2 + 5.4: the split kernel itself takes 2 us longer, every wave rotates its q, and 3 us per layer are saved).  Up to
// 1216 positions, with 56 KV heads and more up to 3072, one launch does it all (attn_short_kernel, attention_one_launch_room);
// beyond, a head's few CUs cannot pull the cache fast enough.
#include "spec_internal.h"

#define NEG_BIG (-1.0e30f)

// Where a forward's new tokens come from: the fused QKV projection y [M][(Hq + 2 Hkv) dh] (fp32) and the (cos, sin)
// table [M][dh / 2] of their positions.
struct AttnNew {
  const float* y;
  const float2* tab;
};

// Row `tok` (valid), head slot `head` of the QKV projection, rotated and rounded: K step j of lane group g4 holds columns
// 32 j + 8 g4 .. + 7, and a lane's columns of step j pair up with its columns of step j + dh / 64.
template <int DH>
struct AttnPair {                       // columns of K step j and of step j + dh / 64, with their angles
  f32x4 x[2][2], t[4];
  __device__ __forceinline__ void load(const AttnNew& nw, int N, bool valid, int tok, int head, int g4, int j) {
#pragma unroll
    for (int h = 0; h < 4; ++h) x[h >> 1][h & 1] = t[h] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (valid) {
      const float* src = nw.y + (size_t)tok * N + (size_t)head * DH + j * 32 + g4 * 8;
      const f32x4* ts = reinterpret_cast<const f32x4*>(nw.tab + (size_t)tok * (DH / 2) + j * 32 + g4 * 8);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        x[0][h] = reinterpret_cast<const f32x4*>(src)[h];
        x[1][h] = reinterpret_cast<const f32x4*>(src + DH / 2)[h];
        t[h * 2] = ts[h * 2];
        t[h * 2 + 1] = ts[h * 2 + 1];
      }
    }
  }
  __device__ __forceinline__ void rotate(bf16x8& lo, bf16x8& hi) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float x0 = x[0][i >> 2][i & 3], x1 = x[1][i >> 2][i & 3];
      const float cs = t[i >> 1][(i & 1) * 2], sn = t[i >> 1][(i & 1) * 2 + 1];
      lo[i] = (__bf16)(x0 * cs - x1 * sn);
      hi[i] = (__bf16)(x0 * sn + x1 * cs);
    }
  }
};
template <int DH>
__device__ __forceinline__ void attn_rotated(bf16x8 (&f)[DH / 32], const AttnNew& nw, int N, bool valid, int tok, int head, int g4) {
#pragma unroll
  for (int j = 0; j < DH / 64; ++j) {
    AttnPair<DH> p;
    p.load(nw, N, valid, tok, head, g4, j);
    p.rotate(f[j], f[j + DH / 64]);
  }
}

// One wave's 16 query rows: running maximum / sum per row and the output accumulator over DV of the head's columns.
template <int DV>
struct AttnAcc {
  f32x4 o[DV / 16];
  float m, l;
  __device__ __forceinline__ void clear() {
    m = NEG_BIG;
    l = 0.f;
#pragma unroll
    for (int dt = 0; dt < DV / 16; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
};

template <int DH>
struct AttnRows : AttnAcc<DH> {
  bf16x8 qf[DH / 32];                   // rotated q fragments
};

template <int DH, int DV>
struct AttnFresh {                      // columns of 16 new tokens as the fragments want them
  AttnPair<DH> k[DH / 64];              // lane (c, g4): columns 32 j + 8 g4 .. + 7 and their partners of position 16 t + c
  float v[4][DV / 16];                  // lane (c, g4): columns 16 dt + c (of this wave's) of positions 16 t + 4 g4 .. + 3
  __device__ __forceinline__ void load(const AttnNew& nw, const KvGeom& g, int t, int M, int Hq, int kvh, int dv0, int lane) {
    const int c = lane & 15, g4 = lane >> 4, N = (Hq + 2 * g.n_kv_heads) * DH;
#pragma unroll
    for (int j = 0; j < DH / 64; ++j) k[j].load(nw, N, true, min(t * 16 + c, M - 1), Hq + kvh, g4, j);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* src = nw.y + (size_t)min(t * 16 + g4 * 4 + e, M - 1) * N + (size_t)(Hq + g.n_kv_heads + kvh) * DH + dv0 + c;
#pragma unroll
      for (int dt = 0; dt < DV / 16; ++dt) v[e][dt] = src[dt * 16];
    }
  }
};

template <int DH, int DV>
struct AttnChunk {                      // K fragments of 32 positions, and V's of DV columns from dv0 on
  u32x4 k[2][DH / 32], v[DV / 16];
  // buffer loads: a head's block of the page behind a scalar descriptor, one offset register for all of them
  static __device__ __forceinline__ __amdgpu_buffer_rsrc_t block(const bf16* pool, int page, const KvGeom& g, int layer, int kv, int kvh) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(pool + g.offset(page, layer, kv, kvh)), 0, SPEC_PAGE_TOKENS * DH * 2, 0x00020000);
  }
  __device__ __forceinline__ void load_k(const bf16* pool, int page, const KvGeom& g, int layer, int kvh, int ch, int lane) {
    const __amdgpu_buffer_rsrc_t r = block(pool, page, g, layer, 0, kvh);
    const int half = (ch & 1) * (DH * 64);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < DH / 32; ++j) k[t][j] = __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16 + (t * (DH / 32) + j) * 1024, half, 0);
  }
  __device__ __forceinline__ void load_v(const bf16* pool, int page, const KvGeom& g, int layer, int kvh, int dv0, int ch, int lane) {
    const __amdgpu_buffer_rsrc_t r = block(pool, page, g, layer, 1, kvh);
    const int from = (ch & 1) * (DH * 64) + dv0 * 64, at = (lane & 15) * 64 + (lane >> 4) * 16;
#pragma unroll
    for (int dt = 0; dt < DV / 16; ++dt) v[dt] = __builtin_amdgcn_raw_buffer_load_b128(r, at + dt * 1024, from, 0);
  }
  __device__ __forceinline__ void load(const bf16* pool, int page, const KvGeom& g, int layer, int kvh, int dv0, int ch, int lane) {
    load_k(pool, page, g, layer, kvh, ch, lane);
    load_v(pool, page, g, layer, kvh, dv0, ch, lane);
  }
  // The new tokens as one chunk (positions beyond M hold zeros), straight from the QKV projection, k rotated.  Loads are
  // unconditional (rows beyond M read the last one); the second 16 positions are skipped as a whole where there are none.
  __device__ __forceinline__ void fresh_tile(const AttnFresh<DH, DV>& f, int t, int M, int lane) {
    const int c = lane & 15, g4 = lane >> 4;
    bf16x8 r[DH / 32];
#pragma unroll
    for (int j = 0; j < DH / 64; ++j) f.k[j].rotate(r[j], r[j + DH / 64]);
#pragma unroll
    for (int j = 0; j < DH / 32; ++j) {
      const u32x4 none = {0u, 0u, 0u, 0u};
      k[t][j] = t * 16 + c < M ? __builtin_bit_cast(u32x4, r[j]) : none;
    }
#pragma unroll
    for (int dt = 0; dt < DV / 16; ++dt) {
      bf16x8 h = __builtin_bit_cast(bf16x8, v[dt]);
#pragma unroll
      for (int e = 0; e < 4; ++e) h[t * 4 + e] = (__bf16)(t * 16 + g4 * 4 + e < M ? f.v[e][dt] : 0.f);
      v[dt] = __builtin_bit_cast(u32x4, h);
    }
  }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < DH / 32; ++j) k[t][j] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int dt = 0; dt < DV / 16; ++dt) v[dt] = u32x4{0u, 0u, 0u, 0u};
  }
  // f: tile 0's columns, requested before
  __device__ __forceinline__ void fresh(AttnFresh<DH, DV>& f, const AttnNew& nw, const KvGeom& g, int M, int Hq, int kvh, int dv0, int lane) {
    clear();
    fresh_tile(f, 0, M, lane);
    if (M > 16) {
      f.load(nw, g, 1, M, Hq, kvh, dv0, lane);
      fresh_tile(f, 1, M, lane);
    }
  }
  // appends the chunk that fresh() made to the pages of positions len .. len + M - 1 (at most two)
  __device__ __forceinline__ void append(bf16* pool, const int* block_table, const KvGeom& g, int layer, int M, int kvh,
                                         int dv0, int len, int lane) const {
    const int c = lane & 15, g4 = lane >> 4;
    const int first = len / SPEC_PAGE_TOKENS, page0 = block_table[first], page1 = block_table[(len + M - 1) / SPEC_PAGE_TOKENS];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t * 16 >= M) continue;
      const int i = t * 16 + c, pos = len + i, rr = pos % SPEC_PAGE_TOKENS;
      if (i < M && dv0 == 0) {
        u32x4* dst = reinterpret_cast<u32x4*>(pool + g.offset(pos / SPEC_PAGE_TOKENS == first ? page0 : page1, layer, 0, kvh)) +
                     (size_t)(rr >> 4) * (DH / 32) * 64 + g4 * 16 + (rr & 15);
#pragma unroll
        for (int j = 0; j < DH / 32; ++j) dst[j * 64] = k[t][j];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int iv = t * 16 + g4 * 4 + e, pv = len + iv, rv = pv % SPEC_PAGE_TOKENS, r32 = rv & 31;
        if (iv < M) {
          __bf16* dst = reinterpret_cast<__bf16*>(pool + g.offset(pv / SPEC_PAGE_TOKENS == first ? page0 : page1, layer, 1, kvh)) +
                        ((size_t)(rv >> 5) * DH + dv0 + c) * 32 + ((r32 & 15) >> 2) * 8 + (r32 >> 4) * 4 + (r32 & 3);
#pragma unroll
          for (int dt = 0; dt < DV / 16; ++dt) dst[(size_t)dt * 16 * 32] = __builtin_bit_cast(bf16x8, v[dt])[t * 4 + e];
        }
      }
    }
  }
};
static_assert(SPEC_PAGE_TOKENS == 64, "two chunks of 32 positions per page");

// scores of a chunk: s[t][i] = position pos0 + 16 t + 4 g4 + i for query row c
template <int DH, int DV, typename Q>
__device__ __forceinline__ void attn_scores(f32x4 (&s)[2], const AttnChunk<DH, DV>& kv, const Q& q) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < DH / 32; ++j)
      s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kv.k[t][j]), q(j), s[t], 0, 0, 0);
  }
}
// online softmax over the scores of a chunk whose first position is pos0; positions beyond `limit` are masked
template <int DH, int DV>
__device__ __forceinline__ void attn_values(AttnAcc<DV>& r, f32x4 (&s)[2], const AttnChunk<DH, DV>& kv, int pos0, int limit, float scale, int g4) {
  float mx = NEG_BIG;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int pos = pos0 + t * 16 + g4 * 4 + i;
      const float v = (pos <= limit) ? s[t][i] * scale : NEG_BIG;
      s[t][i] = v;
      mx = fmaxf(mx, v);
    }
  mx = groups_max(mx);
  const float m_new = fmaxf(r.m, mx);
  const float corr = __expf(r.m - m_new);
  float psum = 0.f;
  bf16x8 pf;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float p = (s[t][i] > 0.5f * NEG_BIG) ? __expf(s[t][i] - m_new) : 0.f;
      psum += p;
      pf[t * 4 + i] = (__bf16)p;
    }
  r.l = r.l * corr + psum;
  r.m = m_new;
#pragma unroll
  for (int dt = 0; dt < DV / 16; ++dt) {
    r.o[dt] *= corr;
    r.o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kv.v[dt]), pf, r.o[dt], 0, 0, 0);
  }
}
template <int DH>
__device__ __forceinline__ void attn_chunk(AttnRows<DH>& r, const AttnChunk<DH, DH>& kv, int pos0, int limit, float scale, int g4) {
  f32x4 s[2];
  attn_scores<DH, DH>(s, kv, [&](int j) { return r.qf[j]; });
  attn_values<DH, DH>(r, s, kv, pos0, limit, scale, g4);
}

// the query row of lane c of row tile `rtile` of a KV head
struct AttnRow {
  bool valid;
  int tok, head;
  __device__ __forceinline__ AttnRow(int Rr, int R, int G, int kvh) {
    valid = Rr < R;
    tok = valid ? Rr / G : 0;
    head = kvh * G + (valid ? Rr % G : 0);
  }
};

// Splits 0 .. nsplit - 2 take the cache's chunks s, s + (nsplit - 1), ..., the last split the new tokens.  A wave's first
// chunk does not depend on the length, so its page lookup and K / V loads go out at once (of a chunk beyond the length
// too: a page of the pool, all masked) and the chain is page id -> K / V -> result.
template <int DH>
__global__ __launch_bounds__(256) void attn_split_kernel(AttnNew nw, bf16* __restrict__ pool,
                                                         const int* __restrict__ block_table,
                                                         const int* __restrict__ len_ptr, KvGeom g, int layer, int M,
                                                         int Hq, int nsplit, int Rpad, float scale,
                                                         float* __restrict__ opart, float* __restrict__ mlpart) {
  const int kvh = blockIdx.y, split = blockIdx.z, S = nsplit - 1;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int Hkv = g.n_kv_heads, G = Hq / Hkv, R = M * G;
  const int rtile = blockIdx.x * (blockDim.x >> 6) + w;
  if (rtile * 16 >= R) return;
  const int c = lane & 15, g4 = lane >> 4;
  const int Rr = rtile * 16 + c;
  const AttnRow row(Rr, R, G, kvh);
  AttnRows<DH> r;
  r.clear();
  AttnChunk<DH, DH> kv[2];
  if (split == S) {
    attn_rotated<DH>(r.qf, nw, (Hq + 2 * Hkv) * DH, row.valid, row.tok, row.head, g4);
    AttnFresh<DH, DH> f;
    f.load(nw, g, 0, M, Hq, kvh, 0, lane);
    kv[0].fresh(f, nw, g, M, Hq, kvh, 0, lane);
    attn_chunk(r, kv[0], 0, row.valid ? row.tok : -1, scale, g4);
  } else {
    // two chunks in flight: while one is multiplied the loads of the next are on their way
    kv[0].load(pool, block_table[split >> 1], g, layer, kvh, 0, split, lane);
    const int len = len_ptr[0], nchunks = (len + 31) >> 5, limit = row.valid ? len - 1 : -1;
    attn_rotated<DH>(r.qf, nw, (Hq + 2 * Hkv) * DH, row.valid, row.tok, row.head, g4);
    int ch = split;
    for (; ch + S < nchunks; ch += 2 * S) {
      kv[1].load(pool, block_table[(ch + S) >> 1], g, layer, kvh, 0, ch + S, lane);
      attn_chunk(r, kv[0], ch << 5, limit, scale, g4);
      if (ch + 2 * S < nchunks) kv[0].load(pool, block_table[(ch + 2 * S) >> 1], g, layer, kvh, 0, ch + 2 * S, lane);
      attn_chunk(r, kv[1], (ch + S) << 5, limit, scale, g4);
    }
    if (ch < nchunks) attn_chunk(r, kv[0], ch << 5, limit, scale, g4);
  }
  r.l = groups_sum(r.l);
  if (row.valid) {
    const size_t at = ((size_t)kvh * Rpad + Rr) * nsplit + split;   // the splits of a query row lie side by side
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) *reinterpret_cast<f32x4*>(opart + at * DH + dt * 16 + g4 * 4) = r.o[dt];
    if (g4 == 0) {
      mlpart[at * 2] = r.m;
      mlpart[at * 2 + 1] = r.l;
    }
  }
  if (split == S && rtile == 0) kv[0].append(pool, block_table, g, layer, M, kvh, 0, len_ptr[0], lane);
}

// Short caches: one workgroup per KV head, row tile and part of the head's columns takes the whole range, wave w < 7 the chunks
// w, w + 7, .. and the eighth wave the new tokens; the waves' parts are merged through LDS, so there is no merge kernel.
//
// Latency, and what one CU pulls in (a head's 262 KB at 512 positions take it 3 us).  So
//   * a head's columns of V and of the result are dealt to up to four workgroups, which all make the scores: K is asked for
//     four times, but a CU pulls 164 KB, and the sums of a column are the same whoever makes them (the bits too);
//   * two waves rotate q for all, requested ahead of the keys, instead of every wave behind its own;
//   * K of a wave's next chunk is requested when the scores of the present one are done, V when its product is.
// A launch of 16 heads, 512 positions, M = 5 (first wave in to last one out, 0.2 us of it the stamps): 8.5 us with every wave
// rotating and one workgroup per head, 6.0 with q shared, 4.7 so; 24 layers of it (d_model 2048) 928 -> 847 us, M = 1 868 -> 801,
// 790 positions 963 -> 866, 30 positions 879 -> 804.  8 parts: 851, three chunks in flight 853, one chunk 853; 12 or 16 waves
// 854 to 863; a chunk for the eighth wave too, behind the new tokens, 36 us slower with one part.
#define SHORT_WAVES 8
#define SHORT_CHUNK_WAVES (SHORT_WAVES - 1)
#define SHORT_DEPTH 2                     // chunks of a wave in flight
template <int DH, int DV>
__global__ __launch_bounds__(SHORT_WAVES * 64, 2) void attn_short_kernel(AttnNew nw, bf16* __restrict__ pool,
                                                                      const int* __restrict__ block_table,
                                                                      const int* __restrict__ len_ptr, KvGeom g, int layer,
                                                                      int M, int Hq, float scale,
                                                                      bf16* __restrict__ out) {
  constexpr int S = SHORT_CHUNK_WAVES;
  __shared__ f32x4 osh[SHORT_WAVES][16][DV / 4 + 1];     // [row][4 columns], a row padded by 16 bytes
  __shared__ float msh[SHORT_WAVES][16], lsh[SHORT_WAVES][16];
  __shared__ bf16x8 qsh[DH / 32][64];
  const int rtile = blockIdx.x, kvh = blockIdx.y, dv0 = blockIdx.z * DV;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int c = lane & 15, g4 = lane >> 4;
  const int Hkv = g.n_kv_heads, G = Hq / Hkv, R = M * G;
  const AttnRow row(rtile * 16 + c, R, G, kvh);
  // (the empty asm in the loop keeps the fragments from being held in registers across it)
  int ql = lane;
  const auto qf = [&](int j) { return qsh[j][ql]; };
  const auto leave = [&](AttnAcc<DV>& r) {
    r.l = groups_sum(r.l);
#pragma unroll
    for (int dt = 0; dt < DV / 16; ++dt) osh[w][c][dt * 4 + g4] = r.o[dt];
    if (g4 == 0) msh[w][c] = r.m, lsh[w][c] = r.l;
    __syncthreads();
  };
  // the two roles share no registers, both pass the same two barriers
  if (w == S) {
    AttnFresh<DH, DV> f;
    f.load(nw, g, 0, M, Hq, kvh, dv0, lane);
    const int len = len_ptr[0];
    __syncthreads();
    AttnChunk<DH, DV> kv;
    kv.fresh(f, nw, g, M, Hq, kvh, dv0, lane);
    AttnAcc<DV> r;
    r.clear();
    f32x4 s[2];
    attn_scores<DH, DV>(s, kv, qf);
    attn_values<DH, DV>(r, s, kv, 0, row.valid ? row.tok : -1, scale, g4);
    leave(r);
    // the page stores come last: the other waves have read what they want of the page (masked slots of it too), and merge meanwhile
    if (rtile == 0) kv.append(pool, block_table, g, layer, M, kvh, dv0, len, lane);
  } else {
    // the first waves rotate q for all; its columns are requested ahead of the keys (a wave's loads come back in order)
    AttnPair<DH> p;
    if (w < DH / 64) p.load(nw, (Hq + 2 * Hkv) * DH, row.valid, row.tok, row.head, g4, w);
    const int len = len_ptr[0], nchunks = (len + 31) >> 5, limit = row.valid ? len - 1 : -1;
    AttnChunk<DH, DV> kv[SHORT_DEPTH];
#pragma unroll
    for (int i = 0; i < SHORT_DEPTH; ++i) {
      const int ch = w + i * S;
      if (ch < nchunks) kv[i].load(pool, block_table[ch >> 1], g, layer, kvh, dv0, ch, lane);
    }
    if (w < DH / 64) {
      bf16x8 lo, hi;
      p.rotate(lo, hi);
      qsh[w][lane] = lo;
      qsh[w + DH / 64][lane] = hi;
    }
    __syncthreads();
    AttnAcc<DV> r;
    r.clear();
    f32x4 s[2];
    for (int ch = w; ch < nchunks; ch += SHORT_DEPTH * S) {
      asm volatile("" : "+v"(ql));
#pragma unroll
      for (int i = 0; i < SHORT_DEPTH; ++i) {
        const int at = ch + i * S, next = at + SHORT_DEPTH * S;
        if (at >= nchunks) continue;             // uniform
        int page = 0;
        if (next < nchunks) page = block_table[next >> 1];
        attn_scores<DH, DV>(s, kv[i], qf);
        if (next < nchunks) kv[i].load_k(pool, page, g, layer, kvh, next, lane);
        attn_values<DH, DV>(r, s, kv[i], at << 5, limit, scale, g4);
        if (next < nchunks) kv[i].load_v(pool, page, g, layer, kvh, dv0, next, lane);
      }
    }
    leave(r);
  }
  const int rr = threadIdx.x / (DV / 4), q = threadIdx.x % (DV / 4);
  if (rr < 16) {
    const AttnRow me(rtile * 16 + rr, R, G, kvh);
    if (me.valid) {
      float m = msh[0][rr];
#pragma unroll
      for (int k = 1; k < SHORT_WAVES; ++k) m = fmaxf(m, msh[k][rr]);
      f32x4 num = {0.f, 0.f, 0.f, 0.f};
      float den = 0.f;
#pragma unroll
      for (int k = 0; k < SHORT_WAVES; ++k) {
        const float e = __expf(msh[k][rr] - m);      // a wave without a chunk holds (NEG_BIG, 0, 0)
        num += e * osh[k][rr][q];
        den += e * lsh[k][rr];
      }
      bf16 o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = __float2bfloat16(num[i] / den);
      *reinterpret_cast<uint2*>(out + ((size_t)me.tok * Hq + me.head) * DH + dv0 + q * 4) = *reinterpret_cast<const uint2*>(o);
    }
  }
}

// out[i][head][e] = sum_s w_s O_s[e] / sum_s w_s l_s,  w_s = exp(m_s - max_s m_s).
// Workgroup = (dh, 8): the eight thread rows take every eighth split and fold them into a running (max, numerator,
// denominator) triple - no pass for the maximum first, and eight splits' loads in flight per thread, so up to 64
// splits cost one memory round trip - then the eight triples are combined through LDS in a fixed order.
#define MERGE_WAYS 8
#define MERGE_UNROLL 8
__global__ __launch_bounds__(128 * MERGE_WAYS) void attn_merge_kernel(const float* __restrict__ opart,
                                                                      const float* __restrict__ mlpart,
                                                                      bf16* __restrict__ out, int M, int Hq, int Hkv,
                                                                      int dh, int nsplit, int Rpad) {
  __shared__ float sm[MERGE_WAYS], snum[MERGE_WAYS][128], sden[MERGE_WAYS];
  const int i = blockIdx.x, head = blockIdx.y, e = threadIdx.x, y = threadIdx.y;
  const int G = Hq / Hkv, kvh = head / G, Rr = i * G + head % G;
  float mrun = NEG_BIG, num = 0.f, den = 0.f;
  for (int s = y; s < nsplit; s += MERGE_UNROLL * MERGE_WAYS) {
    float ms[MERGE_UNROLL], ls[MERGE_UNROLL], os[MERGE_UNROLL];
#pragma unroll
    for (int k = 0; k < MERGE_UNROLL; ++k) {
      const int sk = s + k * MERGE_WAYS;
      const size_t row = ((size_t)kvh * Rpad + Rr) * nsplit + (sk < nsplit ? sk : s);
      const bool in = sk < nsplit;
      ms[k] = in ? mlpart[row * 2] : NEG_BIG;
      ls[k] = in ? mlpart[row * 2 + 1] : 0.f;
      os[k] = in ? opart[row * dh + e] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < MERGE_UNROLL; ++k) {
      const float mnew = fmaxf(mrun, ms[k]);
      const float c0 = __expf(mrun - mnew), c1 = __expf(ms[k] - mnew);
      num = num * c0 + c1 * os[k];
      den = den * c0 + c1 * ls[k];
      mrun = mnew;
    }
  }
  snum[y][e] = num;
  if (e == 0) sm[y] = mrun, sden[y] = den;
  __syncthreads();
  if (y == 0) {
    float mstar = sm[0];
#pragma unroll
    for (int k = 1; k < MERGE_WAYS; ++k) mstar = fmaxf(mstar, sm[k]);
    float n = 0.f, dd = 0.f;
#pragma unroll
    for (int k = 0; k < MERGE_WAYS; ++k) {
      const float c = __expf(sm[k] - mstar);    // a thread row that took no split holds (NEG_BIG, 0, 0): weight 0 or 0 * 1
      n += c * snum[k][e];
      dd += c * sden[k];
    }
    out[((size_t)i * Hq + head) * dh + e] = __float2bfloat16(n / dd);
  }
}

static int attn_nsplit(int Hkv, int nrt, int T) {
  const int nchunks = (T + 31) / 32;
  int ns = (3 * spec_num_cu() + Hkv * nrt - 1) / (Hkv * nrt);   // about three waves per compute unit ...
  if (ns > (nchunks + 1) / 2) ns = (nchunks + 1) / 2;           // ... but at least two chunks per split
  if (ns < 1) ns = 1;
  return ns + 1;                                                // and the new tokens' own
}

size_t attention_workspace_floats(int Hq, int Hkv, int dh, int max_seq) {
  const int G = Hq / Hkv;
  const int Rpad = ((SPEC_MAX_TOKENS * G + 15) / 16) * 16;
  // the split count is largest for a single query tile
  int ns_max = attn_nsplit(Hkv, 1, max_seq + SPEC_MAX_TOKENS);
  return (size_t)ns_max * Hkv * Rpad * (dh + 2);
}

// Most positions of room for which one launch takes the whole range.  It saves a launch and the parts' way through memory, about
// 5 us per layer, and loses what a head's few CUs pull in more slowly than all of them do: the more heads, the later.  Where the
// line lies depends on the heads alone, so that the rows of a window do not depend on their number.  Up to 1216 it is ahead
// wherever the context stands; from 56 heads on (224 workgroups and more with four to a head) up to 3072.  us per layer of a
// forward with small projections, split | whole range, positions in use / new tokens:
//   room for 1216, 16 heads of 128      300/1 24.6 | 21.9   1120/1 26.3 | 25.7   1120/8 29.9 | 28.5   1120/32 48.8 | 40.6
//                  64 over 8 of 128     300/1 28.5 | 25.5   1120/1 29.0 | 28.2   1120/8 38.6 | 33.0   1120/32 58.9 | 45.0
//                  8 over 1 of 64       300/1 22.9 | 20.7   1120/1 23.3 | 22.6   1120/8 26.2 | 24.9   1120/32 36.4 | 34.4
//   room for 4032, 56 heads of 128      2000/1 39.4 | 36.1  3000/1 47.2 | 46.4   3000/17 65.1 | 63.3  3940/1 53.1 | 53.4
//                  128 over 64 of 64    2000/1 34.7 | 32.5                       2000/32 60.9 | 59.8  3940/17 60.8 | 61.7
//   fewer heads:   48 of 128            1700/1 36.1 | 33.6  3000/1 41.3 | 44.1   3370/1 44.5 | 47.0
//                  52 of 128            1700/1 37.3 | 37.9                       3650/1 49.5 | 51.9
// (12 layers, 16 heads, room for 2048, us a forward: 1100/1 456.3 | 440.8, 1890/1 457.7 | 469.8.)  32 heads, where it would be
// ahead up to 1890 too (4 layers 384.8 | 381.3), stay at 1216: beside a draft model's launches its workgroups wait for whole CUs
// (7B / 1B shapes behind 1024 tokens, step 4583 | 4610 us; with 56 heads 33B / 1B level, 15560 to 16190 | 15960 to 16100).
int attention_one_launch_room(int Hkv) { return Hkv < 56 ? 1216 : 3072; }

// Workgroups that share the columns of a head, from the n that there are without: as many as find a CU each (us per layer against
// one, 700 positions; 16 heads, n = 16: two -1.3, four -2.0; 56 heads, n = 56: -0.8, -1.4; n = 112: -0.8, +2.2).  That is for a
// forward that has the GPU to itself.  Beside a draft model's launches the parts of 32 heads gain nothing (7B / 1B shapes behind 600
// tokens, windows of 4, us per step: one part 4492, four 4544, splits and their merge 4548).
static int short_parts(int n) { return 4 * n <= spec_num_cu() ? 4 : 2 * n <= spec_num_cu() ? 2 : 1; }

hipError_t launch_attention(const float* y, const float2* tab, bf16* pool, const int* block_table, const int* len_ptr,
                            KvGeom g, int layer, int M, int Hq, int split_tokens, float* opart, float* mlpart, bf16* out,
                            hipStream_t st) {
  const int Hkv = g.n_kv_heads, G = Hq / Hkv, R = M * G, dh = g.head_dim;
  const int nrt = (R + 15) / 16;
  const int Rpad = ((SPEC_MAX_TOKENS * G + 15) / 16) * 16;
  const float scale = 1.0f / sqrtf((float)dh);
  const AttnNew nw = {y, tab};
  // the kernel and the split count are chosen for the longest context, not the current one, so that the launch is replayable
  if (split_tokens <= attention_one_launch_room(Hkv)) {
    const int parts = short_parts(Hkv * nrt);
    const dim3 grid(nrt, Hkv, parts), block(SHORT_WAVES * 64);
#define SHORT_GO(DH, PARTS) \
  attn_short_kernel<DH, DH / PARTS><<<grid, block, 0, st>>>(nw, pool, block_table, len_ptr, g, layer, M, Hq, scale, out)
    if (dh == 128) {
      if (parts == 4) SHORT_GO(128, 4);
      else if (parts == 2) SHORT_GO(128, 2);
      else SHORT_GO(128, 1);
    } else {
      if (parts == 4) SHORT_GO(64, 4);
      else if (parts == 2) SHORT_GO(64, 2);
      else SHORT_GO(64, 1);
    }
#undef SHORT_GO
    return hipGetLastError();
  }
  const int nsplit = attn_nsplit(Hkv, nrt, split_tokens);
  const int wpb = nrt < 4 ? nrt : 4;
  dim3 grid((nrt + wpb - 1) / wpb, Hkv, nsplit), block(64 * wpb);
  if (dh == 128)
    attn_split_kernel<128><<<grid, block, 0, st>>>(nw, pool, block_table, len_ptr, g, layer, M, Hq, nsplit, Rpad, scale,
                                                   opart, mlpart);
  else
    attn_split_kernel<64><<<grid, block, 0, st>>>(nw, pool, block_table, len_ptr, g, layer, M, Hq, nsplit, Rpad, scale,
                                                  opart, mlpart);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  attn_merge_kernel<<<dim3(M, Hq), dim3(dh, MERGE_WAYS), 0, st>>>(opart, mlpart, out, M, Hq, Hkv, dh, nsplit, Rpad);
  return hipGetLastError();
}

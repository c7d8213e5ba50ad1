// Prompt (prefill) kernels for gfx950: the only compute-bound part of the decoding workload.
//
// A prompt of C tokens goes through every projection as one dense GEMM Y[C][N] = X[C][K] W^T, so the
// contraction has C flop per weight byte pair and belongs on the matrix cores at full tile size,
// unlike the decode-time projections (<= 32 rows, HBM-bound).  W stays in the panel-packed order the decode
// kernels stream (16 output rows x 32 k per 1 KiB block = one A operand of v_mfma_f32_16x16x32_bf16); X is
// row-major bf16, and a 16-token x 32-k block of it gathered with one 16-byte load per lane is exactly one
// B operand.
//
// Tiling: workgroup = 4 waves (one per SIMD, 512 registers each) = 256 tokens x 256 outputs; wave w owns the
// outputs 64 w .. 64 w + 63 for all 256 tokens: 4 x 16 MFMA tiles whose 256 accumulator registers fill the
// AGPR file.  Measured on this part, a CU moves about 25 bytes per clock from L2 and about 62 from LDS, so the
// tile is built to need the least of both per MFMA:
//   * every weight fragment is used by exactly one wave, which loads it straight from global memory into
//     registers three K steps ahead (no LDS traffic, no duplicate loads), through a ring of four register sets;
//   * X is needed by all four waves and goes global -> LDS once per workgroup with the LDS-direct loads of
//     gfx950 (global_load_lds_dwordx4: lane l lands at base + 16 l), whole 128-byte lines at a time (8 token
//     rows x 64 k per instruction, so L2 is asked for every line once); a wave reads each of its 16 fragments
//     back with one ds_read_b128 (free of bank conflicts).
// Per 32-wide K step that is 32 KiB from L2 and 80 KiB through LDS for 64 MFMAs per wave (1024 MFMA cycles).
//
// The inner loop is inline asm with hand-placed waits.  The compiler cannot be trusted with it: it drains every
// load in flight behind an LDS-direct load (vmcnt(0)), shuffles accumulators between register files when all
// 256 AGPRs are live, and sinks LDS reads to just before their use.  Every asm statement names the registers
// it defines or that a wait makes valid, so the compiler still sees all data flow.
#include "spec_internal.h"

#define DG_BM 256
#define DG_BN 256
#define DG_THREADS 256
// LDS ring of X: a stage holds two K steps (64 k) of the tile's tokens, 128 bytes per row, rows one after the other; the
// 16-byte chunk q of row r sits at place q ^ (r % 8).  A load takes 8 rows, 8 consecutive lanes one row's 128 bytes, so
// that the address unit sees whole lines; the XOR keeps a fragment read (16 rows, one chunk per 16 lanes) free of bank
// conflicts.  With a row per lane and 16 bytes of each (and chunk-major blocks in LDS) a 1 KiB load took the unit nearly
// twice as long: 1023 x 4096 x 11008 in 256 x 256 tiles 230 -> 212 us, 4095 x 57344 x 8192 2656 -> 2623.
#define DG_STAGES 3
#define DG_HALF_BYTES 1024
#define DG_TILE_BYTES (2 * DG_HALF_BYTES)
#define DG_STAGE_BYTES (16 * DG_TILE_BYTES)

enum { DG_EPI_STORE = 0, DG_EPI_RESID = 1, DG_EPI_SWIGLU = 2, DG_EPI_ROPE128 = 3, DG_EPI_ROPE64 = 4 };

// What the QKV epilogue needs to rotate q and k and to append k and v to the paged cache.
struct DenseRope {
  bf16* q;                    // [M][Hq][dh]
  bf16* pool;                 // KV pages
  const int* block_table;
  const int* len_ptr;         // position of token 0 of the block
  const float2* tab;          // [M][dh/2] (cos, sin) for positions len .. len + M - 1
  KvGeom g;
  int layer, Hq;
};

typedef __attribute__((address_space(3))) u32x4 dg_lds_u32x4;

// What a projection does with its sums, two panels (16 outputs each) of 16 tokens at a time:
//   STORE  Y[m][n] = sum (fp32);  RESID  Y[m][n] += sum;  SWIGLU  Z[m][f] = silu(gate) * up (bf16), the even panels gate
//   rows, the odd ones the matching up rows, N = 2F;  ROPE128 / ROPE64 (fused QKV projection, head_dim 128 / 64): rotate
//   the q and k heads, store q as bf16 and k, v into the paged cache in operand order.
// The panels of pair p: for a rotation columns e and e + dh/2 of a head, else neighbours.
template <int EPI>
__device__ __forceinline__ int dense_panel(int p, int second) {
  if (EPI == DG_EPI_ROPE128) return (p >> 2) * 8 + (p & 3) + second * 4;
  if (EPI == DG_EPI_ROPE64) return (p >> 1) * 4 + (p & 1) + second * 2;
  return p * 2 + second;
}

// x0[r] = Y[m][16 panel(p, 0) + 4 kb + r], x1[r] the same of panel(p, 1); m < M
template <int EPI>
__device__ __forceinline__ void dense_pair(f32x4 x0, f32x4 x1, int m, int p, int kb, float* __restrict__ Y, bf16* __restrict__ Z,
                                           int N, int ldz, int len, const DenseRope& ra) {
  if (EPI == DG_EPI_ROPE128 || EPI == DG_EPI_ROPE64) {
    constexpr int DH = EPI == DG_EPI_ROPE128 ? 128 : 64;
    const int Hkv = ra.g.n_kv_heads;
    const int head = p / (DH / 32);
    if (head >= ra.Hq + 2 * Hkv) return;
    const int pos = len + m;
    const int e0 = p % (DH / 32) * 16 + kb * 4;                   // column inside the head, < dh/2; x1: + dh/2
    if (head < ra.Hq + Hkv) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float2 cs = ra.tab[(size_t)m * (DH / 2) + e0 + r];
        const float y0 = x0[r] * cs.x - x1[r] * cs.y, y1 = x0[r] * cs.y + x1[r] * cs.x;
        x0[r] = y0; x1[r] = y1;
      }
    }
    bf16 o0[4], o1[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) o0[r] = __float2bfloat16(x0[r]), o1[r] = __float2bfloat16(x1[r]);
    if (head < ra.Hq) {
      bf16* dst = ra.q + ((size_t)m * ra.Hq + head) * DH + e0;
      *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(o0);
      *reinterpret_cast<uint2*>(dst + DH / 2) = *reinterpret_cast<const uint2*>(o1);
      return;
    }
    const int page = ra.block_table[pos / SPEC_PAGE_TOKENS];
    const int rr = pos % SPEC_PAGE_TOKENS;
    if (head < ra.Hq + Hkv) {       // K block: [16-token tile][dh/32 steps][64 lanes][8]
      bf16* blk = ra.pool + ra.g.offset(page, ra.layer, 0, head - ra.Hq);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int e = e0 + t * (DH / 2);
        const size_t off = ((size_t)(((rr >> 4) * (DH / 32) + (e >> 5)) * 64 + ((e & 31) >> 3) * 16 + (rr & 15))) * 8 + (e & 7);
        *reinterpret_cast<uint2*>(blk + off) = *reinterpret_cast<const uint2*>(t ? o1 : o0);
      }
    } else {                        // V block: [32-token chunk][dh][32 slots]
      bf16* blk = ra.pool + ra.g.offset(page, ra.layer, 1, head - ra.Hq - Hkv);
      const int r32 = rr & 31;
      const int slot = ((r32 & 15) >> 2) * 8 + (r32 >> 4) * 4 + (r32 & 3);
      bf16* base = blk + ((size_t)(rr >> 5) * DH + e0) * 32 + slot;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        base[(size_t)r * 32] = o0[r];
        base[(size_t)(r + DH / 2) * 32] = o1[r];
      }
    }
    return;
  }
  if (EPI == DG_EPI_SWIGLU) {
    if (p * 32 + 32 > N) return;
    bf16 out[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = __float2bfloat16(x0[q] / (1.0f + __expf(-x0[q])) * x1[q]);
    *reinterpret_cast<uint2*>(Z + (size_t)m * ldz + p * 16 + kb * 4) = *reinterpret_cast<const uint2*>(out);
    return;
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int n = (p * 2 + t) * 16 + kb * 4;
    if (n >= N) continue;
    f32x4* dst = reinterpret_cast<f32x4*>(Y + (size_t)m * N + n);
    const f32x4 v = t ? x1 : x0;
    if (EPI == DG_EPI_RESID) *dst = *dst + v;
    else *dst = v;
  }
}

// A wave's 64 outputs (group wn of them) x 16 MTN tokens from m0 on.  Rotated, tiles nt and nt + 2 pair up (with head_dim
// 128 the two waves of a head take the panels {0, 1, 4, 5} and {2, 3, 6, 7}), else nt and nt + 1.
template <int EPI, int MTN>
__device__ __forceinline__ void dense_epilogue(const f32x4 (&acc)[4][MTN], int m0, int wn, int c, int kb, float* __restrict__ Y,
                                               bf16* __restrict__ Z, int M, int N, int ldz, const DenseRope& ra) {
  constexpr bool ROPE = EPI == DG_EPI_ROPE128 || EPI == DG_EPI_ROPE64;
  const int len = ROPE ? ra.len_ptr[0] : 0;
#pragma unroll
  for (int mt = 0; mt < MTN; ++mt) {
    const int m = m0 + mt * 16 + c;
    if (m >= M) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      dense_pair<EPI>(acc[ROPE ? i : 2 * i][mt], acc[ROPE ? i + 2 : 2 * i + 1][mt], m, wn * 2 + i, kb, Y, Z, N, ldz, len, ra);
  }
}

template <int EPI>
__global__ __launch_bounds__(DG_THREADS, 1) void dense_gemm_kernel(const bf16* __restrict__ X,
                                                                   const u32x4* __restrict__ Wp,
                                                                   float* __restrict__ Y, bf16* __restrict__ Z, int M,
                                                                   int N, int K, int ldz, int NT, int steps, int TM, int cx,
                                                                   DenseRope ra) {
  extern __shared__ u32x4 lds[];          // DG_STAGES * DG_STAGE_BYTES
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // w: wave-uniform
  // Workgroups are dealt to the 8 XCDs round-robin; XCD x owns tile columns [x cx, (x+1) cx) and walks them in
  // groups of 4 columns x all row tiles, so the 32 workgroups an XCD runs together share 8 x 4 operand strips
  // in its L2.
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int TN = (NT + 15) >> 4;
  int nx = TN - x * cx;
  if (nx > cx) nx = cx;
  const int grp = j / (TM * 4), idx = j % (TM * 4);
  int gw = nx - grp * 4;          // columns in this group; its tiles are numbered row-major over them
  if (gw > 4) gw = 4;
  if (gw <= 0 || idx >= TM * gw) return;
  const int tm = idx / gw, tn = x * cx + grp * 4 + idx % gw;

  const int c = lane & 15, kb = lane >> 4;
  // Addresses are a wave-uniform base (scalar registers) plus a 32-bit per-lane offset.
  const char* wbase[4];                   // this wave's 4 weight panels (clamped rows are computed, never stored)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int panel = tn * 16 + w * 4 + i;
    if (EPI == DG_EPI_ROPE128) panel = tn * 16 + (w >> 1) * 8 + (w & 1) * 2 + (i & 1) + (i >> 1) * 4;
    if (panel > NT - 1) panel = NT - 1;
    wbase[i] = reinterpret_cast<const char*>(Wp + (size_t)panel * steps * 64);
  }
  const unsigned woff = lane * 16;
  const char* xbase = reinterpret_cast<const char*>(X);
  // X moves global -> LDS in whole 128-byte lines: one LDS-direct load covers 8 token rows x 64 k, so that L2 sees every
  // line of X once (a 16-row x 32-k load would ask for each line twice, half used).  Per stage the wave issues 8 of them: token tiles 4w .. 4w+3, rows 0-7 and 8-15 of each.
  const int xchunk = (lane & 7) ^ (lane >> 3);
  unsigned xoff[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    int m = tm * DG_BM + (w * 4 + i / 2) * 16 + (i & 1) * 8 + (lane >> 3);
    if (m > M - 1) m = M - 1;
    xoff[i] = (unsigned)m * (unsigned)K * 2u + xchunk * 16;          // < 2^32: checked by the launcher
  }
  // fragment (tile mt, step half h) of lane (c, kb): row c of tile mt, chunk 4 h + kb
  const unsigned lds_rd = (unsigned)(size_t)(dg_lds_u32x4*)lds + c * 128 + (kb ^ (c & 7)) * 16;

  f32x4 acc[4][16];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 16; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Load schedule per wave: iteration j issues 4 of the 8 LDS-direct loads of X stage j/2 + 2 (K steps 2(j/2)+4
  // and +5) and the 4 register loads of W step j+3, alternating, one after every second token tile, i.e. 8 MFMAs
  // apart: the address unit takes about 30 cycles per 1 KiB wave load, and a wave that issues loads back to back
  // sits in the issue stage (issuing no MFMAs) until the unit has taken them all.  Vector-memory operations
  // complete in order.  Steps past the end reload the last step (into a free buffer / a dead register set),
  // which keeps the count of outstanding loads uniform so that one vmcnt threshold serves every iteration.
  u32x4 wq[4][4];      // W fragments of steps j .. j+3 (set = step % 4)
  u32x4 bq[16];        // X fragments of the current step; each is refilled for the next step once consumed
  const unsigned xfix = (xchunk >> 2) * 64;   // lanes of the second K step of a stage: fall back to the first one
#define DG_LOAD_X(PG, J)   /* instruction J (0..7) of X stage PG: token tile 4w + J/2, rows 8 (J%2) .. + 7 */    \
  {                                                                                                          \
    const int st_ = 2 * (PG) < steps ? 2 * (PG) : (steps - 1) & ~1;                                          \
    const unsigned fix_ = st_ + 1 < steps ? 0u : xfix;   /* odd K-step count: never read past the row's end */ \
    __builtin_amdgcn_global_load_lds(                                                                        \
        xbase + (size_t)st_ * 64 + (xoff[J] - fix_),                                                         \
        lds + (((PG) % DG_STAGES) * DG_STAGE_BYTES + (w * 4 + (J) / 2) * DG_TILE_BYTES + ((J) & 1) * DG_HALF_BYTES) / 16, \
        16, 0, 0);                                                                                           \
  }
#define DG_LOAD_W(STEP, SET, I)                                                                              \
  {                                                                                                          \
    const int st_ = (STEP) < steps ? (STEP) : steps - 1;                                                     \
    asm volatile("global_load_dwordx4 %0, %1, %2"                                                            \
                 : "=v"(wq[SET][I]) : "v"(woff), "s"(wbase[I] + (size_t)st_ * 1024) : "memory");             \
  }
#define DG_MFMA(ACC, A, B)                                                                                   \
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(ACC) : "v"(A), "v"(B))
  // One iteration = K step KS (KS % 4 == U, so that the register sets are compile-time names).  At its top: this
  // wave's loads issued up to iteration KS-2 have landed (the 8 of iteration KS-1 may be in flight), i.e. W step
  // KS+1 and X step KS+1's stage, then the barrier: that stage is in LDS for everybody, and everybody is past
  // reading the stage this iteration's LDS-direct loads refill.  The 16 token tiles follow; fragment mt of step
  // KS was read 16 LDS reads ago (lgkmcnt(15)), feeds 4 MFMAs and is at once re-read for step KS+1, so that every
  // LDS read has 60 MFMAs to arrive.
#define DG_ITER(KS, U)                                                                                       \
  {                                                                                                          \
    asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier"                                                            \
                 : "+v"(wq[((U) + 1) % 4][0]), "+v"(wq[((U) + 1) % 4][1]), "+v"(wq[((U) + 1) % 4][2]),       \
                   "+v"(wq[((U) + 1) % 4][3])::"memory");                                                    \
    const unsigned rd_ = (lds_rd ^ (((KS) + 1) & 1) * 64) + ((((KS) + 1) >> 1) % DG_STAGES) * DG_STAGE_BYTES;  \
    _Pragma("unroll") for (int mt = 0; mt < 16; ++mt) {                                                      \
      asm volatile("s_waitcnt lgkmcnt(15)" : "+v"(bq[mt]));                                                  \
      _Pragma("unroll") for (int nt = 0; nt < 4; ++nt) DG_MFMA(acc[nt][mt], wq[U][nt], bq[mt]);              \
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(bq[mt]) : "v"(rd_), "n"(mt * DG_TILE_BYTES));      \
      if (mt % 4 == 1) DG_LOAD_X((KS) / 2 + 2, ((U) & 1) * 4 + mt / 4)                                       \
      if (mt % 4 == 3) DG_LOAD_W((KS) + 3, ((U) + 3) % 4, mt / 4)                                            \
    }                                                                                                        \
  }
  // prologue: X stages 0 and 1 (K steps 0..3) and W steps 0..2, all landed before the first iteration
#pragma unroll
  for (int j8 = 0; j8 < 8; ++j8) {
    DG_LOAD_X(0, j8)
    DG_LOAD_X(1, j8)
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    DG_LOAD_W(0, 0, i)
    DG_LOAD_W(1, 1, i)
    DG_LOAD_W(2, 2, i)
  }
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier"
               : "+v"(wq[0][0]), "+v"(wq[0][1]), "+v"(wq[0][2]), "+v"(wq[0][3]), "+v"(wq[1][0]), "+v"(wq[1][1]),
                 "+v"(wq[1][2]), "+v"(wq[1][3]), "+v"(wq[2][0]), "+v"(wq[2][1]), "+v"(wq[2][2]), "+v"(wq[2][3])::"memory");
#pragma unroll
  for (int mt = 0; mt < 16; ++mt)
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(bq[mt]) : "v"(lds_rd), "n"(mt * DG_TILE_BYTES));
  int ks = 0;
  for (; ks + 4 <= steps; ks += 4) {
    DG_ITER(ks, 0)
    DG_ITER(ks + 1, 1)
    DG_ITER(ks + 2, 2)
    DG_ITER(ks + 3, 3)
  }
  if (ks < steps) DG_ITER(ks, 0)
  if (ks + 1 < steps) DG_ITER(ks + 1, 1)
  if (ks + 2 < steps) DG_ITER(ks + 2, 2)
#undef DG_ITER
#undef DG_MFMA
#undef DG_LOAD_X
#undef DG_LOAD_W
  // The redundant tail loads must not outlive the workgroup's LDS, and the registers they (and the last LDS
  // reads) target must not be handed to anything else while they are in flight: naming them here keeps them
  // allocated until everything has landed.  The s_nops cover the distance the hardware wants between the last
  // MFMA and a read of its accumulator; the compiler does not know that the asm statements above are MFMAs and
  // would otherwise be free to read an accumulator right behind the one that wrote it, so every accumulator is
  // passed through a statement that follows the s_nops.
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15"
               : "+v"(wq[0][0]), "+v"(wq[0][1]), "+v"(wq[0][2]), "+v"(wq[0][3]), "+v"(wq[1][0]), "+v"(wq[1][1]),
                 "+v"(wq[1][2]), "+v"(wq[1][3]), "+v"(wq[2][0]), "+v"(wq[2][1]), "+v"(wq[2][2]), "+v"(wq[2][3])::"memory");
  asm volatile("" : "+v"(wq[3][0]), "+v"(wq[3][1]), "+v"(wq[3][2]), "+v"(wq[3][3]));
  asm volatile("" : "+v"(bq[0]), "+v"(bq[1]), "+v"(bq[2]), "+v"(bq[3]), "+v"(bq[4]), "+v"(bq[5]), "+v"(bq[6]),
               "+v"(bq[7]), "+v"(bq[8]), "+v"(bq[9]), "+v"(bq[10]), "+v"(bq[11]), "+v"(bq[12]), "+v"(bq[13]),
               "+v"(bq[14]), "+v"(bq[15]));
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
    asm volatile("" : "+a"(acc[nt][0]), "+a"(acc[nt][1]), "+a"(acc[nt][2]), "+a"(acc[nt][3]), "+a"(acc[nt][4]),
                 "+a"(acc[nt][5]), "+a"(acc[nt][6]), "+a"(acc[nt][7]), "+a"(acc[nt][8]), "+a"(acc[nt][9]),
                 "+a"(acc[nt][10]), "+a"(acc[nt][11]), "+a"(acc[nt][12]), "+a"(acc[nt][13]), "+a"(acc[nt][14]),
                 "+a"(acc[nt][15]));

  dense_epilogue<EPI, 16>(acc, tm * DG_BM, tn * 4 + w, c, kb, Y, Z, M, N, ldz, ra);
}

// Grids that 256 x 256 tiles do not fill.  dense_small: 128 tokens x 128 outputs per workgroup of 8 waves, a wave has
// 64 x 64 (4 x 4 MFMA tiles) of every second K step; waves w and w + 4 hold the even and the odd steps of the same outputs
// and exchange halves at the end.  Both operands go global -> LDS with LDS-direct loads, each byte once per workgroup; a
// stage is two K steps, 16 KiB of X (as in the large tile) and 16 KiB of W (lane-linear), in a ring of 4.
// Bound by what a CU pulls in: loads alone take 0.26 us per K step (61 bytes per ns and CU, the same with 3, 4 and 5 stages;
// all of it from L2 0.17), LDS and MFMAs alone 0.17, all together 0.27.  What counts is that consecutive lanes of a load of X
// take whole lines (with a row per lane, 16 bytes of each, X took 0.23 us of a K step instead of 0.13), that loads are issued
// between MFMAs and that every SIMD has a second wave: 1023 x 4096 x 11008 124 -> 100 us; 511 x 6144 x 2048 28 -> 23 from
// HBM and 26.4 -> 18 to 19 from the memory-side cache.
// PN: panels of a tile, 8 (128 outputs) or 6 (96: a wave has 32 x 96, a stage 12 KiB of W), see dense_tile, dense_epi_tile.
#define DS_WAVES 8
#define DS_THREADS (DS_WAVES * 64)
#define DS_STAGES 4
#define DS_LOADS 4                        // per wave and stage
#define DS_X_BYTES (8 * DG_TILE_BYTES)
#define DS_STAGE_BYTES(PN) (DS_X_BYTES + (PN) * 2048)
// The tile of this workgroup: XCD x takes the tiles [x chunk, (x + 1) chunk), numbered row-major inside groups of 4
// columns, so that what an XCD runs together shares operand strips in its L2.
__device__ __forceinline__ bool dense_tile_of(int TM, int TN, int chunk, int* tm, int* tn) {
  const int j = blockIdx.x >> 3, tile = (blockIdx.x & 7) * chunk + j;
  if (j >= chunk || tile >= TM * TN) return false;
  const int grp = tile / (TM * 4), idx = tile % (TM * 4), gw = min(4, TN - grp * 4);
  *tm = idx / gw;
  *tn = grp * 4 + idx % gw;
  return true;
}

template <int EPI, int PN>
__global__ __launch_bounds__(DS_THREADS, 2) void dense_small_kernel(const bf16* __restrict__ X, const u32x4* __restrict__ Wp,
                                                                    float* __restrict__ Y, bf16* __restrict__ Z, int M, int N,
                                                                    int K, int ldz, int NT, int panel_steps, int TM, int TN,
                                                                    int chunk, int slice, DenseRope ra) {
  static_assert(PN == 8 || PN == 6, "panels of a tile");
  constexpr int WN = PN == 8 ? 2 : 1, WM = 4 / WN;         // waves side by side, of the four that share a K step
  constexpr int NP = PN / WN, MT = 8 / WM;                 // a wave's panels and token tiles
  constexpr int STAGE = DS_X_BYTES + PN * 2048;
  constexpr bool ROPE = EPI == DG_EPI_ROPE128 || EPI == DG_EPI_ROPE64;
  extern __shared__ u32x4 lds[];          // DS_STAGES * STAGE
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int tm, tn;
  if (!dense_tile_of(TM, TN, chunk, &tm, &tn)) return;
  // this workgroup's slice of the K axis; the slices of a split projection leave their sums side by side
  const int step0 = blockIdx.y * slice, steps = min(slice, panel_steps - step0);
  if (EPI == DG_EPI_STORE) Y += (size_t)blockIdx.y * M * N;
  const int c = lane & 15, kb = lane >> 4;
  const int kg = w >> 2, wm = (w & 3) / WN, wn = (w & 3) % WN;
  // Per stage a wave loads token tile w (8 rows x 64 k at a time) and, of 8 panels, two K steps of panel w, of 6 the blocks w and
  // (the first four waves) w + 8 of 1 KiB; rows and panels past the end are clamped, computed and never stored.  6 panels lie
  // in the order of the pairs that the epilogue wants.
  const int loads = PN == 8 || w < 4 ? DS_LOADS : DS_LOADS - 1;
  const char* wbase[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int blk = PN == 8 ? 2 * w + i : (w + 8 * i) % 12;
    int panel = PN == 8 ? tn * 8 + w : dense_panel<EPI>(tn * 3 + (blk >> 2), (blk >> 1) & 1);
    if (panel > NT - 1) panel = NT - 1;
    wbase[i] = reinterpret_cast<const char*>(Wp + ((size_t)panel * panel_steps + step0) * 64) + lane * 16;
  }
  const char* xbase = reinterpret_cast<const char*>(X) + (size_t)step0 * 64;
  const int xchunk = (lane & 7) ^ (lane >> 3);
  unsigned xoff[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    int m = tm * 128 + (w * 2 + i) * 8 + (lane >> 3);
    if (m > M - 1) m = M - 1;
    xoff[i] = (unsigned)m * (unsigned)K * 2u + xchunk * 16;          // < 2^32: checked by the launcher
  }
  const unsigned xfix = (xchunk >> 2) * 64;   // lanes of the second K step of a stage: fall back to the first one
  const int stages = (steps + 1) >> 1;
  // load i of this wave for stage st; past the end: the last stage again, into a slot that nobody reads
  auto issue = [&](int st, int slot, int i) {
    if (st > stages - 1) st = stages - 1;
    const bool whole = st * 2 + 1 < steps;  // odd K-step count: never read past a row's or a panel's end
    if (i < 2) {
      __builtin_amdgcn_global_load_lds(xbase + (size_t)st * 128 + (xoff[i] - (whole ? 0u : xfix)),
                                       lds + (slot * STAGE + w * 2048 + i * 1024) / 16, 16, 0, 0);
    } else if (i < loads) {          // uniform
      const int blk = PN == 8 ? 2 * w + (i & 1) : w + 8 * (i & 1);
      __builtin_amdgcn_global_load_lds(wbase[i & 1] + (size_t)st * 2048 + ((blk & 1) && whole ? 1024 : 0),
                                       lds + (slot * STAGE + DS_X_BYTES + blk * 1024) / 16, 16, 0, 0);
    }
  };
  // fragment addresses inside a stage: token tiles MT wm + mt, and this wave's panels
  const unsigned lds0 = (unsigned)(size_t)(dg_lds_u32x4*)lds;
  const unsigned xrd = lds0 + wm * MT * DG_TILE_BYTES + c * 128 + ((kg * 4 + kb) ^ (c & 7)) * 16;
  const unsigned wrd = lds0 + DS_X_BYTES + wn * (PN == 8 && EPI == DG_EPI_ROPE128 ? 2 : NP) * 2048 + lane * 16 + kg * 1024;
  f32x4 acc[NP][MT];
#pragma unroll
  for (int a = 0; a < NP; ++a)
#pragma unroll
    for (int b = 0; b < MT; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 fw[2][NP], fx[2][MT];                 // fragments of this wave's current and next K step
#define DS_READ(B, SLOT)                                                                                     \
  {                                                                                                          \
    const unsigned so_ = (SLOT) * STAGE;                                                                     \
    _Pragma("unroll") for (int i = 0; i < MT; ++i)                                                           \
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fx[B][i]) : "v"(xrd + so_), "n"(i * DG_TILE_BYTES)); \
    _Pragma("unroll") for (int i = 0; i < NP; ++i)                                                           \
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fw[B][i]) : "v"(wrd + so_),                        \
                   "n"((PN == 8 && EPI == DG_EPI_ROPE128 ? (i & 1) + (i >> 1) * 4 : i) * 2048));                        \
  }
#define DS_WAIT(B)                                                                                           \
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fx[B][0]), "+v"(fx[B][1]), "+v"(fw[B][0]), "+v"(fw[B][1]),      \
               "+v"(fw[B][2]), "+v"(fw[B][3])::"memory");                                                    \
  _Pragma("unroll") for (int i = 2; i < MT; ++i) asm volatile("" : "+v"(fx[B][i]));                          \
  _Pragma("unroll") for (int i = 4; i < NP; ++i) asm volatile("" : "+v"(fw[B][i]));
// this wave's loads of all but the last N stages have landed, then everybody's
#define DS_LANDED(N)                                                                                         \
  if (PN == 8 || w < 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((N) * DS_LOADS) : "memory");                \
  else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((N) * (DS_LOADS - 1)) : "memory");                           \
  asm volatile("s_barrier" ::: "memory");
  // Stage ST: stage ST + 1 has landed for this wave, then for everybody, and everybody holds its half of stage ST in
  // registers, so that slot is refilled, one load after every fourth MFMA: no wave sits in the issue stage behind the
  // address unit while its matrix core idles.  MULTIPLY: whether this wave has a K step in the stage.
#define DS_STAGE(B, ST, MULTIPLY)                                                                            \
  {                                                                                                          \
    DS_LANDED(DS_STAGES - 2)                                                                                 \
    DS_READ(1 - (B), ((ST) + 1) % DS_STAGES)                                                                 \
    if (MULTIPLY) {                                                                                          \
      _Pragma("unroll") for (int mt = 0; mt < MT; ++mt) {                                                    \
        __builtin_amdgcn_sched_barrier(0);                                                                   \
        _Pragma("unroll") for (int nt = 0; nt < NP; ++nt)                                                    \
          acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[B][nt]),       \
                                                                __builtin_bit_cast(bf16x8, fx[B][mt]), acc[nt][mt], 0, 0, 0); \
        __builtin_amdgcn_sched_barrier(0);                                                                   \
        _Pragma("unroll") for (int i = 0; i < DS_LOADS / MT; ++i)                                            \
          issue((ST) + DS_STAGES, (ST) % DS_STAGES, mt * (DS_LOADS / MT) + i);                               \
      }                                                                                                      \
    }                                                                                                        \
    DS_WAIT(1 - (B))                                                                                         \
  }
#pragma unroll
  for (int s = 0; s < DS_STAGES; ++s)
#pragma unroll
    for (int i = 0; i < DS_LOADS; ++i) issue(s, s, i);
  DS_LANDED(DS_STAGES - 1)                  // stage 0 is in LDS for everybody
  DS_READ(0, 0)
  DS_WAIT(0)
  const bool last = kg == 0 || !(steps & 1);
  int st = 0;
  for (; st + 2 < stages; st += 2) {
    DS_STAGE(0, st, true)
    DS_STAGE(1, st + 1, true)
  }
  if (st + 1 < stages) {
    DS_STAGE(0, st, true)
    DS_STAGE(1, st + 1, last)
  } else {
    DS_STAGE(0, st, last)
  }
#undef DS_STAGE
#undef DS_READ
#undef DS_WAIT
  // The redundant tail loads must neither outlive the workgroup's LDS nor land on what is exchanged there.
  DS_LANDED(0)
#undef DS_LANDED
  // waves w and w + 4 hold the even and the odd K steps of the same outputs: each adds up and stores half of the tokens
  f32x4* ex = reinterpret_cast<f32x4*>(lds);
  constexpr int H = MT / 2;
  f32x4 sum[NP][H];
#pragma unroll
  for (int nt = 0; nt < NP; ++nt)
#pragma unroll
    for (int mt = 0; mt < H; ++mt) {
      sum[nt][mt] = kg ? acc[nt][mt + H] : acc[nt][mt];
      ex[(w * NP * H + nt * H + mt) * 64 + lane] = kg ? acc[nt][mt] : acc[nt][mt + H];
    }
  __syncthreads();
#pragma unroll
  for (int nt = 0; nt < NP; ++nt)
#pragma unroll
    for (int mt = 0; mt < H; ++mt) sum[nt][mt] += ex[((w ^ 4) * NP * H + nt * H + mt) * 64 + lane];
  const int m0 = tm * 128 + wm * MT * 16 + kg * H * 16;
  if constexpr (PN == 8) {
    dense_epilogue<EPI, H>(sum, m0, tn * 2 + wn, c, kb, Y, Z, M, N, ldz, ra);
  } else {
    const int len = ROPE ? ra.len_ptr[0] : 0, m = m0 + c;
    if (m >= M) return;
#pragma unroll
    for (int i = 0; i < NP / 2; ++i) dense_pair<EPI>(sum[2 * i][0], sum[2 * i + 1][0], m, tn * 3 + i, kb, Y, Z, N, ldz, len, ra);
  }
}

// dense_wide: 256 tokens x 192 outputs by 8 waves of 64 tokens x 6 panels, for grids that deal out more evenly so.  Operands
// and ring as in dense_small, X (from L2 or the memory-side cache: the other tile columns read it too) two stages deep, W
// (from HBM) three.  0.6 us per K step with every CU busy: 28 KiB of it 0.46 us of loads, and X has one stage to arrive.
// A third stage of it does not fit LDS beside 256 x 192, and 256 x 128 with three of both takes 0.39 us for two thirds.
#define DW_PANELS 6                        // of a wave
#define DW_X_BYTES (16 * DG_TILE_BYTES)
#define DW_W_BYTES (DW_PANELS * 4096)
template <int EPI>
__global__ __launch_bounds__(DS_THREADS, 2) void dense_wide_kernel(const bf16* __restrict__ X, const u32x4* __restrict__ Wp,
                                                                   float* __restrict__ Y, bf16* __restrict__ Z, int M, int N,
                                                                   int K, int ldz, int NT, int steps, int TM, int TN, int chunk,
                                                                   DenseRope ra) {
  constexpr int PN = DW_PANELS, XS = DW_X_BYTES, WS = DW_W_BYTES, WL = PN / 2;
  extern __shared__ u32x4 lds[];          // 2 stages of X, 3 of W
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int tm, tn;
  if (!dense_tile_of(TM, TN, chunk, &tm, &tn)) return;
  const int c = lane & 15, kb = lane >> 4, wm = w >> 1, wn = w & 1;
  const char* wbase[WL];
  unsigned xoff[4];
  const int xchunk = (lane & 7) ^ (lane >> 3);
#pragma unroll
  for (int i = 0; i < WL; ++i) {                 // load i: K step q & 1 of the tile's panel q >> 1
    const int q = w * WL + i;
    int panel = dense_panel<EPI>(tn * PN + (q >> 2), (q >> 1) & 1);
    if (panel > NT - 1) panel = NT - 1;
    wbase[i] = reinterpret_cast<const char*>(Wp + (size_t)panel * steps * 64) + lane * 16;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int m = tm * 256 + (w * 4 + i) * 8 + (lane >> 3);
    if (m > M - 1) m = M - 1;
    xoff[i] = (unsigned)m * (unsigned)K * 2u + xchunk * 16;          // < 2^32: checked by the launcher
  }
  const char* xbase = reinterpret_cast<const char*>(X);
  const unsigned xfix = (xchunk >> 2) * 64;
  const int stages = (steps + 1) >> 1;
  auto issue_x = [&](int st, int slot, int i) {
    if (st > stages - 1) st = stages - 1;
    const bool whole = st * 2 + 1 < steps;
    __builtin_amdgcn_global_load_lds(xbase + (size_t)st * 128 + (xoff[i] - (whole ? 0u : xfix)),
                                     lds + (slot * XS + (w * 4 + i) * DG_HALF_BYTES) / 16, 16, 0, 0);
  };
  auto issue_w = [&](int st, int slot, int i) {
    if (st > stages - 1) st = stages - 1;
    const bool whole = st * 2 + 1 < steps;
    const int q = w * WL + i;
    __builtin_amdgcn_global_load_lds(wbase[i] + (size_t)st * 2048 + ((q & 1) && whole ? 1024 : 0),
                                     lds + (2 * XS + slot * WS + q * 1024) / 16, 16, 0, 0);
  };
  const unsigned lds0 = (unsigned)(size_t)(dg_lds_u32x4*)lds;
  const unsigned xrd = lds0 + wm * 4 * DG_TILE_BYTES + c * 128 + (kb ^ (c & 7)) * 16;
  const unsigned wrd = lds0 + 2 * XS + wn * PN * 2048 + lane * 16;
  f32x4 acc[PN][4];
#pragma unroll
  for (int a = 0; a < PN; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 fw[2][PN], fx[2][4];
#define DW_READ(B, XSLOT, WSLOT, H)                                                                          \
  {                                                                                                          \
    const unsigned xo_ = (xrd ^ ((H) * 64)) + (XSLOT) * XS, wo_ = wrd + (WSLOT) * WS;                        \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                            \
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fx[B][i]) : "v"(xo_), "n"(i * DG_TILE_BYTES));     \
    _Pragma("unroll") for (int i = 0; i < PN; ++i)                                                           \
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fw[B][i]) : "v"(wo_), "n"(i * 2048 + (H) * 1024)); \
  }
#define DW_WAIT(B)                                                                                           \
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fx[B][0]), "+v"(fx[B][1]), "+v"(fx[B][2]), "+v"(fx[B][3])::"memory"); \
  _Pragma("unroll") for (int i = 0; i < PN; ++i) asm volatile("" : "+v"(fw[B][i]));
#define DW_MMA(B, ISSUE)                                                                                     \
  _Pragma("unroll") for (int mt = 0; mt < 4; ++mt) {                                                         \
    __builtin_amdgcn_sched_barrier(0);                                                                       \
    _Pragma("unroll") for (int nt = 0; nt < PN; ++nt)                                                        \
      acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[B][nt]),           \
                                                            __builtin_bit_cast(bf16x8, fx[B][mt]), acc[nt][mt], 0, 0, 0); \
    __builtin_amdgcn_sched_barrier(0);                                                                       \
    ISSUE;                                                                                                   \
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) issue_x(0, 0, i);
#pragma unroll
  for (int i = 0; i < WL; ++i) issue_w(0, 0, i), issue_w(1, 1, i);
#pragma unroll
  for (int i = 0; i < 4; ++i) issue_x(1, 1, i);
#pragma unroll
  for (int i = 0; i < WL; ++i) issue_w(2, 2, i);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(4 + WL) : "memory");        // stage 0 is in LDS for everybody
  DW_READ(0, 0, 0, 0)
  DW_WAIT(0)
  const int pairs = steps >> 1;
  int wc = 0;                                      // W slot of stage st
  for (int st = 0; st < pairs; ++st) {
    const int wnx = wc == 2 ? 0 : wc + 1, wpv = wc == 0 ? 2 : wc - 1, xc = st & 1;
    DW_READ(1, xc, wc, 1)
    // W of stage st + 2 into the slot of stage st - 1 (the first time: the same bytes again)
    DW_MMA(0, if (mt < WL) issue_w(st + 2, wpv, mt))
    DW_WAIT(1)
    // Stage st + 1 has landed for this wave (W of st + 2 may be in flight), then for everybody; everybody holds what it
    // needs of stage st in registers, so X of st + 2 may take its place.
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(WL) : "memory");
    DW_READ(0, xc ^ 1, wnx, 0)
    DW_MMA(1, if (mt < 2) { issue_x(st + 2, xc, 2 * mt); issue_x(st + 2, xc, 2 * mt + 1); })
    DW_WAIT(0)
    wc = wnx;
  }
  if (steps & 1) {
    DW_MMA(0, )
  }
#undef DW_READ
#undef DW_WAIT
#undef DW_MMA
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the redundant tail loads must not outlive the workgroup's LDS
  constexpr bool ROPE = EPI == DG_EPI_ROPE128 || EPI == DG_EPI_ROPE64;
  const int len = ROPE ? ra.len_ptr[0] : 0;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    const int m = tm * 256 + wm * 64 + mt * 16 + c;
    if (m >= M) continue;
#pragma unroll
    for (int i = 0; i < PN / 2; ++i)
      dense_pair<EPI>(acc[2 * i][mt], acc[2 * i + 1][mt], m, tn * PN + wn * (PN / 2) + i, kb, Y, Z, N, ldz, len, ra);
  }
}

// Tile by the time a launch takes (us): rounds of one workgroup per CU, each a fixed part and a time per K step that grows
// with the share of CUs in use, fitted to these (large | small | wide; the launch itself, about 6, is in all of them):
//   66 x 4096 x 4096        76 |  32 |  63     1023 x 4096 x 11008   213 | 101 | 171     2047 x 4096 x 11008   217 | 185 | 178
//   511 x 6144 x 2048       49 |  23 |  40     1023 x 12288 x 4096    91 | 117 |  88     2500 x 6144 x 2048     56 |  79 |  80
//   511 x 22016 x 4096      88 | 111 |  84     1023 x 22016 x 4096   173 | 211 | 159     4095 x 8192 x 8192    430 | 540 | 476
//   1500 x 3072 x 2048      49 |  35 |  41     1023 x 8192 x 8192    166 | 149 | 137     4095 x 57344 x 8192  2634 | 3470 | 2945
// Of 34 shapes measured it takes the fastest in 30, else one at most 6 % (once 16 %) behind and ahead of what it replaces.
// The fit is low where a full row tile meets few CUs: 128 x 4096 x 11008, 32 tiles of 128 x 128, 0.28 us per K step (fit 0.196).
// Large and wide tiles add K as one chain per output, the same bits; 128 x 128 tiles and slices (below) group it otherwise, so
// the last bits of a prompt's K and V depend on its length, as they do between the dense pass and forwards over 32 tokens.
int dense_tile(int M, int NT, int steps) {
  static const struct { int tokens, panels; float round, step, busy; } T[3] = {
      {256, 16, 4.f, 0.50f, 0.23f}, {128, 8, 2.f, 0.185f, 0.085f}, {256, 12, 2.f, 0.405f, 0.205f}};
  const int ncu = spec_num_cu();
  int best = 0;
  float best_us = 0.f;
  for (int i = 0; i < 3; ++i) {
    const int tiles = (M + T[i].tokens - 1) / T[i].tokens * ((NT + T[i].panels - 1) / T[i].panels), rounds = (tiles + ncu - 1) / ncu;
    const float us = rounds * (T[i].round + steps * (T[i].step + T[i].busy * tiles / ((float)rounds * ncu)));
    if (i == 0 || us < best_us) best = i, best_us = us;
  }
  // 128 x 96 where one round of them fills three quarters of the CUs or more and 128 x 128 would be taken (the same round with
  // fewer, larger tiles): what a CU pulls in per K step falls by an eighth, what all of them pull in together rises by a sixth.  So
  // it gains while each CU waits for its own loads, and loses where the level they share is the limit.  Not below 16 K steps,
  // where it is all launch.
  //   us, 128 x 128 | 128 x 96, bf16 results, W from HBM:
  //     256 tiles: 511 x 6144 x 2048  21.1 | 19.9   511 x 6144 x 4096  38.9 | 34.1   255 x 12288 x 4096 40.7 | 36.5
  //                1023 x 3072 x 2048 20.2 | 19.1   1023 x 3072 x 4096 37.0 | 32.4   400 x 6144 x 2048  18.1 | 18.0
  //     224, 192:  511 x 5376 x 2048  20.6 | 19.1   511 x 5376 x 4096  38.8 | 33.2   511 x 4608 x 2048  20.4 | 19.0
  //   a single W in the memory-side cache: 511 x 6144 x 2048 16.8 | 17.1   511 x 6144 x 4096 28.9 | 28.3   255 x 12288 x 4096 28.7 | 29.6
  //   two rounds of them gain nothing (fp32): 511 x 11264 x 2048 37.0 | 38.4     2047 x 3072 x 2048 38.8 | 39.0
  // The sums are those of 128 x 128 tiles, bit for bit.
  const int narrow = (M + 127) / 128 * ((NT + 5) / 6);
  if (best == DENSE_SMALL && steps >= 16 && narrow <= ncu && 4 * narrow >= 3 * ncu) best = DENSE_NARROW;
  return best;
}

// With fp32 results 128 x 96 stays out: their stores go to the shared level too, and with operands from the memory-side cache it
// falls behind (three sets of operands in turn, 128 x 128 | 128 x 96):
//   fp32: 511 x 6144 x 2048 (256 tiles) 20.22 | 20.47   511 x 6144 x 4096 32.55 | 32.78   1023 x 2688 x 4096 (224) 30.84 | 31.34
//   bf16: 511 x 6144 x 2048             18.44 | 18.42   511 x 6144 x 4096 31.31 | 31.16   1023 x 2688 x 4096       29.82 | 29.86
// Prompt passes with them for QKV and gate/up: small pair, 511 tokens through 24 layers 2984 | 2924 us, 7B shape, 255 through 4
// 653 | 639, 1B draft, 255 through 22 1894 | 1857; weights in that cache (small, 2 layers) 189 | 187.
int dense_epi_tile(int M, int NT, int steps, int epi) {
  const int t = dense_tile(M, NT, steps);
  return t == DENSE_NARROW && (epi == DG_EPI_STORE || epi == DG_EPI_RESID) ? (int)DENSE_SMALL : t;
}

template <typename F>
static hipError_t dense_lds(F* kernel, int bytes, bool* set) {      // more than the default dynamic LDS
  if (*set) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  *set = e == hipSuccess;
  return e;
}

template <int EPI>
static hipError_t dense_launch_epi(const bf16* x, const u32x4* w, int M, int N, int K, float* y, bf16* z, int ldz,
                                   const DenseRope& ra, hipStream_t st) {
  static bool set[4] = {};
  const int NT = N / 16, steps = K / 32, tile = dense_epi_tile(M, NT, steps, EPI);
  hipError_t e;
  if (tile == DENSE_LARGE) {
    constexpr int lds_bytes = DG_STAGES * DG_STAGE_BYTES;
    if ((e = dense_lds(dense_gemm_kernel<EPI>, lds_bytes, &set[0])) != hipSuccess) return e;
    const int TM = (M + DG_BM - 1) / DG_BM, TN = (NT + 15) / 16;
    const int cx = (TN + 7) / 8, groups = (cx + 3) / 4;
    dense_gemm_kernel<EPI><<<8 * groups * TM * 4, DG_THREADS, lds_bytes, st>>>(x, w, y, z, M, N, K, ldz, NT, steps, TM, cx, ra);
  } else if (tile == DENSE_SMALL) {
    constexpr int lds_bytes = DS_STAGES * DS_STAGE_BYTES(8);
    if ((e = dense_lds(dense_small_kernel<EPI, 8>, lds_bytes, &set[1])) != hipSuccess) return e;
    const int TM = (M + 127) / 128, TN = (NT + 7) / 8, chunk = (TM * TN + 7) / 8;
    dense_small_kernel<EPI, 8><<<8 * chunk, DS_THREADS, lds_bytes, st>>>(x, w, y, z, M, N, K, ldz, NT, steps, TM, TN, chunk, steps, ra);
  } else if (tile == DENSE_NARROW) {
    if constexpr (EPI != DG_EPI_STORE && EPI != DG_EPI_RESID) {
      constexpr int lds_bytes = DS_STAGES * DS_STAGE_BYTES(6);
      if ((e = dense_lds(dense_small_kernel<EPI, 6>, lds_bytes, &set[3])) != hipSuccess) return e;
      const int TM = (M + 127) / 128, TN = (NT + 5) / 6, chunk = (TM * TN + 7) / 8;
      dense_small_kernel<EPI, 6><<<8 * chunk, DS_THREADS, lds_bytes, st>>>(x, w, y, z, M, N, K, ldz, NT, steps, TM, TN, chunk, steps, ra);
    }
  } else {
    constexpr int lds_bytes = 2 * DW_X_BYTES + 3 * DW_W_BYTES;
    if ((e = dense_lds(dense_wide_kernel<EPI>, lds_bytes, &set[2])) != hipSuccess) return e;
    const int TM = (M + 255) / 256, TN = (NT + 2 * DW_PANELS - 1) / (2 * DW_PANELS), chunk = (TM * TN + 7) / 8;
    dense_wide_kernel<EPI><<<8 * chunk, DS_THREADS, lds_bytes, st>>>(x, w, y, z, M, N, K, ldz, NT, steps, TM, TN, chunk, ra);
  }
  return hipGetLastError();
}

// K slices of a prompt projection whose consumer (launch_norm) adds them, 1 = none: where 128 x 128 tiles leave at least half of
// the CUs idle.  A slice's time falls with its length; the sums cost their way through memory, about 3 MB per us and a few us
// (measured, us, whole | in slices, with what the norm behind them takes longer: 128 x 4096 x 11008 101 | 30, 511 x 2048 x 5504
// 50 | 23, 128 x 4096 x 4096 35 | 17; a prompt of 100 tokens through four layers of 4096 x 11008 1411 | 976 with the last layer's
// dead part gone).  time() is the fit of dense_tile, low for whole launches on few CUs, and 0.85 asks for a clear gain on top:
// what is cut gains, some of what is left whole would.
#define DENSE_SLICES_MAX 16
int dense_slices(int M, int N, int K) {
  const int ncu = spec_num_cu(), steps = K / 32, tiles = (M + 127) / 128 * ((N + 127) / 128);
  if (2 * tiles > ncu || dense_epi_tile(M, N / 16, steps, DG_EPI_RESID) != DENSE_SMALL) return 1;
  auto time = [&](int S, int slice) { return slice * (0.185f + 0.085f * S * tiles / ncu) + (S > 1 ? 3.f + S * (float)M * N * 4.f / 3e6f : 0.f); };
  int best = 1;
  float best_us = 0.85f * time(1, steps);
  for (int S = 2; S <= DENSE_SLICES_MAX && S * tiles <= ncu; ++S) {
    const int slice = ((steps + S - 1) / S + 1) & ~1;
    if (slice < 4 || (steps + slice - 1) / slice != S) continue;
    if (time(S, slice) < best_us) best = S, best_us = time(S, slice);
  }
  return best;
}
size_t dense_slices_floats() { return (size_t)spec_num_cu() * 128 * 128; }

// P[s][m][n] = slice s of X W^T, S = dense_slices(M, N, K) > 1 of them
hipError_t launch_dense_slices(const bf16* x, const void* wp, int M, int N, int K, int S, float* P, hipStream_t st) {
  if ((double)M * K * 2.0 >= 4294967296.0 || S < 2) return hipErrorInvalidValue;
  constexpr int lds_bytes = DS_STAGES * DS_STAGE_BYTES(8);
  static bool set = false;
  hipError_t e = dense_lds(dense_small_kernel<DG_EPI_STORE, 8>, lds_bytes, &set);
  if (e != hipSuccess) return e;
  const int NT = N / 16, steps = K / 32, slice = ((steps + S - 1) / S + 1) & ~1;      // whole stages
  if ((steps + slice - 1) / slice != S) return hipErrorInvalidValue;
  const int TM = (M + 127) / 128, TN = (NT + 7) / 8, chunk = (TM * TN + 7) / 8;
  dense_small_kernel<DG_EPI_STORE, 8><<<dim3(8 * chunk, S), DS_THREADS, lds_bytes, st>>>(x, (const u32x4*)wp, P, nullptr, M, N, K, 0, NT,
                                                                                      steps, TM, TN, chunk, slice, DenseRope{});
  return hipGetLastError();
}

static hipError_t dense_gemm_launch(const bf16* x, const void* wp, int M, int N, int K, int epi, float* y, bf16* z,
                                    int ldz, const DenseRope& ra, hipStream_t st) {
  if ((double)M * K * 2.0 >= 4294967296.0) return hipErrorInvalidValue;   // per-lane activation offsets are 32-bit
  const u32x4* w4 = (const u32x4*)wp;
  switch (epi) {
    case DG_EPI_STORE: return dense_launch_epi<DG_EPI_STORE>(x, w4, M, N, K, y, z, ldz, ra, st);
    case DG_EPI_RESID: return dense_launch_epi<DG_EPI_RESID>(x, w4, M, N, K, y, z, ldz, ra, st);
    case DG_EPI_SWIGLU: return dense_launch_epi<DG_EPI_SWIGLU>(x, w4, M, N, K, y, z, ldz, ra, st);
    case DG_EPI_ROPE128: return dense_launch_epi<DG_EPI_ROPE128>(x, w4, M, N, K, y, z, ldz, ra, st);
    default: return dense_launch_epi<DG_EPI_ROPE64>(x, w4, M, N, K, y, z, ldz, ra, st);
  }
}

hipError_t launch_dense_gemm(const bf16* x, const void* wp, int M, int N, int K, int epi, float* y, bf16* z,
                             hipStream_t st, int ldz) {
  DenseRope none = {};
  return dense_gemm_launch(x, wp, M, N, K, epi, y, z, ldz ? ldz : N / 2, none, st);
}

// The fused QKV projection of a prompt block: q (rotated, bf16) to `q`, k (rotated) and v into the pages of
// positions len .. len + M - 1.  `tab` from launch_rope_table for the same block.
hipError_t launch_dense_qkv_rope(const bf16* x, const void* wp, int M, int K, bf16* q, bf16* pool, const int* block_table,
                                 const int* len_ptr, const float2* tab, KvGeom g, int layer, int Hq, hipStream_t st) {
  DenseRope ra = {q, pool, block_table, len_ptr, tab, g, layer, Hq};
  const int N = (Hq + 2 * g.n_kv_heads) * g.head_dim;
  return dense_gemm_launch(x, wp, M, N, K, g.head_dim == 128 ? DG_EPI_ROPE128 : DG_EPI_ROPE64, nullptr, nullptr, 0, ra, st);
}

// ---------------------------------------------------------------------------------------------------------
// Causal attention of a block of M prompt tokens over the paged KV cache (positions 0 .. len + M - 1, the
// block's own K / V already appended).  Rows are the M*G (token, query head) pairs of one KV head, token-major,
// as in the decode kernel; a workgroup of 8 waves owns 128 consecutive rows, a wave one tile of 16, and two
// workgroups share a CU, so that four waves per SIMD cover each other's softmax arithmetic and waits.  K and V pages
// are in MFMA operand order, so every 64-position chunk (= one page) is 32 KiB (head_dim 128) that the workgroup brings
// into LDS once with LDS-direct loads and each wave reads as ready-made fragments: S^T = K Q^T, online softmax
// per query row in the base-2 domain, O^T += V^T P^T.  Chunks beyond the last position a workgroup's rows may
// see are never touched (causal skip), and the workgroups with the longest ranges are scheduled first.
//
// The vector ALU bounds it, about 1900 cycles of it per chunk of two tiles beside 1024 of MFMAs: so only chunks on the
// diagonal are masked, the scale goes into the exponent's fma, and the accumulator is rescaled where a maximum moved
// (traced, two tiles per wave: 64 heads over 8, 4095 tokens 499 -> 442 us; 32 heads, 1023 tokens 37.6 -> 34.0).  Waves
// of one tile instead of two, twice as many of them on a CU: 442 -> 377 and 34.0 -> 31.6; 16 heads, 511 tokens 16.4 ->
// 15.0, 1500 tokens 40.6 -> 35.7; 32 heads over 4 of head_dim 64, 4000 tokens 158 -> 130.
// ---------------------------------------------------------------------------------------------------------
#define PA_WAVES 8                               // one 16-row tile each
#define PA_ROWS (PA_WAVES * 16)
#define PA_STAGES 2
#define PA_NEG_BIG (-1.0e30f)

// Brings chunk `ch` (64 positions = page block_table[ch]) of one KV head into an LDS stage.  Block b of a chunk:
// b < KB -> K block b (lane-linear in the page), else V block b - KB, whose lane (c, g4) sits at byte
// c*64 + g4*16 of the block.
template <int DH>
__device__ __forceinline__ void pa_issue(const bf16* __restrict__ pool, const int* __restrict__ block_table,
                                         const KvGeom& g, int layer, int kvh, int ch, u32x4* lds_stage, int w,
                                         int lane) {
  constexpr int KB = 4 * (DH / 32), VB = 2 * (DH / 16), LPW = (KB + VB) / PA_WAVES;
  const int c = lane & 15, g4 = lane >> 4;
  const int page = block_table[ch];
  const u32x4* kblk = reinterpret_cast<const u32x4*>(pool + g.offset(page, layer, 0, kvh)) + lane;
  const bf16* vblk = pool + g.offset(page, layer, 1, kvh);
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int b = w * LPW + i;
    const void* src = (b < KB) ? (const void*)(kblk + (size_t)b * 64)
                               : (const void*)(vblk + ((size_t)((b - KB) * 16 + c) * 32 + g4 * 8));
    __builtin_amdgcn_global_load_lds(src, lds_stage + b * 64, 16, 0, 0);
  }
}

template <int DH>
__global__ __launch_bounds__(PA_WAVES * 64, 4) void prefill_attn_kernel(const bf16* __restrict__ q,
                                                                        const bf16* __restrict__ pool,
                                                                        const int* __restrict__ block_table,
                                                                        const int* __restrict__ len_ptr, KvGeom g,
                                                                        int layer, int M, int Hq, float scale_log2e,
                                                                        bf16* __restrict__ out) {
  constexpr int KS = DH / 32;                    // K steps per 16-position tile
  constexpr int KB = 4 * KS;                     // K blocks (1 KiB) per chunk
  constexpr int VB = 2 * (DH / 16);              // V blocks per chunk
  constexpr int NB = KB + VB;
  __shared__ u32x4 lds[PA_STAGES][NB][64];
  const int kvh = blockIdx.y;
  const int rb = gridDim.x - 1 - blockIdx.x;     // longest ranges first
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int c = lane & 15, g4 = lane >> 4;
  const int Hkv = g.n_kv_heads, G = Hq / Hkv, R = M * G;
  const int len = len_ptr[0];
  const int r0 = rb * PA_ROWS;
  int rlast = r0 + PA_ROWS - 1;
  if (rlast > R - 1) rlast = R - 1;
  const int nch = ((len + rlast / G) >> 6) + 1;  // chunks this workgroup needs
  int wlast = r0 + (w + 1) * 16 - 1;
  if (wlast > R - 1) wlast = R - 1;
  const int wave_limit = (r0 + w * 16 < R) ? len + wlast / G : -1;
  const int wave_open = len + (r0 + w * 16) / G;     // positions up to here are visible to all of the wave's rows

  // row of this lane, its visibility limit and its Q fragments.  Rows past the end behave like
  // unmasked rows of zeros (finite arithmetic, never stored).
  const int Rr = r0 + w * 16 + c;
  const bool valid = Rr < R;
  const int tok = valid ? Rr / G : 0;
  const int head = kvh * G + (valid ? Rr % G : 0);
  const int limit = valid ? len + tok : 0x7fffffff;
  bf16x8 qf[KS];
#pragma unroll
  for (int j = 0; j < KS; ++j) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (valid) v = *reinterpret_cast<const u32x4*>(q + ((size_t)tok * Hq + head) * DH + j * 32 + g4 * 8);
    qf[j] = __builtin_bit_cast(bf16x8, v);
  }

  float m_run = PA_NEG_BIG, l_run = 0.f;        // running max (base-2 domain) and sum of the query row
  f32x4 o[DH / 16];
#pragma unroll
  for (int dt = 0; dt < DH / 16; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};

  pa_issue<DH>(pool, block_table, g, layer, kvh, 0, &lds[0][0][0], w, lane);
  for (int ch = 0; ch < nch; ++ch) {
    // chunk ch has landed for this wave, then for everybody; all waves are done with the other stage
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    pa_issue<DH>(pool, block_table, g, layer, kvh, ch + 1 < nch ? ch + 1 : nch - 1, &lds[(ch + 1) % PA_STAGES][0][0], w,
                 lane);
    const int pos0 = ch << 6;
    if (pos0 > wave_limit) continue;           // nothing visible for this wave's rows (uniform per wave)
    const u32x4(*st)[64] = lds[ch % PA_STAGES];

    // scores of the 64 positions: s[t4][r] = position pos0 + 16 t4 + 4 g4 + r for query row c
    f32x4 s[4];
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) {
      s[t4] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < KS; ++j)
        s[t4] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, st[t4 * KS + j][lane]), qf[j], s[t4], 0, 0, 0);
    }
    if (pos0 + 63 > wave_open) {                // uniform per wave: chunks on the diagonal only
#pragma unroll
      for (int t4 = 0; t4 < 4; ++t4)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[t4][r] = pos0 + t4 * 16 + g4 * 4 + r <= limit ? s[t4][r] : PA_NEG_BIG;
    }
    float mx = PA_NEG_BIG;
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[t4][r]);
    // position 0 is visible to every row, so after the first chunk the running max is a real score and a
    // masked entry (-1e30) underflows to exactly 0
    const float m_new = fmaxf(m_run, groups_max(mx) * scale_log2e);
    const float corr = __builtin_amdgcn_exp2f(m_run - m_new);
    float psum = 0.f;
    bf16x8 pf[2];                               // P fragments of the two 32-position halves
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pv = __builtin_amdgcn_exp2f(fmaf(s[t4][r], scale_log2e, -m_new));
        psum += pv;
        pf[t4 >> 1][(t4 & 1) * 4 + r] = (__bf16)pv;
      }
    l_run = l_run * corr + psum;
    m_run = m_new;
    if (!__all(corr == 1.0f)) {                 // maxima settle after a few chunks
#pragma unroll
      for (int dt = 0; dt < DH / 16; ++dt) o[dt] *= corr;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int dt = 0; dt < DH / 16; ++dt)
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, st[KB + h * (DH / 16) + dt][lane]), pf[h], o[dt], 0, 0, 0);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the redundant tail loads must not outlive the workgroup's LDS

  const float inv = 1.0f / groups_sum(l_run);
  if (!valid) return;
  bf16* dst = out + ((size_t)tok * Hq + head) * DH + g4 * 4;
#pragma unroll
  for (int dt = 0; dt < DH / 16; ++dt) {
    bf16 v4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v4[r] = __float2bfloat16(o[dt][r] * inv);
    *reinterpret_cast<uint2*>(dst + dt * 16) = *reinterpret_cast<const uint2*>(v4);
  }
}

hipError_t launch_prefill_attention(const bf16* q, const bf16* pool, const int* block_table, const int* len_ptr,
                                    KvGeom g, int layer, int M, int Hq, bf16* out, hipStream_t st) {
  const int Hkv = g.n_kv_heads, G = Hq / Hkv, R = M * G, dh = g.head_dim;
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)dh);
  const dim3 grid((R + PA_ROWS - 1) / PA_ROWS, Hkv), block(PA_WAVES * 64);
  if (dh == 128) prefill_attn_kernel<128><<<grid, block, 0, st>>>(q, pool, block_table, len_ptr, g, layer, M, Hq, scale_log2e, out);
  else prefill_attn_kernel<64><<<grid, block, 0, st>>>(q, pool, block_table, len_ptr, g, layer, M, Hq, scale_log2e, out);
  return hipGetLastError();
}

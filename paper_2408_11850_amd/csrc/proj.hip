// Whole-K projection kernels for gfx950: y[M][N] = x[M][K] W^T with M <= 32 new tokens, the K axis inside one
// workgroup, so that whatever follows the projection element by element happens in its epilogue.
//
// Every weight is read once per forward, so the kernel is bound by HBM and by what each launch costs besides the
// stream: ramp, tail, and the kernels that would have to add K slices afterwards.  A workgroup of 8 waves owns a
// contiguous range of panels (16 outputs x K, packed in MFMA operand order, see gemm.hip); the K steps of a panel are
// dealt evenly to the 8 waves, a wave takes RP panels at a time and streams weights and activations through a ring of
// D register stages (one K step of RP panels each).  All ring loads are buffer loads whose range check turns "past the
// end" (steps, panels, rows, ragged K) into zeros without memory traffic: they are unconditional, so the compiler
// counts them exactly and a stage waits for its own loads only (behind branches it waits for everything in flight).
// The ring runs on across panel groups.  Per group the 8 wave sums are added through LDS in a fixed order: the sums
// depend on the shape only, not on the number of workgroups or on timing.
//
// What counts next to HBM is the address unit: a 1 KiB wave load takes it 16 cycles whether its lanes count or not, so
// loads of x are packed (PAIR, HALF below) and a load that would bring nothing is not issued where it can be helped.
// Measured against K slices plus the kernel that adds them (us, weights from HBM, back to back in a graph):
//   2048 x 2048, M = 5     6.5 -> 4.1     8192 x 28672, M = 7   76.9 -> 71.5 (6.6 TB/s; a long plain read: 6.7)
//   2048 x 5632, M = 5     8.7 -> 6.3     57344 x 8192, M = 7  149.8 -> 141.2    M = 17  205.8 -> 150.8
//   4096 x 11008, M = 1   19.9 -> 16.3    38400 x 7168, M = 17 106.1 -> 96.1
//
// Epilogues: STORE  y = sum * 1/rms(row);  RESID  h += sum, x' = bf16(h * gain) for the next projection and the
// sums of squares of every 16 columns of h;  SWIGLU  z = bf16(silu(gate) * up) of interleaved gate / up panels.
#include <cstring>

#include "spec_internal.h"

#define PROJ_WAVES 8
#define PROJ_THREADS (PROJ_WAVES * 64)
#define PROJ_NT 2                     // cache policy of the weight stream: non-temporal
#define PROJ_SKIP 0x7f000000u         // an offset beyond every buffer: the load returns zeros

__device__ __forceinline__ __amdgpu_buffer_rsrc_t proj_rsrc(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

// How the 16 columns of the B operand (rows of x) and the 16 rows of the A operand (outputs) are used:
//   FULL   column c = token c: one K step per load of x (9..16 tokens; with MT = 2 up to 32)
//   PAIR   up to 8 tokens: one load of x brings two K steps, columns 0-7 the even and 8-15 the odd one.  The same
//          operand multiplies the weights of both steps into two accumulators; of the even one columns 0-7 count, of
//          the odd one columns 8-15.
//   HALF   as PAIR, and the work unit is half a panel (8 outputs): rows 0-7 of the A operand take the even step, rows
//          8-15 the odd one, and of the product the two diagonal blocks count.  Twice the workgroups for narrow
//          matrices.
enum { PROJ_FULL = 0, PROJ_PAIR = 1, PROJ_HALF = 2 };

// A lane's outputs: the 8 waves' pieces (PAIR, HALF: even + odd steps of each) added as a tree of pairs; few LDS reads
// at a time, the ring holds most registers.
template <int MODE, int STRIDE>
__device__ __forceinline__ f32x4 proj_sum(const f32x4* red, int lane) {
  constexpr int PARTNER = MODE == PROJ_PAIR ? 8 : MODE == PROJ_HALF ? 40 : 0;   // lane that holds the odd steps' part
  static_assert(PROJ_WAVES == 8, "two halves of four waves");
  f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int h = 0; h < PROJ_WAVES; h += 4) {
    f32x4 s[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const f32x4* r = red + (h + k * 2) * STRIDE;
      s[k] = r[lane];
      f32x4 u = r[STRIDE + lane];
      if (PARTNER) {
        s[k] += r[(lane + PARTNER) & 63];
        u += r[STRIDE + ((lane + PARTNER) & 63)];
      }
      s[k] += u;
    }
    t += s[0] + s[1];
  }
  return t;
}

template <int MODE, int MT, int RP, int D, int EPI, bool FIRST>
__global__ __launch_bounds__(PROJ_THREADS, RP * MT > 4 ? 2 : 4) void proj_kernel(ProjArgs a) {
  static_assert(MODE == PROJ_FULL || MT == 1, "two row tiles only with one token per column");
  static_assert(MODE != PROJ_HALF || RP == (EPI == PROJ_SWIGLU ? 2 : 1), "half panels are taken one unit at a time");
  constexpr int Q = MODE == PROJ_FULL ? 1 : 2;          // K steps per stage
  constexpr int WL = MODE == PROJ_HALF ? 1 : Q;         // weight loads per stage and panel
  constexpr int AC = RP * MT > 2 && MODE == PROJ_FULL && !(RP == 2 && MT == 2) ? 1 : 2;   // accumulators per panel and row tile: chains half as long
  constexpr int NBUF = RP * MT <= 4 ? 2 : 1;            // two reduction buffers while they fit: one barrier per group
  __shared__ f32x4 red[NBUF][PROJ_WAVES][RP][MT][64];
  __shared__ float inv_sh[SPEC_MAX_TOKENS];
  // Of two overlapped chains the favoured one issues first (runtime.hip, favoured_chain), from its first instruction on.
  if (FIRST) __builtin_amdgcn_s_setprio(3);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int c = lane & 15, kb = lane >> 4;
  if (a.stamp && threadIdx.x == 0)
    atomicMax(a.stamp + 2 * (blockIdx.x % STAMP_WAYS), ~(unsigned long long)wall_clock64());
  // this workgroup's units (panel pairs, panels or half panels): the first `rem` workgroups take one more
  const int b = blockIdx.x;
  const int u0 = b * a.per + (b < a.rem ? b : a.rem), u1 = u0 + a.per + (b < a.rem ? 1 : 0);
  constexpr int UP = EPI == PROJ_SWIGLU ? 2 : 1;        // panels per unit; two units of half panels per panel (pair)
  const int p0 = u0 * UP, p1 = u1 * UP;                 // HALF: counted in half panels
  // this wave's K steps, dealt in stages of Q
  const int stages = (a.steps + Q - 1) / Q;
  const int s0 = w * stages / PROJ_WAVES, ns = (w + 1) * stages / PROJ_WAVES - s0;
  const int niter = ns > D ? (ns + D - 1) / D : 1;
  const int left = a.steps - s0 * Q;                    // K steps behind this wave's first one

  const unsigned pbytes = (unsigned)a.steps * 1024u;    // a panel
  const unsigned xrow = (unsigned)a.K * 2u;
  const __amdgpu_buffer_rsrc_t xr = proj_rsrc(reinterpret_cast<const char*>(a.x) + (size_t)s0 * Q * 64,
                                              (unsigned)a.M * xrow - (unsigned)(s0 * Q) * 64u);
  const int xc = MODE == PROJ_FULL ? c : (c & 7), xq0 = MODE == PROJ_FULL ? 0 : (c >> 3);
  unsigned xlane = (unsigned)xc * xrow + xq0 * 64 + kb * 16;
  // stages in which this lane has columns of x (ragged K, odd step count)
  const int xlim = (a.K - kb * 8 - (s0 * Q + xq0) * 32 + 31) >> 5;           // its K steps, counted from its first
  const int xst = min(ns, (xlim + Q - 1) / Q);
  unsigned wlane = MODE == PROJ_HALF ? (unsigned)((c >> 3) * 1024 + kb * 256 + (c & 7) * 16) : lane * 16u;

  u32x4 wq[D][RP][WL], xq[D][MT];
  // (the empty asm keeps the compiler from working out all the offsets of a refill once and holding them in registers)
#define PROJ_LOAD(DD, WR, J)                                                                                     \
  {                                                                                                              \
    asm volatile("" : "+v"(wlane), "+v"(xlane));                                                                 \
    _Pragma("unroll") for (int q = 0; q < WL; ++q) {                                                             \
      const int st_ = (J) * Q + q;                                                                               \
      unsigned so_ = ((J) < ns && st_ < left) ? (unsigned)st_ * 1024u : PROJ_SKIP;                               \
      if (MODE == PROJ_HALF && (c >> 3) + st_ >= left) so_ = PROJ_SKIP;                                          \
      _Pragma("unroll") for (int rp = 0; rp < RP; ++rp)                                                          \
        wq[DD][rp][q] = __builtin_amdgcn_raw_buffer_load_b128(WR, wlane + so_ + rp * pbytes, 0, PROJ_NT);        \
    }                                                                                                            \
    const unsigned xo_ = (J) < xst ? xlane + (unsigned)(J) * (Q * 64u) : PROJ_SKIP;                              \
    _Pragma("unroll") for (int mt = 0; mt < MT; ++mt)                                                            \
      xq[DD][mt] = __builtin_amdgcn_raw_buffer_load_b128(xr, xo_ + mt * 16u * xrow, 0, 0);                       \
    __builtin_amdgcn_sched_barrier(0);   /* a stage is refilled before the next one is waited for */             \
  }
  auto group_rsrc = [&](int p) {
    int n = p1 - p;
    if (n > RP) n = RP;
    const size_t panel = MODE == PROJ_HALF ? p / (2 * UP) * UP : p;
    const unsigned half = MODE == PROJ_HALF ? (p / UP & 1) * 128u : 0u;
    const unsigned bytes = n > 0 ? (unsigned)(n - 1) * pbytes + (unsigned)left * 1024u - half : 0u;
    return proj_rsrc(reinterpret_cast<const char*>(a.w) + (panel * a.steps + s0 * Q) * 1024 + half, bytes);
  };
  __amdgpu_buffer_rsrc_t wr = group_rsrc(p0);
  // 1 / rms of every row from its sums of squares (ssq_w pieces, added in a fixed order).  A wave's first row is
  // requested ahead of the ring, so that it is not waited for behind the weights, and summed once the ring is on its way.
  const bool scaled = EPI != PROJ_RESID && a.ssq;
  f32x4 sq[2] = {};
  const int row_bytes = (a.ssq_w + 3) / 4 * 16;   // whole vectors; what lies behind the pieces is masked below
  if (EPI != PROJ_RESID) {
    const __amdgpu_buffer_rsrc_t sr = proj_rsrc(a.ssq + (size_t)w * SSQ_STRIDE, scaled && w < a.M ? row_bytes : 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) sq[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(sr, lane * 16 + i * 1024, 0, 0));
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int d = 0; d < D; ++d) {
    PROJ_LOAD(d, wr, d)
    __builtin_amdgcn_sched_barrier(0);
  }

  if (scaled) {
    for (int m = w; m < a.M; m += PROJ_WAVES) {
      const float* row = a.ssq + (size_t)m * SSQ_STRIDE;
      float s = 0.f;
      for (int i = lane * 4, k = 0; i < a.ssq_w; i += 256, ++k) {
        f32x4 t = m == w && k == 0 ? sq[0] : m == w && k == 1 ? sq[1] : *reinterpret_cast<const f32x4*>(row + i);
#pragma unroll
        for (int r = 0; r < 4; ++r) s += i + r < a.ssq_w ? t[r] : 0.f;
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
      if (lane == 0) inv_sh[m] = 1.0f / sqrtf(s / (float)a.K + a.eps);
    }
  }

  int rb = 0;
  for (int p = p0; p < p1; p += RP) {
    f32x4 acc[RP][MT][AC];
#pragma unroll
    for (int rp = 0; rp < RP; ++rp)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < AC; ++q) acc[rp][mt][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    // what the epilogue's thread needs besides the sums is requested ahead of them
    const int it_mt = w % MT, it_rp = w / MT, g4 = kb;
    const int m = it_mt * 16 + c;
    const int col = MODE == PROJ_HALF ? p * 8 + g4 * 4 : (p + it_rp) * 16 + g4 * 4;
    const bool mine = w < RP * MT && p + it_rp < p1 && m < a.M && (MODE == PROJ_FULL || c < 8) && (MODE != PROJ_HALF || g4 < 2);
    f32x4 hv = {0.f, 0.f, 0.f, 0.f};
    bf16x4u gv = {0, 0, 0, 0};
    if (EPI == PROJ_RESID && mine) {
      hv = *reinterpret_cast<const f32x4*>(a.h + (size_t)m * a.N + col);
      gv = *reinterpret_cast<const bf16x4u*>(a.gain + col);
    }
    // accumulator of weight load q of stage DD: PAIR by step parity (see above), else alternating stages
#define PROJ_MMA(DD)                                                                                             \
  _Pragma("unroll") for (int mt = 0; mt < MT; ++mt)                                                              \
    _Pragma("unroll") for (int q = 0; q < WL; ++q)                                                               \
      _Pragma("unroll") for (int rp = 0; rp < RP; ++rp) {                                                        \
        f32x4& t_ = acc[rp][mt][MODE == PROJ_PAIR ? q : (DD) % AC];                                              \
        t_ = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wq[DD][rp][q]),                  \
                                                     __builtin_bit_cast(bf16x8, xq[DD][mt]), t_, 0, 0, 0);       \
      }
    // After every iteration (every second one if D is small and the range long) the accumulators go to this wave's
    // slots of the reduction buffer and start again at zero: chains of 2 to 8 additions, added up in a second level,
    // keep the rounding error at or below that of K slices (8192 x 28672, M = 7: 2.6e-7 with one chain per wave,
    // 1.2e-7 in K slices, 1.1e-7 so).
    const int fmask = D <= 4 && ns > 32 ? 1 : 0;
    auto flush = [&](bool first) {
#pragma unroll
      for (int rp = 0; rp < RP; ++rp)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          f32x4 v = acc[rp][mt][0];
          if (MODE == PROJ_PAIR) {
            const f32x4 odd = acc[rp][mt][AC - 1];
            asm volatile("" ::"v"(v), "v"(odd));   // a second use keeps the choice one of values, not of addresses
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = c >= 8 ? odd[r] : v[r];
          } else if (AC == 2) {
            v += acc[rp][mt][AC - 1];
          }
          f32x4* slot = &red[rb][w][rp][mt][lane];
          if (!first) v += *slot;
          *slot = v;
#pragma unroll
          for (int q = 0; q < AC; ++q) acc[rp][mt][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // An iteration has D stages; those past the wave's range hold zeros.  The last one refills from the next group, and
    // that of the last group not at all: a copy of its own, so that every load is unconditional.
    const bool more = p + RP < p1;
    const __amdgpu_buffer_rsrc_t wn = group_rsrc(p + RP);
    const int full = more ? niter : niter - 1;
    bool first = true;
    for (int it = 0; it < full; ++it) {
      const bool last = it + 1 == niter;
      const __amdgpu_buffer_rsrc_t lr = last ? wn : wr;
      const int j0 = last ? 0 : (it + 1) * D;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        PROJ_MMA(d)
        PROJ_LOAD(d, lr, j0 + d)
      }
      if ((it & fmask) == fmask) {
        flush(first);
        first = false;
      }
    }
    if (!more) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        PROJ_MMA(d)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (!more || fmask) flush(first);
    wr = wn;
    __syncthreads();
    if (w < RP * MT) {
      f32x4 t = proj_sum<MODE, RP * MT * 64>(&red[rb][0][it_rp][it_mt][0], lane);
      if (EPI == PROJ_STORE) {
        if (mine) {
          if (a.ssq) t *= inv_sh[m];
          *reinterpret_cast<f32x4*>(a.y + (size_t)m * a.N + col) = t;
        }
      } else if (EPI == PROJ_RESID) {
        t += hv;
        float ss = t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w;
        ss += __shfl_xor(ss, 16);
        if (MODE != PROJ_HALF) ss += __shfl_xor(ss, 32);
        if (mine) {
          *reinterpret_cast<f32x4*>(a.h + (size_t)m * a.N + col) = t;
          bf16 o[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r] = __float2bfloat16(t[r] * bf16x4_at(gv, r));
          *reinterpret_cast<uint2*>(a.xo + (size_t)m * a.N + col) = *reinterpret_cast<const uint2*>(o);
          if (g4 == 0) a.ssq_out[(size_t)m * SSQ_STRIDE + p + it_rp] = ss;
        }
      } else if ((it_rp & 1) == 0) {
        f32x4 u = proj_sum<MODE, RP * MT * 64>(&red[rb][0][it_rp + 1][it_mt][0], lane);
        if (mine) {
          const float inv = a.ssq ? inv_sh[m] : 1.0f;
          bf16 o[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float g = t[r] * inv;
            o[r] = __float2bfloat16(g / (1.0f + __expf(-g)) * (u[r] * inv));
          }
          const int f = MODE == PROJ_HALF ? (p >> 1) * 8 + g4 * 4 : ((p + it_rp) >> 1) * 16 + g4 * 4;
          *reinterpret_cast<uint2*>(a.xo + (size_t)m * (a.N / 2) + f) =
              *reinterpret_cast<const uint2*>(o);
        }
      }
    }
    // with two buffers the next group writes the other one, and nobody can reach the group after that before every
    // thread has passed the next barrier, i.e. has finished reading this buffer
    if (NBUF == 2) rb ^= 1;
    else __syncthreads();
  }
#undef PROJ_LOAD
#undef PROJ_MMA
  if (a.stamp && threadIdx.x == 0)
    atomicMax(a.stamp + 2 * (blockIdx.x % STAMP_WAYS) + 1, (unsigned long long)wall_clock64());
}

// Whether this kernel is the faster one; else K slices (gemm.hip) and a kernel that adds them.  What counts against it:
//   narrow and deep, K > 4 N: few workgroups, long ranges           512 x 8192, M = 12    8.1 (slices) | 10.9 (this kernel)
//   activations: the slices keep theirs in registers, here every panel group loads them again, M / (16 RP) of the weights'
//   traffic on top, in one workgroup's single long group where panels are fewer than CUs
//                      1024 x 4096: M = 9 1.14 times as fast as slices, M = 16 0.95, M = 17 0.81, M = 32 0.66
//                      4096 x 11008: M = 8 1.18, M = 9 1.11, M = 16 0.93, M = 32 0.74
//   uneven shares of panels, which slices deal in smaller pieces (`share`: part of the CUs' time in use if every CU takes as
//   many panels as the busiest; slower from longer K on)
//                      4608 x 4096, 5120 x 4096 (0.56, 0.63): M = 8 0.94; x 11008 0.85, 0.89; 6144 x 16384 (0.75) 0.86
//                      10240 x 11008 (0.83): M = 16 0.98, M = 24 0.91, M = 32 0.84; 14336 x 11008 (0.88): M = 32 0.99
// The limits lie where the ratio falls below 1 on a grid of 30 N x 18 K x 11 M (weights from HBM, back to back in a graph).
bool proj_whole_k(int M, int N, int K) {
  if (K > 4 * N) return false;
  const int NT = N / 16, ncu = spec_num_cu();
  const int share = (int)(100LL * NT / ((long long)(NT + ncu - 1) / ncu * ncu));
  if (M <= 8) return NT <= ncu || NT > 2 * ncu || share >= 80 || K < (share < 70 ? 4096 : 12288);
  if (NT <= ncu) {
    if (M <= 12) return K <= (share >= 95 ? 16384 : share >= 85 ? 8192 : 4096);
    if (M <= 16) return K <= (share >= 95 ? 8192 : 4096);
    if (M <= 24) return K <= (share >= 90 ? 4096 : share >= 30 ? 3072 : 2048);
    return K <= (share >= 90 ? 4096 : share >= 60 ? 2048 : 1024);
  }
  if (NT <= 2 * ncu) {
    if (M <= 16) return K <= 4096 || (share >= 80 && (K <= 8192 || M <= 12 || share >= 95));
    if (M <= 24) return K <= 4096 || share >= 95 || (share >= 80 && M <= 20);
    return K <= (share < 80 ? 2048 : 4096);
  }
  return K <= 4096 || share >= (M <= 24 ? 80 : 86);
}

// Layout, panels at a time (RP) and workgroups.  The layout and RP set the order of the sums; up to 8 tokens they follow from
// N, K and the epilogue alone, so that the rows of a forward do not depend on how many of them there are (behind the same cache;
// a token that stands in the cache instead of among the new ones is attended in another order).  The number of workgroups
// does not touch the sums; it depends on the launch mode too.
//
// Up to 8 tokens.  Shares come first: as many workgroups as give each the same number of units, one per CU, or two where
// that fills both places (`full`) (us, weights from HBM, back to back in a graph; two per CU with shares as they fall | now):
//   6144 x 2048, M = 5   384 of 1  7.1 | 192 of 2  6.2        22016 x 4096, M = 5   512 of 2, 1  33.7 | 230 of 3   31.1
//   14336 x 4096, M = 1  RP 4     22.3 | 448 of 2 20.6        10240 x 8192, M = 7   256 of 3, 2  30.3 | 214 of 3   28.7
// Then, by units per CU (`one`) and length of a wave's range (an eighth of K), the layout that costs least over 1 to 8 tokens:
//   up to 6 K steps per wave: several panels at a time save barriers; rings of 3 (RP 4) or, for 4 steps, of 4 (RP 2)
//                              8192 x 512, M = 7    4.5 (RP 1  5.3)     57344 x 512, SWIGLU  12.9 (half panels 22.4)
//   half a panel per CU: half panels            2048 x 5632, M = 5   6.3 (panels  7.7)
//   one: what pads the range least              4096 x 4096, M = 7   7.4 (RP 1, range 16 = 2 rings of 8; PAIR 2 of 12: 8.9)
//   two: both at once (short and long ranges)   5120 x 2048, M = 7   6.1 (RP 1  6.5)      7168 x 19200, M = 7  44.1 (PAIR 47.4)
//     between, half panels where two per CU would not be full, else single ones, two workgroups per CU
//                                               8192 x 8192, M = 7  24.0 (PAIR 24.3, half panels 25.1), M = 1 23.6 (23.7, 23.3)
//   three: RP 1                                 12288 x 4096, M = 7  18.9 (RP 4 18.1), M = 1 17.6 (17.9)
//   four: the same, two workgroups per CU       16384 x 4096, M = 7  23.4 (RP 4 26.2), M = 1 23.1 (25.6)
//   three and four from K = 6144 on PAIR, one per CU, for its loads of x, up to K = 12288 and 8192; beyond RP 4
//     10240 x 8192, M = 7  28.7 (RP 4 28.0, half panels 30.6), M = 1 27.2 (27.6, 26.3)
//     16384 x 8192, M = 7  43.7 (RP 4 47.2), M = 1 44.0 (47.8)     14176 x 10904, M = 8  49.5 (PAIR 56.5)
//     (three per CU are close; beside a second stream's launches a step of the 70B/7B pair takes 38.9 ms with these two, 39.2 with
//     either in RP 4)
//   five, six: RP 2                             21504 x 7168, M = 7  49.9 (PAIR 53.4), M = 1 48.7 (48.8)
//   more: PAIR                                  32000 x 8192, M = 7  79.1 (RP 2 81.2), M = 1 78.9 (80.6)
// SWIGLU pairs a gate and an up panel, so shares get coarser: half panels where that costs more than their loads of x.
//                              28672 x 8192, M = 1  72.4 (panels 79.0)  22016 x 4096, M = 7  34.1 (panels 31.3)
// Over 515 shapes (M 1..8, N 256..57344, K 256..28672) 6 % faster in the mean than two workgroups per CU with shares as they
// fall, 1 % behind the best layout measured for each; 13 of them more than 1 % slower, none more than 5 %.
//
// From 9 tokens on (FULL): RP as large as the panels fill; one workgroup per CU streams as fast as two and has the
// fewer loads of x                                 38400 x 7168, M = 12  90 (two per CU: 99)
ProjPlan proj_plan(int M, int N, int K, int epi, int wgs_per_cu) {
  ProjPlan p;
  const int ncu = spec_num_cu();
  p.M = M; p.N = N; p.K = K; p.epi = epi;
  p.steps = (K + 31) / 32;
  p.NT = N / 16;
  const bool sw = epi == PROJ_SWIGLU;
  const int units = sw ? p.NT / 2 : p.NT;                // of whole panels
  p.mode = PROJ_FULL;
  p.units = units;
  if (M > 8) {
    int G = ncu * wgs_per_cu;
    p.RP = sw ? (p.NT <= 2 * ncu ? 2 : 4) : p.NT <= ncu ? 1 : p.NT <= 2 * ncu ? 2 : 4;
    if (p.NT < 4 * ncu || (sw ? p.NT == 4 * ncu : p.NT <= 2 * ncu || p.NT > 6 * ncu)) G = ncu;
    if (M > 16 && epi == PROJ_RESID) p.RP = 2;
    if (M > 16 && p.RP == 4) G = ncu;                    // a workgroup's registers fill a CU
    p.G = units < G ? units : G;
    return p;
  }
  auto share = [](int n, int places) { return (n + places - 1) / places; };
  const int one = share(units, ncu), range = share(p.steps, PROJ_WAVES);
  const bool brief = range <= 6, full = units * 100 >= one * ncu * 85;
  const int brief_rp = range == 4 ? 2 : 4;
  auto pad = [&](int ring, int q) { return share(share(range, q), ring) * ring * q; };
  bool two = false;        // two workgroups per CU
  bool uneven = false;     // ... with shares as they fall: as fast or faster there
  p.RP = sw ? 2 : 1;
  if (2 * units <= ncu) {
    if (!sw || K >= 1024) p.mode = PROJ_HALF;
  } else if (sw) {
    if (one > 1 && brief) {
      p.RP = brief_rp;
    } else if (one == 1) {
      if (K >= 6144 || (K >= 3072 && full)) p.mode = PROJ_HALF, two = full;
    } else if (one == 2) {
      if (K >= 3072) p.mode = PROJ_HALF, two = full && K < 6144;
      else if (full) two = true;
      else p.mode = PROJ_HALF, uneven = true;
    } else if (one <= 4) {
      if (K >= (one == 4 ? 3072 : 6144)) p.mode = PROJ_HALF;
    } else if (K >= 8192 || (K >= 6144 && one > 6)) {
      p.mode = PROJ_HALF, two = true;
    } else if (K >= 6144) {
      uneven = true;
    }
  } else if (one == 1) {
    if (range < 4) p.RP = 2;
    else if (brief || K >= 6144 || pad(6, 2) < pad(8, 1)) p.mode = PROJ_PAIR;
  } else if (one == 2) {
    if (K < 3072 || (K >= 6144 && pad(6, 1) < pad(8, 1))) p.RP = 2;
    else if (K >= 6144 && K < 12288 && !full) p.mode = PROJ_HALF;
    else two = full, p.mode = K >= 12288 ? PROJ_PAIR : PROJ_FULL;
  } else if (one <= 4) {
    if (brief) p.RP = brief_rp;
    else if (K >= 12288 || (one == 4 && K > 8192)) p.RP = 4;
    else if (K >= 6144) p.mode = PROJ_PAIR;
    else two = one == 4;
  } else if (one <= 6) {
    if (brief) p.RP = 4, uneven = true;
    else p.RP = 2;
  } else {
    if (brief) p.RP = brief_rp;
    else p.mode = PROJ_PAIR;
  }
  // half panels: a residual add leaves a piece of sums of squares per unit, at most 2 x 2 per CU (a row holds SSQ_STRIDE)
  if (p.mode == PROJ_HALF) p.units = 2 * units;
  const int places = ncu * (wgs_per_cu > 1 && (two || uneven) ? 2 : 1);
  p.G = uneven ? (p.units < places ? p.units : places) : share(p.units, share(p.units, places));
  return p;
}

// What launch_epi has kernels for.  HALF and PAIR keep two K steps in a load of x and so at most 8 tokens; a residual add
// with two row tiles streams at most two panels at a time (registers); SWIGLU needs whole gate / up pairs.
bool proj_plan_ok(const ProjPlan& p) {
  if (p.M < 1 || p.M > SPEC_MAX_TOKENS || p.N < 16 || (p.N & 15) || p.K < 8 || (p.K & 7) || p.G < 1 || p.units < p.G) return false;
  if (p.steps != (p.K + 31) / 32 || p.NT != p.N / 16 || (double)p.steps * 4096.0 >= (double)PROJ_SKIP) return false;
  if (p.epi != PROJ_STORE && p.epi != PROJ_RESID && p.epi != PROJ_SWIGLU) return false;
  const bool sw = p.epi == PROJ_SWIGLU;
  if (sw && (p.N & 31)) return false;
  switch (p.mode) {
    case PROJ_HALF:                  // a residual add leaves a sum of squares per half panel, SSQ_STRIDE at most
      return p.M <= 8 && p.RP == (sw ? 2 : 1) && p.units == (sw ? p.NT : p.NT * 2) && !(p.epi == PROJ_RESID && p.units > SSQ_STRIDE);
    case PROJ_PAIR: return p.M <= 8 && !sw && p.RP == 1 && p.units == p.NT;
    case PROJ_FULL:
      if (p.units != (sw ? p.NT / 2 : p.NT)) return false;
      if (p.RP == 1) return !sw;
      return p.RP == 2 || (p.RP == 4 && !(p.M > 16 && p.epi == PROJ_RESID));
  }
  return false;
}

template <int EPI, bool FIRST>
static hipError_t launch_epi(const ProjPlan& p, const ProjArgs& a, hipStream_t st) {
  dim3 g(p.G), b(PROJ_THREADS);
#define PROJ_GO(MODE, MT, RP, D)                                    \
  {                                                                 \
    proj_kernel<MODE, MT, RP, D, EPI, FIRST><<<g, b, 0, st>>>(a);    \
    return hipGetLastError();                                       \
  }
  constexpr int SW = EPI == PROJ_SWIGLU ? 2 : 1;
  // Stages of the ring: 6, or 4 where a wave's range has 4 or 8 of them (K <= 2048) and every third load would bring
  // nothing (24 layers of d_model 2048, M = 5: 1000 us with 6, 949 with 4).
  const bool brief = p.steps <= 8 * PROJ_WAVES;
  if (p.mode == PROJ_HALF) {
    if (brief) PROJ_GO(PROJ_HALF, 1, SW, 4)
    PROJ_GO(PROJ_HALF, 1, SW, 6)
  } else if (p.mode == PROJ_PAIR) {
    if constexpr (EPI != PROJ_SWIGLU) {
      if (brief) PROJ_GO(PROJ_PAIR, 1, 1, 4)
      PROJ_GO(PROJ_PAIR, 1, 1, 6)
    }
  } else if (p.M > 16) {
    if (p.RP <= 2) PROJ_GO(PROJ_FULL, 2, 2, 4)
    if constexpr (EPI != PROJ_RESID) PROJ_GO(PROJ_FULL, 2, 4, 4)
  } else if (p.RP == 4) {
    PROJ_GO(PROJ_FULL, 1, 4, 3)
  } else if (p.RP == 2) {
    if (brief) PROJ_GO(PROJ_FULL, 1, 2, 4)
    PROJ_GO(PROJ_FULL, 1, 2, 6)
  } else if constexpr (EPI != PROJ_SWIGLU) {
    PROJ_GO(PROJ_FULL, 1, 1, 8)
  }
#undef PROJ_GO
  return hipErrorInvalidValue;      // nothing was launched
}

template <bool FIRST>
static hipError_t launch_first(const ProjPlan& p, const ProjArgs& a, hipStream_t st) {
  if (p.epi == PROJ_STORE) return launch_epi<PROJ_STORE, FIRST>(p, a, st);
  if (p.epi == PROJ_RESID) return launch_epi<PROJ_RESID, FIRST>(p, a, st);
  return launch_epi<PROJ_SWIGLU, FIRST>(p, a, st);
}

hipError_t launch_proj(const ProjPlan& p, ProjArgs a, hipStream_t st, int prio) {
  if (!proj_plan_ok(p)) return hipErrorInvalidValue;
  a.M = p.M; a.N = p.N; a.K = p.K; a.steps = p.steps;
  a.per = p.units / p.G; a.rem = p.units % p.G;
  if (prio == 2 && p.epi != PROJ_STORE) return hipErrorInvalidValue;      // stand-alone calls store
  return prio == 1 ? launch_first<true>(p, a, st) : launch_first<false>(p, a, st);
}

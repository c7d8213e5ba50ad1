// Fused logits -> probability kernels (gfx950): the draft's draw x_i ~ q_i and the target's
// accept / reject with residual resampling (paper Section 2, Eq. (1); Algorithm 2).
//
// A distribution is softmax(mult * logits) in fp32 (mult = logit_scale / temperature), or the
// one-hot at the arg-max (lowest id on ties) for greedy decoding.  A draw is an inverse-CDF walk in
// ascending token id with one uniform u: the first k whose running sum (fp64) exceeds u * total.
// The acceptance test is evaluated without a division, in fp64: accept iff r * q[x] <= p[x].
//
// What bounds them is one compute unit's vector ALU and the latency of dependent passes, so
//   * up to 32768 ids one workgroup of 1024 threads holds a row in registers and reads it once (the reg_* functions);
//   * longer rows are cut into pieces of 8192 ids, one workgroup each; what the pieces have to know of each other (row
//     maximum, sums) goes through a kernel boundary;
//   * wave reductions and scans run on DPP row shifts and broadcasts, not on LDS permutes.
#include <cstring>

#include "spec_internal.h"

#define SAMP_THREADS 1024
#define SAMP_WAVES (SAMP_THREADS / 64)

struct MaxIdx { float v; int i; };

// ---- wave reductions and scans on DPP ------------------------------------------------------------
// A lane receives x of the lane that CTRL names (row_shr:n inside rows of 16 lanes; row_bcast:15 / :31 = the last lane
// of the row(s) before, into the rows of mask RM), or `none` where there is none.
template <int CTRL, int RM>
__device__ __forceinline__ int dpp_i(int none, int x) {
  return __builtin_amdgcn_update_dpp(none, x, CTRL, RM, 0xf, false);
}
template <int CTRL, int RM>
__device__ __forceinline__ float dpp_f(float none, float x) {
  return __int_as_float(dpp_i<CTRL, RM>(__float_as_int(none), __float_as_int(x)));
}
template <int CTRL, int RM>
__device__ __forceinline__ double dpp_d(double x) {
  return __hiloint2double(dpp_i<CTRL, RM>(0, __double2hiint(x)), dpp_i<CTRL, RM>(0, __double2loint(x)));
}
// inclusive sum over the lanes 0 .. this one; lane 63 holds the total
__device__ __forceinline__ double wave_scan_d(double x) {
  x += dpp_d<0x111, 0xf>(x);
  x += dpp_d<0x112, 0xf>(x);
  x += dpp_d<0x114, 0xf>(x);
  x += dpp_d<0x118, 0xf>(x);
  x += dpp_d<0x142, 0xa>(x);
  x += dpp_d<0x143, 0xc>(x);
  return x;
}
__device__ __forceinline__ double lane_d(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane), __builtin_amdgcn_readlane(__double2loint(x), lane));
}
__device__ __forceinline__ MaxIdx better(MaxIdx a, float v, int i) {
  // larger value wins; on equal values the lower index wins
  const bool take = (v > a.v) | ((v == a.v) & (i < a.i));
  a.v = take ? v : a.v;
  a.i = take ? i : a.i;
  return a;
}
// larger value, then lower index, over the wave; to every lane
__device__ __forceinline__ MaxIdx wave_argmax(MaxIdx m) {
  float v = m.v;
  v = fmaxf(v, dpp_f<0x111, 0xf>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x112, 0xf>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x114, 0xf>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x118, 0xf>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x142, 0xa>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x143, 0xc>(-INFINITY, v));
  MaxIdx r;
  r.v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
  int i = m.v == r.v ? m.i : 0x7fffffff;
  i = min(i, dpp_i<0x111, 0xf>(0x7fffffff, i));
  i = min(i, dpp_i<0x112, 0xf>(0x7fffffff, i));
  i = min(i, dpp_i<0x114, 0xf>(0x7fffffff, i));
  i = min(i, dpp_i<0x118, 0xf>(0x7fffffff, i));
  i = min(i, dpp_i<0x142, 0xa>(0x7fffffff, i));
  i = min(i, dpp_i<0x143, 0xc>(0x7fffffff, i));
  r.i = __builtin_amdgcn_readlane(i, 63);
  return r;
}

__device__ __forceinline__ MaxIdx block_argmax(MaxIdx m, MaxIdx* sh) {
  const int lane = threadIdx.x & 63;
  m = wave_argmax(m);
  if (lane == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  MaxIdx r;
  r.v = -INFINITY; r.i = 0x7fffffff;
  if (lane < SAMP_WAVES) r = sh[lane];
  r = wave_argmax(r);
  __syncthreads();
  return r;
}

// largest value of the workgroup (NaN counts as none), to every thread
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f<0x111, 0xf>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x112, 0xf>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x114, 0xf>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x118, 0xf>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x142, 0xa>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x143, 0xc>(-INFINITY, v));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float block_max(float v, float* sh) {
  const int lane = threadIdx.x & 63;
  v = wave_max(v);
  if (lane == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return wave_max(lane < SAMP_WAVES ? sh[lane] : -INFINITY);
}

__device__ __forceinline__ double block_sum_d(double v, double* sh) {
  const int lane = threadIdx.x & 63;
  v = wave_scan_d(v);
  if (lane == 63) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  const double r = lane_d(wave_scan_d(lane < SAMP_WAVES ? sh[lane] : 0.0), 63);
  __syncthreads();
  return r;
}

// Four consecutive values, at any 4-byte alignment (rows of a vocabulary that is no multiple of four), `fill` beyond V.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4 load4(const float* __restrict__ row, int j, int V, float fill) {
  f32x4 v = {fill, fill, fill, fill};
  if (j + 4 <= V) {
    v = *reinterpret_cast<const f32x4u*>(row + j);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (j + i < V) v[i] = row[j + i];
  }
  return v;
}
__device__ __forceinline__ void store4(float* __restrict__ row, int j, int V, f32x4 v) {
  if ((V & 3) == 0) {
    if (j < V) *reinterpret_cast<f32x4u*>(row + j) = v;
  } else if (j + 4 <= V) {
    *reinterpret_cast<f32x4u*>(row + j) = v;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (j + i < V) row[j + i] = v[i];
  }
}

// ---- a row, or a piece of one, in the registers of a workgroup ------------------------------------
// Wave w owns the ids [w R 256, (w + 1) R 256), lane l of it the four ids w R 256 + 256 k + 4 l .. + 3 of every k < R.
#define SAMP_CHUNKS_MAX 8
#define SAMP_REG_VOCAB_MAX (SAMP_CHUNKS_MAX * 4 * SAMP_THREADS)
#define SAMP_PIECE 8192
#define SAMP_PIECE_CHUNKS (SAMP_PIECE / (4 * SAMP_THREADS))
struct RegGeom {
  int R, w, lane, j0;
  __device__ __forceinline__ int id(int k) const { return j0 + 256 * k; }
};
__device__ __forceinline__ RegGeom reg_geom(int V) {
  RegGeom g;
  g.R = (V + 4 * SAMP_THREADS - 1) / (4 * SAMP_THREADS);
  g.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  g.lane = threadIdx.x & 63;
  g.j0 = g.w * g.R * 256 + g.lane * 4;
  return g;
}
// probability of a logit given the row's statistics: hardware exp2 (1 ulp) of a product rounded once, times the
// reciprocal of the sum: relative error below 1e-5 for exponents down to -100, two orders under what the bf16
// logits carry.  Every kernel of the register path forms p and q with this one expression.
__device__ __forceinline__ float reg_prob(float l, float mult, float zmax, float inv) { return __expf(fmaf(l, mult, -zmax)) * inv; }
// max(0, p - q) of the rounded p that a draft's q is compared with: fused with the product behind p, the subtraction would leave
// the product's rounding error where p and q are the same bits, and a residual without mass would seem to have some.
__device__ __forceinline__ float residual(float p, float q) {
#pragma clang fp contract(off)
  return fmaxf(p - q, 0.f);
}

// A thread's chunks of a row, `fill` beyond V.  Where no vector straddles the end the loads are unconditional (lanes
// beyond the end read the last vector): behind branches each would be waited for before the next goes out.
template <int CH>
__device__ __forceinline__ void reg_fetch(const float* __restrict__ row, int V, const RegGeom& g, float fill, f32x4 (&e)[CH]) {
  if ((V & 3) == 0) {
#pragma unroll
    for (int k = 0; k < CH; ++k) e[k] = *reinterpret_cast<const f32x4u*>(row + min(g.id(k), V - 4));
#pragma unroll
    for (int k = 0; k < CH; ++k)
      if (k >= g.R || g.id(k) >= V) e[k] = f32x4{fill, fill, fill, fill};
  } else {
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      e[k] = f32x4{fill, fill, fill, fill};
      if (k < g.R) e[k] = load4(row, g.id(k), V, fill);
    }
  }
}
template <int CH>
__device__ __forceinline__ MaxIdx reg_load(const float* __restrict__ row, int V, const RegGeom& g, f32x4 (&e)[CH]) {
  MaxIdx m;
  m.v = -INFINITY; m.i = 0x7fffffff;
  reg_fetch(row, V, g, __builtin_nanf(""), e);     // which wins no comparison
  // a thread's ids ascend, so the larger value alone decides; where nothing is larger than -inf, the first that is -inf
#pragma unroll
  for (int k = 0; k < CH; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool take = e[k][i] > m.v;
      m.v = take ? e[k][i] : m.v;
      m.i = take ? g.id(k) + i : m.i;
    }
  if (m.i == 0x7fffffff && g.j0 < V) {
#pragma unroll
    for (int k = 0; k < CH; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) m = better(m, e[k][i], g.id(k) + i);
  }
  return m;
}
// the largest value alone; beyond V e holds -inf, which has no mass whatever the largest value is (mult > 0)
template <int CH>
__device__ __forceinline__ float reg_load_max(const float* __restrict__ row, int V, const RegGeom& g, f32x4 (&e)[CH]) {
  float m = -INFINITY;
  reg_fetch(row, V, g, -INFINITY, e);
#pragma unroll
  for (int k = 0; k < CH; ++k) m = fmaxf(fmaxf(m, fmaxf(e[k][0], e[k][1])), fmaxf(e[k][2], e[k][3]));
  return m;
}

// arg-max of a row of any length by the whole workgroup, a vector per thread and pass
__device__ __forceinline__ MaxIdx row_argmax(const float* logits, int V, MaxIdx* shm) {
  MaxIdx m;
  m.v = -INFINITY; m.i = 0x7fffffff;
#pragma unroll 4
  for (int j = 4 * threadIdx.x; j < V; j += 4 * SAMP_THREADS) {
    const f32x4 v = load4(logits, j, V, -INFINITY);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (j + i < V) m = better(m, v[i], j + i);
  }
  return block_argmax(m, shm);
}

// Clears what lies beyond V where mult leaves mass there: 0 at an infinite temperature, or a negative scale.
template <int CH>
__device__ __forceinline__ void reg_clear_rest(int V, float mult, const RegGeom& g, f32x4 (&e)[CH]) {
  if (mult > 0.f) return;
#pragma unroll
  for (int k = 0; k < CH; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k >= g.R || g.id(k) + i >= V) e[k][i] = 0.f;
}

// Loads the row once; returns its maximum, sum_j exp(mult l_j - zmax) and e[k] = exp(mult l - zmax) (0 outside V).  What
// `between` loads is under way while the sum is formed.
template <int CH, typename F>
__device__ __forceinline__ void reg_softmax(const float* __restrict__ row, int V, float mult, const RegGeom& g, f32x4 (&e)[CH],
                                            float& top, float& sum, float* shm, double* shd, F between) {
  top = block_max(reg_load_max(row, V, g, e), shm);
  between();
  const float zmax = top * mult;
  float acc = 0.f;
#pragma unroll
  for (int k = 0; k < CH; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) e[k][i] = __expf(fmaf(e[k][i], mult, -zmax));
  reg_clear_rest(V, mult, g, e);
#pragma unroll
  for (int k = 0; k < CH; ++k) acc += (e[k][0] + e[k][1]) + (e[k][2] + e[k][3]);
  sum = (float)block_sum_d((double)acc, shd);
}

__device__ __forceinline__ double sum4_d(f32x4 v) { return ((double)v[0] + (double)v[1]) + ((double)v[2] + (double)v[3]); }

// One wave's part of the walk: the first id of its chunks whose running sum, from `base` on, exceeds target; the last
// id with mass if rounding lets the search run off its end, or if `clamp` asks for that one.  The wave has mass.
template <int CH>
__device__ __forceinline__ int wave_walk(const f32x4 (&e)[CH], int j0, int lane, double base, double target, bool clamp) {
  int tok = -1;
#pragma unroll
  for (int k = 0; k < CH; ++k) {
    if (tok >= 0 || clamp) continue;             // uniform over the wave
    f32x4 v = e[k];
    asm volatile("" : "+v"(v));                  // keeps the fp64 values of reg_draw's sums from being held for here
    const double s = sum4_d(v);
    const double incl = wave_scan_d(s);
    const double tot = lane_d(incl, 63);
    if (tot > 0.0 && base + tot > target) {
      const unsigned long long pos = __ballot(s > 0.0), hit = __ballot(s > 0.0 && base + incl > target);
      const int l = hit ? __ffsll((long long)hit) - 1 : 63 - __clzll((long long)pos);
      double run = base + (incl - s);
      int mine = -1, lastm = -1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        run += (double)v[i];
        const bool mass = v[i] > 0.f;
        lastm = mass ? j0 + 256 * k + i : lastm;
        mine = (mass & (mine < 0) & (run > target)) ? lastm : mine;
      }
      tok = __builtin_amdgcn_readlane(mine >= 0 ? mine : lastm, l);
    }
    base += tot;
  }
  if (tok >= 0) return tok;
  int last = -1;
#pragma unroll
  for (int k = 0; k < CH; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) last = e[k][i] > 0.f ? j0 + 256 * k + i : last;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o));
  return last;
}

// Inverse-CDF draw over the non-negative weights e[] (0 outside V): first the wave (scan of the 16 wave totals), then
// its chunks of 256 ids, the lane, the id, all sums in fp64.  Returns the id to every thread, -1 if the weights have no
// mass; *total_out = their sum.  `before` and `target` serve a caller whose weights are a piece of a longer row: the
// sum ahead of the piece and the value to exceed (target < 0: u times the total).  shd: SAMP_WAVES doubles, shi: 1 int.
// Every thread of the workgroup must call it (two barriers inside).
template <int CH>
__device__ __forceinline__ int reg_draw(const f32x4 (&e)[CH], const RegGeom& g, float u, double before, double target,
                                        double* shd, int* shi, double* total_out) {
  double mine = 0.0;
#pragma unroll
  for (int k = 0; k < CH; ++k) mine += sum4_d(e[k]);
  const double winc = wave_scan_d(mine);
  if (g.lane == 63) shd[g.w] = winc;
  __syncthreads();
  const double wt = g.lane < SAMP_WAVES ? shd[g.lane] : 0.0;
  const double wincl = wave_scan_d(wt);
  const double total = lane_d(wincl, SAMP_WAVES - 1);
  if (total_out) *total_out = total;
  if (target < 0.0) target = (double)u * total;
  const unsigned long long wmass = __ballot(g.lane < SAMP_WAVES && wt > 0.0);
  const unsigned long long whit = __ballot(g.lane < SAMP_WAVES && wt > 0.0 && before + wincl > target);
  // rounding can leave the target at or beyond the total: then the draw is the last id with mass
  const bool clamp = whit == 0;
  const int owner = !wmass ? -1 : (clamp ? 63 - __clzll((long long)wmass) : __ffsll((long long)whit) - 1);
  if (threadIdx.x == 0 && owner < 0) shi[0] = -1;      // no mass at all
  if (g.w == owner) {
    const double base = before + (owner > 0 ? lane_d(wincl, owner > 0 ? owner - 1 : 0) : 0.0);
    const int tok = wave_walk(e, g.j0, g.lane, base, target, clamp);
    if (g.lane == 0) shi[0] = tok;
  }
  __syncthreads();
  return shi[0];
}

// ---- draft: q = softmax(mult*logits), x = invCDF(q, u) -------------------------------------
// What bounds these kernels up to 32768 ids is the vector ALU of one compute unit (16 waves, a row's every id in each phase) and
// the trips between them, so a kernel is built for 1, 2, 4 and 8 chunks of 4096 ids (a thread's work follows CH, not the ids that
// are there), a draw looks for the largest value and not for its id, and nothing is worked out ahead for the case that rounding
// runs off the end.  Draws from Python 25.1 -> 23.8 us (32000 ids), 24.4 -> 20.4 (8000); acceptance on the device, 5 rows of 32000 14.4 -> 11.4, of 5000
// 14.7 -> 7.2, 2 rows of 1024 13.2 -> 5.9.
// q_out may be the logits themselves: a workgroup has read all it needs of them before it writes.
template <int CH>
__global__ __launch_bounds__(SAMP_THREADS) void sample_row_reg_kernel(const float* logits, int V, float mult, int greedy,
                                                                      float u, float* q_out, int* __restrict__ tok_out) {
  __shared__ MaxIdx shm[SAMP_WAVES];
  __shared__ float shf[SAMP_WAVES];
  __shared__ double shd[SAMP_WAVES];
  __shared__ int shi[1];
  const RegGeom g = reg_geom(V);
  f32x4 e[CH];
  if (greedy) {
    const MaxIdx top = block_argmax(reg_load(logits, V, g, e), shm);
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      f32x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = g.id(k) + i == top.i ? 1.0f : 0.0f;
      if (k < g.R) store4(q_out, g.id(k), V, o);
    }
    if (threadIdx.x == 0) tok_out[0] = top.i;
    return;
  }
  float top, sum;
  reg_softmax(logits, V, mult, g, e, top, sum, shf, shd, [] {});
  const float inv = 1.0f / sum;
#pragma unroll
  for (int k = 0; k < CH; ++k) {
#pragma unroll
    for (int i = 0; i < 4; ++i) e[k][i] *= inv;
    if (k < g.R) store4(q_out, g.id(k), V, e[k]);
  }
  const int tok = reg_draw(e, g, u, 0.0, -1.0, shd, shi, nullptr);
  if (threadIdx.x == 0) tok_out[0] = tok;
}

// ---- rows beyond the registers of a workgroup -----------------------------------------------------
// The draft's q and the target's p of one row are the same bits if its logits are: both sides form the row's maximum and sum
// with the functions of this section, in the same order.  A row is cut into pieces of SAMP_PIECE ids; a piece has a maximum
// and a sum of exp relative to it, and the row's are put together from the pieces'.
struct PieceStat { float top, sum; int i; };     // maximum, sum of exp(mult l - mult top); greedy: arg-max in the row
__device__ __forceinline__ int row_pieces(int V) { return (V + SAMP_PIECE - 1) / SAMP_PIECE; }
__device__ __forceinline__ float long_prob(float l, float mult, float zmax, float sum) { return expf(fmaf(l, mult, -zmax)) / sum; }
// Piece p of a row by the whole workgroup, to every thread (barriers inside).
__device__ __forceinline__ PieceStat piece_stat(const float* row, int V, int p, float mult, int greedy, MaxIdx* shm, float* shf, double* shd) {
  const int first = p * SAMP_PIECE, n = min(SAMP_PIECE, V - first);
  const RegGeom g = reg_geom(SAMP_PIECE);
  f32x4 e[SAMP_PIECE_CHUNKS];
  PieceStat r;
  r.sum = 0.f;
  if (greedy) {
    const MaxIdx top = block_argmax(reg_load(row + first, n, g, e), shm);
    r.top = top.v;
    r.i = top.i == 0x7fffffff ? top.i : first + top.i;
  } else {
    r.top = block_max(reg_load_max(row + first, n, g, e), shf);
    r.i = first;                     // a draw has no use for it
    const float zmax = r.top * mult;
    float acc = 0.f;
#pragma unroll
    for (int k = 0; k < SAMP_PIECE_CHUNKS; ++k) {
#pragma unroll
      for (int j = 0; j < 4; ++j)    // -inf has no mass, also where it is the maximum; NaN stays NaN
        e[k][j] = g.id(k) + j < n && e[k][j] != -INFINITY ? expf(fmaf(e[k][j], mult, -zmax)) : 0.f;
      acc += (e[k][0] + e[k][1]) + (e[k][2] + e[k][3]);
    }
    r.sum = (float)block_sum_d((double)acc, shd);
  }
  return r;
}
// a piece's term of the row's sum
__device__ __forceinline__ double piece_term(PieceStat s, float mult, double zmax) {
  return s.sum != 0.f ? (double)s.sum * exp((double)(s.top * mult) - zmax) : 0.0;
}
// A row's maximum, arg-max and sum from the statistics of its P pieces, by one wave (lane l adds the terms of the pieces
// l, l + 64, ..), to every lane.
__device__ __forceinline__ MaxIdx row_stat(const PieceStat* s, int P, float mult, int greedy, float* sum) {
  const int lane = threadIdx.x & 63;
  MaxIdx m;
  m.v = -INFINITY; m.i = 0x7fffffff;
  for (int p = lane; p < P; p += 64) m = better(m, s[p].top, s[p].i);
  const MaxIdx top = wave_argmax(m);
  *sum = 1.f;
  if (!greedy) {
    const double zmax = (double)(top.v * mult);
    double t = 0.0;
    for (int p = lane; p < P; p += 64) t += piece_term(s[p], mult, zmax);
    *sum = (float)lane_d(wave_scan_d(t), 63);
  }
  return top;
}

// statistics of piece blockIdx.x of row blockIdx.y to stats[row][piece]
__global__ __launch_bounds__(SAMP_THREADS) void piece_stat_kernel(const float* __restrict__ logits, int V, float mult,
                                                                  int greedy, PieceStat* __restrict__ stats) {
  __shared__ MaxIdx shm[SAMP_WAVES];
  __shared__ float shf[SAMP_WAVES];
  __shared__ double shd[SAMP_WAVES];
  const PieceStat s = piece_stat(logits + (size_t)blockIdx.y * V, V, blockIdx.x, mult, greedy, shm, shf, shd);
  if (threadIdx.x == 0) stats[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// Draft draws over a long row: piece_stat_kernel leaves the statistics where the first ids of q go, this kernel writes q
// behind those (a piece per workgroup), draw_kernel the first ids, then draws: 15.4 us at 32769 ids, 19.4 at 128256 (16.1 and
// 36.9 with one launch for q whose workgroups each add up the whole row: bound by the exponentials of one compute unit).
__host__ __device__ static constexpr int sample_head(int P) { return (P * (int)(sizeof(PieceStat) / sizeof(float)) + 3) & ~3; }
__global__ __launch_bounds__(SAMP_THREADS) void sample_piece_kernel(const float* __restrict__ logits, int V, float mult,
                                                                    float* q_out) {
  float sum;
  const float zmax = row_stat(reinterpret_cast<const PieceStat*>(q_out), gridDim.x, mult, 0, &sum).v * mult;
  const int first = blockIdx.x * SAMP_PIECE, end = min(first + SAMP_PIECE, V);
  for (int j = max(first, sample_head(gridDim.x)) + 4 * threadIdx.x; j < end; j += 4 * SAMP_THREADS) {
    f32x4 v = load4(logits, j, V, -INFINITY);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = long_prob(v[i], mult, zmax, sum);
    store4(q_out, j, V, v);
  }
}

// Greedy: every workgroup finds the row's arg-max (the row comes from L2) and writes its piece of the one-hot.  Where that
// takes the place of the logits one workgroup writes all of it: nobody else may still be reading the row.
__global__ __launch_bounds__(SAMP_THREADS) void sample_greedy_kernel(const float* logits, int V, float* q_out, int* __restrict__ tok_out) {
  __shared__ MaxIdx shm[SAMP_WAVES];
  const int first = gridDim.x == 1 ? 0 : blockIdx.x * SAMP_PIECE, end = gridDim.x == 1 ? V : min(first + SAMP_PIECE, V);
  const MaxIdx top = row_argmax(logits, V, shm);
  for (int j = first + 4 * threadIdx.x; j < end; j += 4 * SAMP_THREADS) {
    f32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = j + i == top.i ? 1.0f : 0.0f;
    store4(q_out, j, V, o);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) tok_out[0] = top.i;
}

// q in the place of its logits (nowhere to leave statistics): one workgroup, piece after piece, the same sums
__global__ __launch_bounds__(SAMP_THREADS) void sample_in_place_kernel(const float* logits, int V, float mult, float* q_out) {
  __shared__ MaxIdx shm[SAMP_WAVES];
  __shared__ float shf[SAMP_WAVES];
  __shared__ double shd[SAMP_WAVES];
  const float zmax = row_argmax(logits, V, shm).v * mult;
  double t = 0.0;
  for (int p = 0; p < row_pieces(V); ++p) {
    const PieceStat s = piece_stat(logits, V, p, mult, 0, shm, shf, shd);
    if ((p & 63) == (threadIdx.x & 63)) t += piece_term(s, mult, (double)zmax);
  }
  const float sum = (float)lane_d(wave_scan_d(t), 63);
  for (int j = 4 * threadIdx.x; j < V; j += 4 * SAMP_THREADS) {
    f32x4 v = load4(logits, j, V, -INFINITY);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = long_prob(v[i], mult, zmax, sum);
    store4(q_out, j, V, v);
  }
}

// Inverse-CDF draw from the non-negative weights w[0 .. V) in memory by one workgroup: 16 ranges, one per wave, whose
// sums find the owner; its range again in 16, and so on until a range fits the registers of the workgroup.  Returns
// the id to every thread, -1 if there is no mass.  The barriers inside also separate it from what wrote w.
__device__ int block_draw(const float* __restrict__ w, int V, float u, double* shd, int* shi) {
  __threadfence_block();
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int first = 0, n = V;
  double before = 0.0, target = -1.0;
  while (n > SAMP_PIECE) {
    const int per = ((n + SAMP_WAVES - 1) / SAMP_WAVES + 255) / 256 * 256;
    const int b = first + wv * per, e = min(b + per, first + n);
    double mine = 0.0;
#pragma unroll 4
    for (int j = b + 4 * lane; j < e; j += 256) mine += sum4_d(load4(w, j, e, 0.f));
    mine = wave_scan_d(mine);
    if (lane == 63) shd[wv] = mine;
    __syncthreads();
    const double wt = lane < SAMP_WAVES ? shd[lane] : 0.0;
    __syncthreads();
    const double wincl = wave_scan_d(wt);
    const double total = lane_d(wincl, SAMP_WAVES - 1);
    if (target < 0.0) target = (double)u * total;
    const unsigned long long wmass = __ballot(lane < SAMP_WAVES && wt > 0.0);
    const unsigned long long whit = __ballot(lane < SAMP_WAVES && wt > 0.0 && before + wincl > target);
    if (!wmass) return -1;
    const int owner = whit ? __ffsll((long long)whit) - 1 : 63 - __clzll((long long)wmass);
    if (owner > 0) before += lane_d(wincl, owner - 1);
    const int nb = first + owner * per;
    n = min(per, first + n - nb);
    first = nb;
  }
  const RegGeom g = reg_geom(n);
  f32x4 e[SAMP_PIECE_CHUNKS];
  reg_fetch(w + first, n, g, 0.f, e);
  const int tok = reg_draw(e, g, u, before, target, shd, shi, nullptr);
  return tok < 0 ? -1 : first + tok;
}

// logits: those of sample_piece_kernel (its first ids of q are still missing), or null: all of q is there
__global__ __launch_bounds__(SAMP_THREADS) void draw_kernel(const float* __restrict__ logits, float* q, int V, float mult, float u,
                                                            int* __restrict__ tok_out) {
  __shared__ double shd[SAMP_WAVES];
  __shared__ int shi[1];
  if (logits) {
    const int P = row_pieces(V);
    float sum;
    const float zmax = row_stat(reinterpret_cast<const PieceStat*>(q), P, mult, 0, &sum).v * mult;
    __syncthreads();     // everybody has read the statistics
    for (int j = 4 * threadIdx.x; j < sample_head(P); j += 4 * SAMP_THREADS) {
      f32x4 v = load4(logits, j, V, -INFINITY);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = long_prob(v[i], mult, zmax, sum);
      *reinterpret_cast<f32x4u*>(q + j) = v;
    }
  }
  const int tok = block_draw(q, V, u, shd, shi);
  if (threadIdx.x == 0) tok_out[0] = tok;
}

// GO(CH): the kernel for rows of V ids, V <= SAMP_REG_VOCAB_MAX
#define SAMP_BY_CHUNKS(V, GO)                               \
  switch (((V) + 4 * SAMP_THREADS - 1) / (4 * SAMP_THREADS)) { \
    case 1: GO(1); break;                                   \
    case 2: GO(2); break;                                   \
    case 3: case 4: GO(4); break;                           \
    default: GO(8); break;                                  \
  }
static_assert(SAMP_CHUNKS_MAX == 8, "every length up to SAMP_REG_VOCAB_MAX has its kernel");
hipError_t launch_sample_row(const float* logits, int V, float mult, int greedy, float u, float* q_out, int* tok_out,
                             hipStream_t st) {
  if (V <= SAMP_REG_VOCAB_MAX) {
#define SAMP_GO(CH) sample_row_reg_kernel<CH><<<1, SAMP_THREADS, 0, st>>>(logits, V, mult, greedy, u, q_out, tok_out)
    SAMP_BY_CHUNKS(V, SAMP_GO)
#undef SAMP_GO
    return hipGetLastError();
  }
  const bool in_place = q_out < logits + V && logits < q_out + V;
  const int P = (V + SAMP_PIECE - 1) / SAMP_PIECE;
  if (greedy) {
    sample_greedy_kernel<<<in_place ? 1 : P, SAMP_THREADS, 0, st>>>(logits, V, q_out, tok_out);
    return hipGetLastError();
  }
  if (in_place) {
    sample_in_place_kernel<<<1, SAMP_THREADS, 0, st>>>(logits, V, mult, q_out);
  } else {
    piece_stat_kernel<<<P, SAMP_THREADS, 0, st>>>(logits, V, mult, 0, reinterpret_cast<PieceStat*>(q_out));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    sample_piece_kernel<<<P, SAMP_THREADS, 0, st>>>(logits, V, mult, q_out);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  draw_kernel<<<1, SAMP_THREADS, 0, st>>>(in_place ? nullptr : logits, q_out, V, mult, u, tok_out);
  return hipGetLastError();
}

// ---- target: per-row test, then first rejection + resampling ---------------------------------
// Scratch of an acceptance: [0, 256) four statistics per row: max logit, sum exp, arg-max (as int bits), accept flag;
// then, for vocabularies beyond SAMP_REG_VOCAB_MAX, a PieceStat per (row, piece); the pieces' weight sums (doubles); and the row of V weights a draw walks over.
__host__ __device__ static constexpr int accept_pieces(int V) { return V <= SAMP_REG_VOCAB_MAX ? 0 : (V + SAMP_PIECE - 1) / SAMP_PIECE; }
__host__ __device__ static constexpr size_t accept_sums_at(int V) {
  return 256 + (size_t)accept_pieces(V) * SPEC_MAX_TOKENS * (sizeof(PieceStat) / sizeof(float));
}
__host__ __device__ static constexpr size_t accept_weights_at(int V) { return accept_sums_at(V) + (size_t)accept_pieces(V) * 2; }
static constexpr size_t accept_scratch_floats_of(int V) { return accept_weights_at(V) + (size_t)V; }
size_t accept_scratch_floats(int V) { return accept_scratch_floats_of(V); }

// The draft that row i tests (0 where it tests none), its logit and its q.  A kernel asks for them long before the test: an id and
// then two values behind it are two round trips to memory.
__device__ __forceinline__ int accept_id(int i, const int* __restrict__ ring, const int* __restrict__ x_direct, const AcceptArgs& a) {
  return i >= a.n_test ? 0 : x_direct ? x_direct[i] : ring[a.slot[i]];
}
struct AcceptPair {
  float l = 0.f, q = 0.f;
  __device__ __forceinline__ void load(const float* __restrict__ row, int i, int x, int V, const float* __restrict__ qcache,
                                       const int* __restrict__ x_direct, const AcceptArgs& a) {
    if (i >= a.n_test) return;
    l = row[x];
    q = qcache[(size_t)(x_direct ? i : a.slot[i]) * V + x];
  }
};
// row i's test from its statistics, by one thread
__device__ __forceinline__ int accept_test(int x, const AcceptPair& at, int i, int V, float mult, int greedy, float top, float sum,
                                           int amax, const AcceptArgs& a) {
  if (i >= a.n_test) return 0;
  int acc;
  if (greedy) {
    acc = x == amax;
  } else {
    const float px = V <= SAMP_REG_VOCAB_MAX ? reg_prob(at.l, mult, top * mult, 1.0f / sum) : long_prob(at.l, mult, top * mult, sum);
    acc = (double)a.r[i] * (double)at.q <= (double)px;
  }
  if (a.force_mask >= 0) acc = (int)((a.force_mask >> i) & 1);
  return acc;
}

template <int CH>
__global__ __launch_bounds__(SAMP_THREADS) void accept_rows_kernel(const float* __restrict__ logits, int V, float mult,
                                                                   int greedy, const float* __restrict__ qcache,
                                                                   const int* __restrict__ ring,
                                                                   const int* __restrict__ x_direct, AcceptArgs a,
                                                                   float* __restrict__ stats) {
  __shared__ MaxIdx shm[SAMP_WAVES];
  __shared__ float shf[SAMP_WAVES];
  __shared__ double shd[SAMP_WAVES];
  const int i = blockIdx.x;
  const float* row = logits + (size_t)i * V;
  const RegGeom g = reg_geom(V);
  const int x = accept_id(i, ring, x_direct, a);
  AcceptPair at;
  MaxIdx top = {0.f, 0};
  float sum = 1.f;
  f32x4 e[CH];
  if (greedy) top = block_argmax(reg_load(row, V, g, e), shm);
  else reg_softmax(row, V, mult, g, e, top.v, sum, shf, shd, [&] { at.load(row, i, x, V, qcache, x_direct, a); });
  if (threadIdx.x == 0) {
    stats[i * 4 + 0] = top.v;
    stats[i * 4 + 1] = sum;
    stats[i * 4 + 2] = __int_as_float(top.i);
    stats[i * 4 + 3] = __int_as_float(accept_test(x, at, i, V, mult, greedy, top.v, sum, top.i, a));
  }
}

// long rows: every row's statistics from its pieces', by the whole workgroup, into `st` (LDS, four floats per row)
__device__ void accept_combine(const float* __restrict__ logits, int V, float mult, int greedy,
                               const float* __restrict__ qcache, const int* __restrict__ ring,
                               const int* __restrict__ x_direct, const AcceptArgs& a, const float* __restrict__ scratch,
                               float* st) {
  const int lane = threadIdx.x & 63, P = accept_pieces(V);
  for (int i = threadIdx.x >> 6; i < a.n_rows; i += SAMP_WAVES) {
    float sum;
    const int x = accept_id(i, ring, x_direct, a);
    AcceptPair at;
    if (!greedy) at.load(logits + (size_t)i * V, i, x, V, qcache, x_direct, a);
    const MaxIdx top = row_stat(reinterpret_cast<const PieceStat*>(scratch + 256) + (size_t)i * P, P, mult, greedy, &sum);
    if (lane == 0) {
      st[i * 4 + 0] = top.v;
      st[i * 4 + 1] = sum;
      st[i * 4 + 2] = __int_as_float(top.i);
      st[i * 4 + 3] = __int_as_float(accept_test(x, at, i, V, mult, greedy, top.v, sum, top.i, a));
    }
  }
  __syncthreads();
}

// n = first rejection.  *off_path: a guided test ended at a draft that left the guessed path (row n >= 1 is the
// target's distribution after x_1..x_n only if those are the guesses).
__device__ __forceinline__ int accept_count(const AcceptArgs& a, const int* __restrict__ ring, const float* stats, bool* off_path) {
  int n = 0;
  *off_path = false;
  while (n < a.n_test) {
    if (a.guided && n >= 1 && ring[a.slot[n - 1]] != a.guess[n - 1]) {
      *off_path = true;
      break;
    }
    if (__float_as_int(stats[n * 4 + 3]) == 0) break;
    ++n;
  }
  return n;
}

// long rows: the weights of the draw, norm(max(0, p_n - q_n)) after a rejection, p_n for the row after the last test
__global__ __launch_bounds__(SAMP_THREADS) void accept_weights_kernel(const float* __restrict__ logits, int V, float mult,
                                                                      const float* __restrict__ qcache,
                                                                      const int* __restrict__ ring,
                                                                      const int* __restrict__ x_direct, AcceptArgs a,
                                                                      float* __restrict__ scratch) {
  __shared__ double shd[SAMP_WAVES];
  __shared__ float st[4 * SPEC_MAX_TOKENS];
  accept_combine(logits, V, mult, 0, qcache, ring, x_direct, a, scratch, st);
  if (blockIdx.x == 0 && threadIdx.x < 4 * a.n_rows) scratch[threadIdx.x] = st[threadIdx.x];     // for accept_finish_kernel
  bool off_path;
  const int n = accept_count(a, ring, st, &off_path);
  const bool rejected = !off_path && n < a.n_test;
  if (!rejected && (a.guided || n >= a.n_rows)) return;
  const int p = blockIdx.x, first = p * SAMP_PIECE, m = min(SAMP_PIECE, V - first);
  const float* row = logits + (size_t)n * V + first;
  const float* qrow = nullptr;
  if (rejected) qrow = (x_direct ? qcache + (size_t)n * V : qcache + (size_t)a.slot[n] * V) + first;
  const float zmax = st[n * 4] * mult, sum = st[n * 4 + 1];
  float* wbuf = scratch + accept_weights_at(V) + first;
  const RegGeom g = reg_geom(SAMP_PIECE);
  f32x4 e[SAMP_PIECE_CHUNKS], q[SAMP_PIECE_CHUNKS];
  reg_fetch(row, m, g, 0.f, e);
  if (qrow) reg_fetch(qrow, m, g, 0.f, q);
  double mine = 0.0;
#pragma unroll
  for (int k = 0; k < SAMP_PIECE_CHUNKS; ++k) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float pv = long_prob(e[k][i], mult, zmax, sum);
      e[k][i] = g.id(k) + i < m ? (qrow ? residual(pv, q[k][i]) : pv) : 0.f;
    }
    store4(wbuf, g.id(k), m, e[k]);
    mine += sum4_d(e[k]);
  }
  const double t = block_sum_d(mine, shd);
  if (threadIdx.x == 0) reinterpret_cast<double*>(scratch + accept_sums_at(V))[p] = t;
}

// The draw over row n in registers: residual weights max(0, p - q) (one rounding of the difference of rounded values), or p itself
// (qrow == nullptr; also where the residual has no mass in floating point).
template <int CH>
__device__ __forceinline__ int accept_draw(const float* __restrict__ row, const float* __restrict__ qrow, int V, float mult,
                                           float zmax, float sum, float u, double* shd, int* shi) {
  const float inv = 1.0f / sum;
  int token = -1;
#pragma unroll 1
  for (int attempt = 0; attempt < 2; ++attempt) {
    RegGeom g = reg_geom(V);
    asm volatile("" : "+v"(g.j0));     // keeps the addresses of both rows from being worked out for both attempts
    f32x4 e[CH];
    reg_fetch(row, V, g, -INFINITY, e);
    constexpr int H = CH < 4 ? 1 : CH / 4;
#pragma unroll
    for (int h = 0; h < CH / H; ++h) {      // q in parts: registers
      RegGeom gh = g;
      gh.j0 = g.id(h * H);
      gh.R = g.R - h * H;
      f32x4 q[H];
      if (qrow) reg_fetch(qrow, V, gh, 0.f, q);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < H; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = reg_prob(e[h * H + k][i], mult, zmax, inv);
          e[h * H + k][i] = qrow ? residual(p, q[k][i]) : p;
        }
    }
    reg_clear_rest(V, mult, g, e);
    double total = 0.0;
    token = reg_draw(e, g, u, 0.0, -1.0, shd, shi, &total);
    if (!qrow || total > 0.0) break;
    qrow = nullptr;
    __syncthreads();
  }
  return token;
}

// The same for a long row: the piece the draw falls into (accept_weights_kernel left the weights and their sums), then
// the walk inside it.
__device__ __forceinline__ int accept_draw_long(const float* __restrict__ row, bool rejected, int V, float mult, float zmax,
                                                float sum, float u, float* __restrict__ scratch, double* shd, int* shi) {
  float* wbuf = scratch + accept_weights_at(V);
  const double* sums = reinterpret_cast<const double*>(scratch + accept_sums_at(V));
  const int P = accept_pieces(V), lane = threadIdx.x & 63;
  double total = 0.0;
  for (int p0 = 0; p0 < P; p0 += 64) total += lane_d(wave_scan_d(p0 + lane < P ? sums[p0 + lane] : 0.0), 63);
  if (rejected && !(total > 0.0)) {   // no residual mass in floating point: draw from p itself
    for (int j = threadIdx.x; j < V; j += SAMP_THREADS) wbuf[j] = long_prob(row[j], mult, zmax, sum);
    return block_draw(wbuf, V, u, shd, shi);
  }
  const double target = (double)u * total;
  double before = 0.0, ahead = 0.0;
  int piece = -1, last = -1;
  for (int p0 = 0; p0 < P && piece < 0; p0 += 64) {
    const double s = p0 + lane < P ? sums[p0 + lane] : 0.0;
    const double incl = wave_scan_d(s);
    const unsigned long long mass = __ballot(s > 0.0), hit = __ballot(s > 0.0 && before + incl > target);
    const int l = hit ? __ffsll((long long)hit) - 1 : (mass ? 63 - __clzll((long long)mass) : -1);
    if (l >= 0) {
      last = p0 + l;
      ahead = before + (lane_d(incl, l) - lane_d(s, l));
      if (hit) piece = last;
    }
    before += lane_d(incl, 63);
  }
  if (piece < 0) piece = last;      // rounding: the last piece with mass
  if (piece < 0) return -1;
  const int first = piece * SAMP_PIECE, m = min(SAMP_PIECE, V - first);
  const RegGeom g = reg_geom(SAMP_PIECE);
  f32x4 e[SAMP_PIECE_CHUNKS];
  reg_fetch(wbuf + first, m, g, 0.f, e);
  const int t = reg_draw(e, g, u, ahead, target, shd, shi, nullptr);
  return t < 0 ? -1 : first + t;
}

// One workgroup: n = first rejection; draw from norm(max(0, p_n - q_n)) (from p_n if that has no
// mass), or the bonus / autoregressive token from the row after the last test.  CH: chunks of a row, 0 for a long one.
template <int CH>
__global__ __launch_bounds__(SAMP_THREADS) void accept_finish_kernel(const float* __restrict__ logits, int V,
                                                                     float mult, int greedy,
                                                                     const float* __restrict__ qcache,
                                                                     const int* __restrict__ ring,
                                                                     const int* __restrict__ x_direct, AcceptArgs a,
                                                                     float* __restrict__ scratch,
                                                                     AcceptResult* __restrict__ res,
                                                                     int* __restrict__ out2) {
  __shared__ double shd[SAMP_WAVES];
  __shared__ int shi[1];
  __shared__ float st[4 * SPEC_MAX_TOKENS];
  constexpr bool LONG = CH == 0;
  if (LONG && greedy) accept_combine(logits, V, mult, greedy, qcache, ring, x_direct, a, scratch, st);
  const float* stats = LONG && greedy ? st : scratch;
  bool off_path;
  const int n = accept_count(a, ring, stats, &off_path);
  const bool rejected = !off_path && n < a.n_test;
  int token = -1;
  if (rejected || (!a.guided && n < a.n_rows)) {   // a row to draw from exists: the rejecting row, or the bonus row
    const float* row = logits + (size_t)n * V;
    const float zmax = stats[n * 4 + 0] * mult, sum = stats[n * 4 + 1];
    if (greedy) {
      token = __float_as_int(stats[n * 4 + 2]);   // residual of two one-hots, or the one-hot itself, is the target's arg-max
    } else if constexpr (LONG) {
      token = accept_draw_long(row, rejected, V, mult, zmax, sum, a.u_resample, scratch, shd, shi);
    } else {
      const float* qrow = nullptr;
      if (rejected) qrow = x_direct ? qcache + (size_t)n * V : qcache + (size_t)a.slot[n] * V;
      token = accept_draw<CH>(row, qrow, V, mult, zmax, sum, a.u_resample, shd, shi);
    }
  }
  if (threadIdx.x == 0) {
    res->n_accepted = n;
    res->token = token;
    res->rejected = rejected ? 1 : 0;
    res->off_path = off_path ? 1 : 0;
    if (out2) {   // callers that want the outcome in device memory of their own
      out2[0] = n;
      out2[1] = token;
    }
  }
  if (ring && threadIdx.x < SPEC_RING_MAX) res->ring[threadIdx.x] = ring[threadIdx.x];
}

hipError_t launch_accept(const float* logits, int V, float mult, int greedy, const float* qcache, const int* ring,
                         const int* x_direct, AcceptArgs a, float* scratch, AcceptResult* result_dev,
                         hipStream_t st, int* out2) {
  if (a.guided && !ring) return hipErrorInvalidValue;   // guided tests compare ring tokens with the guesses
  const int P = accept_pieces(V);
  if (!P) {
#define ROWS_GO(CH) accept_rows_kernel<CH><<<a.n_rows, SAMP_THREADS, 0, st>>>(logits, V, mult, greedy, qcache, ring, x_direct, a, scratch)
    SAMP_BY_CHUNKS(V, ROWS_GO)
#undef ROWS_GO
  } else {
    piece_stat_kernel<<<dim3(P, a.n_rows), SAMP_THREADS, 0, st>>>(logits, V, mult, greedy, reinterpret_cast<PieceStat*>(scratch + 256));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!greedy) accept_weights_kernel<<<P, SAMP_THREADS, 0, st>>>(logits, V, mult, qcache, ring, x_direct, a, scratch);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
#define FINISH_GO(CH) \
  accept_finish_kernel<CH><<<1, SAMP_THREADS, 0, st>>>(logits, V, mult, greedy, qcache, ring, x_direct, a, scratch, result_dev, out2)
  if (P) FINISH_GO(0);
  else SAMP_BY_CHUNKS(V, FINISH_GO)
#undef FINISH_GO
  return hipGetLastError();
}

// ---- acceptance without any allocation ---------------------------------------------------------
// The scratch of the two acceptance kernels (row statistics, one row of draw weights, the result record) in a
// file-scope device array instead of memory from hipMalloc: for callers that must not allocate (code under HIP
// graph capture, tight serving loops).  Every GPU the library runs on holds its own copy of the array until the
// process ends; its address on a device is looked up once, with that device current.  All calls on one GPU share
// the array, so calls that overlap on one GPU (two streams, two threads) race; nothing in it has to start at zero
// (every word a call reads was written by that call before).
#define ACCEPT_STATIC_FLOATS accept_scratch_floats_of(SPEC_STATIC_VOCAB_MAX)
#define ACCEPT_STATIC_BYTES (ACCEPT_STATIC_FLOATS * 4 + 512)
static __device__ __align__(256) unsigned char scratch[ACCEPT_STATIC_BYTES];

#include <mutex>
#define ACCEPT_STATIC_MAX_DEVICES 64
static void* g_scratch_ptr[ACCEPT_STATIC_MAX_DEVICES];
static std::mutex g_scratch_mutex;

// device address of `scratch` on the current device (nullptr and an error message on failure)
static void* static_scratch_ptr() {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= ACCEPT_STATIC_MAX_DEVICES) {
    spec_set_error("hipGetDevice failed or device id %d above %d: %s", dev, ACCEPT_STATIC_MAX_DEVICES - 1,
                   hipGetErrorString(e));
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      spec_set_error("hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
      return nullptr;
    }
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

extern "C" int spec_accept_rows_static(const float* p_logits, int n_rows, const float* q_rows, const int32_t* x,
                                       int n_test, int vocab, float temperature, float logit_scale, const float* r,
                                       float u_resample, int32_t* result_dev, void* stream) {
  if (!p_logits || !result_dev || vocab < 1 || n_rows < 1 || n_rows > SPEC_MAX_TOKENS || n_test < 0 || n_test > n_rows) {
    spec_set_error("bad argument");
    return SPEC_E_INVAL;
  }
  if (vocab > SPEC_STATIC_VOCAB_MAX) {
    spec_set_error("vocabulary of %d ids is above the %d the static scratch holds; use spec_accept_rows", vocab,
                   SPEC_STATIC_VOCAB_MAX);
    return SPEC_E_INVAL;
  }
  if (n_test > 0 && (!q_rows || !x || !r)) {
    spec_set_error("null pointer");
    return SPEC_E_INVAL;
  }
  if (!(temperature >= 0.0f) || !(logit_scale > 0.0f) || !(u_resample >= 0.0f && u_resample < 1.0f)) {
    spec_set_error("bad temperature / logit_scale / uniform");
    return SPEC_E_INVAL;
  }
  static_assert(4 * SPEC_MAX_TOKENS <= 256, "four statistics per row");
  static_assert(sizeof(AcceptResult) <= 512, "the result record sits in the last 512 bytes");
  unsigned char* base = (unsigned char*)static_scratch_ptr();
  if (!base) return SPEC_E_HIP;
  AcceptArgs a;
  memset(&a, 0, sizeof(a));
  a.n_rows = n_rows;
  a.n_test = n_test;
  a.u_resample = u_resample;
  a.force_mask = -1;
  for (int i = 0; i < n_test; ++i) {
    if (!(r[i] >= 0.0f && r[i] < 1.0f)) {
      spec_set_error("uniform outside [0,1)");
      return SPEC_E_INVAL;
    }
    a.r[i] = r[i];
  }
  const bool greedy = temperature == 0.0f;
  float* stats = (float*)base;   // all of the scratch
  AcceptResult* res = (AcceptResult*)(base + ACCEPT_STATIC_FLOATS * 4);
  hipError_t e = launch_accept(p_logits, vocab, greedy ? 1.0f : logit_scale / temperature, greedy ? 1 : 0, q_rows,
                               nullptr, x, a, stats, res, (hipStream_t)stream, result_dev);
  if (e != hipSuccess) {
    spec_set_error("accept kernels failed to launch: %s", hipGetErrorString(e));
    return SPEC_E_HIP;
  }
  return SPEC_OK;
}

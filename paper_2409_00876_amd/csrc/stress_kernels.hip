// Stress kernels for gfx950: the sampled path stress of Eq. 2 with its CI95
// (one pass), the differentiable loss and its adjoint, the initial layout and a
// fused Adam step.
//
// Stress terms are evaluated in FP64 from the float32 coordinates with FMA
// contraction off, so each term is the exactly rounded value of
// ((|v_i - v_j| - d)/d)^2; block partials are FP64 and reduced in a fixed
// order, so results are deterministic for a given launch shape.
#include <algorithm>
#include <type_traits>

#include "device.h"
#include "internal.h"
#include "stress.h"

namespace pgsgd {

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sums over the block; the result is valid in thread 0.
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* scratch) {
  v = wave_sum(v);
  const uint32_t w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if ((threadIdx.x & 63u) == 0) scratch[w] = v;
  __syncthreads();
  T r = 0;
  if (threadIdx.x == 0)
    for (uint32_t k = 0; k < nw; ++k) r += scratch[k];
  __syncthreads();
  return r;
}

__device__ __forceinline__ void fill_offsets(uint64_t* off, const StressLaunch& P) {
  for (uint32_t k = threadIdx.x; k < P.path_slots; k += blockDim.x) off[k] = k <= P.n_paths ? P.path_off[k] : ~0ull;
}

// Stress of one pair of slots in FP64.  Returns false when d == 0.
__device__ __forceinline__ bool pair_terms(const StepRec* __restrict__ rec, uint64_t i, uint64_t j, uint32_t ei,
                                           uint32_t ej, uint64_t& a, uint64_t& b, double& d) {
  const StepRec si = load_rec(rec, i);
  const StepRec sj = load_rec(rec, j);
  const int64_t dd = endpoint_pos(si, ei) - endpoint_pos(sj, ej);
  a = 2ull * (si.node_rev & kNodeMask) + ei;
  b = 2ull * (sj.node_rev & kNodeMask) + ej;
  d = (double)(dd < 0 ? -dd : dd);
  return dd != 0;
}

// ((|v_a - v_b| - d)/d)^2 in FP64 from the two endpoints' float32 coordinates.
__device__ __forceinline__ double stress_xy(float xa, float ya, float xb, float yb, double d) {
#pragma clang fp contract(off)
  const double dx = (double)xa - (double)xb;
  const double dy = (double)ya - (double)yb;
  const double mag = sqrt(dx * dx + dy * dy);
  const double e = (mag - d) / d;
  return e * e;
}

// sqrt(x) for x = 0 or in [2^-300, 2^260], and n / d for quotients well inside
// FP64's range (float32 coordinates and lengths below 2^63 cannot leave
// either), correctly rounded as by sqrt and /: the compiler's own sequences
// without their scaling, Goldschmidt's iteration for the root and Newton's for
// the reciprocal, each with a last step on the residual (Markstein, IBM J. Res.
// Dev. 34, 1990).  NaN where an argument is infinite.
__device__ __forceinline__ double root64(double x) {
  const double y = __builtin_amdgcn_rsq(__builtin_fmax(x, 0x1p-1000));  // x = 0 gives 0 below
  double g = x * y, h = 0.5 * y;
  const double r = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
  return __builtin_fma(__builtin_fma(-g, g, x), h, g);
}

__device__ __forceinline__ double quotient64(double n, double d) {
#pragma clang fp contract(off)
  double c = __builtin_amdgcn_rcp(d);
  c = __builtin_fma(c, __builtin_fma(-d, c, 1.0), c);
  c = __builtin_fma(c, __builtin_fma(-d, c, 1.0), c);
  const double q = n * c;
  return __builtin_fma(__builtin_fma(-d, q, n), c, q);
}

// ((|v| - d) / d)^2 for v = (dx, dy) and 1 <= d < 2^63; NaN where |v| is infinite.
__device__ __forceinline__ double exact_stress(double dx, double dy, double d) {
#pragma clang fp contract(off)
  const double e = quotient64(root64(dx * dx + dy * dy) - d, d);
  return e * e;
}

// stress_xy by the short sequences, taken again the general way where it is not finite.
__device__ __forceinline__ double pair_stress(float2 va, float2 vb, double d) {
  const double st = exact_stress((double)va.x - (double)vb.x, (double)va.y - (double)vb.y, d);
  return st - st == 0.0 ? st : stress_xy(va.x, va.y, vb.x, vb.y, d);
}

// v_a - v_b in FP64; returns |v_a - v_b|.
__device__ __forceinline__ double delta_xy(float2 va, float2 vb, double& dx, double& dy) {
#pragma clang fp contract(off)
  dx = (double)va.x - (double)vb.x;
  dy = (double)va.y - (double)vb.y;
  return root64(dx * dx + dy * dy);
}

// scale (mag - d) / d^2 / mag, the factor of (dx, dy) in a pair's gradient;
// taken again the general way where it is not finite (an infinite grad_out).
__device__ __forceinline__ double gradient_factor(double scale, double mag, double d) {
#pragma clang fp contract(off)
  const double c = quotient64(quotient64(scale * (mag - d), d * d), mag);
  return c - c == 0.0 ? c : scale * (mag - d) / (d * d) / mag;
}

// The stress of endpoints a and b of the interleaved copy (W[e] = (x, y) of endpoint e).
__device__ __forceinline__ double stress_work(const float2* __restrict__ W, uint64_t a, uint64_t b, double d) {
  return pair_stress(W[a], W[b], d);
}

// Outlier collection: a pair whose stress exceeds the threshold is
// appended (slot from one atomic; the first out_max are kept).
__device__ __forceinline__ void keep_outlier(const StressLaunch& P, uint64_t i, uint64_t j, uint32_t e, double st) {
  if (!P.out_count || !(st > P.out_threshold)) return;
  const unsigned long long k = atomicAdd(reinterpret_cast<unsigned long long*>(P.out_count), 1ull);
  if (k < P.out_max) {
    P.out_i[k] = i;
    P.out_j[k] = j;
    P.out_e[k] = (uint8_t)e;
    P.out_s[k] = st;
  }
}

// A running sum with its rounding errors: hi is the plain FP64 sum, lo the sum
// of what its additions rounded away (two-sum), so hi + lo carries about twice
// FP64's digits.  hi is never renormalised, so infinities and NaN come out of
// it as they would of the plain sum.
struct Sum2 {
  double hi = 0.0, lo = 0.0;
  __device__ __forceinline__ void add(double x) {
#pragma clang fp contract(off)
    const double s = hi + x, b = s - hi;
    lo += (hi - (s - b)) + (x - b);
    hi = s;
  }
  __device__ __forceinline__ void add_product(double x, double y) {
#pragma clang fp contract(off)
    const double p = x * y;
    add(p);
    lo += __builtin_fma(x, y, -p);
  }
  __device__ __forceinline__ void add(const Sum2& o) {
    add(o.hi);
    lo += o.lo;
  }
};

// What one pass over the pairs leaves of the sampled path stress: the sums and
// the sums of squares and products of the stress a of a layout and, kPair, of
// the stress b of a second one on the same pairs.  The deviations about a mean
// or a ratio, sum (a - mean)^2 and sum (a - R b)^2, follow from them on the
// host; the sums carry enough digits for the cancellation (equal stresses give
// 0), which a second pass over the pairs paid for before.
constexpr size_t kSpsLds = (5 * 2 + 2) * 16 * 8;

template <bool kPair>
struct SpsAcc {
  static constexpr uint32_t kSums = kPair ? 5 : 2;  // a, aa[, b, bb, ab]
  Sum2 v[kSums];
  uint64_t nv = 0, ns = 0;

  // The stress of endpoints a and b, and with two layouts the second one's (sb).
  // The two layouts' coordinates lie side by side, one line an endpoint: a pair's
  // lines, not its arithmetic, bound the kernel (2.9e7 power-law pairs, 303K nodes: 1.91 ms apart, 1.32 so).
  static __device__ __forceinline__ double stress(const StressLaunch& P, uint64_t a, uint64_t b, double d, double& sb) {
    if constexpr (kPair) {
      const float4* lo = reinterpret_cast<const float4*>(P.work);
      const float4* hi = reinterpret_cast<const float4*>(P.work2) - P.n_nodes;
      const float4 va = (a < P.n_nodes ? lo : hi)[a], vb = (b < P.n_nodes ? lo : hi)[b];
      sb = pair_stress(make_float2(va.z, va.w), make_float2(vb.z, vb.w), d);
      return pair_stress(make_float2(va.x, va.y), make_float2(vb.x, vb.y), d);
    }
    return stress_work(P.work, a, b, d);
  }

  __device__ __forceinline__ void take(double st, double sb) {
    ++nv;
    v[0].add(st);
    v[1].add_product(st, st);
    if constexpr (kPair) {
      v[2].add(sb);
      v[3].add_product(sb, sb);
      v[4].add_product(st, sb);
    }
  }

  // Block sums into column `block` of the rows (row q * 2 + {hi, lo}) of part_f
  // and into the counts, by way of the block's dynamic LDS (kSpsLds bytes),
  // whose tables are no longer read.
  __device__ __forceinline__ void write(char* lds, uint32_t block, uint32_t stride, double* __restrict__ part_f,
                                        uint64_t* __restrict__ part_n, uint64_t* __restrict__ part_skip) {
    double(*red)[2][16] = reinterpret_cast<double(*)[2][16]>(lds);  // [kSums]
    uint64_t(*red_n)[16] = reinterpret_cast<uint64_t(*)[16]>(lds + kSums * 2 * 16 * 8);
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (uint32_t q = 0; q < kSums; ++q) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        Sum2 x;
        x.hi = __shfl_xor(v[q].hi, o, 64);
        x.lo = __shfl_xor(v[q].lo, o, 64);
        v[q].add(x);
      }
      if (lane == 0) {
        red[q][0][w] = v[q].hi;
        red[q][1][w] = v[q].lo;
      }
    }
    nv = wave_sum(nv);
    ns = wave_sum(ns);
    if (lane == 0) {
      red_n[0][w] = nv;
      red_n[1][w] = ns;
    }
    __syncthreads();
    if (threadIdx.x < kSums) {
      Sum2 t;
      for (uint32_t k = 0; k < nw; ++k) {
        t.add(red[threadIdx.x][0][k]);
        t.lo += red[threadIdx.x][1][k];
      }
      part_f[(size_t)(2 * threadIdx.x) * stride + block] = t.hi;
      part_f[(size_t)(2 * threadIdx.x + 1) * stride + block] = t.lo;
    } else if (threadIdx.x - kSums < 2) {
      uint64_t t = 0;
      for (uint32_t k = 0; k < nw; ++k) t += red_n[threadIdx.x - kSums][k];
      (threadIdx.x == kSums ? part_n : part_skip)[block] = t;
    }
  }
};

// ---------------------------------------------------------------------------
// Sampled path stress; step s owns pairs q = m*s .. m*s+m-1, which all belong
// to the path of s.  A thread takes `per` consecutive pairs of a step: per = m
// on graphs with a step for every thread of the chip, fewer on smaller ones,
// whose few steps would otherwise leave it idle while each thread waits for
// one pair's memory after another (14K steps, m = 100: a call took 198 us with
// 57 busy blocks and a second pass, 43 us with chunks of 3 pairs and one pass;
// 2.9e6 steps in 16 paths, m = 10, two layouts: 3.9 and 1.9 ms).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void fill_loss_lds(char* lds, const StressLaunch& P, uint64_t*& off, uint32_t*& zipf,
                                              uint16_t*& guide);

// mode 0: uniform partner in the path (Eq. 2); mode 1: the power-law partner
// of the layout's cooling phase (same draw words; no partner in a single-step
// path: the pair is skipped).
template <bool kPair>
__global__ __launch_bounds__(kPair ? 1024 : 512) void k_sps(StressLaunch P, int mode, uint32_t per, uint32_t chunks,
                                                            double* __restrict__ part_f,
                                                            uint64_t* __restrict__ part_n,
                                                            uint64_t* __restrict__ part_skip) {
  extern __shared__ __align__(16) char lds[];
  uint64_t* off;
  uint32_t* zipf;
  uint16_t* guide;
  if (mode == 1) {
    fill_loss_lds(lds, P, off, zipf, guide);
  } else {
    off = reinterpret_cast<uint64_t*>(lds);
    zipf = nullptr;
    guide = nullptr;
    fill_offsets(off, P);
  }
  __syncthreads();
  SpsAcc<kPair> acc;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t total = P.S * chunks;  // at most the threads of the grid when chunks > 1
  for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < total; u += stride) {
    const uint32_t chunk = chunks > 1 ? (uint32_t)u / (uint32_t)P.S : 0u;
    const uint64_t s = u - (uint64_t)chunk * P.S;
    const uint32_t p = find_path(off, P.path_top, s);
    const uint64_t start = off[p], len = off[p + 1] - start;
    const uint32_t k_end = (uint32_t)min((uint64_t)P.m, ((uint64_t)chunk + 1) * per);
    for (uint32_t k = chunk * per; k < k_end; ++k) {
      const uint64_t q = (uint64_t)P.m * s + k;
      const Rand4 r = philox10((uint32_t)q, (uint32_t)(q >> 32), 0u, P.c3, P.k0, P.k1);
      const uint64_t i = start + mulhi64(r.r0, r.r1, (uint32_t)len);
      uint64_t j;
      if (mode == 1) {
        if (!partner_power_law(i, start, len, r.r2, r.r3, zipf, guide, P.W, j)) {
          ++acc.ns;
          continue;
        }
      } else {
        j = start + mulhi32(r.r2, (uint32_t)len);
      }
      uint64_t a, b;
      double d;
      if (!pair_terms(P.rec, i, j, r.r3 & 1u, (r.r3 >> 1) & 1u, a, b, d)) {
        ++acc.ns;
        continue;
      }
      double sb = 0.0;
      const double st = acc.stress(P, a, b, d, sb);
      keep_outlier(P, i, j, r.r3 & 3u, st);
      acc.take(st, sb);
    }
  }
  acc.write(lds, blockIdx.x, gridDim.x, part_f, part_n, part_skip);
}

// ---------------------------------------------------------------------------
// Sampled path stress in window-major order.  The pairs of Eq. 2 keep their
// law (path p receives m|p| pairs, i and j independent and uniform in p) and
// are listed segment by segment: segment g (a window of 2^win_shift steps cut
// at path boundaries) receives the number n_g of the plain pair draws whose
// step i falls in it, and slot u (numbered consecutively over the segments)
// draws i uniformly in its segment and j uniformly in its path from the slot
// stream at counter u.  XCD x (blocks b with b mod 8 = x) walks the segments
// of run x with all its waves, 64 slots per wave and item, so the i side of
// the pairs (records and coordinates of one window) stays in the XCD's L2 and
// only the j side reaches into the rest of the path.  The waves take their
// items from one counter per run, so they all stay near the same window (a
// static share per wave drifts apart over thousands of items); the FP64
// block sums then depend on which wave took which item, so a result is
// reproducible up to the rounding of that sum order.
// ---------------------------------------------------------------------------
namespace {

constexpr uint64_t kSpsGrab = 4;  // items a wave takes from its run's counter at once

// loads at wave-uniform addresses through the constant address space (scalar loads)
template <typename T>
__device__ __forceinline__ T uload(const T* p) {
  return *(const __attribute__((address_space(4))) T*)(p);
}

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
  return ((uint64_t)uniform_u32((uint32_t)(v >> 32)) << 32) | uniform_u32((uint32_t)v);
}

}  // namespace

// The segment histogram: step s owns the plain pairs q = m*s .. m*s+m-1 (all
// of the path of s); each draws its i as k_sps does and counts its segment.
// With loss_pairs set, the loss's plain pairs q < loss_pairs are counted
// instead.  The segments start at the window starts and the path starts, so
// step i of path p lies in segment (i >> win_shift) + path_extra[p], the path
// starts inside windows up to that of p (a search of the window's segments,
// with three random loads, bound the count of 1e7 loss pairs: 70 us, now 54).
__global__ __launch_bounds__(1024) void k_sps_win_count(SpsWinLaunch W) {
  extern __shared__ __align__(16) char lds[];
  const StressLaunch& P = W.P;
  uint64_t* off = reinterpret_cast<uint64_t*>(lds);
  uint32_t* hist = reinterpret_cast<uint32_t*>(lds + (size_t)P.path_slots * 8);
  fill_offsets(off, P);
  for (uint32_t k = threadIdx.x; k < W.n_seg; k += blockDim.x) hist[k] = 0;
  __syncthreads();
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  // the loss's pairs (reading R22): pair q < loss_pairs draws i uniformly over all steps
  for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < W.loss_pairs; q += stride) {
    const Rand4 r = philox10((uint32_t)q, (uint32_t)(q >> 32), P.word2, P.c3, P.k0, P.k1);
    const uint64_t i = uniform_mulhi64(r.r0, r.r1, P.S);
    const uint32_t p = find_path(off, P.path_top, i);
    atomicAdd(&hist[W.path_extra[p] + (uint32_t)(i >> W.win_shift)], 1u);
  }
  const uint64_t sps_steps = W.loss_pairs ? 0 : P.S;
  for (uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; s < sps_steps; s += stride) {
    const uint32_t p = find_path(off, P.path_top, s);
    const uint64_t start = off[p], len = off[p + 1] - start;
    const uint32_t extra = W.path_extra[p];
    for (uint32_t k = 0; k < P.m; ++k) {
      const uint64_t q = (uint64_t)P.m * s + k;
      const Rand4 r = philox10((uint32_t)q, (uint32_t)(q >> 32), 0u, P.c3, P.k0, P.k1);
      const uint64_t i = start + mulhi64(r.r0, r.r1, (uint32_t)len);
      atomicAdd(&hist[extra + (uint32_t)(i >> W.win_shift)], 1u);
    }
  }
  __syncthreads();
  for (uint32_t k = threadIdx.x; k < W.n_seg; k += blockDim.x)
    if (hist[k]) atomicAdd(&W.count[k], hist[k]);
}

// One wave: out[k] = before + the sum of f(0 .. k - 1) for k < n, 256 at a time; returns before + the sum of all.
template <typename F>
__device__ __forceinline__ uint64_t wave_prefix(uint32_t n, uint64_t before, uint64_t* __restrict__ out, F f) {
  const uint32_t lane = threadIdx.x & 63u;
  for (uint32_t k0 = 0; k0 < n; k0 += 256) {
    const uint32_t k = k0 + 4 * lane;
    uint64_t v[4], x = 0;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      v[u] = x;
      x += k + u < n ? f(k + u) : 0;
    }
    const uint64_t mine = x;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
      const uint64_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u)
      if (k + u < n) out[k + u] = before + x - mine + v[u];
    before += __shfl(x, 63, 64);
  }
  return before;
}

// One wave: the sum of f(0 .. n - 1), in every lane.
template <typename F>
__device__ __forceinline__ uint64_t wave_total(uint32_t n, F f) {
  uint64_t v = 0;
  for (uint32_t k = threadIdx.x & 63u; k < n; k += 64) v += f(k);
#pragma unroll
  for (uint32_t d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// One block of 1024 threads: seg_off = exclusive prefix of the counts and, with
// `runs`, the per-run item prefixes and zeroed item counters (the passes by
// tiles read seg_off alone).  The histogram is read into LDS (and cleared for
// the next use); each of the 16 waves then scans a contiguous part, 256
// neighbours at a time (four a lane), and each half of a run's items the same
// way, so loads and stores are coalesced (a chunk per thread stored 64 lines a
// wave): 24 us
// for the 1e7 loss pairs of a million backbone nodes, now 13.
__global__ __launch_bounds__(1024) void k_sps_win_scan(SpsWinLaunch W, uint32_t runs) {
  extern __shared__ __align__(16) char lds[];
  __shared__ uint64_t sums[16];
  uint32_t* cnt = reinterpret_cast<uint32_t*>(lds);
  const uint32_t n = W.n_seg;
  constexpr uint32_t kBatch = 8;  // loads in flight
  for (uint32_t k = threadIdx.x; k < n; k += kBatch * 1024) {
    uint32_t c[kBatch];
#pragma unroll
    for (uint32_t u = 0; u < kBatch; ++u) c[u] = k + u * 1024 < n ? W.count[k + u * 1024] : 0;
#pragma unroll
    for (uint32_t u = 0; u < kBatch; ++u)
      if (k + u * 1024 < n) {
        cnt[k + u * 1024] = c[u];
        W.count[k + u * 1024] = 0;
      }
  }
  if (runs && threadIdx.x < 2 * kXcds) W.queue[(size_t)threadIdx.x * 16] = 0;
  __syncthreads();
  const uint32_t wave = uniform_u32(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  const uint32_t part = (n + 15) / 16;
  const uint32_t k0 = min(n, wave * part), nk = min(n, k0 + part) - k0;
  const uint64_t mine = wave_total(nk, [&](uint32_t k) { return (uint64_t)cnt[k0 + k]; });
  if (lane == 0) sums[wave] = mine;
  __syncthreads();
  uint64_t before = 0;
  for (uint32_t w = 0; w < wave; ++w) before += sums[w];
  const uint64_t end = wave_prefix(nk, before, W.seg_off + k0, [&](uint32_t k) { return (uint64_t)cnt[k0 + k]; });
  if (wave == 15 && lane == 0) W.seg_off[n] = end;
  if (!runs) return;
  static_assert(2 * kXcds == 16, "two waves of the block per run");
  const uint32_t run = wave >> 1;  // run x: segments [sbeg[x], sbeg[x + 1])
  const uint32_t b = W.sbeg[run], nq = W.sbeg[run + 1] - b, half = (nq + 1) / 2;
  uint64_t* xi = W.xitem + (size_t)run * W.xstride;
  auto items = [&](uint32_t q) { return ((uint64_t)cnt[b + q] + 63) >> 6; };
  if ((wave & 1) == 0) {
    wave_prefix(half, 0, xi, items);
  } else {
    const uint64_t all = wave_prefix(nq - half, wave_total(half, items), xi + half,
                                     [&](uint32_t q) { return items(half + q); });
    if (lane == 0) xi[nq] = all;
  }
}

// The waves of XCD x take the items of run x from its counter,
// kSpsGrab at a time; every wave leaves once the counter has passed the run's
// last item.
template <bool kPair>
__global__ __launch_bounds__(kPair ? 1024 : 512) void k_sps_win(SpsWinLaunch W, double* __restrict__ part_f,
                                                                uint64_t* __restrict__ part_n,
                                                                uint64_t* __restrict__ part_skip) {
  extern __shared__ __align__(16) char lds[];
  const StressLaunch& P = W.P;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t x = blockIdx.x % kXcds;
  const uint32_t gb = uload(W.sbeg + x);
  const uint32_t nq = uload(W.sbeg + x + 1) - gb;
  const uint64_t* __restrict__ xi = W.xitem + (size_t)x * W.xstride;
  const uint64_t n_items = uniform_u64(uload(xi + nq));
  unsigned long long* ctr = reinterpret_cast<unsigned long long*>(W.queue + (size_t)x * 16);
  SpsAcc<kPair> acc;
  uint32_t q = 0;
  for (uint64_t m = 0, m_end = 0;; ++m) {
    if (m >= m_end) {
      uint64_t base = 0;
      if (lane == 0) base = atomicAdd(ctr, (unsigned long long)kSpsGrab);
      m = uniform_u64(base);
      if (m >= n_items) break;
      m_end = min(m + kSpsGrab, n_items);
    }
    while (q + 1 < nq && uniform_u64(uload(xi + q + 1)) <= m) q = uniform_u32(q + 1);
    const uint32_t g = gb + q;
    const uint64_t u0 = uniform_u64(uload(W.seg_off + g)) + (m - uniform_u64(uload(xi + q))) * 64;
    const uint64_t u_end = uniform_u64(uload(W.seg_off + g + 1));
    const uint64_t sst = uniform_u64(uload(W.seg_start + g));
    const uint64_t slen = uniform_u64(uload(W.seg_start + g + 1)) - sst;
    const uint32_t p = uniform_u32(uload(W.seg_path + g));
    const uint64_t pst = uniform_u64(uload(P.path_off + p));
    const uint64_t plen = uniform_u64(uload(P.path_off + p + 1)) - pst;
    const uint64_t u = u0 + lane;
    if (u < u_end) {
      const Rand4 r = philox10((uint32_t)u, (uint32_t)(u >> 32), 0u, W.slot_c3, P.k0, P.k1);
      const uint64_t i = sst + mulhi64(r.r0, r.r1, (uint32_t)slen);
      const uint64_t j = pst + mulhi32(r.r2, (uint32_t)plen);
      uint64_t a, b;
      double d;
      if (!pair_terms(P.rec, i, j, r.r3 & 1u, (r.r3 >> 1) & 1u, a, b, d)) {
        ++acc.ns;
      } else {
        double sb = 0.0;
        const double st = acc.stress(P, a, b, d, sb);
        keep_outlier(P, i, j, r.r3 & 3u, st);
        acc.take(st, sb);
      }
    }
  }
  acc.write(lds, blockIdx.x, gridDim.x, part_f, part_n, part_skip);
}

// ---------------------------------------------------------------------------
// Path stress, Eq. 1: for every path and every step pair i < j of it, the mean
// of the stress over the endpoint combinations with d > 0; averaged over all
// pairs.  O(sum |p|^2) work: for small graphs and for validating the sampled
// metric; bound by the FP64 units.
//
// A unit of work is kExactRows rows i (one per thread) against kExactCols
// columns j, whose endpoint positions and coordinates the block stages in LDS
// as doubles and every wave reads as broadcasts; the units of all rows together
// tile the triangles, so no thread carries a long row to its end alone.  Only
// the pair (i, i + 1) can have d = 0 (node lengths are at least 1) and takes
// the general way; all others have d >= 1 and take exact_stress, whose square
// root and quotient are the compiler's own sequences without their scaling for
// arguments near the ends of FP64's range, which float32 coordinates and
// lengths below 2^63 cannot reach: the same rounding, fewer instructions.  A
// sum that is not finite (infinite or NaN coordinates) is taken again the
// general way.  1.3e9 pairs: 19.3 ms with one row per thread and the
// compiler's sequences, now 5.9 ms (four combinations a pair: 8.9e11 a second).
// part_f: per-block sum of the pair means; part_n: per-block pair count.
// ---------------------------------------------------------------------------
constexpr uint32_t kExactRows = 256, kExactCols = 512;

// Pos: double (differences of positions below 2^53 are exact: one instruction instead of six), or int64_t.
template <typename Pos>
__global__ __launch_bounds__(kExactRows) void k_path_stress_exact(StressLaunch P, uint32_t col_chunks,
                                                                  double* __restrict__ part_f,
                                                                  uint64_t* __restrict__ part_n) {
  extern __shared__ __align__(16) char lds[];
  uint64_t* off = reinterpret_cast<uint64_t*>(lds);
  __shared__ double red_f[16];
  __shared__ uint64_t red_n[16];
  __shared__ Pos s_pos[kExactCols][2];
  __shared__ double s_xy[kExactCols][4];
  fill_offsets(off, P);
  __syncthreads();
  // both endpoints of a node are 16 contiguous bytes of the interleaved copy
  const float4* __restrict__ W4 = reinterpret_cast<const float4*>(P.work);
  double acc = 0.0;
  uint64_t np = 0;
  const uint64_t units = (P.S + kExactRows - 1) / kExactRows * col_chunks;
  for (uint64_t u = blockIdx.x; u < units; u += gridDim.x) {
    const uint64_t r0 = u / col_chunks * kExactRows;
    const uint64_t j0 = r0 + (u % col_chunks) * kExactCols;
    const uint64_t last = min(r0 + kExactRows, P.S) - 1;
    const uint64_t j1 = min(j0 + kExactCols, off[find_path(off, P.path_top, last) + 1]);
    if (j0 >= j1) continue;  // the same for the whole block
    const uint32_t n = (uint32_t)(j1 - j0);
    __syncthreads();  // the columns of the unit before are no longer read
    for (uint32_t c = threadIdx.x; c < n; c += kExactRows) {
      const StepRec sj = load_rec(P.rec, j0 + c);
      const float4 v = W4[sj.node_rev & kNodeMask];
      s_pos[c][0] = (Pos)endpoint_pos(sj, 0);
      s_pos[c][1] = (Pos)endpoint_pos(sj, 1);
      s_xy[c][0] = v.x;
      s_xy[c][1] = v.y;
      s_xy[c][2] = v.z;
      s_xy[c][3] = v.w;
    }
    __syncthreads();
    const uint64_t i = r0 + threadIdx.x;
    if (i >= P.S) continue;
    const uint64_t end = min(off[find_path(off, P.path_top, i) + 1], j1);
    const StepRec si = load_rec(P.rec, i);
    const float4 ci = W4[si.node_rev & kNodeMask];
    const Pos p0 = (Pos)endpoint_pos(si, 0), p1 = (Pos)endpoint_pos(si, 1);
    const double x0 = ci.x, y0 = ci.y, x1 = ci.z, y1 = ci.w;
    // the mean over the combinations with d > 0
    auto general = [&](uint32_t c, double& sum) -> bool {
      uint32_t nv = 0;
      sum = 0.0;
      for (uint32_t e = 0; e < 4; ++e) {
        const Pos dd = ((e & 1u) ? p1 : p0) - s_pos[c][e >> 1];
        if (dd == 0) continue;
        sum += stress_xy((e & 1u) ? ci.z : ci.x, (e & 1u) ? ci.w : ci.y, (float)s_xy[c][(e >> 1) * 2],
                         (float)s_xy[c][(e >> 1) * 2 + 1], (double)(dd < 0 ? -dd : dd));
        ++nv;
      }
      sum = nv ? sum / (double)nv : 0.0;
      return nv != 0;
    };
    if (i + 1 >= j0 && i + 1 < end) {
      double sum;
      np += general((uint32_t)(i + 1 - j0), sum);
      acc += sum;
    }
    const uint32_t lo = (uint32_t)(i + 2 > j0 ? min(i + 2 - j0, (uint64_t)n) : 0);
    const uint32_t hi = end > j0 ? (uint32_t)(end - j0) : 0u;
    if (lo >= hi) continue;
    double unit = 0.0;
    for (uint32_t c = lo; c < hi; ++c) {
#pragma clang fp contract(off)
      const Pos q0 = s_pos[c][0], q1 = s_pos[c][1];
      const double u0 = s_xy[c][0], v0 = s_xy[c][1], u1 = s_xy[c][2], v1 = s_xy[c][3];
      double sum = exact_stress(x0 - u0, y0 - v0, (double)(q0 - p0));
      sum += exact_stress(x1 - u0, y1 - v0, (double)(q0 - p1));
      sum += exact_stress(x0 - u1, y0 - v1, (double)(q1 - p0));
      sum += exact_stress(x1 - u1, y1 - v1, (double)(q1 - p1));
      unit += sum * 0.25;
    }
    if (!(unit - unit == 0.0)) {
      unit = 0.0;
      for (uint32_t c = lo; c < hi; ++c) {
        double sum;
        general(c, sum);
        unit += sum;
      }
    }
    acc += unit;
    np += hi - lo;
  }
  acc = block_sum(acc, red_f);
  np = block_sum(np, red_n);
  if (threadIdx.x == 0) {
    part_f[blockIdx.x] = acc;
    part_n[blockIdx.x] = np;
  }
}

// One block sums the partials of `sums` Sum2 rows and the two counts in a fixed
// order and writes hi, lo of every sum and the counts (and the outlier counter,
// if there is one) to `out`, host memory that the device can write.
__global__ __launch_bounds__(1024) void k_reduce_sps(const double* __restrict__ part_f,
                                                     const uint64_t* __restrict__ part_n,
                                                     const uint64_t* __restrict__ part_skip, uint32_t n_parts,
                                                     uint32_t sums, const uint64_t* __restrict__ out_count,
                                                     SpsHostSums* out) {
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;  // one wave per row
  if (w < sums) {
    Sum2 t;
    for (uint32_t k = lane; k < n_parts; k += 64) {
      Sum2 x;
      x.hi = part_f[(size_t)(2 * w) * n_parts + k];
      x.lo = part_f[(size_t)(2 * w + 1) * n_parts + k];
      t.add(x);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      Sum2 x;
      x.hi = __shfl_xor(t.hi, o, 64);
      x.lo = __shfl_xor(t.lo, o, 64);
      t.add(x);
    }
    if (lane == 0) {
      out->hi[w] = t.hi;
      out->lo[w] = t.lo;
    }
  } else if (w < sums + 2) {
    const uint64_t* part = w == sums ? part_n : part_skip;
    uint64_t t = 0;
    for (uint32_t k = lane; k < n_parts; k += 64) t += part[k];
    t = wave_sum(t);
    if (lane == 0) out->n[w - sums] = t;
  }
  if (threadIdx.x == 0) out->outliers = out_count ? *out_count : 0;
}

// One block sums the partials in a fixed order.
__global__ __launch_bounds__(1024) void k_reduce_parts(const double* __restrict__ part_f,
                                                       const uint64_t* __restrict__ part_n, uint32_t n_parts,
                                                       double* out_f, uint64_t* out_n, float* loss_out,
                                                       uint64_t* n_valid_out) {
  __shared__ double red_f[16];
  __shared__ uint64_t red_n[16];
  double f = 0.0;
  uint64_t n = 0;
  for (uint32_t k = threadIdx.x; k < n_parts; k += blockDim.x) {
    f += part_f[k];
    n += part_n[k];
  }
  f = block_sum(f, red_f);
  n = block_sum(n, red_n);
  if (threadIdx.x == 0) {
    if (out_f) out_f[0] = f;
    if (out_n) out_n[0] = n;
    if (loss_out) loss_out[0] = n ? (float)(f / (double)n) : 0.0f;
    if (n_valid_out) n_valid_out[0] = n;
  }
}

// ---------------------------------------------------------------------------
// Differentiable loss: pairs q in [0, count) from the power-law sampler.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool loss_pair(const StressLaunch& P, const uint64_t* off, const uint32_t* zipf,
                                          const uint16_t* guide, uint64_t q, uint64_t& a, uint64_t& b, double& d) {
  const Rand4 r = philox10((uint32_t)q, (uint32_t)(q >> 32), P.word2, P.c3, P.k0, P.k1);
  const uint64_t i = mulhi64((uint64_t)r.r0 | ((uint64_t)r.r1 << 32), P.S);
  const uint32_t p = find_path(off, P.path_top, i);
  const uint64_t start = off[p], len = off[p + 1] - start;
  uint64_t j;
  if (!partner_power_law(i, start, len, r.r2, r.r3, zipf, guide, P.W, j)) return false;
  if (!pair_terms(P.rec, i, j, r.r3 & 1u, (r.r3 >> 1) & 1u, a, b, d)) return false;
  return a != b;
}

__device__ __forceinline__ void fill_loss_lds(char* lds, const StressLaunch& P, uint64_t*& off, uint32_t*& zipf,
                                              uint16_t*& guide) {
  off = reinterpret_cast<uint64_t*>(lds);
  zipf = reinterpret_cast<uint32_t*>(lds + (size_t)P.path_slots * 8);
  guide = reinterpret_cast<uint16_t*>(lds + (size_t)P.path_slots * 8 + (size_t)(P.W + 1) * 4);
  fill_offsets(off, P);
  for (uint32_t k = threadIdx.x; k <= P.W; k += blockDim.x) zipf[k] = P.zipf[k];
  for (uint32_t k = threadIdx.x; k <= kGuideSize; k += blockDim.x) guide[k] = P.guide[k];
}

__global__ __launch_bounds__(256) void k_stress_fwd(StressLaunch P, double* __restrict__ part_f,
                                                    uint64_t* __restrict__ part_n) {
  extern __shared__ __align__(16) char lds[];
  __shared__ double red_f[16];
  __shared__ uint64_t red_n[16];
  uint64_t* off;
  uint32_t* zipf;
  uint16_t* guide;
  fill_loss_lds(lds, P, off, zipf, guide);
  __syncthreads();
  double acc = 0.0;
  uint64_t nv = 0;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < P.count; q += stride) {
    uint64_t a, b;
    double d;
    if (!loss_pair(P, off, zipf, guide, q, a, b, d)) continue;
    acc += stress_work(P.work, a, b, d);
    ++nv;
  }
  acc = block_sum(acc, red_f);
  nv = block_sum(nv, red_n);
  if (threadIdx.x == 0) {
    part_f[blockIdx.x] = acc;
    part_n[blockIdx.x] = nv;
  }
}

// The adjoint, scattered with float32 atomics into the planar gradient
// (atomics are served per 4-byte word, so an interleaved scratch would not
// make them cheaper); the coordinates come from the interleaved copy.
__global__ __launch_bounds__(256) void k_stress_bwd(StressLaunch P, const float* __restrict__ grad_out,
                                                    const uint64_t* __restrict__ n_valid,
                                                    float* __restrict__ grad) {
  extern __shared__ __align__(16) char lds[];
  uint64_t* off;
  uint32_t* zipf;
  uint16_t* guide;
  fill_loss_lds(lds, P, off, zipf, guide);
  __syncthreads();
  const uint64_t n = n_valid[0];
  if (n == 0) return;
  const double scale = (double)grad_out[0] * 2.0 / (double)n;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < P.count; q += stride) {
    uint64_t a, b;
    double d;
    if (!loss_pair(P, off, zipf, guide, q, a, b, d)) continue;
    double dx, dy;
    const double mag = delta_xy(P.work[a], P.work[b], dx, dy);
    if (mag == 0.0) continue;
    const double c = gradient_factor(scale, mag, d);
    const float gx = (float)(c * dx), gy = (float)(c * dy);
    float* __restrict__ GX = grad;
    float* __restrict__ GY = grad + 2ull * P.n_nodes;
    if (P.inv) {  // the gradient is in the caller's node order
      a = 2ull * P.inv[a >> 1] + (a & 1);
      b = 2ull * P.inv[b >> 1] + (b & 1);
    }
    unsafeAtomicAdd(&GX[a], gx);
    unsafeAtomicAdd(&GY[a], gy);
    unsafeAtomicAdd(&GX[b], -gx);
    unsafeAtomicAdd(&GY[b], -gy);
  }
}

// ---------------------------------------------------------------------------
// The loss over its window-major pairs (reading R22): the waves of XCD x take
// the items (64 slots of one segment) of run x from the counter of row
// `kGrad` of the queue; slot u draws Philox stream 7 (W.slot_c3) at counter u
// with word 2 = the optimiser step: i uniform in the segment, j its power-law
// partner, endpoint coins.  A segment's steps, their partners (at most W steps
// away) and the coordinates and gradient entries of the nodes they visit stay
// in the XCD's L2 while the XCD works on it.  Forward: per-block sums of the
// stress and the valid-pair count; adjoint: as k_stress_bwd.
// ---------------------------------------------------------------------------
template <bool kGrad>
__global__ __launch_bounds__(256) void k_loss_win(SpsWinLaunch W, const float* __restrict__ grad_out,
                                                  const uint64_t* __restrict__ n_valid, float* __restrict__ grad,
                                                  double* __restrict__ part_f, uint64_t* __restrict__ part_n) {
  extern __shared__ __align__(16) char lds[];
  __shared__ double red_f[16];
  __shared__ uint64_t red_n[16];
  const StressLaunch& P = W.P;
  uint32_t* zipf = reinterpret_cast<uint32_t*>(lds);
  uint16_t* guide = reinterpret_cast<uint16_t*>(lds + (size_t)(P.W + 1) * 4);
  for (uint32_t k = threadIdx.x; k <= P.W; k += blockDim.x) zipf[k] = P.zipf[k];
  for (uint32_t k = threadIdx.x; k <= kGuideSize; k += blockDim.x) guide[k] = P.guide[k];
  __syncthreads();
  double scale = 0.0;
  if (kGrad) {
    const uint64_t n = n_valid[0];
    if (n == 0) return;
    scale = (double)grad_out[0] * 2.0 / (double)n;
  }
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t x = blockIdx.x % kXcds;
  const uint32_t gb = uload(W.sbeg + x);
  const uint32_t nq = uload(W.sbeg + x + 1) - gb;
  const uint64_t* __restrict__ xi = W.xitem + (size_t)x * W.xstride;
  const uint64_t n_items = uniform_u64(uload(xi + nq));
  unsigned long long* ctr = reinterpret_cast<unsigned long long*>(W.queue + ((size_t)(kGrad ? 1 : 0) * kXcds + x) * 16);
  float* __restrict__ GX = grad;
  float* __restrict__ GY = grad + 2ull * P.n_nodes;
  double acc = 0.0;
  uint64_t nv = 0;
  uint32_t q = 0;
  for (uint64_t m = 0, m_end = 0;; ++m) {
    if (m >= m_end) {
      uint64_t base = 0;
      if (lane == 0) base = atomicAdd(ctr, (unsigned long long)kSpsGrab);
      m = uniform_u64(base);
      if (m >= n_items) break;
      m_end = min(m + kSpsGrab, n_items);
    }
    while (q + 1 < nq && uniform_u64(uload(xi + q + 1)) <= m) q = uniform_u32(q + 1);
    const uint32_t g = gb + q;
    const uint64_t u0 = uniform_u64(uload(W.seg_off + g)) + (m - uniform_u64(uload(xi + q))) * 64;
    const uint64_t u_end = uniform_u64(uload(W.seg_off + g + 1));
    const uint64_t sst = uniform_u64(uload(W.seg_start + g));
    const uint64_t slen = uniform_u64(uload(W.seg_start + g + 1)) - sst;
    const uint32_t p = uniform_u32(uload(W.seg_path + g));
    const uint64_t pst = uniform_u64(uload(P.path_off + p));
    const uint64_t plen = uniform_u64(uload(P.path_off + p + 1)) - pst;
    const uint64_t u = u0 + lane;
    if (u >= u_end) continue;
    const Rand4 r = philox10((uint32_t)u, (uint32_t)(u >> 32), P.word2, W.slot_c3, P.k0, P.k1);
    const uint64_t i = sst + mulhi64(r.r0, r.r1, (uint32_t)slen);
    uint64_t j, a, b;
    double d;
    if (!partner_power_law(i, pst, plen, r.r2, r.r3, zipf, guide, P.W, j)) continue;
    if (!pair_terms(P.rec, i, j, r.r3 & 1u, (r.r3 >> 1) & 1u, a, b, d) || a == b) continue;
    if (!kGrad) {
      acc += stress_work(P.work, a, b, d);
      ++nv;
    } else {
      double dx, dy;
      const double mag = delta_xy(P.work[a], P.work[b], dx, dy);
      if (mag == 0.0) continue;
      const double c = gradient_factor(scale, mag, d);
      const float gx = (float)(c * dx), gy = (float)(c * dy);
      if (P.inv) {  // the gradient is in the caller's node order
        a = 2ull * P.inv[a >> 1] + (a & 1);
        b = 2ull * P.inv[b >> 1] + (b & 1);
      }
      unsafeAtomicAdd(&GX[a], gx);
      unsafeAtomicAdd(&GY[a], gy);
      unsafeAtomicAdd(&GX[b], -gx);
      unsafeAtomicAdd(&GY[b], -gy);
    }
  }
  if (!kGrad) {
    acc = block_sum(acc, red_f);
    nv = block_sum(nv, red_n);
    if (threadIdx.x == 0) {
      part_f[blockIdx.x] = acc;
      part_n[blockIdx.x] = nv;
    }
  }
}

// ---------------------------------------------------------------------------
// The loss adjoint by tiles.  The ~30 paths through a node each add to its
// gradient, from their own segments; a tile gathers the segments of all paths
// whose steps start in one range of device node ids (the ids follow the
// paths), so most of a tile's adjoint lands in an LDS image of that range and
// reaches memory once per touched entry instead of once per pair.
// ---------------------------------------------------------------------------
static size_t tile_tables_bytes(uint32_t W) {
  return ((size_t)(W + 1) * 4 + (size_t)(kGuideSize + 1) * 2 + 15) & ~(size_t)15;
}
static size_t tile_entry_bytes(TileForm f) {
  return (tile_grad(f) ? 2 * (tile_double(f) ? sizeof(double) : sizeof(float)) : 0) +
         (tile_staged(f) ? sizeof(float2) : 0);
}

// The least entries that a form is taken for.  4e6 pairs over 300,000 backbone
// nodes, by window W: the adjoint staged 67 / 113 / 129 / 158 us for W = 1,000 /
// 4,000 / 6,000 / 9,000 (6,144 / 5,632 / 5,312 / 4,800 entries), not staged 79 /
// 116 / 130 / 144, with the image in float 148 / 150 / 156 / 166; not staged in
// double 173 and 214 for W = 17,000 and 20,000 (5,184 and 4,416 entries), in
// float 176 and 179.  Forward staged and not: 51 / 57 / 60 / 66 and 63 / 72 / 75 / 77.
uint32_t loss_tile_entries(uint32_t W, TileForm form, size_t lds_limit) {
  if (form == kTileFwd) return 0;
  const uint32_t least = form == kTileFwdStaged ? kTileRange : tile_double(form) ? 5120 : 2 * kTileRange;
  const size_t have = lds_limit / tile_blocks(form), head = tile_tables_bytes(W) + kTileStaticLds;
  const size_t fit = have > head ? (have - head) / tile_entry_bytes(form) : 0;
  const uint32_t n = (uint32_t)std::min<size_t>(2 * kTileRange, fit & ~(size_t)63);
  return n >= least ? n : 0;
}

// kTileFwd, kTileFwdStaged: the forward pass (per-block sums of the stress and
// the valid-pair count).  kTileBwd32, kTileBwd64, kTileBwd64Staged: the adjoint,
// its image in float or in double.
//
// Staged: the coordinates of the tile's ids are copied to LDS first by coalesced
// loads, all in flight at once.  A pair's two records and two coordinates are
// scattered 8 and 16-byte loads, 64 cache-line requests each for a wave: of the
// 161 us of the forward pass over 1e7 pairs, draws take 62, records 52, staged
// coordinates 8 (96 us if they are not staged) and the units' tables and copies
// 36.  More pairs of a thread in flight do not help (two: 170 us).
//
// The image: a wave's ds_add_f32 at scattered addresses takes 185 cycles here,
// ds_add_f64 21 (and ds_add_u32 7), so the double image is the faster one and
// rounds once, at the flush; the float image remains where the tables leave the
// double one too little room.  x and y have planes of their own, so the adds of a
// wave use all banks.  Adjoint over 1e7 pairs: 360 us with staging and the image
// in float, 278 in double without staging, 206 with both (214 from the caller's
// planes, which saves the copy's 12).
//
// A unit of work is one of T.split equal parts of a tile's pairs (see
// loss_tile_split for where a tile is cut).
template <TileForm kForm>
__global__ __launch_bounds__(kTileThreads, tile_blocks(kForm) * 4) void k_loss_tile(SpsWinLaunch W, TileLaunch T,
                                                           const float* __restrict__ grad_out,
                                                           const uint64_t* __restrict__ n_valid,
                                                           float* __restrict__ grad, double* __restrict__ part_f,
                                                           uint64_t* __restrict__ part_n) {
  constexpr bool kGrad = tile_grad(kForm);
  constexpr bool kStage = tile_staged(kForm);
  using Acc = typename std::conditional<tile_double(kForm), double, float>::type;
  __shared__ double red_f[16];
  __shared__ uint64_t red_n[16];
  extern __shared__ __align__(16) char lds[];
  __shared__ uint32_t s_flat[kTileMaxSeg + 1];  // slot prefix over the tile's segments (fewer than 2^32 pairs)
  __shared__ uint32_t s_slot[kTileMaxSeg];      // first slot of each segment
  __shared__ uint64_t s_start[kTileMaxSeg];     // first step of each segment
  __shared__ uint64_t s_pst[kTileMaxSeg];       // first step of its path
  __shared__ uint32_t s_len[kTileMaxSeg];       // steps of each segment
  __shared__ uint32_t s_plen[kTileMaxSeg];      // steps of its path
  __shared__ uint8_t s_near[kTileGuide];        // the segment of slots 0, 1 << shift, 2 << shift, ...
  __shared__ uint32_t s_unit;
  const StressLaunch& P = W.P;
  uint32_t* zipf = reinterpret_cast<uint32_t*>(lds);
  uint16_t* guide = reinterpret_cast<uint16_t*>(lds + (size_t)(P.W + 1) * 4);
  const uint32_t n_acc = T.entries;  // endpoints of the tile's range: n_acc / 2 nodes x 2
  char* image = lds + (((size_t)(P.W + 1) * 4 + (size_t)(kGuideSize + 1) * 2 + 15) & ~(size_t)15);
  Acc* acc_x = reinterpret_cast<Acc*>(image);
  Acc* acc_y = acc_x + n_acc;
  float2* xy = reinterpret_cast<float2*>(image + (kGrad ? (size_t)n_acc * 2 * sizeof(Acc) : 0));
  for (uint32_t k = threadIdx.x; k <= P.W; k += blockDim.x) zipf[k] = P.zipf[k];
  for (uint32_t k = threadIdx.x; k <= kGuideSize; k += blockDim.x) guide[k] = P.guide[k];
  double scale = 0.0;
  if (kGrad) {
    const uint64_t n = n_valid[0];
    if (n == 0) return;  // uniform over the grid: no block waits at a barrier below
    scale = (double)grad_out[0] * 2.0 / (double)n;
  }
  double sum = 0.0;
  uint64_t nv = 0;
  float* __restrict__ GX = grad;
  float* __restrict__ GY = grad + 2ull * P.n_nodes;
  auto global_add = [&](uint64_t a, float gx, float gy) {
    if (P.inv) a = 2ull * P.inv[a >> 1] + (a & 1);  // the gradient is in the caller's node order
    unsafeAtomicAdd(&GX[a], gx);
    unsafeAtomicAdd(&GY[a], gy);
  };
  const float* __restrict__ px = T.planes;
  const float* __restrict__ py = T.planes + 2ull * P.n_nodes;
  const uint32_t n_units = T.n_tiles * T.split;
  uint32_t unit = blockIdx.x;  // the first one; the others from the queue
  while (unit < n_units) {
    const uint32_t t = unit / T.split, part = unit % T.split;
    const uint64_t base = T.base[t];
    const uint32_t k0 = T.off[t];
    const uint32_t nk = T.off[t + 1] - k0;
    if (kGrad)
      for (uint32_t e = threadIdx.x; e < 2 * n_acc; e += blockDim.x) acc_x[e] = 0;
    // the coordinates of the range, a node (two endpoints) a load, all in flight at once
    constexpr uint32_t kLoads = kTileRange / kTileThreads;
    using Pair2 = float __attribute__((ext_vector_type(2)));
    using Node = float __attribute__((ext_vector_type(4)));  // float4 arrays go to scratch
    Node node[kLoads];
    const uint32_t nodes = (uint32_t)min((uint64_t)(n_acc / 2), P.n_nodes - base);
    if (kStage && px) {
#pragma unroll
      for (uint32_t q = 0; q < kLoads; ++q) {
        const uint32_t e = threadIdx.x + q * kTileThreads;
        const uint64_t k = 2 * (base + e);
        if (e < nodes) node[q] = Node{px[k], py[k], px[k + 1], py[k + 1]};
      }
    } else if (kStage) {
      const Node* __restrict__ work = reinterpret_cast<const Node*>(P.work) + base;
#pragma unroll
      for (uint32_t q = 0; q < kLoads; ++q) {
        const uint32_t e = threadIdx.x + q * kTileThreads;
        if (e < nodes) node[q] = work[e];
      }
    }
    auto coords = [&](uint64_t a) -> float2 {
      const uint64_t e = a - 2 * base;  // wraps to huge below the base
      if (!kStage || e >= n_acc) return px ? make_float2(px[a], py[a]) : P.work[a];
      const Pair2 v = ((const __attribute__((address_space(3))) Pair2*)xy)[e];  // or both became flat loads
      return make_float2(v.x, v.y);
    };
    for (uint32_t k = threadIdx.x; k < nk; k += blockDim.x) {
      const uint32_t g = T.seg[k0 + k];
      s_slot[k] = (uint32_t)W.seg_off[g];
      s_flat[k + 1] = (uint32_t)(W.seg_off[g + 1] - W.seg_off[g]);
      s_start[k] = W.seg_start[g];
      s_len[k] = (uint32_t)(W.seg_start[g + 1] - W.seg_start[g]);
      const uint32_t p = W.seg_path[g];
      s_pst[k] = P.path_off[p];
      s_plen[k] = (uint32_t)(P.path_off[p + 1] - P.path_off[p]);
    }
    if (kStage) {
#pragma unroll
      for (uint32_t q = 0; q < kLoads; ++q) {
        const uint32_t e = threadIdx.x + q * kTileThreads;
        if (e < nodes) reinterpret_cast<Node*>(xy)[e] = node[q];
      }
    }
    __syncthreads();
    if (threadIdx.x < 64) {  // inclusive prefix by one wave, 64 segments at a time
      uint32_t carry = 0;
      if (threadIdx.x == 0) s_flat[0] = 0;
      for (uint32_t k = 0; k < nk; k += 64) {
        uint32_t x = k + threadIdx.x < nk ? s_flat[k + threadIdx.x + 1] : 0;
#pragma unroll
        for (uint32_t d = 1; d < 64; d <<= 1) {
          const uint32_t y = __shfl_up(x, d, 64);
          if (threadIdx.x >= d) x += y;
        }
        x += carry;
        if (k + threadIdx.x < nk) s_flat[k + threadIdx.x + 1] = x;
        carry = __shfl(x, 63, 64);
      }
    }
    __syncthreads();
    const uint32_t total = s_flat[nk];
    uint32_t shift = 6;  // the guide's step: it spans the tile's slots
    while ((total >> shift) >= kTileGuide) ++shift;
    for (uint32_t e = threadIdx.x; ((uint64_t)e << shift) < total; e += blockDim.x) {
      uint32_t lo = 0, hi = nk;  // the segment k with s_flat[k] <= e << shift < s_flat[k + 1]
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (s_flat[mid] <= (uint64_t)e << shift) lo = mid;
        else hi = mid;
      }
      s_near[e] = (uint8_t)lo;
    }
    __syncthreads();
    const uint64_t f_end = (uint64_t)total * (part + 1) / T.split;
    for (uint64_t f = (uint64_t)total * part / T.split + threadIdx.x; f < f_end; f += blockDim.x) {
      uint32_t lo = s_near[f >> shift];  // the segment k with s_flat[k] <= f < s_flat[k + 1]
      while (s_flat[lo + 1] <= f) ++lo;
      const uint64_t u = s_slot[lo] + (f - s_flat[lo]);
      const uint64_t pst = s_pst[lo], plen = s_plen[lo];
      const Rand4 r = philox10((uint32_t)u, (uint32_t)(u >> 32), P.word2, W.slot_c3, P.k0, P.k1);
      const uint64_t i = s_start[lo] + mulhi64(r.r0, r.r1, s_len[lo]);
      uint64_t j, a, b;
      double d;
      if (!partner_power_law(i, pst, plen, r.r2, r.r3, zipf, guide, P.W, j)) continue;
      if (!pair_terms(P.rec, i, j, r.r3 & 1u, (r.r3 >> 1) & 1u, a, b, d) || a == b) continue;
      const float2 va = coords(a), vb = coords(b);
      if (!kGrad) {
        sum += pair_stress(va, vb, d);
        ++nv;
        continue;
      }
      double dx, dy;
      const double mag = delta_xy(va, vb, dx, dy);
      if (mag == 0.0) continue;
      const double c = gradient_factor(scale, mag, d);
      const Acc gx = (Acc)(c * dx), gy = (Acc)(c * dy);
      const uint64_t ea = a - 2 * base, eb = b - 2 * base;  // wrap to huge below the base
      if (ea < n_acc) {
        unsafeAtomicAdd(&acc_x[ea], gx);
        unsafeAtomicAdd(&acc_y[ea], gy);
      } else {
        global_add(a, (float)gx, (float)gy);
      }
      if (eb < n_acc) {
        unsafeAtomicAdd(&acc_x[eb], -gx);
        unsafeAtomicAdd(&acc_y[eb], -gy);
      } else {
        global_add(b, (float)-gx, (float)-gy);
      }
    }
    if (kGrad) __syncthreads();  // the image is complete
    const bool more = n_units > gridDim.x;
    if (more && threadIdx.x == 0) s_unit = gridDim.x + atomicAdd(T.queue, 1u);
    if (kGrad)
      for (uint32_t e = threadIdx.x; e < n_acc; e += blockDim.x) {
        const float vx = (float)acc_x[e], vy = (float)acc_y[e];
        if ((vx != 0.0f || vy != 0.0f) && 2 * base + e < 2 * P.n_nodes) global_add(2 * base + e, vx, vy);
      }
    if (!more) break;
    __syncthreads();  // the tile's tables and image are free again
    unit = uniform_u32(s_unit);
  }
  // the block that is the last to leave the queue leaves it as it found it
  if (n_units > gridDim.x && threadIdx.x == 0 && atomicAdd(T.queue + kTileDone, 1u) == gridDim.x - 1) {
    T.queue[0] = 0;
    T.queue[kTileDone] = 0;
  }
  if (!kGrad) {
    sum = block_sum(sum, red_f);
    nv = block_sum(nv, red_n);
    if (threadIdx.x == 0) {
      part_f[blockIdx.x] = sum;
      part_n[blockIdx.x] = nv;
    }
  }
}

__global__ __launch_bounds__(256) void k_segment_min_node(const StepRec* __restrict__ rec,
                                                          const uint64_t* __restrict__ start, uint32_t nseg,
                                                          uint32_t* __restrict__ out) {
  const uint32_t g = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);  // one wave per segment
  if (g >= nseg) return;
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t m = 0xFFFFFFFFu;
  for (uint64_t k = start[g] + lane; k < start[g + 1]; k += 64) m = min(m, rec[k].node_rev & kNodeMask);
  for (int o = 32; o > 0; o >>= 1) m = min(m, (uint32_t)__shfl_xor((int)m, o, 64));
  if (lane == 0) out[g] = m;
}

// ---------------------------------------------------------------------------
// Initial layout and first visits
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_fill_u64(uint64_t* __restrict__ p, uint64_t n, uint64_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += stride) p[k] = v;
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* __restrict__ p, uint64_t n, uint32_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += stride) p[k] = v;
}

__global__ __launch_bounds__(256) void k_first_visit(const StepRec* __restrict__ rec, uint64_t S,
                                                     uint64_t* __restrict__ first) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; s < S; s += stride) {
    const uint32_t node = rec[s].node_rev & kNodeMask;
    atomicMin(reinterpret_cast<unsigned long long*>(&first[node]), (unsigned long long)s);
  }
}

// Thread k handles endpoint k = 2m + e of device node m (caller id inv[m] on a
// renumbered graph); the jitter draw is keyed by the caller's endpoint index.
__global__ __launch_bounds__(256) void k_init_coords(const StepRec* __restrict__ rec,
                                                     const uint64_t* __restrict__ first, uint64_t n_nodes,
                                                     const uint32_t* __restrict__ inv, uint32_t k0, uint32_t k1,
                                                     uint32_t c3, float jitter, float* __restrict__ coords) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  float* __restrict__ X = coords;
  float* __restrict__ Y = coords + 2 * n_nodes;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < 2 * n_nodes; k += stride) {
    const uint64_t s = first[k >> 1];
    const uint64_t c = inv ? 2ull * inv[k >> 1] + (k & 1) : k;
    float x = 0.0f;
    if (s != ~0ull) {
      const StepRec r = load_rec(rec, s);
      x = (float)(r.pos + (int64_t)r.len * (int64_t)(k & 1));
    }
    X[c] = x;
    const Rand4 rn = philox10((uint32_t)c, (uint32_t)(c >> 32), 0u, c3, k0, k1);
    const float u = (float)(rn.r0 >> 8) * (1.0f / 16777216.0f);
    Y[c] = jitter * (u - 0.5f);
  }
}

// ---------------------------------------------------------------------------
// Adam (Kingma and Ba, 2015); c1 = 1 - beta1^t, c2 = 1 - beta2^t.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ x, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, uint64_t n, float lr,
                                              float b1, float b2, float eps, float c1, float c2) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += stride) {
    const float gk = g[k];
    const float mk = b1 * m[k] + (1.0f - b1) * gk;
    const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    x[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static size_t loss_lds_bytes(const StressLaunch& P) {
  return (size_t)P.path_slots * 8 + (size_t)(P.W + 1) * 4 + (size_t)(kGuideSize + 1) * 2;
}

static uint32_t grid_for(uint64_t n, uint32_t cap) {
  const uint64_t b = (n + 255) / 256;
  return (uint32_t)(b < 1 ? 1 : (b > cap ? cap : b));
}

hipError_t launch_sps(const StressLaunch& P, int mode, double* part_f, uint64_t* part_n, uint64_t* part_skip,
                      uint32_t* n_parts, hipStream_t s) {
  const size_t lds = std::max(kSpsLds, mode == 1 ? loss_lds_bytes(P) : (size_t)P.path_slots * 8);
  const uint32_t threads = P.work2 ? kSpsPairThreads : kSpsThreads;
  const uint32_t cap = P.work2 ? kSpsPairBlocks : kSpsBlocks;
  const SpsSplit split = sps_split(P.S, P.m, (uint64_t)cap * threads);
  const uint32_t per = split.per, chunks = split.chunks;
  const uint64_t blocks = (P.S * chunks + threads - 1) / threads;
  *n_parts = (uint32_t)std::min<uint64_t>(cap, std::max<uint64_t>(1, blocks));
  if (P.work2)
    hipLaunchKernelGGL(k_sps<true>, dim3(*n_parts), dim3(threads), lds, s, P, mode, per, chunks, part_f, part_n,
                       part_skip);
  else
    hipLaunchKernelGGL(k_sps<false>, dim3(*n_parts), dim3(threads), lds, s, P, mode, per, chunks, part_f, part_n,
                       part_skip);
  return hipGetLastError();
}

hipError_t launch_reduce_sps(const StressLaunch& P, const double* part_f, const uint64_t* part_n,
                             const uint64_t* part_skip, uint32_t n_parts, SpsHostSums* out, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_sps, dim3(1), dim3(1024), 0, s, part_f, part_n, part_skip, n_parts, P.work2 ? 5u : 2u,
                     P.out_count, out);
  return hipGetLastError();
}

hipError_t launch_sps_win_count_scan(const SpsWinLaunch& W, bool runs, hipStream_t s) {
  const size_t lds = (size_t)W.P.path_slots * 8 + (size_t)W.n_seg * 4;
  hipLaunchKernelGGL(k_sps_win_count, dim3(W.count_blocks), dim3(1024), lds, s, W);
  hipError_t e = hipGetLastError();
  if (e) return e;
  hipLaunchKernelGGL(k_sps_win_scan, dim3(1), dim3(1024), (size_t)W.n_seg * 4, s, W, runs ? 1u : 0u);
  return hipGetLastError();
}

hipError_t launch_sps_win(const SpsWinLaunch& W, double* part_f, uint64_t* part_n, uint64_t* part_skip,
                          uint32_t* n_parts, hipStream_t s) {
  *n_parts = W.P.work2 ? kSpsPairBlocks : kSpsBlocks;
  if (W.P.work2)
    hipLaunchKernelGGL(k_sps_win<true>, dim3(*n_parts), dim3(kSpsPairThreads), kSpsLds, s, W, part_f, part_n, part_skip);
  else
    hipLaunchKernelGGL(k_sps_win<false>, dim3(*n_parts), dim3(kSpsThreads), kSpsLds, s, W, part_f, part_n, part_skip);
  return hipGetLastError();
}

hipError_t launch_path_stress_exact(const StressLaunch& P, uint64_t max_path_steps, int64_t d_max, double* part_f,
                                    uint64_t* part_n, uint32_t* n_parts, hipStream_t s) {
  const uint32_t chunks = (uint32_t)((max_path_steps + kExactRows + kExactCols - 1) / kExactCols);
  const size_t lds = (size_t)P.path_slots * 8;
  // a block for every unit at most: each fills its path table before it looks for one
  const uint64_t units = (P.S + kExactRows - 1) / kExactRows * chunks;
  *n_parts = (uint32_t)std::min<uint64_t>(kStressBlocks, std::max<uint64_t>(1, units));
  // any line up to 2^53 is exact; 2^40 leaves genomes a factor of 100 and lets a path of 256 long nodes cross it
  if (d_max < (1ll << 40))
    hipLaunchKernelGGL(k_path_stress_exact<double>, dim3(*n_parts), dim3(kExactRows), lds, s, P, chunks, part_f,
                       part_n);
  else
    hipLaunchKernelGGL(k_path_stress_exact<int64_t>, dim3(*n_parts), dim3(kExactRows), lds, s, P, chunks, part_f,
                       part_n);
  return hipGetLastError();
}

hipError_t launch_reduce_parts(const double* part_f, const uint64_t* part_n, uint32_t n_parts, double* out_f,
                               uint64_t* out_n, float* loss_out, uint64_t* n_valid_out, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_parts, dim3(1), dim3(1024), 0, s, part_f, part_n, n_parts, out_f, out_n, loss_out,
                     n_valid_out);
  return hipGetLastError();
}

hipError_t launch_stress_fwd(const StressLaunch& P, double* part_f, uint64_t* part_n, hipStream_t s) {
  hipLaunchKernelGGL(k_stress_fwd, dim3(kStressBlocks), dim3(kStressThreads), loss_lds_bytes(P), s, P, part_f,
                     part_n);
  return hipGetLastError();
}

hipError_t launch_stress_bwd(const StressLaunch& P, const float* grad_out, const uint64_t* n_valid, float* grad,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_stress_bwd, dim3(kStressBlocks), dim3(kStressThreads), loss_lds_bytes(P), s, P, grad_out,
                     n_valid, grad);
  return hipGetLastError();
}

hipError_t launch_loss_win_fwd(const SpsWinLaunch& W, double* part_f, uint64_t* part_n, uint32_t blocks,
                               hipStream_t s) {
  const size_t lds = (size_t)(W.P.W + 1) * 4 + (size_t)(kGuideSize + 1) * 2;
  hipLaunchKernelGGL(k_loss_win<false>, dim3(blocks), dim3(kStressThreads), lds, s, W, nullptr, nullptr, nullptr,
                     part_f, part_n);
  return hipGetLastError();
}

hipError_t launch_loss_win_bwd(const SpsWinLaunch& W, const float* grad_out, const uint64_t* n_valid, float* grad,
                               uint32_t blocks, hipStream_t s) {
  const size_t lds = (size_t)(W.P.W + 1) * 4 + (size_t)(kGuideSize + 1) * 2;
  hipLaunchKernelGGL(k_loss_win<true>, dim3(blocks), dim3(kStressThreads), lds, s, W, grad_out, n_valid, grad,
                     nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_loss_tile(const SpsWinLaunch& W, const TileLaunch& T, const float* grad_out,
                            const uint64_t* n_valid, float* grad, double* part_f, uint64_t* part_n, uint32_t blocks,
                            hipStream_t s) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kTileThreads),
                       tile_tables_bytes(W.P.W) + T.entries * tile_entry_bytes(T.form), s, W, T, grad_out,
                       n_valid, grad, part_f, part_n);
    return hipGetLastError();
  };
  switch (T.form) {
    case kTileFwd: return go(k_loss_tile<kTileFwd>);
    case kTileFwdStaged: return go(k_loss_tile<kTileFwdStaged>);
    case kTileBwd32: return go(k_loss_tile<kTileBwd32>);
    case kTileBwd64: return go(k_loss_tile<kTileBwd64>);
    default: return go(k_loss_tile<kTileBwd64Staged>);
  }
}

hipError_t launch_segment_min_node(const StepRec* rec, const uint64_t* start, uint32_t nseg, uint32_t* out,
                                   hipStream_t s) {
  hipLaunchKernelGGL(k_segment_min_node, dim3((nseg + 3) / 4), dim3(256), 0, s, rec, start, nseg, out);
  return hipGetLastError();
}

hipError_t launch_first_visit(const StepRec* rec, uint64_t S, uint64_t n_nodes, uint64_t* first_step,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u64, dim3(grid_for(n_nodes, 4096)), dim3(256), 0, s, first_step, n_nodes, ~0ull);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || S == 0) return e;
  hipLaunchKernelGGL(k_first_visit, dim3(grid_for(S, 8192)), dim3(256), 0, s, rec, S, first_step);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n, 4096)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_init_coords(const StepRec* rec, const uint64_t* first_step, uint64_t n_nodes, const uint32_t* inv,
                              uint32_t k0, uint32_t k1, uint32_t c3, float jitter, float* coords, hipStream_t s) {
  hipLaunchKernelGGL(k_init_coords, dim3(grid_for(2 * n_nodes, 8192)), dim3(256), 0, s, rec, first_step, n_nodes,
                     inv, k0, k1, c3, jitter, coords);
  return hipGetLastError();
}

hipError_t launch_adam(float* x, const float* g, float* m, float* v, uint64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3(grid_for(n, 8192)), dim3(256), 0, s, x, g, m, v, n, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace pgsgd

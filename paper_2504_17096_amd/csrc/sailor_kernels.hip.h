// HIP kernels of the batched plan evaluator (gfx950, wave64).
//
// Set-up kernels (once per plan): k_small_tables, k_stage_tables, k_shape_agg, k_group_bounds;
//            k_quota_table    again whenever the availability changes;
//            k_unit_work, k_work_order   in front of the first scan without a running limit.
// Hot path:  k_units<SCAN>    full-space fp32 evaluation + per-unit minima, early pruning
//            k_select_kth     radix select of the k-th smallest fp32 key (k > 128, or minima kept for later calls)
//            k_units<COLLECT> re-evaluates the few units that can hold a winner
//            k_refine, k_rank_topk   fp64 / exact-integer stage-by-stage re-evaluation, ranking
//            k_units<BEST>, k_refine_best   the best plan: the same in two kernels
//            k_eval_rows / k_eval_direct   per-candidate outputs for sailor_eval_batch
//                             (index ranges / index lists)
// Beside it: k_sim_1f1b       event-by-event 1F1B schedule of listed plans
//
// The simulator arithmetic follows Sailor, Sec. 4.3 (memory, iteration time, cost);
// T_pp = sum of stage times + (N_b - 1) * straggler is the 1F1B composition of
// Sec. 4.2.2 with the straggler counted N_b times in total.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sailor_dev.h"

namespace sailor {

// ------------------------------------------------------------------ helpers

// op over a wave's values, in every lane, for an op that may take a value twice (minima, maxima).  By moves
// between lanes within the registers: six trips through the LDS, which __shfl_xor makes, are 0.2 us where a
// wave has nothing else to do.  (Lanes without a source combine their value with itself.)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_word(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false);
}
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_value(T v) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, dpp_word<CTRL>(__builtin_bit_cast(uint32_t, v)));
  } else {
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(T, (uint64_t)dpp_word<CTRL>((uint32_t)(x >> 32)) << 32 | dpp_word<CTRL>((uint32_t)x));
  }
}
template <typename T, typename OP>
__device__ __forceinline__ T wave_fold(T v, OP op) {
  v = op(v, dpp_value<0x111>(v));  // row_shr:1, 2, 4, 8
  v = op(v, dpp_value<0x112>(v));
  v = op(v, dpp_value<0x114>(v));
  v = op(v, dpp_value<0x118>(v));
  v = op(v, dpp_value<0x142>(v));  // row_bcast:15, 31
  v = op(v, dpp_value<0x143>(v));
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
  } else {
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(T, (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), 63) << 32 |
                                     (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63));
  }
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  return wave_fold(v, [](uint32_t a, uint32_t b) { return min(a, b); });
}
__device__ __forceinline__ float wave_min(float v) {
  return wave_fold(v, [](float a, float b) { return fminf(a, b); });
}
__device__ __forceinline__ double wave_min_f64(double v) {
  return wave_fold(v, [](double a, double b) { return fmin(a, b); });
}
__device__ __forceinline__ double wave_max_f64(double v) {
  return wave_fold(v, [](double a, double b) { return fmax(a, b); });
}
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
  return wave_fold(v, [](uint64_t a, uint64_t b) { return a < b ? a : b; });
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
  return wave_fold(v, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
}

// The sum of a wave's values up to and including the lane's own (in the last lane: of all).  Six additions that
// take their operand from another lane, where a shuffle is an LDS operation that is waited for: a search's levels
// (histogram and counts of each) 0.51 -> 0.48 and 0.84 -> 0.74 ms.
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t v) {
  auto from = [&](auto ctrl, auto rows) {  // (0 without a source; rows that a broadcast does not reach keep their sum)
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
  };
  using std::integral_constant;
  from(integral_constant<int, 0x111>(), integral_constant<int, 0xF>());  // row_shr:1, 2, 4, 8
  from(integral_constant<int, 0x112>(), integral_constant<int, 0xF>());
  from(integral_constant<int, 0x114>(), integral_constant<int, 0xF>());
  from(integral_constant<int, 0x118>(), integral_constant<int, 0xF>());
  from(integral_constant<int, 0x142>(), integral_constant<int, 0xA>());  // row_bcast:15, 31
  from(integral_constant<int, 0x143>(), integral_constant<int, 0xC>());
  return v;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_prefix_sum(v), 63); }

// Element j of a three-element array by selects (a lane-dependent subscript would move the
// array to scratch memory).
template <typename T>
__device__ __forceinline__ int at3(const T *v, int j) {
  return j == 0 ? (int)v[0] : (j == 1 ? (int)v[1] : (int)v[2]);
}

// Brings a kernel's arguments into the scalar cache at once.  They lie in device memory that no cache holds
// when a kernel starts, and are read where they are used: every line of 64 bytes a trip of its own, one behind
// the other (half a microsecond each, five of them in front of a re-evaluation's first stage).
template <typename T>
__device__ __forceinline__ void touch_arguments(const T &args) {
  const uint32_t *const w = reinterpret_cast<const uint32_t *>(&args);
  constexpr int kLines = (int)(sizeof(T) / 64);
  static_assert(kLines <= 16, "");
  auto line = [&](int i) { return w[16 * (i < kLines ? i : kLines) < (int)(sizeof(T) / 4) ? 16 * (i < kLines ? i : kLines) : 0]; };
  asm volatile("" ::"s"(line(0)), "s"(line(1)), "s"(line(2)), "s"(line(3)), "s"(line(4)), "s"(line(5)), "s"(line(6)), "s"(line(7)),
               "s"(line(8)), "s"(line(9)), "s"(line(10)), "s"(line(11)), "s"(line(12)), "s"(line(13)), "s"(line(14)), "s"(line(15)));
}

// 24-bit multiply (full rate, unlike the 32-bit one), for table offsets
__device__ __forceinline__ uint32_t mul24(uint32_t a, uint32_t b) { return __umul24(a, b); }

__device__ __forceinline__ size_t agg_slot(const DevPlan &pl, uint32_t shape, int tp, int seg) {
  return ((size_t)shape * pl.TP + tp) * 3 + seg;
}

// Bandwidth a message of `bytes` sees from zone a to zone b: the link's fitted polynomial
// in log2(bytes) (cluster profiling, Sec. 4.1), kept inside [peak / 1000, peak]; the
// constant peak when the problem carries no polynomial.
__device__ __forceinline__ double link_bw(const DevPlan &pl, int a, int b, double bytes) {
  const double peak = pl.bw[a * pl.Z + b];
  if (pl.n_bw_coef <= 0 || bytes < 1.0) return peak;
  const double *c = pl.bw_poly + (size_t)(a * pl.Z + b) * pl.n_bw_coef;
  const double x = log2(bytes);
  double v = c[pl.n_bw_coef - 1];
  for (int k = pl.n_bw_coef - 2; k >= 0; --k) v = v * x + c[k];  // Horner
  // (ordered comparisons: the coefficients are validated finite and the device code is built
  // without NaN support, so the limits must not lean on how a NaN compares)
  if (v >= peak) v = peak;
  if (v <= peak * 1e-3) v = peak * 1e-3;
  return v;
}

// Bit q of the two-word mask of pool p (pool x pool relations for up to 128 pools).
__device__ __forceinline__ bool pool_bit(const uint64_t *mask, int p, int q) {
  return (mask[2 * p + (q >> 6)] >> (q & 63)) & 1ull;
}

// ------------------------------------------------------------------ set-up kernels

// Reciprocal bandwidths, two-way egress, and the per-(mb, dp, tp) scalars of a plan.  link_min (see
// k_group_bounds): per microbatch size the quickest transfer within a zone and between two, and behind
// them the smallest egress between two zones.
__global__ void k_small_tables(DevPlan pl, float *link_min) {
  const int t = threadIdx.x, nt = blockDim.x;
  const int Z = pl.Z;
  for (int i = t; i <= 2 * pl.MB; i += nt) link_min[i] = kPosInf;
  __syncthreads();
  for (int i = t; i < Z * Z; i += nt) {
    int a = i / Z, b = i % Z;
    for (int m = 0; m < pl.MB; ++m) {
      const double bytes = (double)pl.p2p[m], bwv = link_bw(pl, a, b, bytes);
      pl.xsec[m * Z * Z + i] = bytes / bwv;
      pl.tsec_f[m * Z * Z + i] = (float)(bytes / bwv);
      atomicMin(reinterpret_cast<uint32_t *>(&link_min[2 * m + (a != b)]), __float_as_uint((float)(bytes / bwv)));
    }
    double e = 0.0;
    if (pl.egress && a != b) e = pl.egress[a * Z + b] + pl.egress[b * Z + a];
    pl.egs_f[i] = (float)e;
    if (a != b) atomicMin(reinterpret_cast<uint32_t *>(&link_min[2 * pl.MB]), __float_as_uint((float)e));
  }
  for (int g = t; g < pl.GX; g += nt) {
    const int ga = pl.xt[g] & 255, gb = pl.xt[g] >> 8;
    pl.price_f[g] = (float)(ga == gb ? pl.price[ga] : 0.5 * (pl.price[ga] + pl.price[gb]));
  }
  for (int p = t; p < pl.ZG; p += nt) {
    const int x = pl.xt[p % pl.GX], ga = x & 255, gb = x >> 8, z = p / pl.GX;
    uint32_t m = 0;  // H1: tensor parallelism stays inside a node
    for (int k = 0; k < pl.TP; ++k)
      if (pl.tpv[k] > pl.node[ga] || pl.tpv[k] > pl.node[gb]) m |= 1u << k;
    pl.h1m[p] = m;
    uint64_t im[2] = {0, 0};  // pools of the same zone with a real type in common (itself included)
    for (int q = 0; q < pl.ZG; ++q) {
      const int y = pl.xt[q % pl.GX], qa = y & 255, qb = y >> 8;
      if (q / pl.GX == z && (qa == ga || qa == gb || qb == ga || qb == gb)) im[q >> 6] |= 1ull << (q & 63);
    }
    pl.isect[2 * p] = im[0];
    pl.isect[2 * p + 1] = im[1];
  }
  for (int m = t; m < pl.MB; m += nt) {
    // N_b * D = B / mb whenever the batch divides; the product is exact in fp64 for
    // realistic sizes and is rounded once
    pl.xb_f[m] = (float)((double)(pl.B / pl.mbv[m]) * (double)pl.p2p[m]);
    uint32_t bits = 0;
    for (int d = 0; d < pl.DP; ++d) {
      int64_t per = (int64_t)pl.dpv[d] * pl.mbv[m];
      int32_t nb = (pl.B % per == 0) ? (int32_t)(pl.B / per) : 0;
      pl.nb[m * pl.DP + d] = nb;
      pl.nbm1_f[m * pl.DP + d] = (float)(nb - 1);
      if (nb > 0) bits |= 1u << d;
    }
    pl.divis[m] = bits;
  }
  for (int d = t; d < pl.DP; d += nt) {
    double D = (double)pl.dpv[d];
    pl.cd_f[d] = (float)(2.0 * (D - 1.0) / D);
    pl.dph_f[d] = (float)(D / 3600.0);
  }
}

struct StageArgs {
  const uint64_t *layer_params;  // [L]
  const double *t_fwd, *t_bwd;   // [G][MB][TP][Lc]
  const double *t_upd;           // [G][TP][Lc]
  const uint8_t *st_flags;       // bit 0: first stage of its row, bit 1: last
  uint64_t embed, head;
  int L, uniform;
};

// Per stage of every partition row: parameters, summed layer times per (type, mb, tp).
__global__ void k_stage_tables(DevPlan pl, StageArgs a) {
  __shared__ uint64_t s_params;
  __shared__ double s_upd[kMaxTypes * kMaxTP];
  const int rs = blockIdx.x;
  const int n = pl.st_n[rs], first = pl.st_first[rs];
  const int G = pl.G, MB = pl.MB, TP = pl.TP;
  if (threadIdx.x == 0) {
    uint64_t p = 0;
    for (int l = first; l < first + n; ++l) p += a.layer_params[l];
    if (a.st_flags[rs] & 1) p += a.embed;
    if (a.st_flags[rs] & 2) p += a.head;
    s_params = p;
  }
  double *const row = pl.st_row + (size_t)rs * MB * TP * pl.row_w;  // [MB][TP][row_w]
  const int Lc = a.uniform ? 1 : a.L;
  for (int i = threadIdx.x; i < G * MB * TP; i += blockDim.x) {
    double f = 0.0, b = 0.0;
    if (a.uniform) {
      f = (double)n * a.t_fwd[i];
      b = (double)n * a.t_bwd[i];
    } else {
      const double *rf = a.t_fwd + (size_t)i * Lc, *rb = a.t_bwd + (size_t)i * Lc;
      for (int l = first; l < first + n; ++l) { f += rf[l]; b += rb[l]; }
    }
    pl.st_c[(size_t)rs * G * MB * TP + i] = f + b;
    row[(size_t)(i % (MB * TP)) * pl.row_w + i / (MB * TP)] = f + b;
    pl.st_f[(size_t)rs * G * MB * TP + i] = f;
    pl.st_b[(size_t)rs * G * MB * TP + i] = b;
  }
  for (int i = threadIdx.x; i < G * TP; i += blockDim.x) {
    double u = 0.0;
    if (a.uniform) {
      u = (double)n * a.t_upd[i];
    } else {
      const double *ru = a.t_upd + (size_t)i * Lc;
      for (int l = first; l < first + n; ++l) u += ru[l];
    }
    pl.st_u[(size_t)rs * G * TP + i] = u;
    s_upd[i] = u;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < MB * TP; i += blockDim.x) {
    const int k = i % TP;
    const uint64_t shard = (s_params + (uint64_t)pl.tpv[k] - 1) / (uint64_t)pl.tpv[k];
    double *const r = row + (size_t)i * pl.row_w + G;
    for (int g = 0; g < G; ++g) r[g] = s_upd[g * TP + k];
    r[G] = __longlong_as_double((long long)(shard * (uint64_t)pl.bpp));
    r[G + 1] = (double)shard * (double)pl.gb;
  }
}

// activation bytes of a worker: microbatches in flight x layers x bytes of one (validated < 2^62)
__device__ __forceinline__ uint64_t act_bytes(int in_flight, int layers, uint64_t act) {
  return (uint64_t)(uint32_t)in_flight * (uint32_t)layers * act;
}

// makes a wave's LDS writes visible to its own later reads (operations of one wave complete in
// order; the compiler must not move them)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Segment aggregates of one shape: everything of a segment that does not depend on
// the pool it is placed on.  One workgroup per shape; a thread per (degree, segment, ...) entry
// walks the segment's stages.  Bound by the latency of those walks: what a stage contributes is
// read ready-made from its record (st_row; the shard sizes were 64-bit divisions per entry and
// stage), the walks are unrolled so that their loads are in flight together, and eight waves per
// shape shorten them.  What one thread writes and another reads stays within the workgroup: a
// barrier orders it.  (A fence for the whole device behind the tables had every workgroup write its
// die's L2 back: about 1 000 shapes with pairs of types 218 us, without it 64.)
constexpr int kShapeAggThreads = 512;
__global__ __launch_bounds__(kShapeAggThreads) void k_shape_agg(DevPlan pl, DirectMem dm) {
  extern __shared__ float agg_lds[];  // [TP][3][Z], [TP][3][GX]
  const uint32_t shp = blockIdx.x;
  const ShapeRec sh = pl.shapes[shp];
  const int G = pl.G, GX = pl.GX, MB = pl.MB, TP = pl.TP, DP = pl.DP, P = sh.P;
  const int t = threadIdx.x, nt = blockDim.x;
  // (first stage and number of stages, 16 bits a segment: a record indexed by lane lies in scratch memory,
  // 48 bytes a lane, and about 1 000 shapes with pairs of types took 69 us instead of 64)
  const uint64_t los = sh.lo[0] | (uint64_t)sh.lo[1] << 16 | (uint64_t)sh.lo[2] << 32;
  const uint64_t ns = sh.n[0] | (uint64_t)sh.n[1] << 16 | (uint64_t)sh.n[2] << 32;
  auto lo_of = [&](int seg) { return (int)((los >> (16 * seg)) & 0xFFFFu); };
  auto n_of = [&](int seg) { return (int)((ns >> (16 * seg)) & 0xFFFFu); };
  const size_t row_stride = (size_t)MB * TP * pl.row_w;          // from stage to stage
  const double *const rows = pl.st_row + sh.row_stage * row_stride;
  // need[tp][seg][mb][dp], syncz, upd
  for (int it = t; it < TP * 3 * MB * DP; it += nt) {
    int d = it % DP, m = (it / DP) % MB, seg = (it / (DP * MB)) % 3, k = it / (DP * MB * 3);
    uint64_t mx = 0;
    const int64_t nb = pl.nb[m * DP + d];
    if (seg < sh.s && nb > 0) {
      const uint64_t act = pl.act[m * TP + k];
      const double *const shard_bytes = rows + (size_t)k * pl.row_w + 2 * G;
#pragma unroll 4
      for (int i = lo_of(seg); i < lo_of(seg) + n_of(seg); ++i) {
        const int64_t in_flight = (int64_t)(P - i) < nb ? (int64_t)(P - i) : nb;
        const uint64_t b = (uint64_t)__double_as_longlong(shard_bytes[i * row_stride]) +
                           act_bytes((int)in_flight, pl.st_n[sh.row_stage + i], act);
        mx = b > mx ? b : mx;
      }
    }
    pl.need[(agg_slot(pl, shp, k, seg) * MB + m) * DP + d] = mx;
  }
  // slowest all-reduce per zone and slowest update per type, then both by pool
  const size_t slot0 = agg_slot(pl, shp, 0, 0);
  float *const syncz = agg_lds, *const upd = agg_lds + TP * 3 * pl.Z;
  for (int it = t; it < TP * 3 * pl.Z; it += nt) {
    int z = it % pl.Z, seg = (it / pl.Z) % 3, k = it / (pl.Z * 3);
    double mx = 0.0;  // seconds of the slowest stage's gradient buffer over the zone's link
    if (seg < sh.s) {
      const double *const grads = rows + (size_t)k * pl.row_w + 2 * G + 1;
      const int lo = lo_of(seg), hi = lo + n_of(seg);
      if (pl.n_bw_coef > 0) {
        for (int i = lo; i < hi; ++i) {
          const double bytes = grads[i * row_stride];
          mx = fmax(mx, bytes / link_bw(pl, z, z, bytes));
        }
      } else {  // one bandwidth for all: the largest buffer is the slowest (division rounds monotonically)
#pragma unroll 4
        for (int i = lo; i < hi; ++i) mx = fmax(mx, grads[i * row_stride]);
        mx = mx / pl.bw[z * pl.Z + z];
      }
    }
    syncz[it] = (float)mx;
    pl.syncz[slot0 * pl.Z + it] = (float)mx;
  }
  for (int it = t; it < TP * 3 * GX; it += nt) {
    int g = it % GX, seg = (it / GX) % 3, k = it / (GX * 3);
    const int ga = pl.xt[g] & 255, gb = pl.xt[g] >> 8;
    double mx = 0.0;
    if (seg < sh.s) {
#pragma unroll 4
      for (int i = lo_of(seg); i < lo_of(seg) + n_of(seg); ++i) {
        mx = fmax(mx, pl.st_u[((size_t)(sh.row_stage + i) * G + ga) * TP + k]);
        mx = fmax(mx, pl.st_u[((size_t)(sh.row_stage + i) * G + gb) * TP + k]);
      }
    }
    upd[it] = (float)mx;
    pl.upd[slot0 * GX + it] = (float)mx;
  }
  for (int it = t; it < TP * 3 * GX * MB; it += nt) {
    int m = it % MB, g = (it / MB) % GX, seg = (it / (MB * GX)) % 3, k = it / (MB * GX * 3);
    const int ga = pl.xt[g] & 255, gb = pl.xt[g] >> 8;
    float4 v = make_float4(0.f, 0.f, kNegInf, kNegInf);
    if (seg < sh.s) {
      const int lo = lo_of(seg), n = n_of(seg);
      // replicas of two types: the slower one sets the stage's pace (straggler, Sec. 4.3)
      auto stage = [&](int i) {
        return fmax(pl.st_c[(((size_t)(sh.row_stage + i) * G + ga) * MB + m) * TP + k],
                    pl.st_c[(((size_t)(sh.row_stage + i) * G + gb) * MB + m) * TP + k]);
      };
      const double fst = stage(lo), lst = stage(lo + n - 1);
      double sum = fst, mxi = -__builtin_huge_val();
#pragma unroll 4
      for (int i = lo + 1; i < lo + n - 1; ++i) {
        const double c = stage(i);
        sum += c;
        mxi = fmax(mxi, c);
      }
      if (n > 1) sum += lst;
      v = make_float4((float)sum, (float)fst, (float)lst, (float)mxi);
    }
    pl.ta[(agg_slot(pl, shp, k, seg) * GX + g) * MB + m] = v;
  }
  __syncthreads();
  for (int it = t; it < TP * 3 * pl.ZG; it += nt) {
    const int p = it % pl.ZG, ks = it / pl.ZG, seg = ks % 3, k = ks / 3, z = p / GX, g = p - z * GX;
    dm.su[(slot0 + k * 3 + seg) * pl.ZG + p] = make_float2(syncz[ks * pl.Z + z], upd[ks * GX + g]);
  }
  // memok bit d: largest worker of the segment fits the type's memory
  for (int it = t; it < TP * 3 * GX * MB; it += nt) {
    int m = it % MB, g = (it / MB) % GX, seg = (it / (MB * GX)) % 3, k = it / (MB * GX * 3);
    const int ga = pl.xt[g] & 255, gb = pl.xt[g] >> 8;
    uint32_t bits = 0;
    if (seg < sh.s)
#pragma unroll 4
      for (int d = 0; d < DP; ++d) {
        uint64_t need = pl.need[(agg_slot(pl, shp, k, seg) * MB + m) * DP + d];
        if (pl.nb[m * DP + d] > 0 && need + pl.res[ga] <= pl.cap[ga] && need + pl.res[gb] <= pl.cap[gb])
          bits |= 1u << d;
      }
    pl.memok[(agg_slot(pl, shp, k, seg) * GX + g) * MB + m] = bits;
  }
}

// The range evaluation's units, a thread each.  (67 000 of them on 1.1e9 plans: laid out by the host
// and copied, and with allocations in front of the first pass instead of beside it, a new job there took
// 2 850 us, now 2 400.)
__global__ __launch_bounds__(256) void k_eval_units(const EvalBlock *blocks, int n_blocks, uint64_t n_units,
                                                    uint64_t inner, EvalUnit *out) {
  for (uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x; e < n_units; e += (uint64_t)gridDim.x * 256) {
    int lo = 0, hi = n_blocks;  // the last block that starts at or before the unit
    while (hi - lo > 1) {
      const int mid = (lo + hi) / 2;
      if (blocks[mid].first_unit <= e) lo = mid; else hi = mid;
    }
    const EvalBlock b = blocks[lo];
    const uint64_t shape = (e - b.first_unit) / b.per_shape, o = (e - b.first_unit - shape * b.per_shape) * b.chunk;
    EvalUnit u{};
    u.idx_lo = b.off + shape * b.shape_size + o * inner;
    u.shape = b.first_shape + (uint32_t)shape;
    u.o_lo = (uint32_t)o;
    u.o_cnt = (uint32_t)min((uint64_t)b.chunk, b.o_total - o);
    out[e] = u;
  }
}

// ------------------------------------------------------------------ fp32 evaluation

struct Rec {       // one segment placed on one pool, for one (mb, tp); 32 bytes
  float sumT;      // sum of its stage times without the cross-segment transfers
  float tF, tL;    // first / last stage time without the cross-segment transfers
  float tI;        // slowest interior stage
  float syncb;     // slowest stage: gradient bytes / intra-zone bandwidth
  float upd;       // slowest update
  float pricen;    // stages * tp * $/h: rent of one replica of the segment
  uint32_t bits;   // bit d: valid for dp index d (memory, quota, batch, H1)
};

struct LaneC {     // scalars of a (mb, dp) pair
  float nbm1, cd, dph, xb;
};

__device__ __forceinline__ Rec make_rec(float4 ta, float sync, float upd, float price, float w,
                                        int n, int tp, uint32_t bits) {
  Rec r;  // w: seconds of one transfer inside the zone
  r.sumT = fmaf((float)(2 * (n - 1)), w, ta.x);
  r.tF = (n == 1) ? ta.y : ta.y + w;
  r.tL = (n == 1) ? kNegInf : ta.z + w;
  r.tI = (n >= 3) ? fmaf(2.0f, w, ta.w) : kNegInf;
  r.syncb = sync;
  r.upd = upd;
  r.pricen = (float)(n * tp) * price;
  r.bits = bits;
  return r;
}

// A segment record in LDS: two 16-byte halves in arrays of their own (the records a wave reads
// together then lie 16 bytes apart and spread over all banks; 32-byte records leave half of
// them idle) and the validity bits once more in a dense array for the tests that need
// nothing else.
__device__ __forceinline__ void rec_store(float4 *lo, float4 *hi, uint32_t *bits, int i, const Rec &r) {
  lo[i] = make_float4(r.sumT, r.tF, r.tL, r.tI);
  hi[i] = make_float4(r.syncb, r.upd, r.pricen, __uint_as_float(r.bits));
  bits[i] = r.bits;
}

__device__ __forceinline__ Rec rec_load(const float4 *lo, const float4 *hi, int i) {
  const float4 a = lo[i], b = hi[i];
  Rec r;
  r.sumT = a.x; r.tF = a.y; r.tL = a.z; r.tI = a.w;
  r.syncb = b.x; r.upd = b.y; r.pricen = b.z;
  r.bits = __float_as_uint(b.w);
  return r;
}

// Iteration time and cost of a plan, accumulated segment by segment.  Everything that
// depends only on the leading segments is finished before the pool of the next segment
// is known, so the scan hoists it out of its inner loops; the order of the floating
// point additions is fixed here, and both evaluation kernels go through these steps, so
// they return bit-identical values.
struct Acc {
  float tmax;  // slowest stage of the closed segments
  float sum;   // sum of stage times incl. the transfers across closed boundaries
  float syn, up, pr, egs;
  float tf, tl, ti;  // open segment: first / last / slowest interior stage
};

// the first segment
__device__ __forceinline__ Acc acc_begin(const Rec &r) {
  Acc a;
  a.tmax = kNegInf;
  a.sum = r.sumT;
  a.syn = r.syncb;
  a.up = r.upd;
  a.pr = r.pricen;
  a.egs = 0.f;
  a.tf = r.tF;
  a.tl = r.tL;
  a.ti = r.tI;
  return a;
}

// Closes the open segment over a boundary with transfer times wf (activations, sent by the
// open segment's last stage) and wb (gradients, sent by the next segment's first stage),
// and opens segment r behind it.
__device__ __forceinline__ Acc acc_cross(const Acc &p, const Rec &r, float wf, float wb, float eg,
                                         bool open_is_single, bool first_boundary) {
  Acc a;
  // a one-stage segment's only stage also pays the outgoing transfer (fma with an exact
  // 0 / 1 factor equals the plain sum)
  const float tf = fmaf(open_is_single ? 1.0f : 0.0f, wf, p.tf);
  a.tmax = fmaxf(p.tmax, fmaxf(fmaxf(tf, p.tl + wf), p.ti));
  a.sum = (p.sum + r.sumT) + (wf + wb);
  a.syn = fmaxf(p.syn, r.syncb);
  a.up = fmaxf(p.up, r.upd);
  a.pr = p.pr + r.pricen;
  a.egs = first_boundary ? eg : p.egs + eg;
  a.tf = r.tF + wb;
  a.tl = r.tL;
  a.ti = r.tI;
  return a;
}

// Closes the last segment: T_iter = T_pp + T_sync + T_update, C_iter = C_comp + C_comm.
__device__ __forceinline__ void acc_finish(const Acc &p, const LaneC &lc, float &T, float &C) {
  const float tmax = fmaxf(p.tmax, fmaxf(fmaxf(p.tf, p.tl), p.ti));
  const float tpp = fmaf(lc.nbm1, tmax, p.sum);
  T = fmaf(lc.cd, p.syn, tpp) + p.up;
  C = fmaf(p.pr * lc.dph, T, lc.xb * p.egs);
}

// Quota table, rebuilt whenever the availability changes: a replica that takes w GPUs
// from a pool (its stages there times their tensor-parallel degrees) can be placed for
// the data-parallel degrees whose bit is set (Sec. 4: resource quotas).
// A pool that is a pair of types gives half of the replicas from each (an even number of
// them); qh serves plans whose segments draw on one real pool together: x half-GPUs per
// replica of the plan fit the real pool for the degrees whose bit is set.
// gen: the availability generation (0 while the plan is built); when an entry of qh changes,
// row_gen[0] receives it, so that a scan can tell whether the shared-pool checks of a unit's
// last evaluation still hold.  (A captured call passes the largest number: its replays come at any time.)
//
// table: the availability, which travels in the kernel's arguments -- no upload in front of the
// kernel, no trip over the bus inside it and nothing of the host's to wait for before it is used
// again.  mapped: the same in host-mapped memory instead, for a call under stream capture (a replay
// then reads what the host holds at the time).  Left in avail_copy (= pl.avail) for later kernels.
struct AvailTable { int32_t v[kMaxPools]; };

// bit d: dpv[d] replicas of w >= 1 GPUs fit a pool that has `avail` (the degrees ascend)
__device__ __forceinline__ uint32_t quota_bits(const DevPlan &pl, int32_t avail, int w) {
  const int32_t most = (int32_t)((uint32_t)avail / (uint32_t)w);
  uint32_t bits = 0;
  for (int d = 0; d < pl.DP; ++d) bits |= pl.dpv[d] <= most ? 1u << d : 0u;
  return bits;
}

__device__ __forceinline__ void quota_table(const DevPlan &pl, const int32_t *avail, uint32_t gen, uint32_t block,
                                            uint32_t n_blocks);

__global__ void k_quota_table(DevPlan pl, AvailTable table, const int32_t *mapped, int32_t *avail_copy, uint32_t gen) {
  __shared__ int32_t avail[kMaxPools];
  for (int r = threadIdx.x; r < pl.ZGr; r += blockDim.x) {
    avail[r] = mapped ? mapped[r] : table.v[r];
    if (blockIdx.x == 0) avail_copy[r] = avail[r];
  }
  __syncthreads();
  quota_table(pl, avail, gen, blockIdx.x, gridDim.x);
}

// The share of workgroup `block` of n_blocks.
__device__ __forceinline__ void quota_table(const DevPlan &pl, const int32_t *avail, uint32_t gen, uint32_t block,
                                            uint32_t n_blocks) {
  const int n = (pl.W_max + 1) * pl.ZG;
  for (int i = block * blockDim.x + threadIdx.x; i < n; i += n_blocks * blockDim.x) {
    const int p = i % pl.ZG, w = i / pl.ZG;
    const int x = pl.xt[p % pl.GX], ga = x & 255, gb = x >> 8, z = p / pl.GX;
    const int64_t avail_a = avail[z * pl.G + ga], avail_b = avail[z * pl.G + gb];
    uint32_t bits = 0;
    for (int d = 0; d < pl.DP; ++d) {
      const int64_t D = pl.dpv[d];
      if (ga == gb ? (int64_t)w * D <= avail_a
                   : (D % 2 == 0 && (int64_t)w * D <= 2 * avail_a && (int64_t)w * D <= 2 * avail_b))
        bits |= 1u << d;
    }
    pl.qw[i] = bits;
  }
  if (!pl.mixed) return;
  const int nh = (2 * pl.W_max + 1) * pl.ZGr;
  for (int i = block * blockDim.x + threadIdx.x; i < nh; i += n_blocks * blockDim.x) {
    const int r = i % pl.ZGr, x = i / pl.ZGr;
    const int64_t avail2 = 2 * (int64_t)avail[r];
    uint32_t bits = 0;
    for (int d = 0; d < pl.DP; ++d)
      if ((int64_t)x * pl.dpv[d] <= avail2) bits |= 1u << d;
    if (gen == 0u) {
      pl.qh[i] = bits;
    } else if (pl.qh[i] != bits) {
      pl.qh[i] = bits;
      atomicMax(&pl.row_gen[0], gen);
    }
  }
}

// Plans whose segments draw on one real pool together (possible once pairs of types exist):
// bit d is set when dpv[d] replicas of all segments fit every real pool.  p[j], w[j]: pool and
// GPUs per replica of segment j.
__device__ __forceinline__ uint32_t joint_quota_bits(const DevPlan &pl, int n_seg, int p0, int p1,
                                                     int p2, int w0, int w1, int w2) {
  // six slots (two per segment) of (real pool, half-GPUs per replica); constant trip counts,
  // so that everything stays in registers
  int r[6], h[6];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int p = j == 0 ? p0 : (j == 1 ? p1 : p2), w = j == 0 ? w0 : (j == 1 ? w1 : w2);
    const bool used = j < n_seg;
    const int x = pl.xt[used ? p % pl.GX : 0], ga = x & 255, gb = x >> 8, z = used ? p / pl.GX : 0;
    r[2 * j] = z * pl.G + ga;
    r[2 * j + 1] = z * pl.G + gb;
    h[2 * j] = !used ? 0 : (ga == gb ? 2 * w : w);
    h[2 * j + 1] = (!used || ga == gb) ? 0 : w;
  }
  uint32_t bits = 0xFFFFFFFFu;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    int total = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) total += (r[k] == r[i]) ? h[k] : 0;
    // (a pool that several slots name is checked several times against the same total)
    if (h[i] != 0) bits &= pl.qh[(size_t)total * pl.ZGr + r[i]];
  }
  return bits;
}

// SCAN: a unit's smallest key over the candidates strictly / loosely within the constraint.
// COLLECT: a unit's candidates under a threshold.  BEST: as SCAN, and a unit that comes within the tie
// band of the smallest key so far keeps its candidates at once.
enum { MODE_SCAN = 0, MODE_COLLECT = 1, MODE_BEST = 2 };

struct ScanArgs {
  float *umin_s, *umin_l;   // [n_units] minima over strictly / loosely constrained candidates
  uint32_t *counters;       // see Counter
  const uint32_t *tau_src;  // COLLECT: fp32 bits of the threshold, scaled by band ...
  float band;
  float tau_host;           // ... or, when use_tau_host is set, this threshold
  int use_tau_host;
  int count_only;           // COLLECT: count the candidates under the threshold, keep none
  uint32_t n_sub;           // workgroups that share one unit
  float lim_s, lim_l;       // constraint limits (strict, loose) on cost or on time
  SurvRec *surv;
  uint32_t surv_cap;
  const uint32_t *ulist;    // COLLECT, optional: the units to visit and, in counters[CNT_NLIST],
                            // how many; the grid then strides over the list.  SCAN, BEST: the order
                            // in which the units are launched, if it is not their own
  uint32_t *unit_gen;       // SCAN, optional: per unit, the availability generation its minima
  uint32_t cur_gen;         // were computed at; a scan stamps what it computes with cur_gen
  uint32_t *unit_seq;       // SCAN, with unit_gen: per unit, the call that evaluated it last
  uint32_t call_seq;
  int incremental;          // SCAN: units whose validity bits come out as they were at their
                            // last evaluation keep their minima and are not evaluated again
  uint32_t *ubits;          // SCAN, with unit_gen: per unit, the validity bits of its records
  uint32_t ubits_stride;    // (and the shared-pool quota words) as last staged; words per unit
  float near_band;          // BEST: the tie band.  A unit whose loose minimum lies within near_band of
                            // the smallest strict key seen so far appends its candidates up to there;
                            // the running minimum only falls, so every candidate within the band of
                            // the final one is among them.  SCAN with kth: what its keys may err by
  uint32_t kth;             // SCAN, if not 0: only units among which the kth smallest key lies matter; COLLECT
                            // behind it: the threshold is what SCAN's slots give for it (kth_of_slots)
  // Bounds of a unit's plans by data-parallel degree (k_group_bounds), [unit][2][DP]:
  const float *rows_con;    // with a constraint, of the constrained quantity: a degree beyond the loose limit
                            // holds nothing, and a unit without a degree left is not staged at all
                            // (Sec. 4.2.1, H3, applied to a part of the space)
  const float *rows_key;    // optional, of the objective: the same against what is known of the result -- the
                            // running minimum (BEST) or running kth smallest key (SCAN), COLLECT the threshold
  uint32_t n_seeds;         // SCAN, BEST with rows_key: so many units at the front of the order are shared by n_sub
                            // workgroups each
  uint32_t wait_ticks;      // the others wait for what these find, no longer than so many ticks (100 MHz)
  uint64_t most;            // the most replicas of one GPU that any pool holds: a degree D whose largest segment
                            // takes w GPUs a replica needs D w <= most
  int direct;               // COLLECT without a scan before it, BEST: ulist names the only units
  uint32_t n_list_host;     // whose bound meets the limit (n_list_host of them).  COLLECT: every
                            // candidate of theirs that is valid and within the loose limit is kept
  uint32_t fresh;           // BEST: the availability is new and travels with this launch (plain pools only): units
                            // take their quotas from it, and the `fresh` workgroups behind theirs
  int32_t *avail_copy;      // bring the quota table and the device's copy up to date
};

// Two sets, which a plan's calls use in turn; the final kernel of a call resets the next call's.
enum Counter { CNT_SURV = 0, CNT_OWNER = 1,      // number of the call the set belongs to (read with CNT_SURV)
               CNT_REF = 2, CNT_FEAS = 3, CNT_GMIN = 4, CNT_TAU0 = 5, CNT_TAU1 = 6,
               CNT_NLOOSE = 7, CNT_NSTRICT = 8,  // count-only collect passes
               CNT_NLIST = 9,                    // length of the collect pass's unit list
               CNT_DONE = 10,                    // workgroups of the final kernel that have finished
               CNT_COUNT = 16 };
// Behind a set's counters: the smallest keys that SCAN has come across, a word for the waves that share it;
// the same of the candidates that COLLECT keeps, a word for those whose index leads to it; and copies of the running limit, a cache line each, of which a workgroup reads one (thousands of workgroups
// that ask for one word, and the atomics that lower it, wait for one another: 8 us of a scan of 15).
constexpr uint32_t kKeySlots = 256, kLimitCopies = 16, kLimitStride = 32,
                   kKeptSlots = CNT_COUNT + kKeySlots, kCopies = kKeptSlots + kKeySlots,
                   kSetWords = kCopies + kLimitCopies * kLimitStride;
static_assert(CNT_SURV % 2 == 0 && CNT_OWNER == CNT_SURV + 1 && CNT_COUNT % 2 == 0, "one 8-byte word");

// c: a counter of the set that belongs to `call`
__device__ __forceinline__ uint32_t counter_reset_value(int c, uint32_t call) {
  if (c == CNT_OWNER) return call;
  return (c >= CNT_GMIN && c <= CNT_TAU1) || c >= CNT_COUNT ? 0x7f800000u : 0u;  // thresholds start at +inf
}

// zeroes the counters selected by mask (a fill kernel, usable under stream capture)
__global__ void k_zero_counters(uint32_t *c, uint32_t mask) {
  if (threadIdx.x < CNT_COUNT && ((mask >> threadIdx.x) & 1u)) c[threadIdx.x] = 0u;
}

// both sets, before `call`
__global__ void k_init_counters(uint32_t *c, uint32_t call) {
  for (uint32_t i = threadIdx.x; i < 2 * kSetWords; i += blockDim.x)
    c[i] = counter_reset_value((int)(i % kSetWords), call + ((i / kSetWords ^ call) & 1u));
}

struct NoAvail {};
template <int MODE, bool MIXED> constexpr bool kAvailRides = MODE == MODE_BEST && !MIXED;
template <int MODE, bool MIXED> using AvailArg = std::conditional_t<kAvailRides<MODE, MIXED>, AvailTable, NoAvail>;

// The candidates a workgroup keeps of a unit, gathered in LDS and appended to the survivors when the unit has
// been walked: one trip to the counter, where every wave made one for every chunk and pool at
// which it kept something, and waited for it.
constexpr uint32_t kKeptHere = 256;
struct Kept {
  unsigned long long idx[kKeptHere];
  uint32_t key[kKeptHere], where[kKeptHere];  // as in SurvRec (where: without the tp)
  uint32_t n, full, base;
};

__device__ __forceinline__ void survivor(const DevPlan &pl, const ScanArgs &a, const UnitRec &u, uint32_t slot,
                                         unsigned long long idx, uint32_t key, uint32_t where) {
  if (slot >= a.surv_cap) return;
  SurvRec sv;
  sv.idx = idx;
  sv.key = key;
  sv.row_stage = pl.shapes[u.shape].row_stage;
  sv.where = where | (uint32_t)u.tp[0] << 29;
  sv.segs = ((uint32_t)(u.n[0] - 1) & 255u) | ((uint32_t)(u.n[1] - 1) & 255u) << 8 | ((uint32_t)(u.n[2] - 1) & 255u) << 16 |
            (uint32_t)u.s << 24 | (uint32_t)u.tp[1] << 26 | (uint32_t)u.tp[2] << 29;
  a.surv[slot] = sv;
}

// (the workgroup, behind its walk of the unit)  A wave that found the list full has left its place empty
// there: the list ends before it.  drop (the first wave's word counts): none of it matters any more.
__device__ __forceinline__ void keep_flush(const DevPlan &pl, const ScanArgs &a, const UnitRec &u, Kept &kept, bool drop) {
  __syncthreads();
  uint32_t n = kept.n;
  if (n == 0) return;  // uniform
  if (n > kKeptHere) n = kept.full;
  if (threadIdx.x == 0) kept.base = drop ? ~0u : atomicAdd(&a.counters[CNT_SURV], n);
  __syncthreads();
  if (kept.base == ~0u) return;  // uniform
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    const uint32_t key = kept.key[i], idx = (uint32_t)kept.idx[i];
    if (!(key >> 31)) atomicMin(&a.counters[kKeptSlots + (idx * 0x9E3779B1u >> 24)], key);
    survivor(pl, a, u, kept.base + i, kept.idx[i], key, kept.where[i]);
  }
}
static_assert(kKeySlots == 256, "eight bits of a hash");

// One candidate of the scan: update the running minima, or keep it.
template <int MODE, int OBJ, bool HASB>
__device__ __forceinline__ void visit(const DevPlan &pl, const ScanArgs &a, const UnitRec &u, float T, float C, bool feas,
                                      float tau, uint64_t idx, uint32_t where, Kept &kept, float &ms, float &ml) {
  const float key = OBJ == 0 ? T : C;
  const float con = OBJ == 0 ? C : T;
  if (MODE != MODE_COLLECT) {
    const float kf = feas ? key : kPosInf;
    if (HASB) {
      ms = fminf(ms, con <= a.lim_s ? kf : kPosInf);
      ml = fminf(ml, con <= a.lim_l ? kf : kPosInf);
    } else {
      ms = fminf(ms, kf);
    }
  } else {
    const bool loose = feas && (!HASB || con <= a.lim_l);
    if (a.count_only) {  // uniform
      const bool strict = !HASB || con <= a.lim_s;
      const uint64_t m_loose = __builtin_amdgcn_ballot_w64(loose && key <= tau);
      const uint64_t m_strict = __builtin_amdgcn_ballot_w64(loose && strict && key <= tau);
      if (m_loose != 0 && (threadIdx.x & 63) == 0) {
        atomicAdd(&a.counters[CNT_NLOOSE], (uint32_t)__popcll(m_loose));
        if (m_strict != 0) atomicAdd(&a.counters[CNT_NSTRICT], (uint32_t)__popcll(m_strict));
      }
    } else {
      // the first lane that keeps its candidate reserves the places of all: in the workgroup's list, or, when
      // that is full, among the survivors at once
      const bool take = loose && key <= tau;
      const uint64_t m_take = __builtin_amdgcn_ballot_w64(take);
      if (m_take == 0) return;
      const uint32_t lane = threadIdx.x & 63u, n = (uint32_t)__popcll(m_take);
      const int leader = __builtin_ctzll(m_take);
      const bool strict = !HASB || con <= a.lim_s;
      uint32_t base = 0;
      if ((int)lane == leader) base = atomicAdd(&kept.n, n);
      base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
      const bool here = base + n <= kKeptHere;  // uniform over the wave
      if (!here) {
        if ((int)lane == leader && base <= kKeptHere) kept.full = base;  // (the one that crosses the end)
        if ((int)lane == leader) base = atomicAdd(&a.counters[CNT_SURV], n);
        base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
      }
      if (!take) return;
      const uint32_t slot = base + (uint32_t)__popcll(m_take & ((1ull << lane) - 1ull));
      const uint32_t bits = __float_as_uint(key) | (strict ? 0u : 1u << 31);
      if (here) {
        kept.idx[slot] = idx;
        kept.key[slot] = bits;
        kept.where[slot] = where;
      } else {
        survivor(pl, a, u, slot, idx, bits, where);
      }
    }
  }
}

// q = n / d for n * d < 2^32 with m = ceil(2^32 / d) (m = 0 encodes d = 1)
__device__ __forceinline__ uint32_t fast_div(uint32_t n, uint32_t m) {
  return m ? __umulhi(n, m) : n;
}

struct LaneItem {  // what a lane owns for one chunk of the lane space
  int mb, dp, a1;
  bool active;
  LaneC lc;
  uint32_t dpbit;
};

// Lane item e of a lane space laid out as mb + MB * (a1 + n_a1 * i), with i the position of its dp in the
// list s_dp: the dp digit is the slowest, so a wave holds one or two dp values and whole waves drop out
// together when their data-parallel degree cannot be placed.  mg = ceil(2^32 / (MB * n_a1)).
__device__ __forceinline__ LaneItem lane_item(const DevPlan &pl, int e, int n_items, int n_a1,
                                              uint32_t mg, const uint8_t *s_dp) {
  LaneItem it;
  it.active = e < n_items;
  const uint32_t ee = it.active ? (uint32_t)e : 0u;
  const uint32_t i = fast_div(ee, mg), rem = ee - i * (uint32_t)(pl.MB * n_a1), dp = s_dp[i];
  const uint32_t a1 = fast_div(rem, pl.mg_mb);
  it.a1 = (int)a1;
  it.dp = (int)dp;
  it.mb = (int)(rem - a1 * (uint32_t)pl.MB);
  it.lc.nbm1 = pl.nbm1_f[it.mb * pl.DP + it.dp];
  it.lc.cd = pl.cd_f[it.dp];
  it.lc.dph = pl.dph_f[it.dp];
  it.lc.xb = pl.xb_f[it.mb];
  it.dpbit = it.active ? (1u << it.dp) : 0u;
  return it;
}

__device__ __forceinline__ bool wave_any(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// Bounds of a group of units -- one shape, one tp per segment -- by data-parallel degree: rows[group] =
// the smallest iteration time per degree, then the smallest cost, of plans that memory, node size and
// batch allow, whatever the availability.  A segment's pool matters through its type and its zone.  Types
// are gone through exhaustively; of the zones only the best case is kept: the quickest link of the right
// kind (two neighbours of one type lie in different zones), the smallest egress, the quickest all-reduce.
// What the scan computes for a plan goes through the same operations on inputs that are no smaller, and
// fp32 additions, products, fused multiply-adds and maxima of non-negative values round monotonically: so
// a row's entry is at most the fp32 value of every plan it stands for, and needs no slack.  It is infinite
// exactly where there is no such plan.
//
// The types leave (types / pools)^segments of the plans, and what the segments add up to is shared by all
// degrees: MB x types^segments sums a group, bound by vector instructions.  On 1.1e9 plans with pairs of
// types 44 us, where a pass over every plan took 659 for one bound for all degrees.  On 1.0e8 plans as many
// units meet the budget and the cheapest plan by either; of 3 457 within reach of the 64 fastest remain 297
// with these bounds and 167 with exact ones.
constexpr int kGroupThreads = 256;  // (64 where all pairs of types are few)

struct GroupArgs {
  const EvalBlock *blocks;
  int n_blocks;
  const float *link_min;   // [MB] {within a zone, between zones}, egress
  uint64_t most;           // ScanArgs::most of the availability at creation
  float *rows;             // [group][2][DP]
  GroupSum *sums;          // [group]
};

__host__ __device__ inline size_t group_lds_bytes(int GX, int MB, int DP) {
  return (size_t)3 * GX * MB * (2 * sizeof(float4) + sizeof(uint32_t)) + (size_t)MB * DP * sizeof(float);
}

__global__ __launch_bounds__(kGroupThreads) void k_group_bounds(DevPlan pl, GroupArgs a) {
  extern __shared__ uint4 lds_raw[];
  __shared__ uint32_t s_row[2 * kMaxDP], s_seg2[4];
  const int GX = pl.GX, MB = pl.MB, DP = pl.DP, TP = pl.TP, Z = pl.Z, t = threadIdx.x, nt = blockDim.x;
  int blk = 0;
  for (int i = 1; i < a.n_blocks; ++i)
    if (blockIdx.x >= a.blocks[i].first_group) blk = i;
  const uint32_t per_shape = a.blocks[blk].groups, in_block = blockIdx.x - a.blocks[blk].first_group;
  const uint32_t shape = a.blocks[blk].first_shape + in_block / per_shape;
  const ShapeRec sh = pl.shapes[shape];
  const int S = sh.s;
  int k[3];  // tp index of each segment
  {
    uint32_t kk = in_block % per_shape;
    k[0] = (int)(kk % (uint32_t)TP);
    kk /= (uint32_t)TP;
    k[1] = pl.pst ? (int)(kk % (uint32_t)TP) : k[0];
    k[2] = pl.pst ? (int)(kk / (uint32_t)TP) : k[0];
  }
  float4 *const lo = reinterpret_cast<float4 *>(lds_raw), *const hi = lo + 3 * GX * MB;  // [S][GX][MB]
  uint32_t *const bits = reinterpret_cast<uint32_t *>(hi + 3 * GX * MB);
  float *const nbm1 = reinterpret_cast<float *>(bits + 3 * GX * MB);  // [MB][DP]
  uint32_t even = 0;  // degrees that can be halved
  for (int d = 0; d < DP; ++d) even |= pl.dpv[d] % 2 == 0 ? 1u << d : 0u;
  for (int i = t; i < S * GX * MB; i += nt) {
    const int m = i % MB, x = i / MB % GX, seg = i / (MB * GX);
    const int kt = at3(k, seg), n = at3(sh.n, seg);
    const uint32_t sl = (shape * (uint32_t)TP + (uint32_t)kt) * 3u + (uint32_t)seg, gi = (sl * (uint32_t)GX + (uint32_t)x) * (uint32_t)MB + (uint32_t)m;
    float sync = pl.syncz[sl * Z];
    for (int z = 1; z < Z; ++z) sync = fminf(sync, pl.syncz[sl * Z + z]);
    uint32_t b = pl.memok[gi] & pl.divis[m];
    if ((pl.xt[x] & 255) != pl.xt[x] >> 8) b &= even;
    if ((pl.h1m[x] >> kt) & 1u) b = 0;  // (pool x: type x in the first zone)
    rec_store(lo, hi, bits, i, make_rec(pl.ta[gi], sync, pl.upd[sl * GX + x], pl.price_f[x], a.link_min[2 * m], n, pl.vals[DP + kt], b));
  }
  for (int i = t; i < MB * DP; i += nt) nbm1[i] = pl.nbm1_f[i];
  if (t < 2 * DP) s_row[t] = __float_as_uint(kPosInf);
  if (t < 4) s_seg2[t] = S >= 2 ? 0u : ~0u;
  __syncthreads();
  const float eg_out = Z > 1 ? a.link_min[2 * MB] : 0.f;
  float low_t[kMaxDP], low_c[kMaxDP];
#pragma unroll
  for (int d = 0; d < kMaxDP; ++d) low_t[d] = low_c[d] = kPosInf;
  const uint32_t n_items = (uint32_t)MB * (uint32_t)GX * (S >= 2 ? (uint32_t)GX : 1u) * (S == 3 ? (uint32_t)GX : 1u);
  for (uint32_t e = t; e < n_items; e += nt) {
    const uint32_t r1 = fast_div(e, pl.mg_mb), m = e - r1 * (uint32_t)MB;
    const uint32_t r2 = fast_div(r1, pl.mg_g), x0 = r1 - r2 * (uint32_t)GX;
    const uint32_t x2 = fast_div(r2, pl.mg_g), x1 = r2 - x2 * (uint32_t)GX;
    const uint32_t i0 = x0 * MB + m, i1 = (GX + x1) * MB + m, i2 = (2 * GX + x2) * MB + m;
    uint32_t b = bits[i0];
    if (S >= 2) b &= (Z > 1 || x0 != x1) ? bits[i1] : 0u;  // neighbours lie on different pools
    if (S == 3) b &= (Z > 1 || x1 != x2) ? bits[i2] : 0u;
    if (!wave_any(b != 0)) continue;
    const float t_in = a.link_min[2 * m], t_out = Z > 1 ? a.link_min[2 * m + 1] : t_in, t_any = fminf(t_in, t_out);
    Acc p = acc_begin(rec_load(lo, hi, (int)i0));
    if (S >= 2) {
      const float w = x0 == x1 ? t_out : t_any;
      p = acc_cross(p, rec_load(lo, hi, (int)i1), w, w, x0 == x1 ? eg_out : 0.f, sh.n[0] == 1, true);
    }
    if (S == 3) {
      const float w = x1 == x2 ? t_out : t_any;
      p = acc_cross(p, rec_load(lo, hi, (int)i2), w, w, x1 == x2 ? eg_out : 0.f, sh.n[1] == 1, false);
    }
    LaneC lc;
    lc.xb = pl.xb_f[m];
#pragma unroll
    for (int d = 0; d < kMaxDP; ++d) {
      if (d < DP) {  // uniform
        lc.nbm1 = nbm1[m * DP + d];
        lc.cd = pl.cd_f[d];
        lc.dph = pl.dph_f[d];
        float T, C;
        acc_finish(p, lc, T, C);
        const bool ok = (b >> d) & 1u;
        low_t[d] = fminf(low_t[d], ok ? T : kPosInf);
        low_c[d] = fminf(low_c[d], ok ? C : kPosInf);
      }
    }
    if (S >= 2 && b != 0) atomicOr(&s_seg2[x1 >> 5], 1u << (x1 & 31u));
  }
#pragma unroll
  for (int d = 0; d < kMaxDP; ++d) {
    if (d < DP) {
      const uint32_t mt = wave_min_u32(__float_as_uint(low_t[d])), mc = wave_min_u32(__float_as_uint(low_c[d]));
      if ((t & 63) == 0) {
        atomicMin(&s_row[d], mt);
        atomicMin(&s_row[DP + d], mc);
      }
    }
  }
  __syncthreads();
  if (t < 2 * DP) a.rows[(size_t)blockIdx.x * 2 * DP + t] = __uint_as_float(s_row[t]);
  if (t == 0) {
    uint64_t w = 0;
    for (int seg = 0; seg < S; ++seg) w = max(w, (uint64_t)at3(sh.n, seg) * (uint64_t)pl.vals[DP + at3(k, seg)]);
    uint32_t mt = 0x7f800000u, mc = 0x7f800000u, now = 0x7f800000u;
    for (int d = 0; d < DP; ++d) {
      mt = min(mt, s_row[d]);
      mc = min(mc, s_row[DP + d]);
      if ((uint64_t)pl.dpv[d] * w <= a.most) now = min(now, s_row[d]);
    }
    a.sums[blockIdx.x] = GroupSum{__uint_as_float(now), __uint_as_float(mt), __uint_as_float(mc), {s_seg2[0], s_seg2[1], s_seg2[2], s_seg2[3]}};
  }
}

// An upper bound of the k-th smallest of a set's key slots, by one wave: the leading bits of that value,
// the others set.  (+inf while fewer than k slots hold a key.)
__device__ __forceinline__ uint32_t kth_of_slots(const uint32_t *slots, uint32_t k) {
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t v[kKeySlots / 64];
#pragma unroll
  for (uint32_t i = 0; i < kKeySlots / 64; ++i)
    v[i] = __hip_atomic_load(&slots[lane + 64 * i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  auto below = [&](uint32_t x) {  // how many are
    uint32_t n = 0;
#pragma unroll
    for (uint32_t i = 0; i < kKeySlots / 64; ++i) n += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(v[i] < x));
    return n;
  };
  constexpr int kCoarse = 10;  // (13 bits of mantissa: 1e-4 above the value at most)
  if (below(0x7f800000u) < k) return 0x7f800000u;
  uint32_t at = 0;
  for (int bit = 30; bit >= kCoarse; --bit)
    if (below(at | 1u << bit) < k) at |= 1u << bit;
  return at | ((1u << kCoarse) - 1u);
}

// The slot of a workgroup's wave: where those of the first waves would come round to the same ones, they move on by one.
__device__ __forceinline__ uint32_t key_slot(uint32_t workgroup, uint32_t waves, uint32_t wave) {
  return (workgroup * waves + workgroup * (waves & (0u - waves)) / kKeySlots + wave) % kKeySlots;
}

// What a launch knows of the result while it runs.  BEST: the smallest strict key so far.  SCAN with kth: a
// key that at least kth candidates do not exceed.  Keys go to slots, each candidate's to one, and as every
// slot keeps its smallest, kth slots that hold a key up to some value are as many candidates up to it.
__device__ __forceinline__ uint32_t *limit_copy(const ScanArgs &a, uint32_t i) {
  return &a.counters[kCopies + i % kLimitCopies * kLimitStride];
}
__device__ __forceinline__ uint32_t running_limit(const ScanArgs &a) {
  return __hip_atomic_load(limit_copy(a, blockIdx.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// (a wave) the copies, and the smallest key for the kernels behind this one
template <int MODE>
__device__ __forceinline__ void lower_limit(const ScanArgs &a, uint32_t to) {
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t *const word = lane < kLimitCopies ? limit_copy(a, lane) : &a.counters[CNT_GMIN];
  if (lane < kLimitCopies + (MODE == MODE_BEST ? 1u : 0u)) atomicMin(word, to);
}

// The rows of the units' groups, unit by unit, so that a workgroup asks for them together with its record.
__global__ __launch_bounds__(256) void k_unit_rows(const UnitRec *units, const float *rows, uint32_t n_units, uint32_t width,
                                                   float *out) {
  const size_t n = (size_t)n_units * width;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
    out[i] = rows[(size_t)units[i / width].group * width + i % width];
}

// How long each unit takes, roughly, where nothing rules out the plans that are valid under the present
// availability; as a bucket, an eighth of an octave wide, the longest first.  A wave a unit: per segment and degree
// how many pools hold the segment, with any microbatch size; of the lane space that leaves so many chunks alive, each
// of which goes through the pools of the next segments, at four times the price where those hold theirs.  (Bound by
// trips to memory; with the kernel behind it 31 us for 16 037 units and 17 for 7 797, once a plan.  129 cheapest of the
// latter's 1.1e9 plans 335 us in the order of the units' bounds, 243 in this one, 257 in that of a timed pass over
// the space at creation, which took 254.)
constexpr int kWorkBuckets = 256;

__global__ __launch_bounds__(256) void k_unit_work(DevPlan pl, uint8_t *bucket) {
  const int lane = threadIdx.x & 63, ZG = pl.ZG, G = pl.GX, MB = pl.MB;
  const float most_chunks = (float)((MB * ZG + 63) / 64);
  for (uint32_t uidx = blockIdx.x * 4u + (threadIdx.x >> 6); uidx < (uint32_t)pl.n_units; uidx += gridDim.x * 4u) {  // uniform
    const UnitRec &u = pl.units[uidx];
    float holds[3] = {0.f, 0.f, 0.f};  // of degree `lane`
#pragma unroll
    for (int seg = 0; seg < 3; ++seg) {
      if (seg >= u.s) continue;
      const int k = at3(u.tp, seg), w = at3(u.n, seg) * pl.vals[pl.DP + k];
      const uint32_t sl = (u.shape * (uint32_t)pl.TP + (uint32_t)k) * 3u + (uint32_t)seg;
      const int from = seg == 1 ? (int)u.o_lo : 0, to = seg == 1 ? (int)u.o_lo + (int)u.o_cnt : ZG;
      for (int p0 = from; p0 < to; p0 += 64) {
        const int p = p0 + lane;
        uint32_t bits = 0;
        if (p < to) {
          const uint32_t g = (uint32_t)p - fast_div((uint32_t)p, pl.mg_g) * (uint32_t)G;
          for (int mb = 0; mb < MB; ++mb) bits |= pl.memok[(sl * (uint32_t)G + g) * (uint32_t)MB + (uint32_t)mb] & pl.divis[mb];
          bits &= pl.qw[w * ZG + p];
          if ((pl.h1m[p] >> k) & 1u) bits = 0;
        }
        for (int d = 0; d < pl.DP; ++d) {
          const float n = (float)__popcll(__builtin_amdgcn_ballot_w64((bits >> d) & 1u));
          if (lane == d) holds[seg] += n;
        }
      }
    }
    float work = fminf(most_chunks, holds[0]);
    if (u.s == 2) work *= holds[1] > 0.f ? (float)u.o_cnt + 4.f * holds[1] : 0.f;
    if (u.s == 3) work *= holds[2] > 0.f ? holds[1] * ((float)ZG + 4.f * holds[2]) : 0.f;
    for (int off = 32; off >= 1; off >>= 1) work += __shfl_xor(work, off);
    const int at = (int)(__float_as_uint(1.f + work) >> 20) - (127 << 3);
    if (lane == 0) bucket[uidx] = (uint8_t)(kWorkBuckets - 1 - min(at, kWorkBuckets - 1));
  }
}

// The units by bucket.  One workgroup.
__global__ __launch_bounds__(1024) void k_work_order(const uint8_t *bucket, uint32_t n, uint32_t *order) {
  __shared__ uint32_t s_at[kWorkBuckets];
  const uint32_t t = threadIdx.x;
  if (t < (uint32_t)kWorkBuckets) s_at[t] = 0;
  __syncthreads();
  for (uint32_t i = t; i < n; i += 1024) atomicAdd(&s_at[bucket[i]], 1u);
  __syncthreads();
  if (t < 64) {
    uint32_t mine[kWorkBuckets / 64], sum = 0;
    for (int j = 0; j < kWorkBuckets / 64; ++j) { mine[j] = s_at[t * (kWorkBuckets / 64) + (uint32_t)j]; sum += mine[j]; }
    uint32_t at = wave_prefix_sum(sum) - sum;
    for (int j = 0; j < kWorkBuckets / 64; ++j) { s_at[t * (kWorkBuckets / 64) + (uint32_t)j] = at; at += mine[j]; }
  }
  __syncthreads();
  for (uint32_t i = t; i < n; i += 1024) order[atomicAdd(&s_at[bucket[i]], 1u)] = i;
}

// What a workgroup walks of its unit: the degrees listed in s_dp, and its share of the lane space's chunks and
// of the innermost loop.
struct Walk {
  const uint8_t *s_dp;
  int n_dp, chunk, n_chunk, inner, n_inner;
};

// The lanes of a workgroup own the (mb, pool of segment 1, dp) triples; the pools of the
// later segments are walked in uniform loops, so their record addresses, zones and
// transfer terms are the same for the whole wave.
//   one or two segments: lanes cover every pool 1; in the loop over pool 2 a lane whose own
//     pool equals it sits that iteration out;
//   three segments: pool 2 is the outer uniform loop, lanes cover the ZG - 1 other pools,
//     pool 3 is the inner uniform loop.
// Invalid plans are pruned early (cf. H2, Sec. 4.2.1): as soon as the validity bits of the
// segments placed so far are zero in every lane of a wave, the wave skips everything that
// depends on the remaining segments.
// With pairs of types (MIXED) different pools can draw on one real pool; the plans concerned
// (isect) get the joint quota check, the others keep the per-segment bits.
//
// Plans that cannot matter are pruned as early: closing a plan after its leading segments
// (acc_finish on what acc_begin / acc_cross gave so far) bounds its time and cost from below.
// Segments only add to the sums and raise the maxima, and fp32 additions, products and maxima of
// non-negative values round monotonically, so the bound holds for the very values that the full
// evaluation returns, and no minimum and no kept candidate changes.  A lane is dropped when the
// bound lies above the smallest key its workgroup has found (kept in LDS), above the threshold
// the caller knows, or above the loose limit.  For the fastest plan the lane space is walked from the
// largest data-parallel degrees down, for the cheapest from the smallest up: what is small early prunes
// most (cheapest of 1.9e7 plans with a TP degree per segment: 59 us down, 53 up).
//
// live: a degree whose bound (s_rows) lies above the limit falls without a record read.  follows: what other
// workgroups have found counts as well.  The first wave asks for the running limit once per round, and takes
// the answer to the question before, so that no round waits for it.
template <int S, int MODE, int OBJ, bool HASB, bool MIXED>
__device__ __forceinline__ void unit_body(const DevPlan &pl, const ScanArgs &a, const UnitRec &u,
                                          const float4 *rec_lo, const float4 *rec_hi,
                                          const uint32_t *rbits, const float4 *pair,
                                          const uint32_t *q13, const uint64_t *isect, int w0,
                                          int w1, int w2, float tau, const Walk &wk,
                                          const float *s_rows, bool live, bool follows,
                                          uint32_t *s_min, Kept &kept, float &ms, float &ml) {
  // the chunks of the lane space are dealt round-robin to the waves of the workgroups that share the unit
  const int ZG = pl.ZG, G = pl.GX, MB = pl.MB, DP = pl.DP, Z = pl.Z;
  const int lane = threadIdx.x & 63;
  const int wave = (int)(threadIdx.x >> 6) + (int)(blockDim.x >> 6) * wk.chunk;
  const int nwave = (int)(blockDim.x >> 6) * wk.n_chunk;
  const bool single0 = u.n[0] == 1, single1 = u.n[1] == 1;
  const int tp = u.tp[0];
  const uint64_t ubase = u.base;
  // the limit in force: the smallest strict key so far, COLLECT the threshold
  uint32_t asked = 0x7f800000u;
  auto ask = [&]() {  // (in front of a loop without loads from memory: they would wait for it)
    if (MODE != MODE_COLLECT && follows && threadIdx.x < 64)
      asked = running_limit(a);
  };
  auto limit = [&]() {
    if (MODE == MODE_COLLECT) return tau;
    if (follows && threadIdx.x == 0) atomicMin(s_min, __float_as_uint(__uint_as_float(asked) * a.near_band));
    return __uint_as_float(__hip_atomic_load(s_min, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
  };
  // can plans of this degree still matter?
  auto alive_row = [&](int dp, float l0) { return MODE == MODE_COLLECT || !live || s_rows[dp] <= l0; };
  // can a plan that starts like this still matter?
  auto alive = [&](const Acc &p, const LaneC &lc, float l0) {
    float T, C;
    acc_finish(p, lc, T, C);
    const float key = OBJ == 0 ? T : C, con = OBJ == 0 ? C : T;
    return key <= l0 && (!HASB || con <= a.lim_l);
  };
  // (one thread of the waves that improve on what the workgroup has)
  auto report = [&](float l0) {
    if (MODE == MODE_COLLECT) return;
    if (wave_any(ms < l0)) {
      const float m = wave_min(ms);
      if (lane == 0) atomicMin(s_min, __float_as_uint(m));
    }
  };
  if (S <= 2) {
    const int nin = S == 1 && wk.inner != 0 ? 0 : MB * wk.n_dp * ZG;
    const int o_from = u.o_lo + u.o_cnt * wk.inner / wk.n_inner, o_to = u.o_lo + u.o_cnt * (wk.inner + 1) / wk.n_inner;
    const int rounds = (nin - 1 - wave * 64 + nwave * 64) / (nwave * 64);  // (0 for waves beyond the lane space)
    for (int i = 0; i < rounds; ++i) {
      const int e0 = (wave + (OBJ == 0 ? rounds - 1 - i : i) * nwave) * 64;
      const LaneItem it = lane_item(pl, e0 + lane, nin, ZG, pl.mg_mbzg, wk.s_dp);
      const int a1 = it.a1;
      const float l0 = limit();
      uint32_t b0 = alive_row(it.dp, l0) ? rbits[a1 * MB + it.mb] & it.dpbit : 0u;
      if (!wave_any(b0 != 0)) continue;
      const Rec r0 = rec_load(rec_lo, rec_hi, a1 * MB + it.mb);
      const int z1 = (int)fast_div((uint32_t)a1, pl.mg_g);
      const float4 *pair1 = pair + (it.mb * Z + z1) * Z;  // transfers out of this lane's first zone
      const Acc A0 = acc_begin(r0);
      // index of the candidate whose outer digits are all zero
      const uint64_t idx0 = ubase + (uint64_t)(it.mb + MB * (tp + pl.TP * (it.dp + DP * a1)));
      const uint32_t where0 = (uint32_t)a1 | (uint32_t)it.mb << 21 | (uint32_t)it.dp << 24;
      if (S == 1) {
        float T, C;
        acc_finish(A0, it.lc, T, C);
        visit<MODE, OBJ, HASB>(pl, a, u, T, C, b0 != 0, tau, idx0, where0, kept, ms, ml);
        continue;
      }
      if (!alive(A0, it.lc, l0)) b0 = 0;
      if (!wave_any(b0 != 0)) continue;
      ask();
      int z2 = o_from / G, g2 = o_from % G;
      for (int a2 = o_from; a2 < o_to; ++a2) {
        const int i1 = (ZG + a2) * MB + it.mb;
        uint32_t b1 = (a1 != a2) ? (b0 & rbits[i1]) : 0u;
        if (MIXED && b1 != 0 && pool_bit(isect, a2, a1))
          b1 &= joint_quota_bits(pl, 2, a1, a2, 0, w0, w1, 0);
        if (wave_any(b1 != 0)) {
          const Rec r1 = rec_load(rec_lo, rec_hi, i1);
          const float4 p12 = pair1[z2];
          const Acc A1 = acc_cross(A0, r1, p12.x, p12.y, p12.z, single0, true);
          int rel2 = a2 - a1 - 1;
          if (rel2 < 0) rel2 += ZG;
          float T, C;
          acc_finish(A1, it.lc, T, C);
          visit<MODE, OBJ, HASB>(pl, a, u, T, C, b1 != 0, tau,
                                 idx0 + (uint64_t)pl.inner * (uint64_t)rel2, where0 | (uint32_t)a2 << 7, kept, ms, ml);
        }
        if (++g2 == G) { g2 = 0; ++z2; }
      }
      report(l0);
    }
  } else {
    const int nin = MB * wk.n_dp * (ZG - 1);
    const int p_from = ZG * wk.inner / wk.n_inner, p_to = ZG * (wk.inner + 1) / wk.n_inner;
    const int rounds = (nin - 1 - wave * 64 + nwave * 64) / (nwave * 64);
    int z2 = u.o_lo / G, g2 = u.o_lo % G;
    for (int a2 = u.o_lo; a2 < u.o_lo + u.o_cnt; ++a2) {
      for (int i = 0; i < rounds; ++i) {
        const int e0 = (wave + (OBJ == 0 ? rounds - 1 - i : i) * nwave) * 64;
        const LaneItem it = lane_item(pl, e0 + lane, nin, ZG - 1, pl.mg_mbzg1, wk.s_dp);
        const int a1 = it.a1 + (it.a1 >= a2 ? 1 : 0);  // skip the pool of segment 2
        const int i0 = a1 * MB + it.mb, i1 = (ZG + a2) * MB + it.mb;
        const float l0 = limit();
        uint32_t b1 = alive_row(it.dp, l0) ? rbits[i0] & it.dpbit & rbits[i1] : 0u;
        if (!wave_any(b1 != 0)) continue;
        const Rec r0 = rec_load(rec_lo, rec_hi, i0);
        const Rec r1 = rec_load(rec_lo, rec_hi, i1);
        const int z1 = (int)fast_div((uint32_t)a1, pl.mg_g);
        const float4 *pairm = pair + it.mb * Z * Z;
        const float4 p12 = pairm[z1 * Z + z2];
        const Acc A1 = acc_cross(acc_begin(r0), r1, p12.x, p12.y, p12.z, single0, true);
        if (!alive(A1, it.lc, l0)) b1 = 0;
        if (!wave_any(b1 != 0)) continue;
        const uint32_t q13a = MIXED ? 0u : q13[a1];
        int rel2 = a2 - a1 - 1;
        if (rel2 < 0) rel2 += ZG;
        const uint64_t idx0 = ubase + (uint64_t)(it.mb + MB * (tp + pl.TP * (it.dp + DP * a1))) +
                              (uint64_t)pl.inner * (uint64_t)rel2;
        const uint32_t where0 = (uint32_t)a1 | (uint32_t)a2 << 7 | (uint32_t)it.mb << 21 | (uint32_t)it.dp << 24;
        ask();
        int z3 = p_from / G, g3 = p_from % G;
        for (int a3 = p_from; a3 < p_to; ++a3) {
          if (a3 != a2) {  // uniform
            const int i2 = (2 * ZG + a3) * MB + it.mb;
            uint32_t b2 = b1 & rbits[i2];
            if (MIXED) {
              if (b2 != 0 && (pool_bit(isect, a2, a1) || pool_bit(isect, a2, a3) || pool_bit(isect, a3, a1)))
                b2 &= joint_quota_bits(pl, 3, a1, a2, a3, w0, w1, w2);
            } else if (a3 == a1) {
              b2 &= q13a;  // segments 1 and 3 share one pool's quota
            }
            if (wave_any(b2 != 0)) {
              const Rec r2 = rec_load(rec_lo, rec_hi, i2);
              const float4 p23 = pairm[z2 * Z + z3];
              const Acc A2 = acc_cross(A1, r2, p23.x, p23.y, p23.z, single1, false);
              int rel3 = a3 - a2 - 1;
              if (rel3 < 0) rel3 += ZG;
              float T, C;
              acc_finish(A2, it.lc, T, C);
              visit<MODE, OBJ, HASB>(pl, a, u, T, C, b2 != 0, tau,
                                     idx0 + pl.stride3 * (uint64_t)rel3, where0 | (uint32_t)a3 << 14, kept, ms, ml);
            }
          }
          if (++g3 == G) { g3 = 0; ++z3; }
        }
        report(l0);
      }
      if (++g2 == G) { g2 = 0; ++z2; }
    }
  }
}

// The smallest strict key so far, by the way that a call's workgroups make it known.
__device__ __forceinline__ uint32_t smallest_key(const ScanArgs &a, bool live) {
  return live ? running_limit(a) : __hip_atomic_load(&a.counters[CNT_GMIN], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Folds a scanned unit's minima into the global minimum.  One wave.  Returns (best plan) the
// threshold up to which the unit's candidates are kept, or -1 if it has none that near.
__device__ __forceinline__ float unit_publish(const ScanArgs &a, bool live, uint32_t seen, float ms, float ml) {
  // keys are non-negative, so their bit patterns order like unsigned integers
  // (a stale `seen` only costs redundant atomics; most units lose and skip theirs)
  if (__float_as_uint(ms) < seen) {
    if (live) lower_limit<MODE_BEST>(a, __float_as_uint(ms));
    else if ((threadIdx.x & 63u) == 0) atomicMin(&a.counters[CNT_GMIN], __float_as_uint(ms));
  }
  // (a stale `seen` is larger than the true running minimum: more is kept, nothing is lost)
  const float tau = fminf(__uint_as_float(seen), ms) * a.near_band;
  return ml < kPosInf && ml <= tau ? tau : -1.0f;
}

// LDS of a scan workgroup: the records of [3][ZG][MB] (segment, pool, mb) as two float4 arrays
// and a dense array of their validity bits, the transfer table, the shared-pool masks.
__host__ __device__ inline size_t unit_lds_records(int ZG, int MB) {
  return ((size_t)3 * ZG * MB + 3) & ~(size_t)3;  // a multiple of 4, so that what follows stays 16-byte aligned
}

// What a pass leaves behind for a unit.  One thread (sub: of the first of the workgroups that share the
// unit).  The minima are read where a pass follows that visits units by them: a shared unit, whose
// workgroups each know a part of it, is visited in any case.  What the constraint or the running minimum rules
// out is not counted as evaluated; what falls to the availability or to a k-th key is.
template <int MODE>
__device__ __forceinline__ void unit_done(const ScanArgs &a, uint32_t uidx, int sub, uint32_t n_sub, float ms, float ml, bool counts) {
  if (MODE == MODE_COLLECT || (MODE == MODE_BEST && a.direct) || sub != 0) return;
  const bool shared = n_sub > 1;
  a.umin_s[uidx] = shared ? 0.f : ms;
  a.umin_l[uidx] = shared ? 0.f : ml;
  if (a.unit_gen) {
    a.unit_gen[uidx] = a.cur_gen;
    if (counts) a.unit_seq[uidx] = a.call_seq;
  }
}

// A lane's test of a unit: is there a degree that can matter?  (unit_work finds out which, and asks for the
// limit once more.)
template <int MODE, bool HASB>
__device__ __forceinline__ bool unit_test(const DevPlan &pl, const ScanArgs &a, uint32_t uidx, float key_limit) {
  const UnitRec &u = pl.units[uidx];
  const float *const con = a.rows_con + (size_t)uidx * 2 * pl.DP, *const key = a.rows_key + (size_t)uidx * 2 * pl.DP;
  uint64_t w = 0;
#pragma unroll
  for (int j = 0; j < 3; ++j) w = max(w, (uint64_t)u.n[j] * (uint32_t)pl.vals[pl.DP + u.tp[j]]);
  bool any = false, meets = false, near = false;
#pragma unroll 4
  for (int d = 0; d < pl.DP; ++d) {
    const bool m = !HASB || con[d] <= a.lim_l, n = key[d] <= key_limit;
    any |= m && n && (uint64_t)pl.dpv[d] * w <= a.most;
    meets |= m;
    near |= n;
  }
  if (!any) unit_done<MODE>(a, uidx, 0, 1u, kPosInf, kPosInf, meets && (MODE != MODE_BEST || near));
  return any;
}

// One workgroup per unit: stage the unit's segment records in LDS, then every lane walks
// its (mb, dp, pool 1) triple over the unit's outer pool digits.  Everything the staging
// needs comes from the unit record and tables that do not depend on one another, so all of
// its global loads are in flight together and one barrier ends it.  may_wait: for the running limit, if there is
// none yet (GUIDED) and the unit has a degree that could matter.
template <int MODE, int OBJ, bool HASB, bool MIXED, bool GUIDED>
__device__ __forceinline__ void unit_work(const DevPlan &pl, const ScanArgs &a, const AvailArg<MODE, MIXED> &avail,
                                          uint32_t uidx, int sub, uint32_t n_sub, float tau, bool may_wait, uint4 *lds_raw) {
  const UnitRec u = pl.units[uidx];
  const bool fresh = kAvailRides<MODE, MIXED> && a.fresh != 0;
  const bool live = MODE != MODE_COLLECT && a.rows_key != nullptr;
  const bool follows = live && (MODE == MODE_BEST || GUIDED);  // a k-th key has a running limit where seeds find it only
  const int n0 = u.n[0], n1 = u.n[1], n2 = u.n[2];
  const int k0 = u.tp[0], k1 = u.tp[1], k2 = u.tp[2];            // tp index of each segment
  const int tv0 = pl.tpv[k0], tv1 = pl.tpv[k1], tv2 = pl.tpv[k2];
  const int w0 = n0 * tv0, w1 = n1 * tv1, w2 = n2 * tv2;        // GPUs of one replica
  // The degrees that can matter, the same in every wave: the running limit changes while the workgroup
  // reads it, so one thread reads and all follow.
  __shared__ float s_rows[kMaxDP];
  uint32_t degrees, fixed;  // (fixed: those that the workgroups which share a unit agree on)
  bool counts;  // not ruled out by the constraint or the running minimum
  float key_limit = tau;
  {
    __shared__ uint32_t s_seen;
    const int d = threadIdx.x & 63;
    const bool have = d < pl.DP;
    const float con = HASB && have ? a.rows_con[(size_t)uidx * 2 * pl.DP + d] : 0.f;
    const float key = a.rows_key && have ? a.rows_key[(size_t)uidx * 2 * pl.DP + d] : 0.f;
    const uint64_t replicas = have ? (uint64_t)(uint32_t)pl.vals[d] : 0u;
    const bool meets = have && (!HASB || con <= a.lim_l), fits = replicas * (uint64_t)max(w0, max(w1, w2)) <= a.most;
    if (live) {
      if (follows && threadIdx.x < 64) {
        uint32_t seen = running_limit(a);
        if (GUIDED && may_wait && wave_any(meets && fits) && !(__uint_as_float(seen) < kPosInf)) {
          const unsigned long long until = wall_clock64() + a.wait_ticks;
          do {
            __builtin_amdgcn_s_sleep(12);
            seen = running_limit(a);
          } while (!(__uint_as_float(seen) < kPosInf) && wall_clock64() < until);
          if (MODE == MODE_SCAN) {  // (the first bound comes from the quickest of them)
            __builtin_amdgcn_s_sleep(64);
            seen = running_limit(a);
          }
        }
        if (threadIdx.x == 0) s_seen = seen;
      }
      if ((int)threadIdx.x < pl.DP) s_rows[threadIdx.x] = key;
      if (follows) {
        __syncthreads();
        key_limit = __uint_as_float(s_seen) * a.near_band;  // (nothing above it matters to the query)
      }
    }
    const bool near = have && key <= key_limit;
    fixed = (uint32_t)__builtin_amdgcn_ballot_w64(meets && (near || MODE != MODE_COLLECT) && fits);
    degrees = fixed & (uint32_t)__builtin_amdgcn_ballot_w64(near);
    counts = wave_any(meets) && (MODE != MODE_BEST || wave_any(near));
  }
  if (degrees == 0) {
    if (threadIdx.x == 0) unit_done<MODE>(a, uidx, sub, n_sub, kPosInf, kPosInf, counts);
    return;
  }
  // The lane space holds the degrees that matter only: with two of nine a unit takes a quarter of the rounds.
  // Workgroups that share the unit divide its chunks first, a round for each of their waves, and then the
  // innermost loop.  (A part of a unit that was cut has all degrees: chunk c goes to part c / waves mod n_parts,
  // and the collect pass must visit exactly what the scan saw.)
  __shared__ uint8_t s_dp[kMaxDP];
  Walk wk{s_dp, 0, 0, 1, 0, 1};
  {
    const uint32_t dps = u.n_parts > 1 ? (1u << pl.DP) - 1u : (n_sub > 1 ? fixed : degrees);
    wk.n_dp = __popc(dps);
    const uint32_t d = threadIdx.x;
    if (d < (uint32_t)pl.DP && ((dps >> d) & 1u)) s_dp[__popc(dps & ((1u << d) - 1u))] = (uint8_t)d;
    if (u.n_parts > 1) {
      wk.chunk = sub * (int)u.n_parts + (int)u.part;
      wk.n_chunk = (int)(u.n_parts * n_sub);
    } else if (n_sub > 1) {
      const uint32_t rounds = ((uint32_t)(pl.MB * wk.n_dp * pl.ZG) + blockDim.x - 1u) / blockDim.x;
      wk.n_chunk = (int)min(n_sub, rounds);
      wk.n_inner = (int)n_sub / wk.n_chunk;
      wk.chunk = sub % wk.n_chunk;
      wk.inner = sub / wk.n_chunk;
      if (wk.inner >= wk.n_inner) return;  // (the rest of the division; never the first)
    }
  }
  const int ZG = pl.ZG, G = pl.GX, MB = pl.MB, Z = pl.Z, S = u.s;
  const size_t n_rec = unit_lds_records(ZG, MB);
  float4 *rec_lo = reinterpret_cast<float4 *>(lds_raw);               // [S][ZG][MB], first halves
  float4 *rec_hi = rec_lo + n_rec;                                    // second halves
  uint32_t *rbits = reinterpret_cast<uint32_t *>(rec_hi + n_rec);     // validity bits alone
  float4 *pair = reinterpret_cast<float4 *>(rbits + n_rec);           // [MB][Z][Z]
  uint64_t *isect = reinterpret_cast<uint64_t *>(pair + MB * Z * Z);  // [ZG][2]
  uint32_t *q13 = reinterpret_cast<uint32_t *>(isect + 2 * ZG);       // [ZG]
  __shared__ float red[2][kMaxUnitThreads / 64];
  __shared__ uint32_t s_any[kMaxUnitThreads / 64];  // per wave, bit j: a pool can host segment j
  __shared__ uint32_t s_min;  // the smallest key the workgroup has found so far (see unit_body)
  __shared__ Kept kept;
  const int t = threadIdx.x;
  if (MODE != MODE_SCAN && t == 0) kept.n = 0;
  if (MODE != MODE_COLLECT && t == 0) s_min = __float_as_uint(key_limit);

  // Re-planning after an availability change: the unit is staged as always, and if every
  // validity word comes out as at its last evaluation its minima still hold.  With pairs of
  // types the shared-pool table is read during the evaluation, not the staging: a unit of two
  // or three segments is evaluated again whenever that table has changed since.
  const bool joint_changed = MIXED && MODE == MODE_SCAN && a.incremental && S >= 2 &&
                             pl.row_gen[0] > a.unit_gen[uidx];
  const bool keep_bits = (MODE == MODE_SCAN || MODE == MODE_BEST) && a.ubits != nullptr;
  uint32_t *const ub = keep_bits ? a.ubits + (size_t)uidx * a.ubits_stride : nullptr;
  uint32_t any_here = 0;
  for (int i = t; i < S * ZG * MB; i += blockDim.x) {
    const uint32_t sp = fast_div((uint32_t)i, pl.mg_mb), mb = (uint32_t)i - sp * (uint32_t)MB;
    const int seg = sp >= 2u * ZG ? 2 : (sp >= (uint32_t)ZG ? 1 : 0), p = (int)sp - seg * ZG;
    const int z = (int)fast_div((uint32_t)p, pl.mg_g), g = p - z * G;
    const int k = seg == 0 ? k0 : (seg == 1 ? k1 : k2);
    const int w = seg == 0 ? w0 : (seg == 1 ? w1 : w2);
    const uint32_t sl = (u.shape * (uint32_t)pl.TP + (uint32_t)k) * 3u + (uint32_t)seg;
    const uint32_t gi = (sl * (uint32_t)G + (uint32_t)g) * (uint32_t)MB + mb;
    const float4 ta = pl.ta[gi];
    uint32_t q = 0xFFFFFFFFu;
    if (!fresh) q = pl.qw[w * ZG + p];
    if constexpr (kAvailRides<MODE, MIXED>)
      if (fresh) q = quota_bits(pl, avail.v[p], w);
    if ((pl.h1m[p] >> k) & 1u) q = 0;  // H1: tensor parallelism stays inside a node
    const uint32_t bits = pl.memok[gi] & q & pl.divis[mb];
    rec_store(rec_lo, rec_hi, rbits, i,
              make_rec(ta, pl.syncz[sl * Z + z], pl.upd[sl * G + g], pl.price_f[g],
                       pl.tsec_f[(mb * Z + z) * Z + z], seg == 0 ? n0 : (seg == 1 ? n1 : n2),
                       seg == 0 ? tv0 : (seg == 1 ? tv1 : tv2), bits & degrees));
    // a segment that no pool can host validly rules the whole unit out
    const bool counts = seg != 1 || (p >= (int)u.o_lo && p < (int)(u.o_lo + u.o_cnt));
    if ((bits & degrees) != 0 && counts) any_here |= 1u << seg;
    if (keep_bits && counts) {  // (segment 2's pools outside the unit's range do not concern it)
      if (!a.incremental) ub[i] = bits;
      else if (ub[i] != bits) { ub[i] = bits; any_here |= 8u; }
    }
  }
  if (S == 3 && !MIXED)
    for (int p = t; p < ZG; p += blockDim.x) {
      uint32_t q = 0xFFFFFFFFu;
      if (!fresh) q = pl.qw[(w0 + w2) * ZG + p];
      if constexpr (kAvailRides<MODE, MIXED>)
        if (fresh) q = quota_bits(pl, avail.v[p], w0 + w2);
      q13[p] = q;
      if (keep_bits) {
        uint32_t *const uq = ub + a.ubits_stride - ZG;  // behind the records' bits
        if (!a.incremental) uq[p] = q;
        else if (uq[p] != q) { uq[p] = q; any_here |= 8u; }
      }
    }
  if (MIXED)
    for (int p = t; p < 2 * ZG; p += blockDim.x) isect[p] = pl.isect[p];
  for (int i = t; i < MB * Z * Z; i += blockDim.x) {  // per mb: transfer a -> b, b -> a, egress
    const int m = i / (Z * Z), ab = i - m * Z * Z, za = ab / Z, zb = ab % Z;
    pair[i] = make_float4(pl.tsec_f[i], pl.tsec_f[(m * Z + zb) * Z + za], pl.egs_f[ab], 0.f);
  }
  {
    uint32_t wv = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j)  // (bit 3: a validity word differs from the last evaluation's)
      if (__builtin_amdgcn_ballot_w64((any_here >> j) & 1u) != 0) wv |= 1u << j;
    if ((t & 63) == 0) s_any[t >> 6] = wv;
  }
  __syncthreads();
  uint32_t any_all = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) any_all |= s_any[w];
  if (MODE == MODE_SCAN && a.incremental && !(any_all & 8u) && !joint_changed) {
    // every validity bit is what it was: the minima still hold (uniform over the workgroup)
    if (t < 64) unit_publish(a, false, smallest_key(a, false), a.umin_s[uidx], a.umin_l[uidx]);
    return;
  }
  any_all &= 7u;
  if (any_all != (1u << S) - 1u) {  // uniform over the workgroup
    if (t == 0) unit_done<MODE>(a, uidx, sub, n_sub, kPosInf, kPosInf, true);
    return;
  }

  float ms = kPosInf, ml = kPosInf;
  auto walk = [&](auto mode) {
    constexpr int M = decltype(mode)::value;
    if (S == 1) unit_body<1, M, OBJ, HASB, MIXED>(pl, a, u, rec_lo, rec_hi, rbits, pair, q13, isect, w0, w1, w2, tau, wk, s_rows, live, follows, &s_min, kept, ms, ml);
    else if (S == 2) unit_body<2, M, OBJ, HASB, MIXED>(pl, a, u, rec_lo, rec_hi, rbits, pair, q13, isect, w0, w1, w2, tau, wk, s_rows, live, follows, &s_min, kept, ms, ml);
    else unit_body<3, M, OBJ, HASB, MIXED>(pl, a, u, rec_lo, rec_hi, rbits, pair, q13, isect, w0, w1, w2, tau, wk, s_rows, live, follows, &s_min, kept, ms, ml);
  };
  walk(std::integral_constant<int, MODE>());
  if (MODE == MODE_COLLECT && !a.count_only) keep_flush(pl, a, u, kept, false);

  if (MODE != MODE_COLLECT) {
    const bool folds = !(MODE == MODE_SCAN && live);  // (a scan for the kth smallest key has no use for the smallest one)
    const uint32_t seen = folds && t < 64 ? smallest_key(a, live) : 0u;  // (on its way during the reduction)
    if (!HASB) ml = ms;
    ms = wave_min(ms);
    ml = wave_min(ml);
    if ((t & 63) == 0) { red[0][t >> 6] = ms; red[1][t >> 6] = ml; }
    __syncthreads();
    if (t < 64) {
      const bool has = t < (int)(blockDim.x >> 6);
      ms = wave_min(has ? red[0][t] : kPosInf);
      ml = wave_min(has ? red[1][t] : kPosInf);
      if (folds) {
        const float keep = unit_publish(a, live, seen, ms, ml);
        if (MODE == MODE_BEST && t == 0) s_min = __float_as_uint(keep);
      }
      if (t == 0) unit_done<MODE>(a, uidx, sub, n_sub, ms, ml, true);
    }
    if (MODE == MODE_SCAN && live && t < 64) {  // the waves' minima are keys of as many candidates
      const uint32_t m = __float_as_uint(t < (int)(blockDim.x >> 6) ? red[0][t] : kPosInf);
      if (m < 0x7f800000u)
        // (One wave alone reaches every slot: with a degree left, the others of each workgroup often have nothing.  And
        // a workgroup's waves lie side by side, in one trip to memory: 64 best of 9.2e8 plans 79 us if they do not, 74.)
        atomicMin(&a.counters[CNT_COUNT + key_slot(blockIdx.x, blockDim.x >> 6, (uint32_t)t)], m);
      // (by all workgroups this would cost more than it prunes: they would wait for one another)
      if (GUIDED && blockIdx.x % 4u == 0u) {
        const uint32_t at = kth_of_slots(a.counters + CNT_COUNT, a.kth);
        if (at < running_limit(a)) lower_limit<MODE>(a, at);
      }
    }
  }
  if (MODE == MODE_BEST) {
    // The few units near the minimum are walked once more, their records still in LDS, instead of
    // being listed for a kernel of their own (8 to 10 us of a query of 35 to 55): with the threshold
    // known nearly all of it falls to the bounds.
    __syncthreads();
    tau = __uint_as_float(s_min);
    if (tau >= 0.0f) {  // uniform
      // (What comes near is walked at about the same time: a second look at the limit, on its way during the walk,
      // leaves a query some tens of candidates, which one workgroup re-evaluates, where it had 70 to 140.)
      const uint32_t now = t < 64 ? smallest_key(a, live) : 0u;
      walk(std::integral_constant<int, MODE_COLLECT>());
      keep_flush(pl, a, u, kept, ml > __uint_as_float(now) * a.near_band);
    }
  }
}

// How a running limit is used where the units do not fit on the chip at once.  The units at the front of the
// order, which lower it, are short because workgroups share them; the other workgroups wait for what these
// find (a bounded time: about what that takes) and take several units each, so that the waves of all of them
// are launched while the first ones work (a wave costs the dispatcher about a nanosecond: 16 000 workgroups
// 48 us).  Nearly all units then fall in one test of their bounds.  Bound by the chain of a shared unit
// (record, staging, walk, limit: 8 us) and that of the units left alive (10 us).  Scan for the 64
// fastest of 9.2e8 plans with a TP degree per segment 86 -> 28 us, fastest of 1.0e8 28 -> 18, cheapest of
// 1.1e9 with pairs of types 167 -> 19.  Units that do fit at once gain nothing by waiting (1 632 of them: 19
// us, and 15.5 as they come), those with pairs of types apart, which are longer.
// As many each as leave no more than the chip's waves.  (Of 1.1e9 plans with pairs of types: 64 fastest where one pool
// in five is available, which the limit rules out little of, 135 us with 6 144 waves, 121 with 8 192 and 117 with
// 12 288; the cheapest, which it rules out nearly all of, 30, 31 and 34.)
constexpr uint32_t kScanPerWg = 32, kBestSeeds = 16, kBestSeedSub = 16, kKthSeeds = 64, kKthSeedSub = 8;
inline uint32_t scan_workgroups(uint32_t n_units, uint32_t waves, uint32_t chip_waves) {
  const uint64_t per = std::min<uint64_t>(((uint64_t)n_units * waves + chip_waves - 1) / chip_waves, kScanPerWg);
  return (uint32_t)((n_units + per - 1) / per);
}

// SCAN: a workgroup for every unit or every few.  COLLECT: n_sub workgroups share a unit; the grid strides over a list of
// units, or over all of them, of which it visits those whose minimum is within the threshold.  BEST: as SCAN,
// or n_sub workgroups for each of a few listed units.
//
// A new availability rides on the call's first launch (ScanArgs::fresh): a quota table made by a kernel
// of its own in front of it cost 6 of the 44 us that a new table and its fastest plan took on 6.8e6
// candidates.  Only the best plan's pass takes it along: 512 bytes of arguments and the registers of the
// second source of quotas cost a top-64 query, in its scan and its collect pass, 2 to 3 of its 33 to 61 us.
// (Not with pairs of types, whose joint quotas are looked up per plan.)
//
// GUIDED: see scan_workgroups.  (A kernel of its own: what a workgroup keeps over several units made it
// spill 140 scalar registers instead of 20, 9.1 instead of 8 us for the 180 units of a small space.)
template <int MODE, int OBJ, bool HASB, bool MIXED, bool GUIDED>
__global__ __launch_bounds__(kMaxUnitThreads) void k_units(DevPlan pl, ScanArgs a, AvailArg<MODE, MIXED> avail) {
  extern __shared__ uint4 lds_raw[];
  touch_arguments(pl);
  touch_arguments(a);
  if constexpr (kAvailRides<MODE, MIXED>) {
    const uint32_t n_wgs = gridDim.x - a.fresh;
    if (blockIdx.x >= n_wgs) {
      if (blockIdx.x == n_wgs)
        for (int r = threadIdx.x; r < pl.ZGr; r += blockDim.x) a.avail_copy[r] = avail.v[r];
      quota_table(pl, avail.v, 0u, blockIdx.x - n_wgs, a.fresh);
      return;
    }
  }
  if (MODE != MODE_COLLECT && !GUIDED) {
    const uint32_t n_sub = MODE == MODE_BEST && a.direct ? a.n_sub : 1u, e = blockIdx.x / n_sub;
    unit_work<MODE, OBJ, HASB, MIXED, false>(pl, a, avail, a.ulist ? a.ulist[e] : e, (int)(blockIdx.x % n_sub), n_sub, kPosInf, false, lds_raw);
  } else if (MODE != MODE_COLLECT) {
    const uint32_t n_shared = a.n_seeds;
    const bool shared = blockIdx.x < n_shared * a.n_sub;
    const uint32_t n_sub = shared ? a.n_sub : 1u, sub = shared ? blockIdx.x % n_sub : 0u;
    const uint32_t first = shared ? blockIdx.x / n_sub : blockIdx.x - n_shared * (a.n_sub - 1u);  // in the order
    const uint32_t step = gridDim.x - a.fresh - n_shared * a.n_sub, n = (uint32_t)pl.n_units;  // workgroups behind the shared units'
    uint32_t hits = 1;
    bool may_wait = !shared && a.wait_ticks != 0;  // (once: what the shared units find is there by then, or they found nothing)
    for (bool more = !shared && first + step < n; hits != 0;) {  // uniform
      const uint32_t e = first + (uint32_t)__builtin_ctz(hits) * step;
      unit_work<MODE, OBJ, HASB, MIXED, true>(pl, a, avail, a.ulist ? a.ulist[e] : e, (int)sub, n_sub, kPosInf, may_wait, lds_raw);
      may_wait = false;
      hits &= hits - 1;
      if (!more && hits == 0) break;
      __syncthreads();  // the staging area is reused
      if (more) {       // of the units behind the first, `step` apart: those that are alive by now
        __shared__ uint32_t s_hits;
        if (threadIdx.x < 64) {
          const uint32_t mine = first + threadIdx.x * step;
          const bool alive = threadIdx.x > 0 && threadIdx.x < kScanPerWg && mine < n &&
                             unit_test<MODE, HASB>(pl, a, a.ulist ? a.ulist[mine] : mine, __uint_as_float(running_limit(a)) * a.near_band);
          const uint64_t all = __builtin_amdgcn_ballot_w64(alive);
          if (threadIdx.x == 0) s_hits = (uint32_t)all;
        }
        __syncthreads();
        hits = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_hits);
        more = false;
      }
    }
  } else {
    const float tau = a.use_tau_host ? a.tau_host
                      : __uint_as_float(a.kth ? kth_of_slots(a.counters + CNT_COUNT, a.kth) : *a.tau_src) * a.band;
    const uint32_t per_round = gridDim.x / a.n_sub, lane = threadIdx.x & 63u;
    const uint32_t n = !a.ulist ? (uint32_t)pl.n_units : a.direct ? a.n_list_host : a.counters[CNT_NLIST];
    for (uint32_t e = blockIdx.x / a.n_sub; e < n; e += (a.ulist ? 1u : 64u) * per_round) {  // uniform
      uint64_t hits = 1;
      if (!a.ulist) {  // 64 units, a lane each: which of them hold a candidate under the threshold
        const uint32_t mine = e + lane * per_round;
        const float um = mine < n ? a.umin_l[mine] : kPosInf;
        hits = __builtin_amdgcn_ballot_w64(um < kPosInf && um <= tau);
      }
      for (; hits != 0; hits &= hits - 1) {  // uniform
        const uint32_t at = e + (uint32_t)__builtin_ctzll(hits) * per_round;
        unit_work<MODE, OBJ, HASB, MIXED, false>(pl, a, avail, a.ulist ? a.ulist[at] : at, (int)(blockIdx.x % a.n_sub), a.n_sub, tau, false, lds_raw);
        __syncthreads();  // the staging area is reused
      }
    }
  }
}

// ------------------------------------------------------------------ k-th smallest key

// The form that looks for the k-th value by rank (k_select_kth, RANK) is taken for more values than the
// other one keeps in registers and k up to kKthByRank; beyond kKthRanked candidates it, too, takes the digits.
constexpr uint32_t kKthByRank = 128, kKthByRankFrom = 8192, kKthRanked = 512;

// Radix select (11 + 11 + 10 bits) of the k-th smallest non-negative float among
// n = min(*count, cap) values read with a stride; +inf entries are ignored and fewer than
// k finite values yield +inf.  One workgroup of THREADS threads (1024 for thousands of values,
// 256 for a short list: fewer waves make the passes' barriers cheaper).  The result's bit pattern
// goes to *out.
// With a list (1024 threads only): also writes the positions i < n_list_src whose list_src[i] is finite and at
// most result * band to list, and their number to *list_count (in no particular order).
//
// Thousands of values for a small k (the units' minima, where a call keeps them or starts over) take no radix pass: every wave names the
// ceil(k / waves) smallest of its lanes' minima, and the largest value so named has at least k values up
// to it.  Those -- hundreds, units being dealt to lanes by their place in the launch order -- go to LDS,
// where each counts its rank.  The 64th of the minima of 9.2e8 plans' units, and the list: 15.7 -> 9.7 us, of
// a query of 136 -> 132.  Not below 8 192 values, which the other form keeps in registers: 1 to 5 us slower there.
// Nor for a larger k, for which the waves name more and hundreds become thousands, which take the digits after
// all (that query, by digits and by rank: k = 65 137.9 and 134.4 us, 128 144.0 and 143.0, 256 175.5 and 181.4,
// 512 245.9 and 249.1).
template <int THREADS, bool RANK = false>
__global__ __launch_bounds__(THREADS) void k_select_kth(const float *vals, int stride_words,
                                                     const uint32_t *count, uint32_t cap,
                                                     uint32_t k, uint32_t *out,
                                                     const float *list_src, uint32_t n_list_src,
                                                     float band, uint32_t *list,
                                                     uint32_t *list_count) {
  constexpr int kBinsPerThread = 2048 / THREADS, kWaves = THREADS / 64;
  // (the form for survivors is never asked for a list: without that code it takes 5.0 instead of 5.3 us)
  constexpr bool kLists = THREADS == 1024;
  __shared__ __align__(16) uint32_t hist[2048];
  __shared__ uint32_t wsum[kWaves];
  __shared__ uint32_t s_prefix, s_k, s_done, s_nlist;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // The first kSelectKeep values of every thread stay in registers for all three passes.
  // Their loads (and those of the list's source) do not wait for a count that comes from
  // memory: the buffers hold cap values, so the first value of every thread is requested
  // together with the count and taken as +inf afterwards if it lies beyond it (requesting
  // all kKept that way cost more than it saved when the list was short).
  constexpr int kSelectKeep = RANK ? 16 : 8;
  constexpr uint32_t kKept = kSelectKeep * THREADS;
  uint32_t xr[kSelectKeep];
  float lr[kSelectKeep];
  const uint32_t n_early = count ? min(cap, (uint32_t)THREADS) : cap;
#pragma unroll
  for (int q = 0; q < kSelectKeep; ++q) {
    const uint32_t i = t + q * (uint32_t)THREADS;
    xr[q] = i < n_early ? __float_as_uint(vals[(size_t)i * stride_words]) : 0x7f800000u;
    lr[q] = (kLists && list && i < n_list_src) ? list_src[i] : kPosInf;
  }
  const uint32_t n = count ? min(*count, cap) : cap;
  if (t >= n) xr[0] = 0x7f800000u;
  if (count) {
#pragma unroll
    for (int q = 1; q < kSelectKeep; ++q) {
      const uint32_t i = t + q * (uint32_t)THREADS;
      if (i < n) xr[q] = __float_as_uint(vals[(size_t)i * stride_words]);
    }
  }
  if (t == 0) { s_prefix = 0; s_k = k; s_done = 0; s_nlist = 0; }
  bool found = false;  // uniform
  if constexpr (RANK) {
    uint32_t mine = 0x7f800000u;
#pragma unroll
    for (int q = 0; q < kSelectKeep; ++q) mine = min(mine, xr[q]);
    auto beyond = [&](auto &&f) {  // the values that are not kept, eight loads in flight
      for (uint32_t i0 = t + kKept; i0 < n; i0 += 8u * THREADS) {
        uint32_t x8[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const uint32_t i = i0 + q * (uint32_t)THREADS;
          x8[q] = i < n ? __float_as_uint(vals[(size_t)i * stride_words]) : 0x7f800000u;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) f(x8[q]);
      }
    };
    beyond([&](uint32_t x) { mine = min(mine, x); });
    uint32_t upto = 0;
    for (uint32_t r = 0; r < (k + kWaves - 1) / kWaves; ++r) {  // uniform
      upto = wave_min_u32(mine);
      const unsigned long long at = __builtin_amdgcn_ballot_w64(mine == upto);
      if (lane == __builtin_ctzll(at)) mine = 0x7f800000u;
    }
    if (lane == 0) wsum[wv] = upto;
    __syncthreads();
    upto = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) upto = max(upto, wsum[w]);
    auto take = [&](uint32_t x) {  // (s_done counts them)
      if (x <= upto && x < 0x7f800000u) {
        const uint32_t at = atomicAdd(&s_done, 1u);
        if (at < kKthRanked) hist[at] = x;
      }
    };
#pragma unroll
    for (int q = 0; q < kSelectKeep; ++q) take(xr[q]);
    beyond(take);
    __syncthreads();
    const uint32_t c = s_done;
    found = c <= kKthRanked;
    if (found) {
      if (t < 8) hist[c + t] = ~0u;  // (the ranks read eight values at a time)
      __syncthreads();
      const uint32_t x = t < (int)c ? hist[t] : 0u;
      uint32_t less = 0, equal = 0;
      auto rank = [&](uint32_t o) { less += o < x ? 1u : 0u; equal += o == x ? 1u : 0u; };
      for (uint32_t j = 0; j < c; j += 8) {
        const uint4 lo = *reinterpret_cast<const uint4 *>(hist + j), hi = *reinterpret_cast<const uint4 *>(hist + j + 4);
        rank(lo.x); rank(lo.y); rank(lo.z); rank(lo.w);
        rank(hi.x); rank(hi.y); rank(hi.z); rank(hi.w);
      }
      if (t == 0 && c < k) s_prefix = 0x7f800000u;
      if (t < (int)c && less < k && k <= less + equal) s_prefix = x;  // (equal values: the same word)
      __syncthreads();
    } else {
      __syncthreads();
      if (t == 0) s_done = 0;
    }
  }
  const int shifts[3] = {21, 10, 0}, widths[3] = {11, 11, 10};
  for (int pass = 0; pass < 3 && !found; ++pass) {
#pragma unroll
    for (int b = 0; b < kBinsPerThread; ++b) hist[t + b * THREADS] = 0;
    __syncthreads();
    const int sh = shifts[pass], wd = widths[pass];
    const uint32_t prefix = s_prefix, kk = s_k;
    if (s_done) break;  // uniform
    // (RANK comes here with many equal values only, and reads them again)
#pragma unroll
    for (int q = 0; q < (RANK ? 0 : kSelectKeep); ++q) {
      if ((uint32_t)q * (uint32_t)THREADS >= n) break;  // uniform: nothing is kept beyond the count
      const uint32_t x = xr[q];
      const bool match = x < 0x7f800000u && (pass == 0 || (x >> (sh + wd)) == prefix);
      const uint32_t bin = (x >> sh) & ((1u << wd) - 1);
      // Keys of a survivor list lie close together and share their leading digits: the
      // lanes that agree with the wave's first matching lane add to its bin once (hundreds
      // of atomics on one LDS word took 1 us per pass).
      const unsigned long long m = __builtin_amdgcn_ballot_w64(match);
      if (m == 0) continue;  // uniform over the wave
      const uint32_t bin0 = (uint32_t)__shfl((int)bin, __ffsll((long long)m) - 1);
      const bool same = match && bin == bin0;
      const unsigned long long ms = __builtin_amdgcn_ballot_w64(same);
      if (lane == __ffsll((long long)m) - 1) atomicAdd(&hist[bin0], (uint32_t)__popcll(ms));
      if (match && !same) atomicAdd(&hist[bin], 1u);
    }
    for (uint32_t i0 = t + (RANK ? 0u : kKept); i0 < n; i0 += 4u * blockDim.x) {  // four loads in flight
      uint32_t x4[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t i = i0 + q * blockDim.x;
        x4[q] = i < n ? __float_as_uint(vals[(size_t)i * stride_words]) : 0x7f800000u;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t x = x4[q];
        const bool match = x < 0x7f800000u && (pass == 0 || (x >> (sh + wd)) == prefix);
        if (match) atomicAdd(&hist[(x >> sh) & ((1u << wd) - 1)], 1u);
      }
    }
    __syncthreads();
    // inclusive prefix sum over the bins, kBinsPerThread consecutive bins per thread
    uint32_t h[kBinsPerThread], mine = 0;
#pragma unroll
    for (int b = 0; b < kBinsPerThread; ++b) {
      h[b] = hist[kBinsPerThread * t + b];
      mine += h[b];
    }
    uint32_t incl = wave_prefix_sum(mine);
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wv; ++w) before += wsum[w];
    incl += before;
    uint32_t excl = incl - mine;
    if (excl < kk && kk <= incl) {  // exactly one thread: the k-th value lies in its bins
      int bin = 0;
#pragma unroll
      for (int b = 0; b < kBinsPerThread - 1; ++b)  // (constant subscripts: h stays in registers)
        if (bin == b && excl + h[b] < kk) { excl += h[b]; bin = b + 1; }
      s_prefix = (prefix << wd) | (uint32_t)(kBinsPerThread * t + bin);
      s_k = kk - excl;
    }
    if (t == THREADS - 1 && incl < kk) { s_done = 1; s_prefix = 0x7f800000u; }
    __syncthreads();
  }
  if (t == 0) *out = s_prefix;
  if (kLists && list) {
    __syncthreads();
    const float tau = __uint_as_float(s_prefix) * band;
#pragma unroll
    for (int q = 0; q < kSelectKeep; ++q) {
      const uint32_t i = t + q * (uint32_t)THREADS;
      if (lr[q] < kPosInf && lr[q] <= tau) list[atomicAdd(&s_nlist, 1u)] = i;
    }
    for (uint32_t i0 = t + kKept; i0 < n_list_src; i0 += 4u * THREADS) {  // four loads in flight
      float v4[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v4[q] = i0 + q * THREADS < n_list_src ? list_src[i0 + q * THREADS] : kPosInf;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (v4[q] < kPosInf && v4[q] <= tau) list[atomicAdd(&s_nlist, 1u)] = i0 + q * THREADS;
    }
    __syncthreads();
    if (t == 0) *list_count = s_nlist;
  }
}

// ------------------------------------------------------------------ fp64 re-evaluation

struct Cand {
  uint32_t row_stage;
  int P, s, mb, dp;          // indices into the value lists
  int tp[3];                 // tp index of each segment
  int a[3];
  int n[3], k1, k2;          // stages per segment, cut points (P when unused)
};

// Of a kept candidate.
__device__ __forceinline__ Cand candidate(const SurvRec &sv) {
  Cand c;
  c.row_stage = sv.row_stage;
  c.s = (int)((sv.segs >> 24) & 3u);
  c.mb = (int)((sv.where >> 21) & 7u);
  c.dp = (int)((sv.where >> 24) & 31u);
  c.tp[0] = (int)(sv.where >> 29);
  c.tp[1] = (int)((sv.segs >> 26) & 7u);
  c.tp[2] = (int)(sv.segs >> 29);
  c.P = 0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    c.a[j] = j < c.s ? (int)((sv.where >> (7 * j)) & 127u) : -1;
    c.n[j] = j < c.s ? (int)((sv.segs >> (8 * j)) & 255u) + 1 : 0;
    c.P += c.n[j];
  }
  c.k1 = c.n[0];
  c.k2 = c.n[0] + c.n[1];
  return c;
}

// The digits of candidate idx, which lies in the given shape.
__device__ __forceinline__ void decode_in_shape(const DevPlan &pl, uint32_t shape, uint64_t idx,
                                                Cand &c) {
  const ShapeRec sh = pl.shapes[shape];
  const uint64_t rem = idx - sh.base;
  c.row_stage = sh.row_stage;
  c.P = sh.P;
  c.s = sh.s;
#pragma unroll
  for (int j = 0; j < 3; ++j) c.n[j] = sh.n[j];
  c.k1 = sh.k1;
  c.k2 = sh.k2;
  uint32_t o = (uint32_t)(rem / pl.inner);
  uint32_t in = (uint32_t)rem - o * pl.inner;  // below 8 * 8 * 24 * 128: fast_div is exact
  c.a[0] = (int)fast_div(in, pl.mg_mbtpdp);
  in -= (uint32_t)(c.a[0] * pl.MB * pl.TP * pl.DP);
  c.dp = (int)fast_div(in, pl.mg_mbtp);
  in -= (uint32_t)(c.dp * pl.MB * pl.TP);
  const int tp = (int)fast_div(in, pl.mg_mb);
  c.tp[0] = c.tp[1] = c.tp[2] = tp;
  c.mb = (int)in - tp * pl.MB;
  c.a[1] = c.a[2] = -1;
  if (c.s >= 2) {
    c.a[1] = c.a[0] + 1 + (int)(o % (pl.ZG - 1));
    if (c.a[1] >= pl.ZG) c.a[1] -= pl.ZG;
    o /= (pl.ZG - 1);
    if (pl.pst) { c.tp[1] = (int)(o % pl.TP); o /= pl.TP; }
  }
  if (c.s == 3) {
    c.a[2] = c.a[1] + 1 + (int)(o % (pl.ZG - 1));
    if (c.a[2] >= pl.ZG) c.a[2] -= pl.ZG;
    o /= (pl.ZG - 1);
    if (pl.pst) c.tp[2] = (int)o;
  }
}

// Any index: find its block, then its shape.
__device__ __forceinline__ bool decode_index(const DevPlan &pl, uint64_t idx, Cand &c) {
  if (idx >= pl.N) return false;
  int b = 0;
  for (int i = 0; i < pl.n_blocks; ++i)
    if (idx >= pl.blocks[i].off) b = i;  // blocks are ordered and non-empty
  const BlockRec blk = pl.blocks[b];
  decode_in_shape(pl, blk.first_shape + (uint32_t)((idx - blk.off) / blk.shape_size), idx, c);
  return true;
}

constexpr int kRefineWaves = 4;  // waves per workgroup of k_refine

struct RefineLds {  // per-wave staging of the per-stage terms that are summed in stage order
  double t[kMaxStages], dol[kMaxStages], comm[kMaxStages];
};

// The two real types a | b << 8 of extended type x (the plain ones, then the pairs a < b in
// lexicographic order), by arithmetic: what DevPlan::xt holds, without the trip to memory
// in front of the loads that depend on it.
__device__ __forceinline__ int type_pair(int x, int G) {
  if (x < G) return x | (x << 8);
  int r = x - G, a = 0;
  while (a < G - 2 && r >= G - 1 - a) { r -= G - 1 - a; ++a; }
  return a | ((a + 1 + r) << 8);
}

// Stage-by-stage evaluation of one plan in fp64 and exact integers (Sec. 4.3) by one wave:
// lane i takes stages i, i + 64, ...; maxima are reduced across the wave, sums are taken in
// stage order (every lane adds the staged terms in the same order, so all lanes hold the
// same results).
__device__ __forceinline__ void eval_exact_wave(const DevPlan &pl, const Cand &c, int objective,
                                                int has_bound, double bound, RefineLds &lds,
                                                double &T, double &C, uint64_t &peak,
                                                uint32_t &mask) {
  const int G = pl.G, GX = pl.GX, Z = pl.Z, MB = pl.MB, TP = pl.TP, DP = pl.DP, P = c.P;
  const int lane = threadIdx.x & 63;
  const uint32_t rs = c.row_stage;
  const int64_t D = pl.vals[c.dp];
  const int64_t nb = pl.nb[c.mb * DP + c.dp];
  const double p2p = (double)pl.p2p[c.mb];
  const double *xsec = pl.xsec + c.mb * Z * Z;  // seconds of a transfer of p2p bytes
  // quota per pool (GPUs of one replica there, times D; counted in halves: a segment on a pair of types
  // takes half of its replicas from each) and H1, a lane for every segment and real type of its pool.  (One
  // behind the other this was a third of the kernel's instructions, which a kernel of one wave fetches
  // as it goes.)
  int xs[3], zj[3], tpj[3];  // real types of each segment's pool, its zone, tp
  mask = 0;
  peak = 0;
  {
    const int j = lane >= 6 ? 0 : lane >> 1, n_j = at3(c.n, j);
    const bool used = lane < 6 && j < c.s;
    const int a = used ? at3(c.a, j) : 0, z = (int)fast_div((uint32_t)a, pl.mg_g), x = type_pair(a - z * GX, G);
    const int ga = x & 255, gb = x >> 8, g = (lane & 1) ? gb : ga;
    const int tp = pl.vals[DP + at3(c.tp, j)];
    const int64_t av = pl.avail[z * G + g], nd = pl.node[g];
    const int w = used ? n_j * tp : 0;  // (a replica's GPUs there: at most 2^20, validated)
    if (nb == 0) {  // uniform over the wave (tested only now: the loads above need not wait for it)
      mask = 4u;    // batch not divisible
      T = C = __builtin_huge_val();
      return;
    }
    int64_t halves = 0;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      xs[q] = __builtin_amdgcn_readlane(x, 2 * q);
      zj[q] = __builtin_amdgcn_readlane(z, 2 * q);
      tpj[q] = __builtin_amdgcn_readlane(tp, 2 * q);
      const int wq = __builtin_amdgcn_readlane(w, 2 * q), qa = xs[q] & 255, qb = xs[q] >> 8;  // (0 for a segment that is not there)
      if (zj[q] == z) halves += (qa == g ? wq : 0) + (qb == g ? wq : 0);
    }
    const bool counts = used && ((lane & 1) == 0 || ga != gb);
    if (wave_any(counts && (halves * D > 2 * av || (ga != gb && D % 2 != 0)))) mask |= 2u;  // (D replicas halved)
    if (wave_any(counts && tp > nd)) mask |= 8u;
  }
  double max_t = 0.0, t_sync = 0.0, t_upd = 0.0;
  const double ring = 2.0 * (double)(D - 1) / (double)D;
  uint32_t oom = 0;
  for (int i = lane; i < P; i += 64) {
    const int seg = i < c.k1 ? 0 : (i < c.k2 ? 1 : 2);
    const int xg = at3(xs, seg), g = xg & 255, g2 = xg >> 8, z = at3(zj, seg);
    const int k = at3(c.tp, seg);
    const int64_t tp = at3(tpj, seg);
    // the zones of the neighbouring stages (the stage's own where there is none)
    const int sn = (i + 1) < c.k1 ? 0 : ((i + 1) < c.k2 ? 1 : 2);
    const int sp = (i - 1) < c.k1 ? 0 : ((i - 1) < c.k2 ? 1 : 2);
    const int zn = i < P - 1 ? at3(zj, sn) : z, zp = i > 0 ? at3(zj, sp) : z;
    // everything the stage reads from memory, requested together.  Its record (st_row) holds what follows
    // from the layer split: with the shard sizes, transfers and gradient buffers divided out anew this was
    // 2 500 instructions of one wave, most of what a re-evaluation takes
    const double *const row = pl.st_row + ((size_t)(rs + (uint32_t)i) * (uint32_t)(MB * TP) + (uint32_t)(c.mb * TP + k)) * pl.row_w;
    const int32_t layers = pl.st_n[rs + (uint32_t)i];
    const uint64_t act = pl.act[c.mb * TP + k];
    const uint64_t res1 = pl.res[g], res2 = pl.res[g2], cap1 = pl.cap[g], cap2 = pl.cap[g2];
    const double c1 = row[g], c2 = row[g2], u1 = row[G + g], u2 = row[G + g2], shard = row[2 * G], grads = row[2 * G + 1];
    const double price1 = pl.price[g], price2 = pl.price[g2];
    const double x_n = xsec[z * Z + zn], x_p = xsec[z * Z + zp];
    const double eg = pl.egress ? pl.egress[z * Z + zn] + pl.egress[zn * Z + z] : 0.0;
    const uint64_t bytes_i = (uint64_t)__double_as_longlong(shard) + act_bytes((int)((int64_t)(P - i) < nb ? (int64_t)(P - i) : nb), layers, act);
    const uint64_t m = bytes_i + res1, m2 = bytes_i + res2;  // both replica types
    if (m > cap1 || m2 > cap2) oom = 1u;
    peak = m > peak ? m : peak;
    peak = m2 > peak ? m2 : peak;
    double x = 0.0, comm = 0.0;
    if (i < P - 1) {
      x += x_n;
      if (pl.egress && zn != z) comm = (double)nb * (double)D * p2p * eg;
    }
    if (i > 0) x += x_p;
    // the slower replica type sets the stage's pace (straggler, Sec. 4.3)
    const double t = fmax(c1, c2) + x;
    max_t = fmax(max_t, t);
    if (D > 1) t_sync = fmax(t_sync, ring * grads / link_bw(pl, z, z, grads));
    t_upd = fmax(t_upd, u1);
    t_upd = fmax(t_upd, u2);
    lds.t[i] = t;
    lds.dol[i] = g == g2 ? (double)(D * tp) * price1 : (double)(D * tp) * (0.5 * (price1 + price2));
    lds.comm[i] = comm;
  }
  if (__builtin_amdgcn_ballot_w64(oom != 0) != 0) mask |= 1u;
  peak = wave_max_u64(peak);
  max_t = wave_max_f64(max_t);
  t_sync = wave_max_f64(t_sync);
  t_upd = wave_max_f64(t_upd);
  // LDS operations of one wave complete in order; the fence keeps the compiler from
  // moving the reads above the writes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  double sum_t = 0.0, dollars = 0.0, comm = 0.0;
#pragma unroll 8
  for (int i = 0; i < P; ++i) {  // (unrolled so that the LDS reads run ahead of the additions)
    sum_t += lds.t[i];
    dollars += lds.dol[i];
    comm += lds.comm[i];
  }
  T = (sum_t + (double)(nb - 1) * max_t) + t_sync + t_upd;
  C = dollars / 3600.0 * T + comm;
  if (has_bound) {
    if (objective == 0) { if (C > bound) mask |= 32u; }
    else if (1.0 / T < bound) mask |= 32u;
  }
  __builtin_amdgcn_wave_barrier();  // the staging arrays are reused by the next candidate
}

struct RefineArgs {
  const SurvRec *surv;
  uint32_t surv_cap;
  uint32_t *counters;
  uint32_t kth;             // if not 0: the threshold is what COLLECT's slots give for the kth smallest key, else
  const uint32_t *tau_src;  // this; NULL: take every survivor
  float band;
  RefRec *ref;
  uint32_t ref_cap;
  int objective, has_bound;
  double bound;
};

// One wave per survivor.
__global__ __launch_bounds__(kRefineWaves * 64) void k_refine(DevPlan pl, RefineArgs a) {
  __shared__ RefineLds lds[kRefineWaves];
  const uint32_t wave = blockIdx.x * kRefineWaves + (threadIdx.x >> 6);
  const uint32_t n_waves = gridDim.x * kRefineWaves;
  // the wave's first record is requested together with the count (the buffer holds surv_cap
  // records, so the address is valid whatever the count turns out to be)
  SurvRec first{};
  if (wave < a.surv_cap) first = a.surv[wave];
  touch_arguments(pl);
  const uint32_t n = min(a.counters[CNT_SURV], a.surv_cap);
  float tau = kPosInf;
  if (a.kth) tau = __uint_as_float(kth_of_slots(a.counters + kKeptSlots, a.kth)) * a.band;
  else if (a.tau_src) tau = __uint_as_float(*a.tau_src) * a.band;
  for (uint32_t i = wave; i < n; i += n_waves) {
    const SurvRec sv = i == wave ? first : a.surv[i];
    if (!(__uint_as_float(sv.key & 0x7fffffffu) <= tau)) continue;
    const Cand c = candidate(sv);
    RefRec r;
    r.idx = sv.idx;
    r.pad = 0;
    eval_exact_wave(pl, c, a.objective, a.has_bound, a.bound, lds[threadIdx.x >> 6], r.T, r.C,
                    r.mem, r.mask);
    if ((threadIdx.x & 63) == 0) {
      const uint32_t slot = atomicAdd(&a.counters[CNT_REF], 1u);
      if (slot < a.ref_cap) {  // (a record that does not fit is counted in CNT_REF only: the
        a.ref[slot] = r;       // host reports the overflow, the ranking sees what was stored)
        if (r.mask == 0) atomicAdd(&a.counters[CNT_FEAS], 1u);
      }
    }
  }
}

__device__ __forceinline__ bool lex_less(double ka, uint64_t ia, double kb, uint64_t ib) {
  return ka < kb || (ka == kb && ia < ib);
}

// The host waits for the results by polling hdr->seq in host-mapped memory, which saves the
// few microseconds between a kernel's last store and the completion of its dispatch; the
// sequence number is therefore stored last, behind a system-scope fence.
__device__ __forceinline__ void publish(ResultHeader *hdr, uint32_t seq) {
  __threadfence_system();
  __hip_atomic_store(&hdr->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Best plan: fp64 re-evaluation of the survivors within the tie band of the smallest fp32 key, one
// wave each, then the minimum fp64 key over the valid ones and the lowest index within the tie
// tolerance of it; results go to host-mapped memory.
//
// There are rarely more than a few survivors, and what this costs is its chain of trips to memory
// (count and records, shape, stages), so up to kBestAlone of them are one workgroup's: it holds the
// results in LDS and picks at once, where a kernel of its own for the pick started with a cold L2 and
// took 4 to 5 us more.  With more, every workgroup takes its share and the one that finishes last
// picks.
//
// In the first case the host has the result while other workgroups may not have started yet.  By then
// the plan may be in use again, on another stream too, where nothing orders them: the next call but one
// uses the same counters.  So a workgroup other than the first works only if the set belongs to its own
// call.  While it does, the count is this call's, which everyone sees alike; the final kernel of the next
// call gives the set a new owner before the call behind it can count anything; and count and owner come in
// one load, so a late workgroup sees a small count or a foreign owner, and leaves.  (A late one touches
// nothing else but the survivor list, whose records it reads and drops.)
constexpr int kBestWaves = 8;
constexpr uint32_t kBestAlone = 64;  // (a lane each in the selection and the pick)
constexpr unsigned kBestWorkgroups = 64;

__global__ __launch_bounds__(kBestWaves * 64) void k_refine_best(DevPlan pl, RefineArgs a, uint32_t *next_counters,
                                                                ResultHeader *hdr, RefRec *out, uint32_t seq,
                                                                uint32_t call) {
  __shared__ RefineLds lds[kBestWaves];
  __shared__ RefRec s_ref[kBestAlone];
  __shared__ double s_key[kBestWaves];
  __shared__ unsigned long long s_idx[kBestWaves];
  __shared__ uint32_t s_pos[kBestWaves], s_last;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // a lane's survivor is requested together with the counters (the buffer holds surv_cap records,
  // so the address is valid whatever the count turns out to be)
  SurvRec mine{};
  if ((uint32_t)lane < a.surv_cap) mine = a.surv[lane];
  const uint64_t count_owner = __hip_atomic_load(reinterpret_cast<const uint64_t *>(a.counters + CNT_SURV),
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t gmin = a.counters[CNT_GMIN];
  touch_arguments(pl);  // (while these are on their way)
  const uint32_t n_surv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)count_owner),
                 owner = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(count_owner >> 32));
  const uint32_t n = min(n_surv, a.surv_cap);
  const float tau = __uint_as_float(gmin) * a.band;
  const bool alone = n <= kBestAlone;  // uniform over the call's grid
  if (blockIdx.x != 0 && (alone || owner != call)) return;
  auto evaluate = [&](const SurvRec &sv) {
    const Cand c = candidate(sv);
    RefRec r;
    r.idx = sv.idx;
    r.pad = 0;
    eval_exact_wave(pl, c, a.objective, a.has_bound, a.bound, lds[wv], r.T, r.C, r.mem, r.mask);
    return r;
  };
  auto within = [&](const SurvRec &sv) { return __uint_as_float(sv.key & 0x7fffffffu) <= tau; };
  auto key_of = [&](const RefRec &r) { return r.mask != 0 ? __builtin_huge_val() : (a.objective == 0 ? r.T : r.C); };
  uint32_t n_ref, n_feas = 0;
  auto reset_next = [&](uint32_t from) {  // for the next call
    for (uint32_t c = (uint32_t)t - from; c < kSetWords; c += kBestWaves * 64 - from) next_counters[c] = counter_reset_value((int)c, owner + 1);
  };
  if (alone) {
    const unsigned long long near = __builtin_amdgcn_ballot_w64((uint32_t)lane < n && within(mine));
    const uint32_t rank = (uint32_t)__popcll(near & ((1ull << lane) - 1ull));
    n_ref = (uint32_t)__popcll(near);
    for (uint32_t w = wv; w < n_ref; w += kBestWaves) {  // uniform over the wave
      const int from = __builtin_ctzll(__builtin_amdgcn_ballot_w64(((near >> lane) & 1ull) != 0 && rank == w));
      SurvRec sv;
      auto of = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, from); };
      sv.idx = (uint64_t)of((uint32_t)(mine.idx >> 32)) << 32 | of((uint32_t)mine.idx);
      sv.key = 0;
      sv.row_stage = of(mine.row_stage);
      sv.where = of(mine.where);
      sv.segs = of(mine.segs);
      const RefRec r = evaluate(sv);
      if (lane == 0) s_ref[w] = r;
    }
    if (wv != 0) reset_next(64);
    __syncthreads();
    if (wv != 0) return;
    // a lane each: no more barriers
    const bool valid = (uint32_t)lane < n_ref && s_ref[lane].mask == 0;
    const double key = valid ? key_of(s_ref[lane]) : __builtin_huge_val(), limit = wave_min_f64(key) * (1.0 + kTieTol);
    const unsigned long long idx = valid && key <= limit ? s_ref[lane].idx : ~0ull, lowest = wave_min_u64(idx);
    const bool found = lowest != ~0ull;
    const uint32_t at = (uint32_t)__builtin_ctzll(__builtin_amdgcn_ballot_w64(idx == lowest));
    if (found && lane < (int)(sizeof(RefRec) / 8))
      reinterpret_cast<unsigned long long *>(out)[lane] = reinterpret_cast<const unsigned long long *>(&s_ref[at])[lane];
    n_feas = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(valid));
    if (lane == 0) {
      hdr->n_found = found ? 1u : 0u;
      hdr->surv_count = n_surv;
      hdr->ref_count = n_ref;
      hdr->feasible_count = n_feas;
      hdr->gmin_bits = gmin;
      publish(hdr, seq);
    }
    return;
  } else {
    for (uint32_t i = blockIdx.x * kBestWaves + wv; i < n; i += gridDim.x * kBestWaves) {
      const SurvRec sv = a.surv[i];
      if (!within(sv)) continue;
      const RefRec r = evaluate(sv);
      if (lane == 0) {
        const uint32_t slot = atomicAdd(&a.counters[CNT_REF], 1u);
        if (slot < a.ref_cap) {  // (what does not fit is counted only: the host reports it)
          a.ref[slot] = r;
          if (r.mask == 0) atomicAdd(&a.counters[CNT_FEAS], 1u);
        }
      }
    }
    __threadfence();  // visible to the other workgroups before this one counts as done
    __syncthreads();
    if (t == 0) s_last = atomicAdd(&a.counters[CNT_DONE], 1u) == gridDim.x - 1 ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;  // uniform
    __threadfence();      // the last workgroup: see what the others stored
    n_ref = __hip_atomic_load(&a.counters[CNT_REF], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    n_feas = __hip_atomic_load(&a.counters[CNT_FEAS], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  reset_next(0);
  const RefRec *const ref = a.ref;
  const uint32_t stored = min(n_ref, a.ref_cap);
  double best = __builtin_huge_val();
  for (uint32_t i = t; i < stored; i += kBestWaves * 64) best = fmin(best, key_of(ref[i]));
  best = wave_min_f64(best);
  if (lane == 0) s_key[wv] = best;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kBestWaves; ++w) best = fmin(best, s_key[w]);
  const double limit = best * (1.0 + kTieTol);
  unsigned long long bi = ~0ull;
  uint32_t bp = 0;
  for (uint32_t i = t; i < stored; i += kBestWaves * 64)
    if (ref[i].mask == 0 && key_of(ref[i]) <= limit && ref[i].idx < bi) { bi = ref[i].idx; bp = i; }
  {
    const unsigned long long lowest = wave_min_u64(bi);
    bp = (uint32_t)__builtin_amdgcn_readlane((int)bp, __builtin_ctzll(__builtin_amdgcn_ballot_w64(bi == lowest)));
    bi = lowest;
  }
  if (lane == 0) { s_idx[wv] = bi; s_pos[wv] = bp; }
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < kBestWaves; ++w)
      if (s_idx[w] < bi) { bi = s_idx[w]; bp = s_pos[w]; }
    const bool found = bi != ~0ull;
    if (found) out[0] = ref[bp];
    hdr->n_found = found ? 1u : 0u;
    hdr->surv_count = n_surv;
    hdr->ref_count = n_ref;
    hdr->feasible_count = n_feas;
    hdr->gmin_bits = gmin;
    publish(hdr, seq);
  }
}

constexpr uint32_t kRankLds = 1024;  // records the one-workgroup form of k_rank_topk takes

// Top-k: the rank of every valid re-evaluated candidate in ascending (key, index) order.
// Launched as one workgroup of kRankLds threads when few records are expected (small k):
// keys and indices go to LDS, the threads share out the counting of each record's
// predecessors, and the k first are copied to host-mapped memory in rank order.  Otherwise (several workgroups,
// or more than kRankLds records) one wave per candidate: its lanes count, in strides over
// the list, the entries that precede it; ranks below k go to a device-side list, which the
// workgroup that finishes last copies to host-mapped memory in one coalesced pass
// (scattered 40-byte stores over the bus, each behind its own fence, cost 20 us for 500
// records).
__global__ __launch_bounds__(kRankLds) void k_rank_topk(const RefRec *ref, uint32_t ref_cap,
                                                        const uint32_t *counters,
                                                        uint32_t *next_counters, int objective,
                                                        uint32_t k, ResultHeader *hdr, RefRec *out,
                                                        RefRec *staged, uint32_t *done,
                                                        uint32_t seq) {
  __shared__ uint32_t s_last;
  __shared__ double s_key[kRankLds];
  __shared__ unsigned long long s_idx[kRankLds];
  __shared__ uint16_t s_opos[kRankLds];
  __shared__ uint32_t s_before[kRankLds];
  // (one-workgroup form) a thread's record is requested together with the count: the
  // buffer holds ref_cap records, so the address is valid whatever the count turns out to be
  RefRec mine{};
  if (gridDim.x == 1 && threadIdx.x < ref_cap) mine = ref[threadIdx.x];
  const uint32_t n_ref = counters[CNT_REF];
  const uint32_t n = min(n_ref, ref_cap);
  const uint32_t f = counters[CNT_FEAS], call = counters[CNT_OWNER];  // valid stored records (requested with the count)
  const bool overflow = n_ref > ref_cap;  // uniform: the list is incomplete, nothing is ranked
  if (blockIdx.x == 0)
    for (uint32_t c = threadIdx.x; c < kSetWords; c += blockDim.x)
      next_counters[c] = counter_reset_value((int)c, call + 1);  // for the next call
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    hdr->n_found = overflow ? 0u : (f < k ? f : k);
    hdr->surv_count = counters[CNT_SURV];
    hdr->ref_count = n_ref;
    hdr->feasible_count = f;
    hdr->gmin_bits = counters[CNT_GMIN];
  }
  if (overflow) {  // the host turns ref_count > ref_cap into SAILOR_ENOMEM
    if (gridDim.x == 1) {
      if (threadIdx.x == 0) publish(hdr, seq);
      return;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      __threadfence_system();
      s_last = atomicAdd(done, 1u) == gridDim.x - 1 ? 1u : 0u;
      if (s_last) publish(hdr, seq);
    }
    return;
  }
  if (gridDim.x == 1 && n <= kRankLds) {  // uniform
    const uint32_t t = threadIdx.x;
    if (t < n) {
      const bool ok = mine.mask == 0;
      s_key[t] = ok ? (objective == 0 ? mine.T : mine.C) : __builtin_huge_val();
      s_idx[t] = ok ? mine.idx : ~0ull;
    }
    s_before[t] = 0;
    __syncthreads();
    // the workgroup's threads form rows of np >= n threads (a power of two); row r counts,
    // for record q, the predecessors among records r, r + rows, ...
    uint32_t np = 64;
    while (np < n) np <<= 1;
    const uint32_t q = t & (np - 1), row = t / np, rows = kRankLds / np;
    if (q < n && s_idx[q] != ~0ull) {
      const double mk = s_key[q];
      const unsigned long long mi = s_idx[q];
      uint32_t before = 0;
#pragma unroll 4
      for (uint32_t j = row; j < n; j += rows) before += lex_less(s_key[j], s_idx[j], mk, mi) ? 1u : 0u;
      if (before) atomicAdd(&s_before[q], before);
    }
    __syncthreads();
    if (t < n && s_idx[t] != ~0ull && s_before[t] < k) s_opos[s_before[t]] = (uint16_t)t;
    __syncthreads();
    const uint32_t n_out = f < k ? f : k;  // n_out <= n
    constexpr uint32_t kWords = sizeof(RefRec) / 8;
    for (uint32_t w = threadIdx.x; w < n_out * kWords; w += blockDim.x)
      reinterpret_cast<unsigned long long *>(out)[w] =
          reinterpret_cast<const unsigned long long *>(ref + s_opos[w / kWords])[w % kWords];
    // One system-scope fence for the workgroup (each costs a fraction of a microsecond per
    // wave that executes it): the stores above are ordered before thread 0's fence by a
    // workgroup-scope release and the barrier.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();
    if (threadIdx.x == 0) publish(hdr, seq);
    return;
  }
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const uint32_t n_waves = gridDim.x * (blockDim.x >> 6);
  bool wrote = false;
  for (uint32_t i = wave; i < n; i += n_waves) {
    const RefRec r = ref[i];
    if (r.mask != 0) continue;  // uniform over the wave
    const double mk = objective == 0 ? r.T : r.C;
    uint32_t before = 0;
    for (uint32_t j = lane; j < n; j += 64) {
      const RefRec &o = ref[j];
      if (o.mask == 0 && lex_less(objective == 0 ? o.T : o.C, o.idx, mk, r.idx)) ++before;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) before += __shfl_xor(before, off);
    if (lane == 0 && before < k) {
      staged[before] = r;
      wrote = true;
    }
  }
  if (wrote) __threadfence();  // visible to the other workgroups before this one counts as done
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence_system();  // (workgroup 0: the header fields above are on their way)
    s_last = atomicAdd(done, 1u) == gridDim.x - 1 ? 1u : 0u;
  }
  __syncthreads();
  if (!s_last) return;  // uniform
  __threadfence();      // the last workgroup: see what the others staged
  const uint32_t n_out = f < k ? f : k;
  const unsigned long long *src = reinterpret_cast<const unsigned long long *>(staged);
  unsigned long long *dst = reinterpret_cast<unsigned long long *>(out);
  for (uint32_t i = threadIdx.x; i < n_out * (uint32_t)(sizeof(RefRec) / 8); i += blockDim.x)
    dst[i] = __builtin_nontemporal_load(src + i);
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) publish(hdr, seq);
}

// ------------------------------------------------------------------ event-by-event 1F1B

struct SimArgs {
  uint64_t count;
  const uint64_t *indices;
  double *t_event, *t_closed;  // either may be NULL
};

// The value of the lane below / above (0 at the ends of the wave).
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double from_below(double v) { return lane_shift<0x138>(v); }  // wave_shr:1
__device__ __forceinline__ double from_above(double v) { return lane_shift<0x130>(v); }  // wave_shl:1

// The 1F1B schedule of one pipeline of a plan, op by op (warm-up, steady and cool-down phases,
// Sec. 4.3), beside the closed form of Sec. 4.2.2 on the same stage times.  One wave per
// candidate, SPL consecutive stages per lane.  A forward of stage i takes its layers' forward time
// plus the transfer to stage i + 1, a backward its backward time plus the transfer to stage i - 1; a
// forward waits for the previous stage's forward of the same microbatch, a backward for the next
// stage's backward.
//
// The order of a stage's ops is fixed, so an op's end time is max(end of the stage's op before
// it, end of the op it waits for) + duration, and the ops can be computed in any order that
// respects both.  Taken in the rounds of a pipeline whose ops all last one round --
//     F of microbatch m on stage i:  round i + m while m < P - i, round i + 2 m afterwards
//     B of microbatch m on stage i:  round 2 P - 1 - i + 2 m
// -- a stage runs at most one op per round, and whenever an op runs, the last op its neighbour
// ran is the one it waits for (the one forward that waits longer, m = P - i, finds its neighbour
// idle since).  One end time per stage is therefore all the state there is, and it stays in
// registers: no queue of end times, no flags, no barrier.
// From round P on, stages of one parity run forwards in the even rounds and the others
// backwards, and vice versa in the odd ones.  Stages are laid out so that in the odd rounds the
// two of a pair wait for each other, which leaves max, add, add per pair, and only the even
// rounds pass values between lanes.  A position without a stage has durations 0: what it passes
// on never exceeds what its neighbour already has.
//
// Bound by the chain of dependent fp64 operations: 2 (N_b + P) rounds of one or two maxima and
// additions.  The 64 best plans of a 48-layer, 104 256 000-candidate space take 18.5 us where the
// form with end times in LDS rings and two barriers per round took 407 us (same plans, one card).
template <int SPL>
__device__ __forceinline__ double sim_schedule(int P, int M, const double (&fd)[SPL], const double (&bd)[SPL]) {
  const int lane = threadIdx.x & 63, first = lane * SPL - (P & 1);  // stage of this lane's first position
  double x[SPL];         // end of the last op of each position
  int a_lo[SPL], a_n[SPL], b_lo[SPL], b_n[SPL];  // periods in which its even / odd round runs an op
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    const int i = first + s;
    const bool on = i >= 0 && i < P;
    x[s] = 0.0;
    if (s & 1) {  // backward, then forward
      a_lo[s] = b_lo[s] = (P - 1 - i) >> 1;
      a_n[s] = on ? M : 0;
      b_n[s] = on ? ((2 * M - 3 + i - P) >> 1) - b_lo[s] + 1 : 0;
    } else {      // forward, then backward
      a_lo[s] = (P - i) >> 1;
      a_n[s] = on ? ((2 * M - 2 + i - P) >> 1) - a_lo[s] + 1 : 0;
      b_lo[s] = (P - 2 - i) >> 1;
      b_n[s] = on ? M : 0;
    }
    a_n[s] = max(a_n[s], 0);
    b_n[s] = max(b_n[s], 0);
  }
  // warm-up: rounds 0 .. P - 1 run forwards only
  for (int r = 0; r < P; ++r) {
    const double below = from_below(x[SPL - 1]);
#pragma unroll
    for (int s = SPL - 1; s >= 0; --s) {  // downwards: a position reads the one before it unchanged
      const int i = first + s;
      const double y = fmax(x[s], s == 0 ? below : x[s > 0 ? s - 1 : 0]) + fd[s];
      x[s] = (i >= 0 && i <= r && r - i < min(M, P - i)) ? y : x[s];
    }
  }
  // period k: rounds P + 2 k (even) and P + 2 k + 1 (odd)
  const int periods = (2 * M + P - 1) >> 1;
  const int full_lo = min((P + 1) >> 1, periods), full_hi = max(full_lo, min((2 * M - 1 - P) >> 1, periods));
  auto period = [&](int k, auto all) {
    constexpr bool ALL = decltype(all)::value;  // every stage runs an op in both rounds
    double y[SPL];
    const double below = from_below(x[SPL - 1]), above = from_above(x[0]);
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
      const double dep = (s & 1) ? (s == SPL - 1 ? above : x[s < SPL - 1 ? s + 1 : s])
                                 : (s == 0 ? below : x[s > 0 ? s - 1 : 0]);
      y[s] = fmax(x[s], dep) + ((s & 1) ? bd[s] : fd[s]);
      if (!ALL) y[s] = (uint32_t)(k - a_lo[s]) < (uint32_t)a_n[s] ? y[s] : x[s];
    }
#pragma unroll
    for (int s = 0; s < SPL; s += 2) {
      const double later = fmax(y[s], y[s + 1]);
      x[s] = later + bd[s];
      x[s + 1] = later + fd[s + 1];
      if (!ALL) {
        x[s] = (uint32_t)(k - b_lo[s]) < (uint32_t)b_n[s] ? x[s] : y[s];
        x[s + 1] = (uint32_t)(k - b_lo[s + 1]) < (uint32_t)b_n[s + 1] ? x[s + 1] : y[s + 1];
      }
    }
  };
  int k = 0;
  for (; k < full_lo; ++k) period(k, std::false_type());
  for (; k + 4 <= full_hi; k += 4) {  // (by hand: the compiler does not unroll around cross-lane moves)
    period(k, std::true_type());
    period(k, std::true_type());
    period(k, std::true_type());
    period(k, std::true_type());
  }
  for (; k < full_hi; ++k) period(k, std::true_type());
  for (; k < periods; ++k) period(k, std::false_type());
  double end = 0.0;  // makespan: the latest stage (what lies beyond the stages is no later)
#pragma unroll
  for (int s = 0; s < SPL; ++s) end = fmax(end, x[s]);
  return wave_max_f64(end);
}

template <int SPL>
__device__ __forceinline__ void sim_plan(const DevPlan &pl, const SimArgs &a, uint64_t ci, const Cand &c, int M,
                                         double *s_t) {
  const int P = c.P, G = pl.G, GX = pl.GX, Z = pl.Z, MB = pl.MB, TP = pl.TP;
  const int lane = threadIdx.x & 63;
  const uint32_t rs = c.row_stage;
  const double *xsec = pl.xsec + c.mb * Z * Z;
  double fd[SPL], bd[SPL];
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    const int i = lane * SPL - (P & 1) + s;
    fd[s] = bd[s] = 0.0;
    if (i < 0 || i >= P) continue;
    const int seg = i < c.k1 ? 0 : (i < c.k2 ? 1 : 2);
    const int xg = pl.xt[at3(c.a, seg) % GX], g = xg & 255, g2 = xg >> 8, z = at3(c.a, seg) / GX, k = at3(c.tp, seg);
    const size_t at = (((size_t)(rs + i) * G + g) * MB + c.mb) * TP + k;
    const size_t at2 = (((size_t)(rs + i) * G + g2) * MB + c.mb) * TP + k;
    double send_f = 0.0, send_b = 0.0;
    if (i < P - 1) {
      const int sn = (i + 1) < c.k1 ? 0 : ((i + 1) < c.k2 ? 1 : 2);
      send_f = xsec[z * Z + at3(c.a, sn) / GX];
    }
    if (i > 0) {
      const int sp = (i - 1) < c.k1 ? 0 : ((i - 1) < c.k2 ? 1 : 2);
      send_b = xsec[z * Z + at3(c.a, sp) / GX];
    }
    double f = pl.st_f[at], b = pl.st_b[at];
    if (g2 != g && pl.st_f[at2] + pl.st_b[at2] > f + b) {  // the pipeline through the slower type
      f = pl.st_f[at2];
      b = pl.st_b[at2];
    }
    fd[s] = f + send_f;
    bd[s] = b + send_b;
    s_t[i] = f + b + (send_f + send_b);
  }
  __syncthreads();
  if (a.t_closed) {  // sums in stage order
    double sum_t = 0.0, max_t = 0.0;
#pragma unroll 8
    for (int j = 0; j < P; ++j) {
      sum_t += s_t[j];
      max_t = fmax(max_t, s_t[j]);
    }
    if (lane == 0) a.t_closed[ci] = sum_t + (double)(M - 1) * max_t;
  }
  if (a.t_event) {
    const double end = sim_schedule<SPL>(P, M, fd, bd);
    if (lane == 0) a.t_event[ci] = end;
  }
}

__global__ __launch_bounds__(64) void k_sim_1f1b(DevPlan pl, SimArgs a) {
  touch_arguments(pl);
  __shared__ double s_t[kMaxStages];
  const uint64_t ci = blockIdx.x;
  if (ci >= a.count) return;
  const uint64_t idx = a.indices[ci];
  Cand c;
  double none = __builtin_nan("");  // an index outside the space
  int M = 0;
  if (decode_index(pl, idx, c)) {
    M = pl.nb[c.mb * pl.DP + c.dp];
    none = __builtin_huge_val();    // M == 0: the batch does not divide
  }
  if (M == 0) {  // uniform
    if (threadIdx.x == 0) {
      if (a.t_event) a.t_event[ci] = none;
      if (a.t_closed) a.t_closed[ci] = none;
    }
    return;
  }
  // two stages per lane up to 128 positions (two and four positions cost nearly the same per
  // round, their chains run side by side; one per lane would pass values in every round)
  if (c.P + (c.P & 1) <= 128) sim_plan<2>(pl, a, ci, c, M, s_t);
  else sim_plan<4>(pl, a, ci, c, M, s_t);
}

// ------------------------------------------------------------------ eval_batch

// "iterations per second below the floor", decided the same way by both evaluation kernels
// (a product instead of a division; the two differ only for values within rounding of the
// floor)
__device__ __forceinline__ bool throughput_below(float T, float floor_) { return T * floor_ > 1.0f; }

struct EvalArgs {
  uint64_t first, count;
  const uint64_t *indices;
  float *time, *cost;
  uint64_t *mem;
  uint32_t *mask;
  int objective, has_bound;
  float bound;
};

// The small tables of the evaluator of index lists: laid out once per plan in memory
// (k_direct_tables), copied to LDS by every workgroup in one go, the availability behind them.
struct DirectBlock {          // a block of the index space (BlockRec) as an index is decoded with it
  uint64_t off;
  double size, inv_size;      // candidates per shape, and 1 / that
  uint32_t first_shape, s;
};
static_assert(sizeof(DirectBlock) == 32, "whole 8-byte words");
constexpr int kDirectShapes = 2048;  // shapes whose stages fit LDS (8 KB)

struct DirectTables {
  DirectBlock *blocks;        // [n_blocks]
  uint64_t *cap, *res;        // [G]
  float *ts;                  // [MB][Z][Z] transfer seconds
  float *egs;                 // [Z][Z]
  float *price;               // [GX]
  float *xb;                  // [MB]
  float *cd, *dph;            // [DP]
  float *nbm1;                // [MB][DP]
  int32_t *nb;                // [MB][DP]
  int32_t *dp, *tp;           // [DP], [TP] the lists' values
  int32_t *node;              // [G]
  uint32_t *xt;               // [GX]
  uint32_t *n;                // [n_shapes] stages - 1 per segment, a byte each (kDirectShapes of them at most)
  uint32_t *room;             // [DP][ZGr] half-GPUs per replica that a real pool has room for (not part of the copy)
};

__host__ __device__ inline uint32_t direct_copy_words(const DevPlan &pl) {  // 4-byte words laid out in memory
  return (uint32_t)(8 * pl.n_blocks + 4 * pl.G + pl.MB * pl.Z * pl.Z + pl.Z * pl.Z + 2 * pl.GX + pl.MB + 3 * pl.DP +
                    2 * pl.MB * pl.DP + pl.TP + pl.G + (pl.n_shapes <= kDirectShapes ? pl.n_shapes : 0));
}
inline size_t direct_lds_bytes(const DevPlan &pl) {  // (57 KB at the limits of a problem)
  return ((size_t)direct_copy_words(pl) + (size_t)pl.DP * pl.ZGr) * sizeof(uint32_t);
}

__device__ __forceinline__ DirectTables direct_tables_at(const DevPlan &pl, uint32_t *at) {
  DirectTables T;
  T.blocks = reinterpret_cast<DirectBlock *>(at);
  T.cap = reinterpret_cast<uint64_t *>(T.blocks + pl.n_blocks);
  T.res = T.cap + pl.G;
  T.ts = reinterpret_cast<float *>(T.res + pl.G);
  T.egs = T.ts + pl.MB * pl.Z * pl.Z;
  T.price = T.egs + pl.Z * pl.Z;
  T.xb = T.price + pl.GX;
  T.cd = T.xb + pl.MB;
  T.dph = T.cd + pl.DP;
  T.nbm1 = T.dph + pl.DP;
  T.nb = reinterpret_cast<int32_t *>(T.nbm1 + pl.MB * pl.DP);
  T.dp = T.nb + pl.MB * pl.DP;
  T.tp = T.dp + pl.DP;
  T.node = T.tp + pl.TP;
  T.xt = reinterpret_cast<uint32_t *>(T.node + pl.G);
  T.n = T.xt + pl.GX;
  T.room = T.n + (pl.n_shapes <= kDirectShapes ? pl.n_shapes : 0);
  return T;
}

// (after k_small_tables, one workgroup)
__global__ void k_direct_tables(DevPlan pl, DirectMem dm) {
  const DirectTables T = direct_tables_at(pl, pl.direct_tables);
  const int t = threadIdx.x, nt = blockDim.x;
  for (int i = t; i < pl.n_blocks; i += nt) {
    const BlockRec b = pl.blocks[i];
    DirectBlock o;
    o.off = b.off; o.size = (double)b.shape_size; o.inv_size = 1.0 / (double)b.shape_size;
    o.first_shape = b.first_shape; o.s = b.s;
    T.blocks[i] = o;
  }
  for (int i = t; i < pl.G; i += nt) { T.cap[i] = pl.cap[i]; T.res[i] = pl.res[i]; T.node[i] = pl.node[i]; }
  for (int i = t; i < pl.MB * pl.Z * pl.Z; i += nt) T.ts[i] = pl.tsec_f[i];
  for (int i = t; i < pl.Z * pl.Z; i += nt) T.egs[i] = pl.egs_f[i];
  for (int i = t; i < pl.GX; i += nt) { T.price[i] = pl.price_f[i]; T.xt[i] = pl.xt[i]; }
  for (int i = t; i < pl.MB; i += nt) T.xb[i] = pl.xb_f[i];
  for (int i = t; i < pl.DP; i += nt) { T.cd[i] = pl.cd_f[i]; T.dph[i] = pl.dph_f[i]; T.dp[i] = pl.vals[i]; }
  for (int i = t; i < pl.MB * pl.DP; i += nt) { T.nbm1[i] = pl.nbm1_f[i]; T.nb[i] = pl.nb[i]; }
  for (int i = t; i < pl.TP; i += nt) T.tp[i] = pl.vals[pl.DP + i];
  if (pl.n_shapes <= kDirectShapes) for (int i = t; i < pl.n_shapes; i += nt) T.n[i] = dm.shape_n[i];
}

// n / d for n < 2^20 and n d < 2^40 or so by a product in single precision: inv is 1 / d rounded up by two
// units, so the product is never below a whole quotient and above the true one by less than n 2^-21 < 1
// in units of 1 / d.  (Three full-rate instructions; 32-bit integer products run at a quarter of it.)
__device__ __forceinline__ float float_inverse(uint32_t d) { return __uint_as_float(__float_as_uint(1.0f / (float)d) + 2u); }
__device__ __forceinline__ uint32_t float_div(uint32_t n, float inv) { return (uint32_t)((float)n * inv); }

// n / d and the remainder, whole numbers below 2^52 held as doubles, given 1 / d: the quotient of the
// rounded product is off by one at most, and the remainder exact (one rounding, of a whole number).
__device__ __forceinline__ double divide_by(double n, double d, double inv, double &rem) {
  double q = trunc(n * inv), r = fma(-q, d, n);
  const double by = r < 0.0 ? -1.0 : (r >= d ? 1.0 : 0.0);
  rem = fma(-by, d, r);
  return q + by;
}

// One lane per candidate, grid-stride; the segment aggregates come straight from global memory.
// Bound by gathers: every lane of a wave reads another cache line, and a compute unit's address path
// takes a cycle per lane and 8 bytes (54 000 of the kernel's 70 000 cycles; vector instructions 32 000).
// So the small tables, the shapes' stages among them, are in LDS, a candidate of three segments gathers
// nine times (aggregate, seconds of all-reduce and update, bytes of each segment), and no load waits for
// another: an index is decoded from its block's record in LDS, its two 64-bit divisions by products in
// double precision (a space has at most 2^29 units of at most 8 x 24 x 128 x 127 plans: below 2^51).  The lanes of a wave go through the segments together,
// whether they have one, two or three (apart, a wave ran the code of each number it held), quotas
// compare with what the table of degrees and pools has room for, and products are 24-bit or in single
// precision (32-bit ones run at a quarter of the rate).
// 1 000 003 random candidates: 42.7 -> 35.4 us (28 MB of indices and outputs; the same bytes take 5 us as
// a copy).  Held to fewer registers for seven waves per SIMD instead of five it spills: 41.3 us.
constexpr int kDirectThreads = 256;
// (five workgroups fit a compute unit, 1 280 in all; the same time with that many, within 1 %: 1 000 003
// candidates 35.7 us, with 1 280 35.4; 250 000 12.8 and 12.9; 30 000 6.5 and 6.6)
constexpr unsigned kDirectWorkgroups = 2048;
__global__ __launch_bounds__(kDirectThreads) void k_eval_direct(DevPlan pl, EvalArgs a, DirectMem dm) {
  extern __shared__ uint64_t direct_lds[];
  uint32_t *const lds = reinterpret_cast<uint32_t *>(direct_lds);
  const DirectTables L = direct_tables_at(pl, lds);
  const int n_words = (int)direct_copy_words(pl);
  for (int i = threadIdx.x; i < pl.DP * pl.ZGr; i += kDirectThreads) {  // (degrees are at least 1)
    const int d = i / pl.ZGr;
    L.room[i] = 2u * (uint32_t)pl.avail[i - d * pl.ZGr] / (uint32_t)pl.vals[d];
  }
#pragma unroll 4
  for (int i = threadIdx.x; i < n_words; i += kDirectThreads) lds[i] = pl.direct_tables[i];
  __syncthreads();
  const uint32_t GX = pl.GX, Z = pl.Z, ZG = pl.ZG, MB = pl.MB, DP = pl.DP, TP = pl.TP;
  const uint32_t mbtp = MB * TP, mbtpdp = mbtp * DP, gxmb = GX * MB, mbdp = MB * DP, slots = 3 * TP;
  const float inv_mb = float_inverse(MB), inv_mbtp = float_inverse(mbtp), inv_mbtpdp = float_inverse(mbtpdp),
              inv_gx = float_inverse(GX), inv_zg1 = float_inverse(ZG > 1 ? ZG - 1 : 1), inv_tp = float_inverse(TP);
  const bool in_lds = pl.n_shapes <= kDirectShapes;
  const double inv_inner = 1.0 / (double)pl.inner;
  int first_step = 1;  // of the search for an index's block
  while (2 * first_step < pl.n_blocks) first_step *= 2;
  const uint64_t stride = (uint64_t)gridDim.x * kDirectThreads;
  for (uint64_t i = (uint64_t)blockIdx.x * kDirectThreads + threadIdx.x; i < a.count; i += stride) {
    const uint64_t idx = a.indices ? a.indices[i] : a.first + i;
    float T = kPosInf, C = kPosInf;
    uint64_t peak = 0;
    uint32_t mask = 0xFFFFFFFFu;
    if (idx < pl.N) {
      int b = 0;  // the last block that starts at or before the index (blocks are ordered and not empty)
      for (int step = first_step; step > 0; step >>= 1) {
        const int c = min(b + step, pl.n_blocks - 1);
        if (L.blocks[c].off <= idx) b = c;
      }
      const DirectBlock blk = L.blocks[b];
      const int S = (int)blk.s;
      const uint64_t within = idx - blk.off;
      double rem, in_d;
      const uint32_t shape = blk.first_shape + (uint32_t)divide_by((double)within, blk.size, blk.inv_size, rem);
      uint32_t o = (uint32_t)divide_by(rem, (double)pl.inner, inv_inner, in_d), in = (uint32_t)in_d;
      uint32_t p[3], k[3];  // pool and TP index of each segment
      p[0] = float_div(in, inv_mbtpdp);
      in -= mul24(p[0], mbtpdp);
      const uint32_t dp = float_div(in, inv_mbtp);
      in -= mul24(dp, mbtp);
      k[0] = k[1] = k[2] = float_div(in, inv_mb);
      const uint32_t mb = in - mul24(k[0], MB), md = mul24(mb, DP) + dp;
      // the later segments' digits (o < 2^20; zero where there is no such segment, which then names
      // the pool behind: in bounds, not used)
      auto digit = [&](uint32_t radix, float inv) {
        const uint32_t q = float_div(o, inv), d = o - mul24(q, radix);
        o = q;
        return d;
      };
#pragma unroll
      for (int j = 1; j < 3; ++j) {
        if (j >= S) { p[j] = p[0]; k[j] = k[0]; continue; }
        p[j] = p[j - 1] + 1 + digit(ZG - 1, inv_zg1);
        if (p[j] >= ZG) p[j] -= ZG;
        if (pl.pst) k[j] = digit(TP, inv_tp);
      }
      const int nb = L.nb[md];
      mask = nb == 0 ? 4u : 0u;
      if (nb != 0) {
        const uint32_t stages = in_lds ? L.n[shape] : dm.shape_n[shape];
        float4 ta[3];
        float2 su[3];
        uint64_t need[3];
        uint32_t z[3], g[3];
        const uint32_t slot0 = shape * slots;
        const float4 *const ta_at = pl.ta + ((uint64_t)slot0 * gxmb + mb);
        const float2 *const su_at = dm.su + (uint64_t)slot0 * ZG;
        const uint64_t *const need_at = pl.need + ((uint64_t)slot0 * mbdp + md);
#pragma unroll
        for (int j = 0; j < 3; ++j) {  // what comes from memory is requested before any of it is used
          z[j] = float_div(p[j], inv_gx);
          g[j] = p[j] - mul24(z[j], GX);
          if (j >= S) continue;
          const uint32_t sl = 3u * k[j] + (uint32_t)j;
          ta[j] = ta_at[mul24(sl, gxmb) + mul24(g[j], MB)];
          su[j] = su_at[mul24(sl, ZG) + p[j]];
          need[j] = need_at[mul24(sl, mbdp)];
        }
        LaneC lc;
        lc.nbm1 = L.nbm1[md];
        lc.cd = L.cd[dp];
        lc.dph = L.dph[dp];
        lc.xb = L.xb[mb];
        const uint32_t *room = L.room + mul24(dp, pl.ZGr);
        const bool odd = (L.dp[dp] & 1) != 0;
        const float *ts = L.ts + mul24(mb, mul24(Z, Z));  // transfer seconds of this microbatch size
        const int n[3] = {(int)(stages & 255u) + 1, (int)((stages >> 8) & 255u) + 1, (int)((stages >> 16) & 255u) + 1};
        Acc acc;
        int w[3], ra[3], rb[3];  // GPUs of one replica on the pool, the real pools
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          w[j] = 0;
          ra[j] = rb[j] = 0;
          if (j >= S) continue;
          const uint32_t x = L.xt[g[j]];
          const int ga = x & 255, gb = x >> 8, tpv = L.tp[k[j]];
          const Rec r = make_rec(ta[j], su[j].x, su[j].y, L.price[g[j]], ts[mul24(z[j], Z + 1)], n[j], tpv, 0u);
          const uint64_t m = need[j] + L.res[ga];
          if (m > L.cap[ga]) mask |= 1u;
          peak = m > peak ? m : peak;
          if (pl.mixed) {
            const uint64_t m2 = need[j] + L.res[gb];
            if (m2 > L.cap[gb]) mask |= 1u;
            peak = m2 > peak ? m2 : peak;
          }
          w[j] = (int)mul24(n[j], tpv);  // (both below 2^21)
          ra[j] = (int)mul24(z[j], pl.G) + ga;
          rb[j] = (int)mul24(z[j], pl.G) + gb;
          // (a pair gives half of the replicas from each type, an even number of them)
          const uint32_t half = (uint32_t)w[j];
          const bool fits = ga == gb ? 2u * half <= room[ra[j]] : (!odd && half <= room[ra[j]] && half <= room[rb[j]]);
          if (!fits) mask |= 2u;
          if (tpv > L.node[ga] || tpv > L.node[gb]) mask |= 8u;
          if (j == 0) {
            acc = acc_begin(r);
          } else {
            const uint32_t zp = z[j - 1];
            const uint32_t ab = mul24(zp, Z) + z[j], ba = mul24(z[j], Z) + zp;
            acc = acc_cross(acc, r, ts[ab], ts[ba], L.egs[ab], n[j - 1] == 1, j == 1);
          }
        }
        // segments that draw on one real pool together
        if (pl.mixed) {  // half-GPUs per replica that each real pool named by the segments gives in all
          auto taken = [&](int r) {
            int h = 0;
#pragma unroll
            for (int q = 0; q < 3; ++q) h += (ra[q] == r ? w[q] : 0) + (rb[q] == r ? w[q] : 0);
            return h;
          };
          if (S >= 2)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              if (j >= S) continue;
              if ((uint32_t)taken(ra[j]) > room[ra[j]] || (uint32_t)taken(rb[j]) > room[rb[j]]) mask |= 2u;
            }
        } else if (S == 3 && p[0] == p[2]) {
          if (2u * (uint32_t)(w[0] + w[2]) > room[p[0]]) mask |= 2u;
        }
        acc_finish(acc, lc, T, C);
        if (a.has_bound) {
          if (a.objective == 0) { if (C > a.bound) mask |= 32u; }
          else if (throughput_below(T, a.bound)) mask |= 32u;
        }
      }
    }
    if (a.time) a.time[i] = T;
    if (a.cost) a.cost[i] = C;
    if (a.mem) a.mem[i] = peak;
    if (a.mask) a.mask[i] = mask;
  }
}

// Range form of sailor_eval_batch.  One workgroup per EvalUnit: the records of the unit's
// shape for every tp are staged in LDS.  A lane keeps its inner digits (mb, tp, dp, pool 1)
// while the unit's outer digits advance, and consecutive lanes hold consecutive
// candidate indices, so every store instruction writes 64 consecutive elements.
struct PoolInfo {   // per pool, staged in LDS (a pair of types: the tighter of the two)
  uint64_t res;     // reserved bytes (the larger)
  int64_t room;     // capacity - reserved (the smaller; negative when nothing fits)
  int32_t avail;    // GPUs available (plain types only)
  uint32_t meta;    // zone | (bit 8 + k: tp k exceeds the node size) (H1)
  uint64_t pad;     // (32 bytes: the index is a shift)
};
static_assert(sizeof(PoolInfo) == 32, "one pool per 32 bytes of LDS");

// A segment record of the range evaluation, kept in LDS as two 16-byte halves in arrays of
// their own: the records a wave reads together then lie 16 bytes apart, not 32, and collide
// on half as many banks.
__device__ __forceinline__ Rec rec_of(const float4 *lo, const float4 *hi, uint32_t i) {
  const float4 a = lo[i], b = hi[i];
  Rec r;
  r.sumT = a.x; r.tF = a.y; r.tL = a.z; r.tI = a.w;
  r.syncb = b.x; r.upd = b.y; r.pricen = b.z;
  r.bits = 0u;  // validity comes from the masks here
  return r;
}

template <int S, bool PST, bool MIXED>
__device__ __forceinline__ void eval_rows_body(const DevPlan &pl, const EvalArgs &a,
                                               const EvalUnit &u, const ShapeRec &sh,
                                               const float4 *rec_lo, const float4 *rec_hi,
                                               const float4 *pair, const uint32_t *qm,
                                               const uint64_t *need, const PoolInfo *pinfo,
                                               const uint32_t *odec, const int32_t *vals,
                                               const uint64_t *isect) {
  const uint32_t ZG = pl.ZG, MB = pl.MB, TP = pl.TP, DP = pl.DP, Z = pl.Z;
  const uint32_t inner = pl.inner;
  const uint64_t last = a.first + a.count;
  const bool single0 = sh.n[0] == 1, single1 = sh.n[1] == 1;
  // the unit's outputs start here; lanes add a 32-bit offset (a unit that begins before the
  // range only stores where idx >= first, so the wrapped pointer is never used below it)
  const int64_t ubase = (int64_t)(u.idx_lo - a.first);
  float *const o_time = a.time ? a.time + ubase : nullptr;
  float *const o_cost = a.cost ? a.cost + ubase : nullptr;
  uint64_t *const o_mem = a.mem ? a.mem + ubase : nullptr;
  uint32_t *const o_mask = a.mask ? a.mask + ubase : nullptr;
  const bool whole = u.idx_lo >= a.first && u.idx_lo + (uint64_t)u.o_cnt * inner <= last;  // uniform
  const uint32_t tp_rec = mul24(ZG, MB) + 1u;  // records per (segment, tp) slice, one unused
  const uint32_t seg_rec = mul24(TP, tp_rec), seg_need = mul24(mul24(TP, MB), DP),
                 seg_qm = mul24(TP, ZG);
  for (uint32_t in = threadIdx.x; in < inner; in += blockDim.x) {
    const uint32_t a1 = fast_div(in, pl.mg_mbtpdp), rem = in - mul24(a1, MB * TP * DP);
    const uint32_t dp = fast_div(rem, pl.mg_mbtp), rem2 = rem - mul24(dp, MB * TP);
    const uint32_t tp = fast_div(rem2, pl.mg_mb), mb = rem2 - mul24(tp, MB);
    const bool divisible = pl.nb[mb * DP + dp] != 0;
    LaneC lc;
    lc.nbm1 = pl.nbm1_f[mb * DP + dp];
    lc.cd = pl.cd_f[dp];
    lc.dph = pl.dph_f[dp];
    lc.xb = pl.xb_f[mb];
    // this lane's slices of the staged tables; segment j with tp index k on pool p:
    const float4 *recl_lo = rec_lo + mb, *recl_hi = rec_hi + mb;  // [(j * TP + k) * tp_rec + p * MB]
    const uint64_t *needl = need + mul24(mb, DP) + dp;  // [(j * TP + k) * MB * DP]
    const float4 *pairm = pair + mul24(mb, Z * Z);   // transfers of this microbatch size
    // with one tp per plan the later segments use this lane's tp: their slices are fixed
    const uint32_t tpo_rec = mul24(tp, tp_rec), tpo_need = mul24(mul24(tp, MB), DP),
                   tpo_qm = mul24(tp, ZG);
    // segment 1 does not change while the outer digits advance
    const uint32_t p0 = a1;
    const Rec r0 = rec_of(recl_lo, recl_hi, tpo_rec + mul24(p0, MB));
    const Acc A0 = acc_begin(r0);
    const PoolInfo i0 = pinfo[p0];
    const uint64_t need0 = needl[tpo_need], mem0 = need0 + i0.res;
    uint32_t mask0 = 0;
    if ((int64_t)need0 > i0.room) mask0 |= 1u;
    if (i0.meta & (1u << (8 + tp))) mask0 |= 8u;
    const bool q0 = (qm[tpo_qm + p0] >> dp) & 1u;
    const uint32_t z0 = i0.meta & 0xFFu;
    const int64_t D = vals[dp];  // value lists staged in LDS: [DP] dp, then [TP] tp
    const int64_t gpus0 = (int64_t)sh.n[0] * vals[DP + tp];
    // with one tp per plan the bytes segments 2 and 3 need do not change with the outer digits
    const uint64_t need1_lane = (!PST && S >= 2) ? needl[seg_need + tpo_need] : 0;
    const uint64_t need2_lane = (!PST && S == 3) ? needl[2 * seg_need + tpo_need] : 0;
    uint32_t off = in;           // o * inner + in
    for (uint32_t o = 0; o < u.o_cnt; ++o, off += inner) {
      if (!whole) {
        const uint64_t idx = u.idx_lo + off;
        if (idx < a.first || idx >= last) continue;
      }
      const uint32_t od = odec[o];  // outer digits (uniform)
      float T = kPosInf, C = kPosInf;
      uint64_t peak = 0;
      uint32_t mask = 4u;
      if (divisible) {
        mask = mask0;
        peak = mem0;
        Acc acc = A0;
        bool quota_ok = q0;
        if (S >= 2) {
          const uint32_t r2 = od & 127u;
          const uint32_t t1 = PST ? ((od >> 7) & 7u) : tp;
          uint32_t p1 = p0 + 1 + r2;
          if (p1 >= ZG) p1 -= ZG;
          // uniform offsets when the segment has its own tp digit, this lane's otherwise
          const uint32_t o_rec = seg_rec + (PST ? mul24(t1, tp_rec) : tpo_rec);
          const uint32_t o_need = seg_need + (PST ? mul24(mul24(t1, MB), DP) : tpo_need);
          const uint32_t o_qm = seg_qm + (PST ? mul24(t1, ZG) : tpo_qm);
          const Rec r1 = rec_of(recl_lo, recl_hi, o_rec + mul24(p1, MB));
          const PoolInfo i1 = pinfo[p1];
          const uint32_t z1 = i1.meta & 0xFFu;
          const uint64_t need1 = PST ? needl[o_need] : need1_lane, mem1 = need1 + i1.res;
          if ((int64_t)need1 > i1.room) mask |= 1u;
          if (i1.meta & (1u << (8 + t1))) mask |= 8u;
          peak = mem1 > peak ? mem1 : peak;
          const bool q1 = (qm[o_qm + p1] >> dp) & 1u;
          quota_ok = quota_ok && q1;
          if (S == 2 && MIXED && quota_ok && pool_bit(isect, (int)p0, (int)p1))
            quota_ok = (joint_quota_bits(pl, 2, (int)p0, (int)p1, 0, (int)gpus0,
                                         sh.n[1] * vals[DP + t1], 0) >> dp) & 1u;
          const float4 pr = pairm[mul24(z0, Z) + z1];
          acc = acc_cross(acc, r1, pr.x, pr.y, pr.z, single0, true);
          if (S == 3) {
            const uint32_t r3 = (od >> 10) & 127u;
            const uint32_t t2 = PST ? (od >> 17) : tp;
            uint32_t p2 = p1 + 1 + r3;
            if (p2 >= ZG) p2 -= ZG;
            const uint32_t o_rec2 = 2 * seg_rec + (PST ? mul24(t2, tp_rec) : tpo_rec);
            const uint32_t o_need2 = 2 * seg_need + (PST ? mul24(mul24(t2, MB), DP) : tpo_need);
            const uint32_t o_qm2 = 2 * seg_qm + (PST ? mul24(t2, ZG) : tpo_qm);
            const Rec r2r = rec_of(recl_lo, recl_hi, o_rec2 + mul24(p2, MB));
            const PoolInfo i2 = pinfo[p2];
            const uint64_t need2 = PST ? needl[o_need2] : need2_lane, mem2 = need2 + i2.res;
            if ((int64_t)need2 > i2.room) mask |= 1u;
            if (i2.meta & (1u << (8 + t2))) mask |= 8u;
            peak = mem2 > peak ? mem2 : peak;
            if (MIXED) {  // pools that draw on one real pool together get the joint check
              quota_ok = quota_ok && ((qm[o_qm2 + p2] >> dp) & 1u);
              if (quota_ok && (pool_bit(isect, (int)p0, (int)p1) || pool_bit(isect, (int)p1, (int)p2) ||
                               pool_bit(isect, (int)p0, (int)p2)))
                quota_ok = (joint_quota_bits(pl, 3, (int)p0, (int)p1, (int)p2, (int)gpus0,
                                             sh.n[1] * vals[DP + t1], sh.n[2] * vals[DP + t2]) >> dp) & 1u;
            } else if (p2 == p0) {  // segments 1 and 3 share one pool's quota
              const int64_t gpus = gpus0 + (int64_t)sh.n[2] * vals[DP + t2];
              quota_ok = q1 && gpus * D <= (int64_t)i0.avail;
            } else {
              quota_ok = quota_ok && ((qm[o_qm2 + p2] >> dp) & 1u);
            }
            const float4 pr2 = pairm[mul24(z1, Z) + (i2.meta & 0xFFu)];
            acc = acc_cross(acc, r2r, pr2.x, pr2.y, pr2.z, single1, false);
          }
        }
        if (!quota_ok) mask |= 2u;
        acc_finish(acc, lc, T, C);
        if (a.has_bound) {
          if (a.objective == 0) { if (C > a.bound) mask |= 32u; }
          else if (throughput_below(T, a.bound)) mask |= 32u;
        }
      }
      if (o_time) o_time[off] = T;
      if (o_cost) o_cost[off] = C;
      if (o_mem) o_mem[off] = peak;
      if (o_mask) o_mask[off] = mask;
    }
  }
}

template <bool MIXED>
__global__ __launch_bounds__(512) void k_eval_rows(DevPlan pl, EvalArgs a, const EvalUnit *units,
                                                   uint32_t unit0) {
  extern __shared__ uint4 lds_raw[];
  const EvalUnit u = units[unit0 + blockIdx.x];
  const ShapeRec sh = pl.shapes[u.shape];
  const int ZG = pl.ZG, G = pl.GX, MB = pl.MB, TP = pl.TP, DP = pl.DP, Z = pl.Z, S = sh.s;
  // [3][TP][ZG * MB + 1]: a (segment, tp) slice is one record longer than its contents, so
  // that the slices of the tp values a wave reads together do not start on the same LDS banks
  float4 *rec_lo = reinterpret_cast<float4 *>(lds_raw);  // the records' two halves (see rec_of)
  float4 *rec_hi = rec_lo + 3 * TP * (ZG * MB + 1);
  float4 *pair = rec_hi + 3 * TP * (ZG * MB + 1);         // [MB][Z][Z]
  PoolInfo *pinfo = reinterpret_cast<PoolInfo *>(pair + MB * Z * Z);     // [ZG]
  uint64_t *need = reinterpret_cast<uint64_t *>(pinfo + ZG);             // [3][TP][MB][DP]
  uint64_t *isect = need + 3 * TP * MB * DP;                             // [ZG][2]
  uint32_t *qm = reinterpret_cast<uint32_t *>(isect + 2 * ZG);           // [3][TP][ZG]
  uint32_t *odec = qm + 3 * TP * ZG;  // [o_cnt] the outer digits of the unit, unpacked:
  int32_t *vals = reinterpret_cast<int32_t *>(odec + kEvalUnitMaxOuter);  // [DP] dp, [TP] tp
  const int t = threadIdx.x;          // r2 | tp2 << 7 | r3 << 10 | tp3 << 17
  if (t < DP) vals[t] = pl.dpv[t];
  else if (t < DP + TP) vals[t] = pl.tpv[t - DP];
  __syncthreads();
  if (S >= 2)
    for (uint32_t o = t; o < u.o_cnt; o += blockDim.x) {
      uint32_t oa = u.o_lo + o;
      uint32_t d = oa % (uint32_t)(ZG - 1);
      oa /= (uint32_t)(ZG - 1);
      if (pl.pst) { d |= (oa % (uint32_t)TP) << 7; oa /= (uint32_t)TP; }
      if (S == 3) {
        d |= (oa % (uint32_t)(ZG - 1)) << 10;
        oa /= (uint32_t)(ZG - 1);
        if (pl.pst) d |= oa << 17;
      }
      odec[o] = d;
    }
  else
    for (uint32_t o = t; o < u.o_cnt; o += blockDim.x) odec[o] = 0;
  for (int i = t; i < S * TP * ZG; i += blockDim.x) {
    const int p = i % ZG, k = (i / ZG) % TP, seg = i / (ZG * TP);
    const int n = seg == 0 ? sh.n[0] : (seg == 1 ? sh.n[1] : sh.n[2]);
    qm[i] = pl.qw[(size_t)(n * vals[DP + k]) * ZG + p];
  }
  for (int p = t; p < ZG; p += blockDim.x) {
    const int x = pl.xt[p % G], ga = x & 255, gb = x >> 8;
    PoolInfo pi;
    pi.res = max(pl.res[ga], pl.res[gb]);
    pi.room = min((int64_t)pl.cap[ga] - (int64_t)pl.res[ga], (int64_t)pl.cap[gb] - (int64_t)pl.res[gb]);
    pi.avail = pl.mixed ? 0 : pl.avail[p];
    pi.meta = (uint32_t)(p / G) | (pl.h1m[p] << 8);
    pi.pad = 0;
    pinfo[p] = pi;
    isect[2 * p] = pl.isect[2 * p];
    isect[2 * p + 1] = pl.isect[2 * p + 1];
  }
  for (int i = t; i < MB * Z * Z; i += blockDim.x) {  // per mb: transfer a -> b, b -> a, egress
    const int m = i / (Z * Z), ab = i - m * Z * Z, za = ab / Z, zb = ab % Z;
    pair[i] = make_float4(pl.tsec_f[i], pl.tsec_f[(m * Z + zb) * Z + za], pl.egs_f[ab], 0.f);
  }
  for (int i = t; i < S * TP * MB * DP; i += blockDim.x) {
    const int md = i % (MB * DP), k = (i / (MB * DP)) % TP, seg = i / (MB * DP * TP);
    need[i] = pl.need[agg_slot(pl, u.shape, k, seg) * MB * DP + md];
  }
  for (int i = t; i < S * TP * ZG * MB; i += blockDim.x) {
    const int mb = i % MB, p = (i / MB) % ZG, k = (i / (MB * ZG)) % TP, seg = i / (MB * ZG * TP);
    const int g = p % G, z = p / G;
    const size_t sl = agg_slot(pl, u.shape, k, seg);
    const Rec r =
        make_rec(pl.ta[(sl * G + g) * MB + mb], pl.syncz[sl * Z + z], pl.upd[sl * G + g],
                 pl.price_f[g], pl.tsec_f[(mb * Z + z) * Z + z],
                 seg == 0 ? sh.n[0] : (seg == 1 ? sh.n[1] : sh.n[2]), vals[DP + k], 0u);
    const int at = i + seg * TP + k;  // (one unused record behind every slice)
    rec_lo[at] = make_float4(r.sumT, r.tF, r.tL, r.tI);
    rec_hi[at] = make_float4(r.syncb, r.upd, r.pricen, 0.f);
  }
  __syncthreads();
#define SAILOR_ROWS(S_, PST_) \
  eval_rows_body<S_, PST_, MIXED>(pl, a, u, sh, rec_lo, rec_hi, pair, qm, need, pinfo, odec, vals, isect)
  if (S == 1) SAILOR_ROWS(1, false);
  else if (!pl.pst) { if (S == 2) SAILOR_ROWS(2, false); else SAILOR_ROWS(3, false); }
  else { if (S == 2) SAILOR_ROWS(2, true); else SAILOR_ROWS(3, true); }
#undef SAILOR_ROWS
}

}  // namespace sailor

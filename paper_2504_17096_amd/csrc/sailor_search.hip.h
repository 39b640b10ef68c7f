// Search over per-stage placements (gfx950, wave64), on top of the tables of the evaluator.
//
// The planner assigns resources stage by stage (Sailor, Sec. 4.2.2, Eq. (1): stage i gets r,
// the stages behind it R - r, times composed by T_total); the heuristics H3 / H4 (Sec. 4.2.1)
// stop early when nothing better can follow.  Here every stage of a pipeline chooses its pool
// (zone, GPU type) freely -- all D replicas of a stage on that pool (H5), one TP degree per
// plan -- and one workgroup works through one sub-problem (pipeline depth, layer split, TP,
// D, microbatch size) level by level: the frontier of placements of stages 0 .. j-1 is
// extended by every pool for stage j, each extension gets a lower bound on T_iter and C_iter
// (Sec. 4.3) of all its completions, extensions whose bound breaks the constraint or exceeds
// an incumbent are dropped, and a frontier longer than the beam width keeps the smallest
// bounds.  At the last level the bound is the plan's own T_iter / C_iter.
//
// Two wider forms of a stage's choice: half of its replicas on a second pool (a, b), or its own
// TP degree (a, t) -- tp_ij of Sec. 4.2.2 taken per stage; TP then leaves the sub-problem and a
// pool's quota is counted in GPUs of one replica.
//
//   k_search_beam        the level-by-level expansion, one workgroup per sub-problem
//   k_search_pick        smallest (key, sub-problem) over the sub-problems' winners
//   k_eval_placements    the simulator of Sec. 4.3 for listed placements, one wave each, fp64
//   k_eval_replicas      the same for plans in which every replica of every stage names its pool
//
// All arithmetic is fp64 in a fixed order (sums in stage order), so that which extension is
// dropped or kept does not depend on how the work is spread over lanes.
#pragma once

#include <hip/hip_runtime.h>

#include "sailor_kernels.hip.h"

namespace sailor {

constexpr int kSearchThreads = 256;
constexpr int kSearchMaxBeam = 1024;   // longest frontier a sub-problem keeps (half of kSearchBuf at most)
constexpr int kSearchBuf = 2048;       // extensions buffered between two sorts
constexpr int kSearchMaxStages = 255;  // placements count stages per pool in a byte
constexpr int kSearchMaxPools = 64;

struct SearchPP {      // one pipeline depth
  int32_t P;
  uint32_t rs0;        // first entry of its first partition row in the stage tables
  uint32_t sub_off;    // first sub-problem of this depth
  int32_t n_part;
  uint32_t sub_off_t;  // the same when TP is not part of the sub-problem
  uint32_t pad[3];
};

enum : int { SEARCH_PLAIN = 0, SEARCH_SPLIT = 1, SEARCH_STAGE_TP = 2, SEARCH_SPLIT_TP = 3 };

struct SState {        // placement of stages 0 .. j; kStateBytes, followed by the paths (a byte per stage)
  double sum;          // times of the closed stages 0 .. j-1
  double maxt;         // slowest closed stage
  double c_open;       // compute time of stage j (its forward transfer is not known yet)
  double xb_open;      // its backward transfer to stage j-1
  double sum_b, maxt_b, c_open_b, xb_open_b;  // with split stages: the pipelines through the second pools
  double msync, mupd, dol, comm;
  uint16_t cnt[kSearchMaxPools];  // stages placed on each pool (split stages: halves of stages; a
                                  // TP degree per stage: GPUs of one replica)
  uint8_t pool, pool_b, runs, tpi, pad[4];  // tpi: the open stage's TP index (TP per stage)
};
constexpr uint32_t kStateBytes = sizeof(SState);
static_assert(kStateBytes == 232, "twelve doubles, the pool counts, pools, runs and TP index");

struct SubResult {     // winner of one sub-problem (or of the whole search)
  double key, T, C;
  uint32_t found, truncated;
  unsigned long long expanded;
  uint32_t sid, P;
  int32_t desc[6];     // pp index, partition, tp index, dp index, mb index, the search's mode
  int32_t pools[256];  // pool of every stage
  int32_t pools_b[256];  // pool of the other half of its replicas (= pools[i] when not split)
  int32_t tps[256];      // TP index of every stage (= desc[2] unless the stages choose their own)
};

struct SearchArgs {
  int objective, has_bound, has_inc, W, max_runs;
  double bound, inc;
  const SearchPP *pps;
  int n_pp;
  uint32_t n_sub;
  uint8_t *states;        // [workgroups][2][W] states of state_stride bytes
  uint32_t state_stride;  // kStateBytes + three paths of path_stride bytes (pools, second pools, TP indices)
  uint32_t path_stride;   // the deepest pipeline, rounded up to 8
  SubResult *results;     // [n_sub]
};

struct SBound { double T, C; };

// Lower bounds of T_iter and C_iter over the completions of a placement whose stage j is open;
// the plan's own values when j = P - 1 (then every S term is zero).
__device__ __forceinline__ SBound search_bounds(double sum, double maxt, double c_open, double xb_open,
                                                double msync, double mupd, double dol, double comm,
                                                double Ssum, double Smax, double Ssync, double Supd,
                                                double Sdol, double nbm1) {
  const double t_open = c_open + xb_open;
  const double tsum = (sum + t_open) + Ssum;
  const double tmax = fmax(fmax(maxt, t_open), Smax);
  SBound b;
  b.T = ((tsum + nbm1 * tmax) + fmax(msync, Ssync)) + fmax(mupd, Supd);
  b.C = (dol + Sdol) / 3600.0 * b.T + comm;
  return b;
}

__device__ __forceinline__ bool key_id_less(unsigned long long ka, uint32_t ia, unsigned long long kb,
                                            uint32_t ib) {
  return ka < kb || (ka == kb && ia < ib);
}

// Ascending bitonic sort of (key, id) pairs in LDS; m = the power of two >= n, entries
// n .. m-1 are filled with the largest pair first.
__device__ __forceinline__ void search_sort(unsigned long long *key, uint32_t *id, int n) {
  int m = 1;
  while (m < n) m <<= 1;
  for (int i = n + (int)threadIdx.x; i < m; i += blockDim.x) { key[i] = ~0ull; id[i] = ~0u; }
  __syncthreads();
  for (int k = 2; k <= m; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < m; i += blockDim.x) {
        const int x = i ^ j;
        if (x > i) {
          const bool up = (i & k) == 0;
          const unsigned long long ki = key[i], kx = key[x];
          const uint32_t ii = id[i], ix = id[x];
          const bool swap = up ? key_id_less(kx, ix, ki, ii) : key_id_less(ki, ii, kx, ix);
          if (swap) { key[i] = kx; key[x] = ki; id[i] = ix; id[x] = ii; }
        }
      }
      __syncthreads();
    }
}

struct SearchTables {  // LDS of a search workgroup: the sub-problem's and the level's tables
  double S[5][kSearchMaxStages + 1];   // what lies behind stage i: sum, max, sync, upd, $
  double xfer[kMaxZones][kMaxZones], comm[kMaxZones][kMaxZones];
  double comm_half[kMaxZones][kMaxZones];  // traffic of one kind of pipeline (half of the replicas)
  double bw[kMaxZones][kMaxZones], ring_price[kMaxZones][kMaxZones];
  double l_c[kMaxTypes], l_upd[kMaxTypes], l_dol[kMaxTypes], l_price[kMaxTypes], l_sync[kMaxZones];
  double l_ring;                       // bytes the level's stage's ring all-reduce moves over every link
  double smin[4][kSearchMaxStages + 1];  // cheapest admissible choice of every stage
  int cap[kSearchMaxPools];            // stages a pool can host
  int cap_half[kSearchMaxPools];       // halves of stages
  uint32_t l_fit;                      // bit g: the level's stage fits type g
  int dp_even;
  double dtp;                          // D * tp
  // a TP degree per stage: the level's stage on every type / zone at every degree
  double l_c3[kMaxTypes][kMaxTP], l_upd3[kMaxTypes][kMaxTP], l_dol3[kMaxTypes][kMaxTP];
  double l_sync3[kMaxZones][kMaxTP];
  uint32_t l_fit3[kMaxTP];             // bit g: the level's stage fits type g at this degree
  int tpv[kMaxTP];
  int cap_gpus[kSearchMaxPools];       // GPUs one replica can take from a pool
  // ... and two pools per stage as well
  double l_ring3[kMaxTP];              // the level's stage's ring bytes at every degree
  int cap_half_gpus[kSearchMaxPools];  // GPUs of one replica, counted once per half of a stage
  long long dp;                        // D
};

struct SAcc {          // what a placement carries besides its pool counts
  double sum, maxt, c_open, xb_open, sum_b, maxt_b, c_open_b, xb_open_b, msync, mupd, dol, comm;
};

// Stage j on pool a (split stages: half of its replicas on pool b, else b = a) at TP index k (a
// TP degree per stage; else the sub-problem's) behind the placement par (none for j = 0): may
// it be placed, and what the placement then carries.  The order of the operations is part of
// the definition: sums in stage order, a closed stage's transfers forward then backward.
template <int MODE>
__device__ __forceinline__ bool search_step(const SearchTables &T, const SState *par, int j, int a, int b,
                                            int k, int G, int max_runs, SAcc &o, int &runs) {
  constexpr bool SPLIT = MODE == SEARCH_SPLIT;
  if (MODE == SEARCH_SPLIT_TP) {
    const int ga = a % G, za = a / G, gb = b % G, zb = b / G, width = T.tpv[k];
    bool ok = ((T.l_fit3[k] >> ga) & 1u) != 0 && ((T.l_fit3[k] >> gb) & 1u) != 0;
    const int ca = par ? (int)par->cnt[a] : 0, cb = par ? (int)par->cnt[b] : 0;
    if (a == b) ok = ok && ca + 2 * width <= T.cap_half_gpus[a];
    else ok = ok && T.dp_even && ca + width <= T.cap_half_gpus[a] && cb + width <= T.cap_half_gpus[b];
    runs = par ? par->runs + ((a != par->pool || b != par->pool_b || k != par->tpi) ? 1 : 0) : 1;
    if (max_runs != 0 && runs > max_runs) ok = false;
    if (!ok) return false;
    double link = T.bw[za][za];
    if (zb != za) link = fmin(fmin(link, T.bw[zb][zb]), fmin(T.bw[za][zb], T.bw[zb][za]));
    const double sync = T.l_ring3[k] / link;
    const double upd = fmax(T.l_upd3[ga][k], T.l_upd3[gb][k]);
    const double dol = (double)(T.dp * (long long)width) * (0.5 * (T.l_price[ga] + T.l_price[gb]));
    const double ring = zb != za ? T.l_ring3[k] * T.ring_price[za][zb] : 0.0;
    o.c_open = T.l_c3[ga][k];
    o.c_open_b = T.l_c3[gb][k];
    if (!par) {
      o.sum = o.maxt = o.xb_open = o.sum_b = o.maxt_b = o.xb_open_b = 0.0;
      o.msync = sync; o.mupd = upd; o.dol = dol; o.comm = ring;
    } else {
      const int pza = par->pool / G, pzb = par->pool_b / G;
      const double ta = par->c_open + (T.xfer[pza][za] + par->xb_open);  // forward, then backward
      const double tb = par->c_open_b + (T.xfer[pzb][zb] + par->xb_open_b);
      o.sum = par->sum + ta;
      o.maxt = fmax(par->maxt, ta);
      o.sum_b = par->sum_b + tb;
      o.maxt_b = fmax(par->maxt_b, tb);
      o.xb_open = T.xfer[za][pza];
      o.xb_open_b = T.xfer[zb][pzb];
      o.msync = fmax(par->msync, sync);
      o.mupd = fmax(par->mupd, upd);
      o.dol = par->dol + dol;
      double comm = par->comm;
      if (pza != za) comm += T.comm_half[pza][za];
      if (pzb != zb) comm += T.comm_half[pzb][zb];
      o.comm = comm + ring;
    }
    return true;
  }
  if (MODE == SEARCH_STAGE_TP) {
    const int g = a % G, z = a / G, t = k;
    bool ok = ((T.l_fit3[t] >> g) & 1u) != 0;
    const int used = par ? (int)par->cnt[a] : 0;
    ok = ok && used + T.tpv[t] <= T.cap_gpus[a];
    runs = par ? par->runs + ((a != par->pool || t != par->tpi) ? 1 : 0) : 1;
    if (max_runs != 0 && runs > max_runs) ok = false;
    if (!ok) return false;
    o.c_open = T.l_c3[g][t];
    if (!par) {
      o.sum = 0.0; o.maxt = 0.0; o.xb_open = 0.0; o.msync = T.l_sync3[z][t]; o.mupd = T.l_upd3[g][t];
      o.dol = T.l_dol3[g][t]; o.comm = 0.0;
    } else {
      const int pz = par->pool / G;
      const double t_closed = par->c_open + (T.xfer[pz][z] + par->xb_open);  // forward, then backward
      o.sum = par->sum + t_closed;
      o.maxt = fmax(par->maxt, t_closed);
      o.xb_open = T.xfer[z][pz];
      o.msync = fmax(par->msync, T.l_sync3[z][t]);
      o.mupd = fmax(par->mupd, T.l_upd3[g][t]);
      o.dol = par->dol + T.l_dol3[g][t];
      o.comm = pz != z ? par->comm + T.comm[pz][z] : par->comm;
    }
    o.sum_b = o.maxt_b = o.c_open_b = o.xb_open_b = 0.0;
    return true;
  }
  const int ga = a % G, za = a / G, gb = b % G, zb = b / G;
  bool ok = ((T.l_fit >> ga) & 1u) != 0 && ((T.l_fit >> gb) & 1u) != 0;
  const int ca = par ? (int)par->cnt[a] : 0, cb = par ? (int)par->cnt[b] : 0;
  if (!SPLIT) ok = ok && ca + 1 <= T.cap[a];
  else if (a == b) ok = ok && ca + 2 <= T.cap_half[a];
  else ok = ok && T.dp_even && ca + 1 <= T.cap_half[a] && cb + 1 <= T.cap_half[b];
  runs = par ? par->runs + ((a != par->pool || (SPLIT && b != par->pool_b)) ? 1 : 0) : 1;
  if (max_runs != 0 && runs > max_runs) ok = false;
  if (!ok) return false;
  if (!SPLIT) {
    o.c_open = T.l_c[ga];
    if (!par) {
      o.sum = 0.0; o.maxt = 0.0; o.xb_open = 0.0; o.msync = T.l_sync[za]; o.mupd = T.l_upd[ga];
      o.dol = T.l_dol[ga]; o.comm = 0.0;
    } else {
      const int pz = par->pool / G;
      const double t_closed = par->c_open + (T.xfer[pz][za] + par->xb_open);  // forward, then backward
      o.sum = par->sum + t_closed;
      o.maxt = fmax(par->maxt, t_closed);
      o.xb_open = T.xfer[za][pz];
      o.msync = fmax(par->msync, T.l_sync[za]);
      o.mupd = fmax(par->mupd, T.l_upd[ga]);
      o.dol = par->dol + T.l_dol[ga];
      o.comm = pz != za ? par->comm + T.comm[pz][za] : par->comm;
    }
    o.sum_b = o.maxt_b = o.c_open_b = o.xb_open_b = 0.0;
    return true;
  }
  // the stage by itself: all-reduce over the slowest link of a ring through both pools, the
  // slower update, the mean rent, the ring's traffic between the zones
  double link = T.bw[za][za];
  if (zb != za) link = fmin(fmin(link, T.bw[zb][zb]), fmin(T.bw[za][zb], T.bw[zb][za]));
  const double sync = T.l_ring / link;
  const double upd = fmax(T.l_upd[ga], T.l_upd[gb]);
  const double dol = T.dtp * (0.5 * (T.l_price[ga] + T.l_price[gb]));
  const double ring = zb != za ? T.l_ring * T.ring_price[za][zb] : 0.0;
  o.c_open = T.l_c[ga];
  o.c_open_b = T.l_c[gb];
  if (!par) {
    o.sum = o.maxt = o.xb_open = o.sum_b = o.maxt_b = o.xb_open_b = 0.0;
    o.msync = sync; o.mupd = upd; o.dol = dol; o.comm = ring;
  } else {
    const int pza = par->pool / G, pzb = par->pool_b / G;
    const double ta = par->c_open + (T.xfer[pza][za] + par->xb_open);
    const double tb = par->c_open_b + (T.xfer[pzb][zb] + par->xb_open_b);
    o.sum = par->sum + ta;
    o.maxt = fmax(par->maxt, ta);
    o.sum_b = par->sum_b + tb;
    o.maxt_b = fmax(par->maxt_b, tb);
    o.xb_open = T.xfer[za][pza];
    o.xb_open_b = T.xfer[zb][pzb];
    o.msync = fmax(par->msync, sync);
    o.mupd = fmax(par->mupd, upd);
    o.dol = par->dol + dol;
    double comm = par->comm;
    if (pza != za) comm += T.comm_half[pza][za];
    if (pzb != zb) comm += T.comm_half[pzb][zb];
    o.comm = comm + ring;
  }
  return true;
}

// Bounds of a placement whose stage j is open; with split stages the slower of the two kinds
// of pipeline counts (Sec. 4.3).
template <int MODE>
__device__ __forceinline__ SBound search_bound_of(const SearchTables &T, const SAcc &o, int j, double nbm1) {
  if (MODE != SEARCH_SPLIT && MODE != SEARCH_SPLIT_TP)
    return search_bounds(o.sum, o.maxt, o.c_open, o.xb_open, o.msync, o.mupd, o.dol, o.comm, T.S[0][j],
                         T.S[1][j], T.S[2][j], T.S[3][j], T.S[4][j], nbm1);
  const double ta = o.c_open + o.xb_open, tb = o.c_open_b + o.xb_open_b;
  const double pa = ((o.sum + ta) + T.S[0][j]) + nbm1 * fmax(fmax(o.maxt, ta), T.S[1][j]);
  const double pb = ((o.sum_b + tb) + T.S[0][j]) + nbm1 * fmax(fmax(o.maxt_b, tb), T.S[1][j]);
  SBound b;
  b.T = (fmax(pa, pb) + fmax(o.msync, T.S[2][j])) + fmax(o.mupd, T.S[3][j]);
  b.C = (o.dol + T.S[4][j]) / 3600.0 * b.T + o.comm;
  return b;
}

template <int MODE>
__global__ __launch_bounds__(kSearchThreads) void k_search_beam(DevPlan pl, SearchArgs a) {
  constexpr bool BOTH = MODE == SEARCH_SPLIT_TP;
  constexpr bool SPLIT = MODE == SEARCH_SPLIT || BOTH;     // two pools per stage
  constexpr bool STP = MODE == SEARCH_STAGE_TP || BOTH;    // a TP degree per stage
  __shared__ SearchTables T;
  __shared__ unsigned long long b_key[kSearchBuf];
  __shared__ uint32_t b_id[kSearchBuf];
  __shared__ uint32_t s_wave[kSearchThreads / 64];
  __shared__ int s_nbuf, s_bad;
  __shared__ unsigned long long s_bk[kSearchThreads / 64];
  __shared__ uint32_t s_bi[kSearchThreads / 64];
  __shared__ unsigned long long s_expanded;
  __shared__ unsigned char s_fit3[kMaxTypes][kMaxTP];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int G = pl.G, Z = pl.Z, ZG = pl.ZGr, MB = pl.MB, TP = pl.TP, DP = pl.DP;
  // choices per stage: a pool; a pair (a, b) = a * ZG + b; a pool and a TP index (a, t) = a * TP + t;
  // a pair and a TP index ((a * ZG + b) * TP + t)
  const int NCH = BOTH ? ZG * ZG * TP : (SPLIT ? ZG * ZG : (STP ? ZG * TP : ZG));
  // a choice c -> first pool, second pool (= the first without split stages), TP index
  auto choice = [&](int c, int it0, int &ca, int &cb, int &ck) {
    ck = STP ? c % TP : it0;
    const int pools = STP ? c / TP : c;
    ca = SPLIT ? pools / ZG : pools;
    cb = SPLIT ? pools - ca * ZG : ca;
  };
  uint8_t *const buf0 = a.states + (size_t)blockIdx.x * 2 * a.W * a.state_stride;
  uint8_t *const buf1 = buf0 + (size_t)a.W * a.state_stride;

  for (uint32_t sid = blockIdx.x; sid < a.n_sub; sid += gridDim.x) {  // uniform
    __syncthreads();  // the shared tables are reused
    int ip = 0;
    for (int i = 1; i < a.n_pp; ++i)
      if (sid >= (STP ? a.pps[i].sub_off_t : a.pps[i].sub_off)) ip = i;
    const SearchPP pp = a.pps[ip];
    uint32_t rem = sid - (STP ? pp.sub_off_t : pp.sub_off);
    const int im = (int)(rem % (uint32_t)MB); rem /= (uint32_t)MB;
    const int id = (int)(rem % (uint32_t)DP); rem /= (uint32_t)DP;
    const int it = STP ? 0 : (int)(rem % (uint32_t)TP);  // (TP per stage: not part of the sub-problem)
    const int q = STP ? (int)rem : (int)(rem / (uint32_t)TP);
    const int P = pp.P;
    const uint32_t rs = pp.rs0 + (uint32_t)q * (uint32_t)P;
    SubResult *res = a.results + sid;
    const int64_t nb = pl.nb[im * DP + id];
    const int64_t D = pl.dpv[id];
    const int tp = pl.tpv[it];
    if (t == 0) {
      res->found = 0; res->truncated = 0; res->expanded = 0; res->sid = sid; res->P = (uint32_t)P;
      res->desc[0] = ip; res->desc[1] = q; res->desc[2] = it; res->desc[3] = id; res->desc[4] = im;
      res->desc[5] = MODE;
      s_bad = 0;
      s_expanded = 0;
      T.dp_even = (D % 2 == 0) ? 1 : 0;
      T.dtp = (double)(D * tp);
      T.dp = (long long)D;
    }
    __syncthreads();
    if (nb == 0) continue;              // the batch does not divide (uniform)
    const double p2p = (double)pl.p2p[im];
    const double nbm1 = (double)(nb - 1);
    // tables of the sub-problem
    for (int i = t; i < Z * Z; i += blockDim.x) {
      const int z = i / Z, y = i - z * Z;
      T.xfer[z][y] = p2p / pl.bw[z * Z + y];
      T.bw[z][y] = pl.bw[z * Z + y];
      double cm = 0.0, ch = 0.0, rp = 0.0;
      if (pl.egress && z != y) {
        const double both = pl.egress[z * Z + y] + pl.egress[y * Z + z];
        cm = (double)nb * (double)D * p2p * both;
        ch = (double)nb * (0.5 * (double)D) * p2p * both;
        rp = both;
      }
      T.comm[z][y] = cm;
      T.comm_half[z][y] = ch;
      T.ring_price[z][y] = rp;
    }
    for (int p = t; p < ZG; p += blockDim.x) {
      T.cap[p] = (int)((int64_t)pl.avail[p] / ((int64_t)tp * D));
      T.cap_half[p] = (int)(2 * (int64_t)pl.avail[p] / ((int64_t)tp * D));
      T.cap_gpus[p] = (int)((int64_t)pl.avail[p] / D);
      T.cap_half_gpus[p] = (int)(2 * (int64_t)pl.avail[p] / D);
    }
    if (t < TP) T.tpv[t] = pl.tpv[t];
    if (STP) {
      for (int i = t; i < P; i += blockDim.x) {  // the cheapest admissible (type, TP) of stage i
        const uint64_t params = pl.st_params[rs + i];
        double cmin = __builtin_huge_val(), umin = cmin, dmin = cmin, smin = cmin;
        bool any = false;
        for (int k = 0; k < TP; ++k) {
          const int tpk = pl.tpv[k];
          const uint64_t bytes = stage_bytes_of(params, pl.st_n[rs + i], pl.bpp, i, P, tpk, nb, pl.act[im * TP + k]);
          const uint64_t shard = (params + (uint64_t)tpk - 1) / (uint64_t)tpk;
          bool fits_some = false;
          for (int g = 0; g < G; ++g) {
            if (!(bytes + pl.res[g] <= pl.cap[g] && tpk <= pl.node[g])) continue;
            fits_some = true;
            cmin = fmin(cmin, pl.st_c[(((size_t)(rs + i) * G + g) * MB + im) * TP + k]);
            umin = fmin(umin, pl.st_u[((size_t)(rs + i) * G + g) * TP + k]);
            dmin = fmin(dmin, (double)(D * tpk) * pl.price[g]);
          }
          if (!fits_some) continue;
          any = true;
          for (int z = 0; z < Z; ++z) {
            double sync = 0.0;
            if (D > 1) {
              const double grad = (double)shard * (double)pl.gb;
              sync = 2.0 * (double)(D - 1) / (double)D * grad / pl.bw[z * Z + z];
            }
            smin = fmin(smin, sync);
          }
        }
        T.smin[0][i] = cmin; T.smin[1][i] = smin; T.smin[2][i] = umin; T.smin[3][i] = dmin;
        if (!any) s_bad = 1;  // (benign race: every writer stores 1)
      }
    } else
    for (int i = t; i < P; i += blockDim.x) {  // the cheapest admissible choice of stage i
      const uint64_t params = pl.st_params[rs + i];
      const uint64_t bytes = stage_bytes_of(params, pl.st_n[rs + i], pl.bpp, i, P, tp, nb, pl.act[im * TP + it]);
      const uint64_t shard = (params + (uint64_t)tp - 1) / (uint64_t)tp;
      double cmin = __builtin_huge_val(), umin = cmin, dmin = cmin, smin = cmin;
      bool any = false;
      for (int g = 0; g < G; ++g) {
        if (!(bytes + pl.res[g] <= pl.cap[g] && tp <= pl.node[g])) continue;
        any = true;
        cmin = fmin(cmin, pl.st_c[(((size_t)(rs + i) * G + g) * MB + im) * TP + it]);
        umin = fmin(umin, pl.st_u[((size_t)(rs + i) * G + g) * TP + it]);
        dmin = fmin(dmin, (double)(D * tp) * pl.price[g]);
      }
      for (int z = 0; z < Z; ++z) {
        double sync = 0.0;
        if (D > 1) {
          const double grad = (double)shard * (double)pl.gb;
          sync = 2.0 * (double)(D - 1) / (double)D * grad / pl.bw[z * Z + z];
        }
        smin = fmin(smin, sync);
      }
      T.smin[0][i] = cmin; T.smin[1][i] = smin; T.smin[2][i] = umin; T.smin[3][i] = dmin;
      if (!any) s_bad = 1;  // (benign race: every writer stores 1)
    }
    __syncthreads();
    if (s_bad) continue;  // some stage fits no pool (uniform)
    if (t == 0) {  // what lies behind stage i, accumulated from the last stage backwards
      T.S[0][P - 1] = T.S[1][P - 1] = T.S[2][P - 1] = T.S[3][P - 1] = T.S[4][P - 1] = 0.0;
      for (int i = P - 2; i >= 0; --i) {
        T.S[0][i] = T.S[0][i + 1] + T.smin[0][i + 1];
        T.S[1][i] = fmax(T.S[1][i + 1], T.smin[0][i + 1]);
        T.S[2][i] = fmax(T.S[2][i + 1], T.smin[1][i + 1]);
        T.S[3][i] = fmax(T.S[3][i + 1], T.smin[2][i + 1]);
        T.S[4][i] = T.S[4][i + 1] + T.smin[3][i + 1];
      }
    }
    int n_cur = 1;  // frontier length; level 0 extends one empty placement
    bool truncated = false;
    for (int j = 0; j < P; ++j) {  // place stage j (uniform loop)
      uint8_t *const cur = (j & 1) ? buf1 : buf0, *const nxt = (j & 1) ? buf0 : buf1;
      __syncthreads();
      // the level's tables: stage j on every type / zone
      if (STP) {
        if (t < G * TP) {  // (type g, TP index k)
          const int g = t / TP, k = t - g * TP, tpk = pl.tpv[k];
          const uint64_t params = pl.st_params[rs + j];
          const uint64_t bytes = stage_bytes_of(params, pl.st_n[rs + j], pl.bpp, j, P, tpk, nb, pl.act[im * TP + k]);
          T.l_c3[g][k] = pl.st_c[(((size_t)(rs + j) * G + g) * MB + im) * TP + k];
          T.l_upd3[g][k] = pl.st_u[((size_t)(rs + j) * G + g) * TP + k];
          T.l_dol3[g][k] = (double)(D * tpk) * pl.price[g];
          if (k == 0) T.l_price[g] = pl.price[g];
          s_fit3[g][k] = (bytes + pl.res[g] <= pl.cap[g] && tpk <= pl.node[g]) ? 1 : 0;
        } else if (t >= 128 && t < 128 + Z * TP) {  // (zone z, TP index k)
          const int z = (t - 128) / TP, k = (t - 128) - z * TP, tpk = pl.tpv[k];
          const uint64_t params = pl.st_params[rs + j];
          const uint64_t shard = (params + (uint64_t)tpk - 1) / (uint64_t)tpk;
          double sync = 0.0, ring = 0.0;
          if (D > 1) {
            const double grad = (double)shard * (double)pl.gb;
            sync = 2.0 * (double)(D - 1) / (double)D * grad / pl.bw[z * Z + z];
            ring = 2.0 * (double)(D - 1) / (double)D * grad;
          }
          T.l_sync3[z][k] = sync;
          if (z == 0) T.l_ring3[k] = ring;
        }
        __syncthreads();
        if (t < TP) {
          uint32_t m = 0;
          for (int g = 0; g < G; ++g) m |= (uint32_t)s_fit3[g][t] << g;
          T.l_fit3[t] = m;
        }
      } else if (t < G) {
        const uint64_t params = pl.st_params[rs + j];
        const uint64_t bytes = stage_bytes_of(params, pl.st_n[rs + j], pl.bpp, j, P, tp, nb, pl.act[im * TP + it]);
        T.l_c[t] = pl.st_c[(((size_t)(rs + j) * G + t) * MB + im) * TP + it];
        T.l_upd[t] = pl.st_u[((size_t)(rs + j) * G + t) * TP + it];
        T.l_dol[t] = (double)(D * tp) * pl.price[t];
        T.l_price[t] = pl.price[t];
        const bool fits = bytes + pl.res[t] <= pl.cap[t] && tp <= pl.node[t];
        const unsigned long long m = __builtin_amdgcn_ballot_w64(fits);
        if (t == 0) T.l_fit = (uint32_t)m;
      } else if (t >= 64 && t < 64 + Z) {
        const int z = t - 64;
        const uint64_t params = pl.st_params[rs + j];
        const uint64_t shard = (params + (uint64_t)tp - 1) / (uint64_t)tp;
        double sync = 0.0, ring = 0.0;
        if (D > 1) {
          const double grad = (double)shard * (double)pl.gb;
          sync = 2.0 * (double)(D - 1) / (double)D * grad / pl.bw[z * Z + z];
          ring = 2.0 * (double)(D - 1) / (double)D * grad;
        }
        T.l_sync[z] = sync;
        if (z == 0) T.l_ring = ring;
      }
      if (t == 0) s_nbuf = 0;
      __syncthreads();
      const bool last = j == P - 1;
      const int n_total = n_cur * NCH;
      unsigned long long best_k = ~0ull;  // last level: this thread's smallest (key, id)
      uint32_t best_i = ~0u;
      uint32_t my_expanded = 0;
      for (int row = 0; row * kSearchThreads < n_total; ++row) {  // uniform
        const int cand = row * kSearchThreads + t;
        bool keep = false;
        unsigned long long kbits = 0;
        if (cand < n_total) {
          const int r = cand / NCH, c = cand - r * NCH;
          int pa, pb, pk;
          choice(c, it, pa, pb, pk);
          const SState *par = j == 0 ? nullptr : reinterpret_cast<const SState *>(cur + (size_t)r * a.state_stride);
          SAcc o;
          int runs;
          if (search_step<MODE>(T, par, j, pa, pb, pk, G, a.max_runs, o, runs)) {
            my_expanded += 1;
            const SBound b = search_bound_of<MODE>(T, o, j, nbm1);
            const double key = a.objective == 0 ? b.T : b.C;
            bool drop = false;
            if (a.has_bound) drop = a.objective == 0 ? b.C > a.bound : 1.0 / b.T < a.bound;
            if (a.has_inc && key > a.inc) drop = true;
            keep = !drop;
            kbits = (unsigned long long)__double_as_longlong(key);  // non-negative: orders like the value
          }
        }
        if (last) {
          if (keep && key_id_less(kbits, (uint32_t)cand, best_k, best_i)) { best_k = kbits; best_i = (uint32_t)cand; }
          continue;
        }
        // append the row's survivors in candidate order
        const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
        if (lane == 0) s_wave[wv] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t before = 0, row_total = 0;
        for (int w = 0; w < kSearchThreads / 64; ++w) {
          if (w < wv) before += s_wave[w];
          row_total += s_wave[w];
        }
        int nbuf = s_nbuf;
        if (nbuf + (int)row_total > kSearchBuf) {  // uniform: make room, only the W smallest can matter
          __syncthreads();
          search_sort(b_key, b_id, nbuf);
          nbuf = min(nbuf, a.W);
          truncated = true;
        }
        if (keep) {
          const int at = nbuf + (int)before + __popcll(m & ((1ull << lane) - 1ull));
          b_key[at] = kbits;
          b_id[at] = (uint32_t)cand;
        }
        __syncthreads();
        if (t == 0) s_nbuf = nbuf + (int)row_total;
        __syncthreads();
      }
      atomicAdd(&s_expanded, (unsigned long long)my_expanded);
      if (last) {
        // the smallest (key, id) of the workgroup
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
          const unsigned long long ok2 = __shfl_xor(best_k, off);
          const uint32_t oi = __shfl_xor(best_i, off);
          if (key_id_less(ok2, oi, best_k, best_i)) { best_k = ok2; best_i = oi; }
        }
        if (lane == 0) { s_bk[wv] = best_k; s_bi[wv] = best_i; }
        __syncthreads();
        best_k = s_bk[0]; best_i = s_bi[0];
        for (int w = 1; w < kSearchThreads / 64; ++w)
          if (key_id_less(s_bk[w], s_bi[w], best_k, best_i)) { best_k = s_bk[w]; best_i = s_bi[w]; }
        if (best_i != ~0u) {  // uniform
          const int r = (int)best_i / NCH, c = (int)best_i - r * NCH;
          int pa, pb, pk;
          choice(c, it, pa, pb, pk);
          const uint8_t *par_path = cur + (size_t)r * a.state_stride + kStateBytes;
          for (int i = t; i < P - 1; i += blockDim.x) {
            res->pools[i] = par_path[i];
            res->pools_b[i] = SPLIT ? par_path[a.path_stride + i] : par_path[i];
            res->tps[i] = STP ? par_path[2 * a.path_stride + i] : it;
          }
          if (t == 0) {
            const SState *par = j == 0 ? nullptr : reinterpret_cast<const SState *>(cur + (size_t)r * a.state_stride);
            SAcc o;
            int runs;
            search_step<MODE>(T, par, j, pa, pb, pk, G, a.max_runs, o, runs);
            const SBound b = search_bound_of<MODE>(T, o, j, nbm1);
            res->pools[P - 1] = pa;
            res->pools_b[P - 1] = pb;
            res->tps[P - 1] = pk;
            if (STP) res->desc[2] = P > 1 ? (int)par_path[2 * a.path_stride] : pk;  // stage 0's
            res->T = b.T;
            res->C = b.C;
            res->key = a.objective == 0 ? b.T : b.C;
            res->found = 1;
          }
        }
        break;
      }
      __syncthreads();
      int n_next = s_nbuf;
      if (n_next > a.W) {  // uniform: keep the W smallest bounds, in that order
        search_sort(b_key, b_id, n_next);
        n_next = a.W;
        truncated = true;
      }
      if (n_next == 0) break;  // uniform
      // write the next frontier
      for (int k = t; k < n_next; k += blockDim.x) {
        const int cand = (int)b_id[k];
        const int r = cand / NCH, c = cand - r * NCH;
        int pa, pb, pk;
        choice(c, it, pa, pb, pk);
        uint8_t *const out = nxt + (size_t)k * a.state_stride;
        const SState *par = j == 0 ? nullptr : reinterpret_cast<const SState *>(cur + (size_t)r * a.state_stride);
        SAcc o;
        int runs;
        search_step<MODE>(T, par, j, pa, pb, pk, G, a.max_runs, o, runs);
        SState st;
        if (par) {
          st = *par;
          const uint8_t *par_path = cur + (size_t)r * a.state_stride + kStateBytes;
          for (int i = 0; i < j; ++i) {
            out[kStateBytes + i] = par_path[i];
            if (SPLIT) out[kStateBytes + a.path_stride + i] = par_path[a.path_stride + i];
            if (STP) out[kStateBytes + 2 * a.path_stride + i] = par_path[2 * a.path_stride + i];
          }
        } else {
          for (int x = 0; x < kSearchMaxPools; ++x) st.cnt[x] = 0;
        }
        st.sum = o.sum; st.maxt = o.maxt; st.c_open = o.c_open; st.xb_open = o.xb_open;
        st.sum_b = o.sum_b; st.maxt_b = o.maxt_b; st.c_open_b = o.c_open_b; st.xb_open_b = o.xb_open_b;
        st.msync = o.msync; st.mupd = o.mupd; st.dol = o.dol; st.comm = o.comm;
        if (BOTH) {
          st.cnt[pa] = (uint16_t)(st.cnt[pa] + T.tpv[pk]);
          st.cnt[pb] = (uint16_t)(st.cnt[pb] + T.tpv[pk]);
        } else if (STP) {
          st.cnt[pa] = (uint16_t)(st.cnt[pa] + T.tpv[pk]);
        } else if (!SPLIT) {
          st.cnt[pa] = (uint16_t)(st.cnt[pa] + 1);
        } else {
          st.cnt[pa] = (uint16_t)(st.cnt[pa] + 1);
          st.cnt[pb] = (uint16_t)(st.cnt[pb] + 1);
        }
        st.pool = (uint8_t)pa;
        st.pool_b = (uint8_t)pb;
        st.tpi = (uint8_t)pk;
        st.runs = (uint8_t)runs;
        for (int x = 0; x < 4; ++x) st.pad[x] = 0;
        *reinterpret_cast<SState *>(out) = st;
        out[kStateBytes + j] = (uint8_t)pa;
        if (SPLIT) out[kStateBytes + a.path_stride + j] = (uint8_t)pb;
        if (STP) out[kStateBytes + 2 * a.path_stride + j] = (uint8_t)pk;
      }
      n_cur = n_next;
    }
    __syncthreads();
    if (t == 0) {
      res->truncated = truncated ? 1u : 0u;
      res->expanded = s_expanded;
    }
  }
}

// Smallest (key, sub-problem) over the sub-problems' winners; also the totals.
__global__ __launch_bounds__(256) void k_search_pick(const SubResult *results, uint32_t n_sub, SubResult *out) {
  __shared__ unsigned long long s_k[4], s_e[4];
  __shared__ uint32_t s_i[4], s_t[4];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  unsigned long long bk = ~0ull, expanded = 0;
  uint32_t bi = ~0u, trunc = 0;
  for (uint32_t i = t; i < n_sub; i += blockDim.x) {
    const SubResult &r = results[i];
    expanded += r.expanded;
    trunc |= r.truncated;
    if (r.found) {
      const unsigned long long k = (unsigned long long)__double_as_longlong(r.key);
      if (key_id_less(k, i, bk, bi)) { bk = k; bi = i; }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned long long ok = __shfl_xor(bk, off);
    const uint32_t oi = __shfl_xor(bi, off);
    if (key_id_less(ok, oi, bk, bi)) { bk = ok; bi = oi; }
    expanded += __shfl_xor(expanded, off);
    trunc |= __shfl_xor(trunc, off);
  }
  if (lane == 0) { s_k[wv] = bk; s_i[wv] = bi; s_e[wv] = expanded; s_t[wv] = trunc; }
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < 4; ++w) {
      if (key_id_less(s_k[w], s_i[w], bk, bi)) { bk = s_k[w]; bi = s_i[w]; }
      expanded += s_e[w];
      trunc |= s_t[w];
    }
    s_i[0] = bi; s_e[0] = expanded; s_t[0] = trunc;
  }
  __syncthreads();
  bi = s_i[0];
  if (bi == ~0u) {
    if (t == 0) { out->found = 0; out->truncated = s_t[0]; out->expanded = s_e[0]; out->P = 0; }
    return;
  }
  const unsigned long long *src = reinterpret_cast<const unsigned long long *>(results + bi);
  unsigned long long *dst = reinterpret_cast<unsigned long long *>(out);
  for (uint32_t w = t; w < sizeof(SubResult) / 8; w += blockDim.x) dst[w] = src[w];
  __syncthreads();
  if (t == 0) { out->truncated = s_t[0]; out->expanded = s_e[0]; }
}

// ------------------------------------------------------------------ listed placements

// The problem's small tables in LDS: every stage of every listed plan reads a dozen of these
// words, at addresses that differ from lane to lane.  They are laid out once per plan in device
// memory (k_list_tables), so that a workgroup copies them in one go -- a dozen loops, one per
// table, cost a trip to memory each, 5 us in front of every workgroup.
struct ListTables {
  double *xsec;      // [MB][Z][Z] seconds of one activation transfer
  double *bw;        // [Z][Z]
  double *egress;    // [Z][Z] (zeros without egress prices)
  double *price;     // [G]
  double *ring;      // [DP] 2 (D - 1) / D
  double *tpd;       // [TP]
  uint64_t *cap, *res;  // [G]
  uint64_t *act;     // [MB][TP]
  int32_t *nb;       // [MB][DP]
  int32_t *dpv, *tpv, *node;  // [DP], [TP], [G]
  uint32_t *zg;      // [ZGr] zone | type << 8 of a pool
  int32_t *avail;    // [ZGr] (not part of the copy: it changes between calls)
};

__host__ __device__ inline size_t list_copy_words(const DevPlan &pl) {  // 8-byte words laid out in memory
  const size_t ints = (size_t)pl.MB * pl.DP + pl.DP + pl.TP + pl.G + pl.ZGr;
  return (size_t)pl.MB * pl.Z * pl.Z + 2 * (size_t)pl.Z * pl.Z + 3 * (size_t)pl.G + pl.DP + pl.TP +
         (size_t)pl.MB * pl.TP + (ints + 1) / 2;
}
__host__ __device__ inline size_t list_tables_words(const DevPlan &pl) {  // with the availability behind them
  return list_copy_words(pl) + ((size_t)pl.ZGr + 1) / 2;
}

__device__ __forceinline__ ListTables list_tables_at(const DevPlan &pl, double *at) {
  const int G = pl.G, Z = pl.Z, MB = pl.MB, TP = pl.TP, DP = pl.DP;
  ListTables T;
  T.xsec = at;
  T.bw = T.xsec + MB * Z * Z;
  T.egress = T.bw + Z * Z;
  T.price = T.egress + Z * Z;
  T.ring = T.price + G;
  T.tpd = T.ring + DP;
  T.cap = reinterpret_cast<uint64_t *>(T.tpd + TP);
  T.res = T.cap + G;
  T.act = T.res + G;
  T.nb = reinterpret_cast<int32_t *>(T.act + MB * TP);
  T.dpv = T.nb + MB * DP;
  T.tpv = T.dpv + DP;
  T.node = T.tpv + TP;
  T.zg = reinterpret_cast<uint32_t *>(T.node + G);
  T.avail = reinterpret_cast<int32_t *>(at + list_copy_words(pl));
  return T;
}

// Lays the tables out in device memory (once per plan).
__global__ void k_list_tables(DevPlan pl) {
  const int G = pl.G, Z = pl.Z, MB = pl.MB, TP = pl.TP, DP = pl.DP;
  const ListTables T = list_tables_at(pl, pl.list_tables);
  const int t = threadIdx.x, nt = blockDim.x;
  for (int i = t; i < MB * Z * Z; i += nt) T.xsec[i] = pl.xsec[i];
  for (int i = t; i < Z * Z; i += nt) {
    T.bw[i] = pl.bw[i];
    T.egress[i] = pl.egress ? pl.egress[i] : 0.0;
  }
  for (int i = t; i < G; i += nt) {
    T.price[i] = pl.price[i];
    T.cap[i] = pl.cap[i];
    T.res[i] = pl.res[i];
    T.node[i] = pl.node[i];
  }
  for (int i = t; i < DP; i += nt) {
    const double D = (double)pl.vals[i];
    T.ring[i] = 2.0 * (D - 1.0) / D;
    T.dpv[i] = pl.vals[i];
  }
  for (int i = t; i < TP; i += nt) {
    T.tpv[i] = pl.vals[DP + i];
    T.tpd[i] = (double)pl.vals[DP + i];
  }
  for (int i = t; i < MB * TP; i += nt) T.act[i] = pl.act[i];
  for (int i = t; i < MB * DP; i += nt) T.nb[i] = pl.nb[i];
  for (int i = t; i < pl.ZGr; i += nt) T.zg[i] = (uint32_t)(i / G) | (uint32_t)(i % G) << 8;
}

// Needs a barrier before the tables are read.
__device__ __forceinline__ ListTables stage_list_tables(const DevPlan &pl, double *lds) {
  const ListTables T = list_tables_at(pl, lds);
  const int t = threadIdx.x, nt = blockDim.x, n = (int)list_copy_words(pl);
  int32_t avail = 0;
  if (t < pl.ZGr) avail = pl.avail[t];  // (at most 64 pools)
  for (int i = t; i < n; i += 4 * nt) {  // four loads in flight
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = i + q * nt < n ? pl.list_tables[i + q * nt] : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q * nt < n) lds[i + q * nt] = v[q];
  }
  if (t < pl.ZGr) T.avail[t] = avail;
  return T;
}

// the bandwidth a gradient buffer sees between two zones
__device__ __forceinline__ double list_link(const DevPlan &pl, const ListTables &T, int za, int zb, double bytes) {
  return pl.n_bw_coef > 0 ? link_bw(pl, za, zb, bytes) : T.bw[mul24(za, pl.Z) + zb];
}

// activation bytes of a worker: microbatches in flight x layers x bytes of one (validated < 2^62)
__device__ __forceinline__ uint64_t act_bytes(int in_flight, int layers, uint64_t act) {
  return (uint64_t)(uint32_t)in_flight * (uint32_t)layers * act;
}

struct PlaceArgs {
  uint64_t count;
  const int32_t *desc;    // [count][5] pp index, partition, tp index, dp index, mb index
  const int32_t *pools;   // [count][pool_stride] pool of every stage
  const int32_t *pools_b; // SPLIT, same shape: pool of the other half of every stage's replicas
  const int32_t *tps;     // optional, same shape: TP index of every stage (else the descriptor's)
  uint32_t pool_stride;
  uint32_t per_wg;        // plans a workgroup takes, at most kPlaceMaxPlans
  const SearchPP *pps;
  int n_pp;
  int objective, has_bound;
  double bound;
  double *T, *C;
  uint64_t *mem;
  uint32_t *mask;
};

constexpr int kPlaceThreads = 256;
constexpr int kPlaceStages = 512;    // stages a workgroup holds at a time
constexpr int kPlaceMaxPlans = 64;    // a lane each when the stages are added up
static_assert(kPlaceStages >= kMaxStages, "one plan's stages fit");

struct PlacePlan {       // a plan as its stages need it
  uint32_t rs;
  int32_t end;           // stages of the workgroup's plans up to and including this one
  int16_t P;             // 0: an invalid descriptor
  uint8_t it, id, im, pad[3];
  double dpd, half_traffic;  // D; N_b x (replicas of one kind of pipeline) x bytes of a transfer
};
static_assert(sizeof(PlacePlan) == 32, "two 16-byte reads");

struct PlaceLds {
  // what the stages contribute, in plan and stage order (four entries more than there are
  // stages: the sums read four at a time): time in the two kinds of pipeline, rent, traffic
  double term[4][kPlaceStages + 4];
  double sum[4][kPlaceMaxPlans], slowest[2][kPlaceMaxPlans];   // what they add up to
  long long sync[kPlaceMaxPlans], upd[kPlaceMaxPlans];  // bits of the maxima (non-negative values, in
                                                        // which order the bits compare like them)
  unsigned long long peak[kPlaceMaxPlans];
  PlacePlan plan[kPlaceMaxPlans];
  uint32_t flags[kPlaceMaxPlans];  // mask bits 0, 1, 3; bit 31: an index out of range
  uint8_t owner[kPlaceStages];     // the stage's plan
};

__host__ __device__ inline size_t place_lds_bytes(const DevPlan &pl, uint32_t per_wg) {
  return sizeof(PlaceLds) + list_tables_words(pl) * 8 + (size_t)per_wg * pl.ZGr * sizeof(int32_t);
}

// Sum (and maximum) over a plan's stages in stage order, for a lane per plan.
__device__ __forceinline__ void place_sum(const double *v, int P, double &sum, double &slowest) {
  sum = 0.0;
  slowest = 0.0;
  int i = 0;
  for (; i + 4 <= P; i += 4) {
    const double x0 = v[i], x1 = v[i + 1], x2 = v[i + 2], x3 = v[i + 3];
    sum += x0; sum += x1; sum += x2; sum += x3;
    slowest = fmax(fmax(slowest, fmax(x0, x1)), fmax(x2, x3));
  }
  for (; i < P; ++i) {
    const double x = v[i];
    sum += x;
    slowest = fmax(slowest, x);
  }
}

// The simulator (Sec. 4.3) for plans whose stages choose their pools freely.
//
// With SPLIT a stage's D replicas lie on two pools, half on each, also across zones (the D tuples
// of a stage, Sec. 4.2): the replicas on the first pools and those on the second pools form two
// kinds of pipeline; T_iter takes the slower kind (Sec. 4.3: max over pipelines), a split stage's
// all-reduce runs over the slowest link of a ring through both pools, and the traffic between
// zones -- of the pipelines, each kind carrying half of the replicas, and of the ring -- is paid
// for.  With a TP index per stage every per-stage quantity (memory shard, activation bytes,
// profiled times, node size, gradient shard, GPUs against the quota, rent) uses the stage's own
// degree.  A descriptor, pool or TP index out of range yields mask = 0xFFFFFFFF, T = C = +inf, mem = 0.
//
// A workgroup takes per_wg plans and works through their stages, up to 1 024 at a time, plans
// one behind the other without gaps: first a lane per stage -- what is added up in stage order,
// which is part of the definition, goes to LDS, maxima are folded in there -- then a lane per
// plan adds its stages up, a wave per quantity.  A wave per plan leaves most lanes idle where
// pipelines are shorter than 64 stages, and walks every plan's sums by itself: 200 003 plans of 1
// to 48 stages with two pools and a degree per stage took 488 us that way and take 85 us this way
// (vector instructions 35 us of it; the rest is the latency of a workgroup's chain: descriptors,
// pools, stage records, sums).  Measured beside it: requesting two stages' words per lane at a time
// (98 us, the registers cost a workgroup per compute unit), 512 threads (100 us), bounds on the
// registers for more waves (113 us and more).
template <bool SPLIT>
__global__ __launch_bounds__(kPlaceThreads) void k_eval_placements(DevPlan pl, PlaceArgs a) {
  extern __shared__ double place_lds[];
  PlaceLds &S = *reinterpret_cast<PlaceLds *>(place_lds);
  double *const tables = reinterpret_cast<double *>(&S + 1);
  int32_t *const cnt = reinterpret_cast<int32_t *>(tables + list_tables_words(pl));  // [plan][ZG]
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t G = pl.G, Z = pl.Z, ZG = pl.ZGr, MB = pl.MB, TP = pl.TP, DP = pl.DP;
  const uint32_t row_words = mul24(mul24(MB, TP), pl.row_w);  // of a stage's records
  const uint64_t c0 = (uint64_t)blockIdx.x * a.per_wg;
  const int n = (int)min((uint64_t)a.per_wg, a.count - c0);
  if (wv == 0) {  // a lane per plan
    PlacePlan p{};
    if (lane < n) {
      const int32_t *d = a.desc + (c0 + lane) * 5;
      const int ip = d[0], q = d[1], it = d[2], id = d[3], im = d[4];
      if (ip >= 0 && ip < a.n_pp && it >= 0 && it < (int)TP && id >= 0 && id < (int)DP && im >= 0 && im < (int)MB && q >= 0) {
        const SearchPP pp = a.pps[ip];
        if (q < pp.n_part && (uint32_t)pp.P <= a.pool_stride) {
          p.P = (int16_t)pp.P;
          p.rs = pp.rs0 + (uint32_t)q * (uint32_t)pp.P;
          p.it = (uint8_t)it; p.id = (uint8_t)id; p.im = (uint8_t)im;
          p.dpd = (double)pl.vals[id];
          p.half_traffic = (double)pl.nb[im * DP + id] * (SPLIT ? 0.5 * p.dpd : p.dpd) * (double)pl.p2p[im];
        }
      }
    }
    int end = p.P;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(end, off);
      if (lane >= off) end += v;
    }
    p.end = end;
    S.plan[lane] = p;
    S.sync[lane] = S.upd[lane] = 0;
    S.peak[lane] = 0;
    S.flags[lane] = 0;
  }
  for (int x = t; x < (int)(a.per_wg * ZG); x += kPlaceThreads) cnt[x] = 0;
  const ListTables L = stage_list_tables(pl, tables);
  __syncthreads();
  for (int s0 = 0; s0 < n;) {  // uniform: plans s0 .. s1 - 1 make up one pass
    const int base = s0 ? S.plan[s0 - 1].end : 0;
    const int s1 = s0 + __popcll(__builtin_amdgcn_ballot_w64(lane >= s0 && lane < n && S.plan[lane].end - base <= kPlaceStages));
    const int stages = S.plan[s1 - 1].end - base;
    if (lane >= s0 && lane < s1) {  // whose stage is whose: a lane per plan, the waves take turns
      const int P = S.plan[lane].P, at = S.plan[lane].end - P - base;
      for (int i = wv; i < P; i += kPlaceThreads / 64) S.owner[at + i] = (uint8_t)lane;
    }
    __syncthreads();
    for (int e = t; e < stages; e += kPlaceThreads) {
      const uint32_t own = S.owner[e];
      const PlacePlan pn = S.plan[own];
      const int P = pn.P, i = e - (pn.end - P - base);
      const size_t row = (c0 + own) * a.pool_stride + (uint32_t)i;
      const int32_t *pa = a.pools + row, *pb = SPLIT ? a.pools_b + row : pa;
      const int fwd = i < P - 1 ? 1 : 0, back = i > 0 ? -1 : 0;
      const uint32_t ra = (uint32_t)pa[0], ran = (uint32_t)pa[fwd], rap = (uint32_t)pa[back];
      const uint32_t rb = (uint32_t)pb[0], rbn = (uint32_t)pb[fwd], rbp = (uint32_t)pb[back];
      const uint32_t rt = a.tps ? (uint32_t)a.tps[row] : pn.it;
      // (indices out of range: reported by the stage they belong to, kept in bounds everywhere)
      const uint32_t a0 = min(ra, ZG - 1), b0 = min(rb, ZG - 1), ti = min(rt, TP - 1);
      const uint32_t zga = L.zg[a0], za = zga & 255u, ga = zga >> 8;
      const uint32_t zgb = SPLIT ? L.zg[b0] : zga, zb = zgb & 255u, gb = zgb >> 8;
      const uint64_t si = (uint64_t)pn.rs + (uint32_t)i;
      const uint32_t mt = mul24(pn.im, TP) + ti;
      const double *row_st = pl.st_row + si * row_words + mul24(mt, pl.row_w);  // the stage's record
      const int layers = pl.st_n[si];
      const double ca = row_st[ga], ua = row_st[G + ga];
      const double cb = SPLIT ? row_st[gb] : 0.0, ub = SPLIT ? row_st[G + gb] : 0.0;
      const uint64_t model = (uint64_t)__double_as_longlong(row_st[2 * G]);
      const double grad = row_st[2 * G + 1];
      const int tp = L.tpv[ti], nb = L.nb[mul24(pn.im, DP) + pn.id];
      atomicAdd(&cnt[mul24(own, ZG) + a0], tp);  // GPUs of one replica (split: counted once per half)
      if (SPLIT) atomicAdd(&cnt[mul24(own, ZG) + b0], tp);
      const uint64_t bytes = model + act_bytes(min(P - i, nb), layers, L.act[mt]);
      const uint64_t m1 = bytes + L.res[ga], m2 = SPLIT ? bytes + L.res[gb] : m1;
      uint32_t flags = (m1 > L.cap[ga] || (SPLIT && m2 > L.cap[gb])) ? 1u : 0u;
      if (tp > L.node[ga] || (SPLIT && tp > L.node[gb])) flags |= 8u;
      if (SPLIT && a0 != b0 && (L.dpv[pn.id] & 1)) flags |= 2u;  // D replicas cannot be halved
      if (ra >= ZG || (SPLIT && rb >= ZG) || rt >= TP) flags |= 1u << 31;
      const double *xsec = L.xsec + mul24(pn.im, mul24(Z, Z));
      double xa = 0.0, xb = 0.0, traffic = 0.0;
      if (fwd) {
        const uint32_t zna = L.zg[min(ran, ZG - 1)] & 255u;
        xa += xsec[mul24(za, Z) + zna];
        // (each kind of pipeline carries half of the replicas)
        if (zna != za) traffic += pn.half_traffic * (L.egress[mul24(za, Z) + zna] + L.egress[mul24(zna, Z) + za]);
        if (SPLIT) {
          const uint32_t znb = L.zg[min(rbn, ZG - 1)] & 255u;
          xb += xsec[mul24(zb, Z) + znb];
          if (znb != zb) traffic += pn.half_traffic * (L.egress[mul24(zb, Z) + znb] + L.egress[mul24(znb, Z) + zb]);
        }
      }
      if (back) {
        xa += xsec[mul24(za, Z) + (L.zg[min(rap, ZG - 1)] & 255u)];
        if (SPLIT) xb += xsec[mul24(zb, Z) + (L.zg[min(rbp, ZG - 1)] & 255u)];
      }
      double sync = 0.0;
      if (pn.dpd > 1.0) {
        double link = list_link(pl, L, za, za, grad);
        if (SPLIT && zb != za)
          link = fmin(fmin(link, list_link(pl, L, zb, zb, grad)),
                      fmin(list_link(pl, L, za, zb, grad), list_link(pl, L, zb, za, grad)));
        const double ring_bytes = L.ring[pn.id] * grad;
        sync = ring_bytes / link;
        if (SPLIT && zb != za) traffic += ring_bytes * (L.egress[mul24(za, Z) + zb] + L.egress[mul24(zb, Z) + za]);
      }
      S.term[0][e] = ca + xa;
      if (SPLIT) S.term[1][e] = cb + xb;
      const double gpus = pn.dpd * L.tpd[ti];  // (whole numbers below 2^53)
      S.term[2][e] = gpus * (SPLIT ? 0.5 * (L.price[ga] + L.price[gb]) : L.price[ga]);
      S.term[3][e] = traffic;
      atomicMax(&S.sync[own], (long long)__double_as_longlong(sync));
      atomicMax(&S.upd[own], (long long)__double_as_longlong(SPLIT ? fmax(ua, ub) : ua));
      atomicMax(&S.peak[own], (unsigned long long)(m1 > m2 ? m1 : m2));
      if (flags) atomicOr(&S.flags[own], flags);
    }
    __syncthreads();
    const int p = s0 + lane;
    if (wv < 4) {  // a lane per plan, a wave per quantity
      if (p < s1 && (SPLIT || wv != 1)) {
        const PlacePlan pn = S.plan[p];
        double sum, slowest;
        place_sum(S.term[wv] + (pn.end - pn.P - base), pn.P, sum, slowest);
        S.sum[wv][p] = sum;
        if (wv < 2) S.slowest[wv][p] = slowest;
      }
    }
    for (int x = t; x < (int)mul24(s1 - s0, ZG); x += kPlaceThreads) {  // every pool holds what is placed on it
      const int q = (int)((uint32_t)x / ZG), pool = x - (int)mul24(q, ZG);
      if ((int64_t)cnt[mul24(s0 + q, ZG) + pool] * L.dpv[S.plan[s0 + q].id] > (SPLIT ? 2 : 1) * (int64_t)L.avail[pool])
        atomicOr(&S.flags[s0 + q], 2u);
    }
    __syncthreads();
    if (wv == 0 && p < s1) {
      double T = __builtin_huge_val(), C = T;
      uint64_t peak = 0;
      uint32_t mask = 0xFFFFFFFFu;
      const PlacePlan pn = S.plan[p];
      if (pn.P != 0 && !(S.flags[p] >> 31)) {
        const int nb = L.nb[pn.im * DP + pn.id];
        if (nb == 0) {
          mask = 4u;
        } else {
          mask = S.flags[p];
          peak = S.peak[p];
          double t_pp = S.sum[0][p] + (double)(nb - 1) * S.slowest[0][p];
          if (SPLIT) t_pp = fmax(t_pp, S.sum[1][p] + (double)(nb - 1) * S.slowest[1][p]);
          T = (t_pp + __longlong_as_double(S.sync[p])) + __longlong_as_double(S.upd[p]);
          C = S.sum[2][p] / 3600.0 * T + S.sum[3][p];
          if (a.has_bound) {
            if (a.objective == 0) { if (C > a.bound) mask |= 32u; }
            else if (1.0 / T < a.bound) mask |= 32u;
          }
        }
      }
      if (a.T) a.T[c0 + p] = T;
      if (a.C) a.C[c0 + p] = C;
      if (a.mem) a.mem[c0 + p] = peak;
      if (a.mask) a.mask[c0 + p] = mask;
    }
    s0 = s1;
  }
}

// ------------------------------------------------------------------ a pool per replica

constexpr int64_t kReplicaMaxDegree = 65536;  // replicas per stage a listed plan may name one by one
constexpr int kReplicaWaves = 4;
constexpr int kReplicaTile = 512;            // stage times a wave keeps in LDS at a time
constexpr int kReplicaShared = 512;           // plans with more (stage, replica) pairs are shared by the waves
static_assert(kReplicaTile >= kMaxStages, "a pipeline's stages fit");

struct ReplicaArgs {
  uint64_t count;
  const int32_t *desc;    // [count][5] pp index, partition, tp index, dp index, mb index
  const int32_t *pools;   // [count][stride]: the pool of replica r of stage i at i * D + r
  uint64_t stride;
  const int32_t *tps;     // optional, [count][tps_stride]: TP index of every stage (else the descriptor's)
  uint32_t tps_stride;
  const SearchPP *pps;
  int n_pp;
  int objective, has_bound;
  double bound;
  double *T, *C;
  uint64_t *mem;
  uint32_t *mask;
};

struct ReplicaPlan {     // a valid descriptor; P = 0: an invalid one
  int32_t P, D, it, id, im;
  uint32_t rs;
};

struct ReplicaSums {     // of a lane, a wave or a plan
  double t_pipe, t_upd, t_sync, rent, traffic;
  uint64_t peak;
  uint32_t flags;        // mask bits 0, 3; bit 31: an index out of range
  uint32_t pad;
};

struct ReplicaLds {
  double times[kReplicaWaves][kReplicaTile];
  ReplicaPlan plan[kReplicaWaves];
  ReplicaSums part[kReplicaWaves];
};

__host__ __device__ inline size_t replica_lds_bytes(const DevPlan &pl) {
  return sizeof(ReplicaLds) + list_tables_words(pl) * 8 + kReplicaWaves * (size_t)pl.ZGr * sizeof(int32_t);
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// makes a wave's LDS writes visible to its own later reads (operations of one wave complete in
// order; the compiler must not move them)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A plan's (stage, replica) pairs and pipelines, shared by THREADS threads (a wave, or the
// workgroup; tid: which one this is); what this thread's share adds up to.
template <int THREADS>
__device__ __forceinline__ ReplicaSums replica_pairs(const DevPlan &pl, const ReplicaArgs &a, const ListTables &L,
                                                     const ReplicaPlan &pn, uint64_t ci, int tid, double *times,
                                                     int32_t *cnt) {
  const uint32_t G = pl.G, Z = pl.Z, ZG = pl.ZGr, MB = pl.MB, TP = pl.TP, DP = pl.DP;
  const int P = pn.P, D = pn.D, im = pn.im;
  const int32_t *const pools = a.pools + ci * a.stride;
  const int32_t *const tps = a.tps ? a.tps + ci * a.tps_stride : nullptr;
  const int nb = L.nb[mul24(im, DP) + pn.id];
  const double one_traffic = (double)nb * (double)pl.p2p[im], ring = L.ring[pn.id];
  const double *xsec = L.xsec + mul24(im, mul24(Z, Z));
  const uint32_t row_words = mul24(mul24(MB, TP), pl.row_w);  // of a stage's records
  ReplicaSums s{};
  const int tile = min(D, kReplicaTile * (THREADS / 64) / P);
  for (int r0 = 0; r0 < D; r0 += tile) {  // uniform
    const int rt = min(tile, D - r0), n = P * rt;
    const uint32_t mg = rt == 1 ? 0u : (uint32_t)(((1ull << 32) + (uint32_t)rt - 1) / (uint32_t)rt);
    for (int e = tid; e < n; e += THREADS) {
      const int i = (int)fast_div((uint32_t)e, mg), r = r0 + e - i * rt;
      const int k = i * D + r;  // (P x D <= 2^24)
      uint32_t p = (uint32_t)pools[k], pf = (uint32_t)pools[i < P - 1 ? k + D : k],
               pv = (uint32_t)pools[i > 0 ? k - D : k],
               ps = (uint32_t)pools[r + 1 == D ? k + 1 - D : k + 1],  // the ring's next replica
               ti = (uint32_t)(tps ? tps[i] : pn.it);                 // the stage's TP index
      if (p >= ZG || ti >= TP) s.flags |= 1u << 31;
      // (a neighbour out of range is reported by its own lane; its values only must stay in bounds)
      p = min(p, ZG - 1); pf = min(pf, ZG - 1); pv = min(pv, ZG - 1); ps = min(ps, ZG - 1);
      ti = min(ti, TP - 1);
      const uint32_t zg = L.zg[p], z = zg & 255u, g = zg >> 8;
      const uint32_t zn = L.zg[pf] & 255u, zv = L.zg[pv] & 255u, zs = L.zg[ps] & 255u;
      const uint64_t si = (uint64_t)pn.rs + (uint32_t)i;
      const uint32_t mt = mul24(im, TP) + ti;
      const double *row_st = pl.st_row + si * row_words + mul24(mt, pl.row_w);  // the stage's record
      const int layers = pl.st_n[si];
      const double c = row_st[g];
      s.t_upd = fmax(s.t_upd, row_st[G + g]);
      const uint64_t model = (uint64_t)__double_as_longlong(row_st[2 * G]);
      const double grad = row_st[2 * G + 1];
      const int tp = L.tpv[ti];
      atomicAdd(&cnt[p], tp);  // GPUs the pool gives
      const uint64_t m = model + act_bytes(min(P - i, nb), layers, L.act[mt]) + L.res[g];
      if (m > L.cap[g]) s.flags |= 1u;
      if (tp > L.node[g]) s.flags |= 8u;
      s.peak = m > s.peak ? m : s.peak;
      double x = 0.0;
      if (i < P - 1) {
        x += xsec[mul24(z, Z) + zn];
        if (zn != z)  // one replica's microbatches, both directions
          s.traffic += one_traffic * (L.egress[mul24(z, Z) + zn] + L.egress[mul24(zn, Z) + z]);
      }
      if (i > 0) x += xsec[mul24(z, Z) + zv];
      times[e] = c + x;
      s.rent += L.tpd[ti] * L.price[g];
      if (D > 1) {
        const double ring_bytes = ring * grad;
        s.t_sync = fmax(s.t_sync, ring_bytes / list_link(pl, L, z, zs, grad));
        if (zs != z) s.traffic += ring_bytes * L.egress[mul24(z, Z) + zs];
      }
    }
    if (THREADS == 64) wave_lds_fence();
    else __syncthreads();
    for (int r = tid; r < rt; r += THREADS) {  // the tile's pipelines, in stage order
      double total = 0.0, slowest = 0.0;
      const double *v = times + r;
      int i = 0;
      for (; i + 4 <= P; i += 4, v += 4 * rt) {
        const double x0 = v[0], x1 = v[rt], x2 = v[2 * rt], x3 = v[3 * rt];
        total += x0; total += x1; total += x2; total += x3;
        slowest = fmax(fmax(slowest, fmax(x0, x1)), fmax(x2, x3));
      }
      for (; i < P; ++i, v += rt) { total += *v; slowest = fmax(slowest, *v); }
      s.t_pipe = fmax(s.t_pipe, total + (double)(nb - 1) * slowest);
    }
    if (THREADS == 64) wave_lds_fence();  // the next tile's times come after these reads
    else __syncthreads();
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint64_t o = __shfl_xor((unsigned long long)s.peak, off);
    s.peak = o > s.peak ? o : s.peak;
    s.flags |= __shfl_xor(s.flags, off);
  }
  s.t_pipe = wave_max_f64(s.t_pipe);
  s.t_sync = wave_max_f64(s.t_sync);
  s.t_upd = wave_max_f64(s.t_upd);
  s.rent = wave_sum_f64(s.rent);
  s.traffic = wave_sum_f64(s.traffic);
  return s;
}

// The results of a plan from its sums, by one wave.
__device__ __forceinline__ void replica_write(const ReplicaArgs &a, const ListTables &L, const ReplicaPlan &pn,
                                              const ReplicaSums &s, int DP, int ZG, uint64_t ci, const int32_t *cnt) {
  const int lane = threadIdx.x & 63;
  double T = __builtin_huge_val(), C = T;
  uint64_t peak = 0;
  uint32_t mask = 0xFFFFFFFFu;
  if (pn.P != 0 && !(s.flags >> 31)) {
    if (L.nb[pn.im * DP + pn.id] == 0) {
      mask = 4u;
    } else {
      mask = s.flags;
      peak = s.peak;
      bool over = false;
      for (int p = lane; p < ZG; p += 64)
        if ((int64_t)cnt[p] > (int64_t)L.avail[p]) over = true;
      if (__builtin_amdgcn_ballot_w64(over) != 0) mask |= 2u;
      T = (s.t_pipe + s.t_sync) + s.t_upd;
      C = s.rent / 3600.0 * T + s.traffic;
      if (a.has_bound) {
        if (a.objective == 0) { if (C > a.bound) mask |= 32u; }
        else if (1.0 / T < a.bound) mask |= 32u;
      }
    }
  }
  if (lane == 0) {
    if (a.T) a.T[ci] = T;
    if (a.C) a.C[ci] = C;
    if (a.mem) a.mem[ci] = peak;
    if (a.mask) a.mask[ci] = mask;
  }
}

// The plan tuple in full (Sec. 4.2: D tuples per stage): replica r of all stages is pipeline r,
// T_iter = max over the D pipelines + T_sync + T_update (Sec. 4.3); the all-reduce of a stage is
// a ring through its replicas in their order at the pace of its slowest link; traffic between
// zones is paid for where a pipeline or a ring crosses; a pool's quota counts the GPUs it gives.
// A descriptor or pool out of range, fewer than P x D entries per plan or more than 65 536
// replicas yield mask = 0xFFFFFFFF, T = C = +inf, mem = 0.
//
// Four plans per workgroup.  A lane per (stage, replica) in the order of the list -- neighbouring
// lanes read neighbouring entries -- leaves the stage times in LDS, then a lane per pipeline adds
// its stages up in stage order.  The slowest link of a ring needs no pass of its own:
// bytes / min(link) = max(bytes / link), division being monotone.  A wave takes a plan of up to
// 512 pairs; a larger one, of which one can hold as many pairs as hundreds of small plans, is
// shared by the four waves.  With a lane per pipeline that fetched stage after stage (most lanes
// idle at D < 64, a chain of memory trips per stage) 10 007 plans of 1-48 stages and 1-32 replicas
// took 225 us; they take 45 us now, half of the workgroups being done after 12 us: what is left is
// the chain of trips in front of a plan and the workgroups that hold several large plans.
__global__ __launch_bounds__(kReplicaWaves * 64) void k_eval_replicas(DevPlan pl, ReplicaArgs a) {
  extern __shared__ double rep_lds[];
  ReplicaLds &S = *reinterpret_cast<ReplicaLds *>(rep_lds);
  double *const tables = reinterpret_cast<double *>(&S + 1);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int ZG = pl.ZGr, DP = pl.DP;
  int32_t *const cnts = reinterpret_cast<int32_t *>(tables + list_tables_words(pl));
  const uint64_t c0 = (uint64_t)blockIdx.x * kReplicaWaves, ci = c0 + wv;
  ReplicaPlan pn{};
  if (ci < a.count) {
    const int32_t *d = a.desc + ci * 5;
    const int ip = d[0], q = d[1], it = d[2], id = d[3], im = d[4];
    if (ip >= 0 && ip < a.n_pp && it >= 0 && it < pl.TP && id >= 0 && id < DP && im >= 0 && im < pl.MB && q >= 0) {
      const SearchPP pp = a.pps[ip];
      const int64_t D = pl.vals[id];
      if (q < pp.n_part && D <= kReplicaMaxDegree && (uint64_t)pp.P * (uint64_t)D <= a.stride &&
          !(a.tps && (uint32_t)pp.P > a.tps_stride)) {
        pn.P = pp.P;
        pn.D = (int32_t)D;
        pn.it = it; pn.id = id; pn.im = im;
        pn.rs = pp.rs0 + (uint32_t)q * (uint32_t)pp.P;
      }
    }
  }
  if (lane == 0) S.plan[wv] = pn;
  for (int p = threadIdx.x; p < kReplicaWaves * ZG; p += kReplicaWaves * 64) cnts[p] = 0;
  const ListTables L = stage_list_tables(pl, tables);
  __syncthreads();
  const bool own = pn.P * pn.D <= kReplicaShared;
  if (own && ci < a.count) {  // uniform over the wave
    ReplicaSums s{};
    if (pn.P != 0) s = replica_pairs<64>(pl, a, L, pn, ci, lane, S.times[wv], cnts + wv * ZG);
    wave_lds_fence();
    replica_write(a, L, pn, s, DP, ZG, ci, cnts + wv * ZG);
  }
  for (int w = 0; w < kReplicaWaves; ++w) {  // uniform over the workgroup
    const ReplicaPlan big = S.plan[w];
    if (big.P * big.D <= kReplicaShared) continue;
    __syncthreads();  // the waves' times and sums are free
    const ReplicaSums s = replica_pairs<kReplicaWaves * 64>(pl, a, L, big, c0 + w, (int)threadIdx.x, S.times[0], cnts + w * ZG);
    if (lane == 0) S.part[wv] = s;
    __syncthreads();
    if (wv == w) {
      ReplicaSums all = S.part[0];
#pragma unroll
      for (int x = 1; x < kReplicaWaves; ++x) {
        const ReplicaSums &o = S.part[x];
        all.t_pipe = fmax(all.t_pipe, o.t_pipe);
        all.t_upd = fmax(all.t_upd, o.t_upd);
        all.t_sync = fmax(all.t_sync, o.t_sync);
        all.rent += o.rent;
        all.traffic += o.traffic;
        all.peak = o.peak > all.peak ? o.peak : all.peak;
        all.flags |= o.flags;
      }
      replica_write(a, L, big, all, DP, ZG, c0 + w, cnts + w * ZG);
    }
  }
}

}  // namespace sailor

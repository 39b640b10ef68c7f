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
//   k_search_root        first level of every sub-problem, a wave each: the ones that survive it
//                        go to a list, the deepest pipelines to be taken first
//   k_search_beam        the level-by-level expansion, one workgroup per surviving sub-problem
//   k_search_pick        smallest (key, sub-problem) over the workgroups' winners
//   k_eval_placements    the simulator of Sec. 4.3 for listed placements, fp64
//   k_eval_replicas      the same for plans in which every replica of every stage names its pool
//
// All arithmetic is fp64 in a fixed order (sums in stage order), so that which extension is
// dropped or kept does not depend on how the work is spread over lanes.
//
// What bounds it: the levels of one deep sub-problem follow one another (48 for 48 stages),
// while all of a search's candidates together are little work for the chip (6 to 30 million of
// them).  So a level is kept short: frontier, tables and history stay in LDS, the next level's
// inputs are requested a level ahead, appending candidates takes no barrier, the W smallest come
// from a histogram and (up to 512 of them) a count of predecessors instead of a sort of everything, and a wide choice
// (second pool, TP degree) is first reduced to the best of each (state, pool).  On the 48-layer,
// 20-pool problem a search with beam 64 takes 0.48 ms where states in device memory, paths copied
// level by level and a bitonic sort of every level took 2.9 ms; with two pools and a TP degree per
// stage (1 600 choices, beam 8) 0.74 ms against 9.3 ms.  (0.1 and 0.2 ms more with equal layer splits gone
// through one by one: a depth of as many stages as layers has one split, however often it is listed,
// and its sub-problems, 576 of 1 078, shared the compute units with the 8 that take longest.)
#pragma once

#include <hip/hip_runtime.h>

#include "sailor_kernels.hip.h"

namespace sailor {

// threads of a search workgroup (256: 0.70 / 1.18 ms on the two searches named above, 1 024: 0.74 / 1.29)
constexpr int kSearchThreads = 512;
constexpr int kSearchMaxBeam = 1024;   // longest frontier a sub-problem keeps (half of kSearchBuf at most)
constexpr int kSearchBuf = 2048;       // most candidates buffered between two selections
constexpr int kSearchBinBits = 8, kSearchBins = 1 << kSearchBinBits;
constexpr int kSelectKeep = kSearchBuf / kSearchThreads;  // of them per thread
constexpr int kSearchMaxStages = 255;  // placements count runs in a byte
constexpr int kSearchMaxPools = 64;
constexpr int kRootWaves = 4;            // of a k_search_root workgroup, if their tables fit
constexpr size_t kSearchStaticLds = 1024;  // left to the search kernels' static LDS

struct SearchPP {      // one pipeline depth
  int32_t P;
  uint32_t rs0;        // first entry of its first partition row in the stage tables
  uint32_t sub_off;    // first sub-problem of this depth
  int32_t n_part;
  uint32_t sub_off_t;  // the same when TP is not part of the sub-problem
  uint32_t part0;      // its first entry of SearchArgs::alike
  uint32_t pad[2];
};

enum : int { SEARCH_PLAIN = 0, SEARCH_SPLIT = 1, SEARCH_STAGE_TP = 2, SEARCH_SPLIT_TP = 3 };

// Forms of k_search_beam: frontiers in LDS; in device memory; the same for beams above kSearchNarrow,
// whose selections leave more pairs than can be ranked by counting; the same, and with two pools and a
// TP degree per stage all-reduce seconds by (first zone, second zone) instead of (first zone, second
// pool), for problems whose degrees x zones x pools of them do not fit LDS twice (16 zones of 4 types
// at 8 degrees: 131 KB; by zone 33 KB).
enum : int { SEARCH_IN_LDS = 0, SEARCH_IN_MEMORY = 1, SEARCH_WIDE = 2, SEARCH_BY_ZONE = 3 };

struct SPart {         // one kind of pipeline of a placement of stages 0 .. j
  double sum;          // times of the closed stages 0 .. j-1
  double maxt;         // slowest closed stage
  double c_open;       // compute time of stage j (its forward transfer is not known yet)
  double xb_open;      // its backward transfer to stage j-1
};

template <bool SPLIT>
struct SState {        // placement of stages 0 .. j, followed by its pool counts (uint16_t per pool):
                       // stages placed on each pool (split stages: halves of stages; a TP degree per
                       // stage: GPUs of one replica)
  double msync, mupd, dol, comm;
  SPart part[SPLIT ? 2 : 1];  // with split stages: the pipelines through the first / second pools
  uint8_t pool, pool_b, runs, tpi;          // tpi: the open stage's TP index (TP per stage)
  uint8_t zone, zone_b, pad[2];             // of the pools
};
__host__ __device__ inline uint32_t search_state_words(bool split, int ZG) {  // 8-byte words
  return (uint32_t)((split ? sizeof(SState<true>) : sizeof(SState<false>)) / 8) + (uint32_t)(ZG + 3) / 4;
}

struct SubResult {     // winner of a workgroup's sub-problems (or of the whole search)
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
  const uint32_t *alike;  // per layer split: how many splits of its depth are the same, 0 if an earlier one is.
                          // The sub-problems of equal splits take the same course: the first is gone through
                          // and counted for all of them, and on ties it is the one that wins
  int n_pp;
  uint32_t n_sub;
  uint32_t *list;         // [n_sub] surviving sub-problems, those of a depth together
  uint32_t *counters;     // [n_pp] how many per depth; at [n_pp]: how many were taken
  unsigned long long *root_expanded;  // [k_search_root's workgroups]
  uint32_t buf;           // candidates buffered, at most kSearchBuf
  uint32_t block;         // split stages: states whose tables are in LDS at a time
  uint32_t by_zone;       // split stages: k_search_beam keeps all-reduce seconds by pairs of zones
  double *states;         // [workgroups][2][W] states, or NULL: they are in LDS
  uint32_t *history;      // [workgroups][P_max][W], or NULL: it is in LDS
  SubResult *results;     // [workgroups]
};

struct SBound { double T, C; };

__device__ __forceinline__ bool key_id_less(unsigned long long ka, uint32_t ia, unsigned long long kb,
                                            uint32_t ib) {
  return ka < kb || (ka == kb && ia < ib);
}

// ---- tables in LDS ----

struct SearchLds {
  // of the sub-problem
  double *S;            // [5][P_max] what lies behind stage i: sum, max, sync, upd, $
  double *smin;         // [4][P_max] cheapest admissible choice of every stage
  double *xfer, *comm;  // [Z][Z] transfer seconds; price of a boundary (split: of one kind of pipeline)
  double *ring_price;   // [Z][Z] split: egress both ways
  double *link;         // [Z] a zone's own link; split: [Z][Z] slowest link of a ring through both
  double *price, *dtp;  // [G]; [TPn] D * tp
  unsigned long long *act;   // [TPn] activation bytes of a layer and microbatch
  long long *room;      // [G] memory without what is reserved
  int32_t *node;        // [G]
  int32_t *cap;         // [ZG] what a pool can host, in the units of the pool counts
  uint32_t *zg;         // [ZG] zone | type << 8
  int32_t *width;       // [TPn] what a stage (half a stage) takes from a pool
  // of a level, two of each: the next level's are filled while this one's are used
  double *raw;          // [2][TPn][row_w] the stage's records (DevPlan::st_row)
  double *sync;         // [2][TPn][Z]; split: [TPn][Z][ZP] (first zone, second pool; ZP: ZG made even) or,
                        // by zone, [TPn][Z][Z]: seconds of the stage's all-reduce
  double *upd;          // split: [2][TPn][ZP] update seconds by pool
  double *ring;         // [2][TPn] bytes it moves over every link
  uint32_t *fit;        // [2][TPn] bit g: the stage fits type g
  // split, for a block of states: bounds of the two kinds of pipeline by (TP, pool), pools that
  // can take one half / both halves, the maxima a choice is folded into
  double *pa, *pb;      // [block][TPn][ZP]
  unsigned long long *half, *whole;  // [block][TPn]
  double *mx;           // [block][2]
  // the candidates
  unsigned long long *key;  // [buf]
  unsigned long long *okey; // [gather]
  uint32_t *id, *oid, *rank, *sel;  // [buf], [gather], [gather], [W]: a candidate is numbered by its
                        // state << 16 | choice, which orders like the order of generation
  uint32_t *hist;       // [kSearchBins]
  double *states;
  uint32_t *history;    // [P_max][W] the candidates the frontiers are made of
};

// most pairs a selection leaves to be ordered
constexpr uint32_t kSearchSlack = 128;
__host__ __device__ inline uint32_t search_gather(uint32_t W, uint32_t buf) { return W + kSearchSlack < buf ? W + kSearchSlack : buf; }

// Lays the tables out from base on (NULL: only counts); returns the 8-byte words they take.
__host__ __device__ inline size_t search_carve(const DevPlan &pl, bool split, bool stp, bool root, const SearchArgs &a,
                                               double *base, SearchLds &L) {
  const size_t G = pl.G, Z = pl.Z, ZG = pl.ZGr, ZP = ZG + (ZG & 1), TPn = stp ? pl.TP : 1, P = pl.P_max, two = root ? 1 : 2;
  const size_t sync_row = root || a.by_zone ? Z : ZP;
  size_t at = 0;
  auto words = [&](size_t n) { double *p = base + at; at += n; return p; };
  auto ints = [&](size_t n) { return reinterpret_cast<uint32_t *>(words((n + 1) / 2)); };
  L.S = words(5 * P);
  if (root) L.smin = words(4 * P);
  L.xfer = words(root ? 0 : Z * Z);
  L.comm = words(root ? 0 : Z * Z);
  L.ring_price = words(split ? Z * Z : 0);
  L.link = words(split ? Z * Z : Z);
  L.price = words(G);
  L.dtp = words(TPn);
  L.act = reinterpret_cast<unsigned long long *>(words(TPn));
  L.room = reinterpret_cast<long long *>(words(G));
  L.node = reinterpret_cast<int32_t *>(ints(G));
  L.cap = reinterpret_cast<int32_t *>(ints(ZG));
  L.zg = ints(ZG);
  L.width = reinterpret_cast<int32_t *>(ints(TPn));
  L.raw = words(two * TPn * pl.row_w);
  at += at & 1;  // (rows that are read in pairs)
  L.sync = words(two * TPn * (split ? Z * sync_row : Z));
  at += at & 1;
  L.upd = words(split && !root ? two * TPn * ZP : 0);
  L.ring = words(two * TPn);
  L.fit = ints(two * TPn);
  if (root) return at;
  at += at & 1;
  L.pa = words(split ? a.block * TPn * ZP : 0);
  L.pb = words(split ? a.block * TPn * ZP : 0);
  L.half = reinterpret_cast<unsigned long long *>(words(split ? a.block * TPn : 0));
  L.whole = reinterpret_cast<unsigned long long *>(words(split ? a.block * TPn : 0));
  L.mx = words(split ? a.block * 2 : 0);
  const size_t gather = search_gather((uint32_t)a.W, a.buf);
  L.smin = words(0);  // (needed before there are candidates)
  const size_t from = at;
  L.key = reinterpret_cast<unsigned long long *>(words(a.buf));
  L.id = ints(a.buf);
  if (at < from + 4 * P) at = from + 4 * P;
  L.okey = reinterpret_cast<unsigned long long *>(words(gather));
  L.oid = ints(gather);
  L.rank = ints(gather);
  L.sel = ints(a.W);
  L.hist = ints(kSearchBins);
  L.states = words(a.states ? 0 : 2 * (size_t)a.W * search_state_words(split, (int)ZG));
  L.history = ints(a.history ? 0 : (size_t)a.W * P);
  return at;
}

// for fast_div
__device__ __forceinline__ uint32_t search_magic(int d) {
  return d == 1 ? 0u : (uint32_t)(((1ull << 32) + (uint32_t)d - 1) / (uint32_t)d);
}

struct SearchSub {     // a sub-problem
  int ip, q, it, id, im, P, nb;
  int64_t D;
  uint32_t rs, alike;
  double nbm1, ringf;  // N_b - 1; 2 (D - 1) / D
};

template <bool STP>
__device__ __forceinline__ SearchSub search_sub(const DevPlan &pl, const SearchArgs &a, uint32_t sid) {
  SearchSub s;
  s.ip = 0;
  for (int i = 1; i < a.n_pp; ++i)
    if (sid >= (STP ? a.pps[i].sub_off_t : a.pps[i].sub_off)) s.ip = i;
  const SearchPP pp = a.pps[s.ip];
  uint32_t rem = sid - (STP ? pp.sub_off_t : pp.sub_off);
  s.im = (int)(rem % (uint32_t)pl.MB); rem /= (uint32_t)pl.MB;
  s.id = (int)(rem % (uint32_t)pl.DP); rem /= (uint32_t)pl.DP;
  s.it = STP ? 0 : (int)(rem % (uint32_t)pl.TP);  // (TP per stage: not part of the sub-problem)
  s.q = STP ? (int)rem : (int)(rem / (uint32_t)pl.TP);
  s.P = pp.P;
  s.rs = pp.rs0 + (uint32_t)s.q * (uint32_t)pp.P;
  s.alike = a.alike[pp.part0 + (uint32_t)s.q];
  s.nb = pl.nb[s.im * pl.DP + s.id];
  s.D = pl.vals[s.id];
  s.nbm1 = (double)(s.nb - 1);
  s.ringf = 2.0 * (double)(s.D - 1) / (double)s.D;
  return s;
}

// First record of stage i (at the sub-problem's TP, or at every one from the first on).
template <bool STP>
__device__ __forceinline__ const double *search_row(const DevPlan &pl, const SearchSub &s, int i) {
  return pl.st_row + ((size_t)(s.rs + (uint32_t)i) * pl.MB * pl.TP + (size_t)s.im * pl.TP + (STP ? 0 : s.it)) * pl.row_w;
}

// The sub-problem's tables, by nt threads (tid: which one this is); false: some stage fits no
// pool (known to the thread that looked at it).  A barrier (or fence) before S is accumulated.
template <int MODE, bool ROOT>
__device__ __forceinline__ bool search_tables(const DevPlan &pl, const SearchSub &s, const SearchLds &L, int tid, int nt) {
  constexpr bool SPLIT = MODE == SEARCH_SPLIT || MODE == SEARCH_SPLIT_TP;
  constexpr bool STP = MODE == SEARCH_STAGE_TP || MODE == SEARCH_SPLIT_TP;
  const int G = pl.G, Z = pl.Z, ZG = pl.ZGr, TP = pl.TP, TPn = STP ? TP : 1;
  const double D = (double)s.D;
  for (int i = tid; i < Z * Z; i += nt) {
    const int z = i / Z, y = i - z * Z;
    double both = 0.0;
    if (pl.egress && z != y) both = pl.egress[z * Z + y] + pl.egress[y * Z + z];
    if (!ROOT) {
      L.xfer[i] = pl.xsec[s.im * Z * Z + i];
      L.comm[i] = z == y ? 0.0 : (double)s.nb * (SPLIT ? 0.5 * D : D) * (double)pl.p2p[s.im] * both;
    }
    if (SPLIT) {
      L.ring_price[i] = both;
      double link = pl.bw[z * Z + z];
      if (y != z) link = fmin(fmin(link, pl.bw[y * Z + y]), fmin(pl.bw[z * Z + y], pl.bw[y * Z + z]));
      L.link[i] = link;
    } else if (z == y) {
      L.link[z] = pl.bw[z * Z + z];
    }
  }
  for (int p = tid; p < ZG; p += nt) {
    const int64_t per = STP ? s.D : (int64_t)pl.vals[pl.DP + s.it] * s.D;
    L.cap[p] = (int32_t)((SPLIT ? 2 : 1) * (int64_t)pl.avail[p] / per);
    const uint32_t z = fast_div((uint32_t)p, pl.mg_g);
    L.zg[p] = z | ((uint32_t)p - z * (uint32_t)G) << 8;
  }
  for (int g = tid; g < G; g += nt) {
    L.price[g] = pl.price[g];
    L.room[g] = (long long)pl.cap[g] - (long long)pl.res[g];  // (both below 2^62)
    L.node[g] = pl.node[g];
  }
  for (int k = tid; k < TPn; k += nt) {
    const int tp = pl.vals[pl.DP + (STP ? k : s.it)];
    L.dtp[k] = (double)(s.D * (int64_t)tp);
    L.width[k] = STP ? tp : 1;
    L.act[k] = pl.act[s.im * TP + (STP ? k : s.it)];
  }
  bool fine = true;
  for (int i = tid; i < s.P; i += nt) {  // the cheapest admissible (type, TP) of stage i
    const double *row = search_row<STP>(pl, s, i);
    const int layers = pl.st_n[s.rs + i];
    double cmin = __builtin_huge_val(), umin = cmin, dmin = cmin, smin = cmin;
    bool any = false;
    for (int k = 0; k < TPn; ++k, row += pl.row_w) {
      const int kk = STP ? k : s.it, tpk = pl.vals[pl.DP + kk];
      const uint64_t bytes = (uint64_t)__double_as_longlong(row[2 * G]) +
                             act_bytes(min(s.P - i, s.nb), layers, pl.act[s.im * TP + kk]);
      bool fits_some = false;
      for (int g = 0; g < G; ++g) {
        if (!(bytes + pl.res[g] <= pl.cap[g] && tpk <= pl.node[g])) continue;
        fits_some = true;
        cmin = fmin(cmin, row[g]);
        umin = fmin(umin, row[G + g]);
        dmin = fmin(dmin, (double)(s.D * (int64_t)tpk) * pl.price[g]);
      }
      if (!fits_some) continue;
      any = true;
      // (the all-reduce is fastest over the fastest link, division being monotone)
      double sync = 0.0;
      if (s.D > 1) {
        double fastest = 0.0;
        for (int z = 0; z < Z; ++z) fastest = fmax(fastest, pl.bw[z * Z + z]);
        sync = s.ringf * row[2 * G + 1] / fastest;
      }
      smin = fmin(smin, sync);
    }
    const int P = pl.P_max;
    L.smin[i] = cmin; L.smin[P + i] = smin; L.smin[2 * P + i] = umin; L.smin[3 * P + i] = dmin;
    fine = fine && any;
  }
  return fine;
}

// What lies behind every stage, accumulated from the last stage backwards: lanes 0 .. 4 of a
// wave take a quantity each.
__device__ __forceinline__ void search_suffix(const DevPlan &pl, const SearchSub &s, const SearchLds &L, int lane) {
  if (lane >= 5) return;
  const int P = pl.P_max;
  const double *v = L.smin + (lane == 0 || lane == 1 ? 0 : lane - 1) * P;
  double *o = L.S + lane * P, x = 0.0;
  o[s.P - 1] = 0.0;
  for (int i = s.P - 2; i >= 0; --i) {
    const double y = v[i + 1];
    x = (lane == 0 || lane == 4) ? x + y : fmax(x, y);
    o[i] = x;
  }
}

// What follows from a level's records (which must be visible): all-reduce seconds (ZONES: by pairs of
// zones), update seconds (not for the root), fits.  layers: of the level's stage; tp1: the
// sub-problem's TP degree.
template <int MODE, bool ROOT, bool ZONES>
__device__ __forceinline__ void search_level(const DevPlan &pl, const SearchSub &s, const SearchLds &L, int j, int layers,
                                             int tp1, int b, int tid, int nt) {
  constexpr bool SPLIT = MODE == SEARCH_SPLIT || MODE == SEARCH_SPLIT_TP;
  constexpr bool STP = MODE == SEARCH_STAGE_TP || MODE == SEARCH_SPLIT_TP;
  const int G = pl.G, Z = pl.Z, ZG = pl.ZGr, TPn = STP ? pl.TP : 1, ZP = ZG + (ZG & 1);
  const int NS = SPLIT ? Z * (ZONES ? Z : ZP) : Z;
  const double *raw = L.raw + (size_t)b * TPn * pl.row_w;
  for (int i = tid; i < TPn * NS; i += nt) {
    const int k = i / NS, z = i - k * NS;  // split: first zone * ZP + second pool, or first zone * Z + second zone
    const double ring = s.D > 1 ? s.ringf * raw[k * pl.row_w + 2 * G + 1] : 0.0;
    if (!SPLIT || ZONES) {
      L.sync[b * TPn * NS + i] = s.D > 1 ? ring / L.link[z] : 0.0;
    } else {
      const uint32_t zgb = L.zg[min(z % ZP, ZG - 1)];
      L.sync[b * TPn * NS + i] = s.D > 1 ? ring / L.link[z / ZP * Z + (int)(zgb & 255u)] : 0.0;
      if (!ROOT && z < ZP) L.upd[(b * TPn + k) * ZP + z] = raw[k * pl.row_w + G + (zgb >> 8)];
    }
    if (z == 0) L.ring[b * TPn + k] = ring;
  }
  if (SPLIT && ZONES && !ROOT) {
    for (int i = tid; i < TPn * ZP; i += nt) {
      const int k = i / ZP, p = i - k * ZP;
      L.upd[b * TPn * ZP + i] = raw[k * pl.row_w + G + (L.zg[min(p, ZG - 1)] >> 8)];
    }
  }
  for (int k = tid; k < TPn; k += nt) {
    const int tpk = STP ? L.width[k] : tp1;
    const uint64_t bytes = (uint64_t)__double_as_longlong(raw[k * pl.row_w + 2 * G]) +
                           act_bytes(min(s.P - j, s.nb), layers, L.act[k]);
    uint32_t m = 0;
    for (int g = 0; g < G; ++g)
      if ((long long)bytes <= L.room[g] && tpk <= L.node[g]) m |= 1u << g;
    L.fit[b * TPn + k] = m;
  }
}

// ---- one choice ----

struct SAcc {          // what a placement carries besides its pool counts
  SPart part[2];
  double msync, mupd, dol, comm;
};

// One kind of pipeline goes on from pool zone pz to a stage of compute time c in zone z (first: no
// stage before it, par is not read).  The order of the operations is part of the definition: sums in
// stage order, a closed stage's transfers forward then backward.
__device__ __forceinline__ SPart search_close(bool first, const SPart *par, int pz, int z, int Z, double c, const double *xfer) {
  SPart o;
  o.c_open = c;
  if (first) {
    o.sum = o.maxt = o.xb_open = 0.0;
  } else {
    const double closed = par->c_open + (xfer[pz * Z + z] + par->xb_open);
    o.sum = par->sum + closed;
    o.maxt = fmax(par->maxt, closed);
    o.xb_open = xfer[z * Z + pz];
  }
  return o;
}

// Lower bound of a kind of pipeline's time over the completions.
__device__ __forceinline__ double search_pipe(const SPart &o, double Ssum, double Smax, double nbm1) {
  const double t_open = o.c_open + o.xb_open;
  return ((o.sum + t_open) + Ssum) + nbm1 * fmax(fmax(o.maxt, t_open), Smax);
}

// Stage j on pool a (split stages: half of its replicas on pool b, else b = a) at TP index k (a
// TP degree per stage; else 0) behind the placement par (first: j = 0, there is none): may it be
// placed, and what the placement then carries.  ZONES: all-reduce seconds are kept by pairs of zones.
template <int MODE, bool ZONES>
__device__ __forceinline__ bool search_step(const DevPlan &pl, const SearchLds &L, const SearchSub &s,
                                            bool first, const SState<MODE == SEARCH_SPLIT || MODE == SEARCH_SPLIT_TP> *par, int tb,
                                            int a, int b, int k, int max_runs, SAcc &o, int &runs) {
  constexpr bool SPLIT = MODE == SEARCH_SPLIT || MODE == SEARCH_SPLIT_TP;
  constexpr bool STP = MODE == SEARCH_STAGE_TP || MODE == SEARCH_SPLIT_TP;
  const int G = pl.G, Z = pl.Z, TPn = STP ? pl.TP : 1;
  const uint32_t zga = L.zg[a], zgb = SPLIT ? L.zg[b] : zga;
  const int za = zga & 255u, ga = zga >> 8, zb = zgb & 255u, gb = zgb >> 8;
  const uint32_t fit = L.fit[tb * TPn + k];
  const int width = STP ? L.width[k] : 1;
  const uint16_t *cnt = reinterpret_cast<const uint16_t *>(par + 1);
  const int ca = first ? 0 : (int)cnt[a];
  bool ok = ((fit >> ga) & 1u) != 0;
  if (!SPLIT) {
    ok = ok && ca + width <= L.cap[a];
  } else {
    ok = ok && ((fit >> gb) & 1u) != 0;
    if (a == b) ok = ok && ca + 2 * width <= L.cap[a];
    else ok = ok && (s.D & 1) == 0 && ca + width <= L.cap[a] && (first ? 0 : (int)cnt[b]) + width <= L.cap[b];
  }
  runs = first ? 1 : par->runs + ((a != par->pool || (SPLIT && b != par->pool_b) || (STP && k != par->tpi)) ? 1 : 0);
  if (max_runs != 0 && runs > max_runs) ok = false;
  if (!ok) return false;
  const double *raw = L.raw + (size_t)(tb * TPn + k) * pl.row_w;
  const int pza = first ? 0 : (int)par->zone, pzb = SPLIT && !first ? (int)par->zone_b : 0;
  o.part[0] = search_close(first, &par->part[0], pza, za, Z, raw[ga], L.xfer);
  if (SPLIT) o.part[1] = search_close(first, &par->part[SPLIT ? 1 : 0], pzb, zb, Z, raw[gb], L.xfer);
  // the stage by itself: all-reduce over the slowest link of a ring through both pools, the
  // slower update, the mean rent, the ring's traffic between the zones
  double sync;
  if (!SPLIT) sync = L.sync[(tb * TPn + k) * Z + za];
  else if (ZONES) sync = L.sync[((tb * TPn + k) * Z + za) * Z + zb];
  else sync = L.sync[((tb * TPn + k) * Z + za) * (pl.ZGr + (pl.ZGr & 1)) + b];
  const double upd = SPLIT ? fmax(raw[G + ga], raw[G + gb]) : raw[G + ga];
  const double dol = L.dtp[k] * (SPLIT ? 0.5 * (L.price[ga] + L.price[gb]) : L.price[ga]);
  const double ring = SPLIT && zb != za ? L.ring[tb * TPn + k] * L.ring_price[za * Z + zb] : 0.0;
  if (first) {
    o.msync = sync; o.mupd = upd; o.dol = dol; o.comm = ring;
  } else {
    o.msync = fmax(par->msync, sync);
    o.mupd = fmax(par->mupd, upd);
    o.dol = par->dol + dol;
    double comm = par->comm;
    if (pza != za) comm += L.comm[pza * Z + za];
    if (SPLIT && pzb != zb) comm += L.comm[pzb * Z + zb];
    o.comm = SPLIT ? comm + ring : comm;
  }
  return true;
}

// Lower bounds of T_iter and C_iter over the completions of a placement whose stage j is open
// (the plan's own values when j = P - 1, where every S term is zero); with split stages the
// slower of the two kinds of pipeline counts (Sec. 4.3).
template <bool SPLIT>
__device__ __forceinline__ SBound search_bound(const SAcc &o, const double *S, int P_max, int j, double nbm1) {
  double pipe = search_pipe(o.part[0], S[j], S[P_max + j], nbm1);
  if (SPLIT) pipe = fmax(pipe, search_pipe(o.part[1], S[j], S[P_max + j], nbm1));
  SBound b;
  b.T = (pipe + fmax(o.msync, S[2 * P_max + j])) + fmax(o.mupd, S[3 * P_max + j]);
  b.C = (o.dol + S[4 * P_max + j]) / 3600.0 * b.T + o.comm;
  return b;
}

// Whether a bound is dropped, and its sort key (non-negative: its bits order like the value).
__device__ __forceinline__ bool search_keep(const SearchArgs &a, const SBound &b, unsigned long long &kbits) {
  const double key = a.objective == 0 ? b.T : b.C;
  bool drop = false;
  if (a.has_bound) drop = a.objective == 0 ? b.C > a.bound : 1.0 / b.T < a.bound;
  if (a.has_inc && key > a.inc) drop = true;
  kbits = (unsigned long long)__double_as_longlong(key);
  return !drop;
}

// ---- the first level of every sub-problem ----

// One wave per sub-problem, kRootWaves per workgroup or as many as have room for their tables.  Most
// sub-problems end here: their batch does not divide, a stage fits nowhere, or no placement of the
// first stage survives its bound.
template <int MODE>
__global__ __launch_bounds__(kRootWaves * 64) void k_search_root(DevPlan pl, SearchArgs a, uint32_t wave_words) {
  constexpr bool SPLIT = MODE == SEARCH_SPLIT || MODE == SEARCH_SPLIT_TP;
  constexpr bool STP = MODE == SEARCH_STAGE_TP || MODE == SEARCH_SPLIT_TP;
  extern __shared__ __align__(16) double search_lds[];
  __shared__ unsigned long long s_exp[kRootWaves];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, n_waves = (int)(blockDim.x >> 6);
  const int ZG = pl.ZGr, TPn = STP ? pl.TP : 1, NCH = SPLIT ? ZG * ZG * TPn : ZG * TPn;
  SearchLds L;
  search_carve(pl, SPLIT, STP, true, a, search_lds + wv * wave_words, L);
  unsigned long long expanded = 0;
  for (uint32_t sid = blockIdx.x * n_waves + wv; sid < a.n_sub; sid += gridDim.x * n_waves) {
    const SearchSub s = search_sub<STP>(pl, a, sid);
    if (s.nb == 0 || s.alike == 0) continue;  // (uniform over the wave, like what follows)
    wave_lds_fence();         // the tables are reused
    for (int i = lane; i < TPn * (int)pl.row_w; i += 64) L.raw[i] = search_row<STP>(pl, s, 0)[i];
    const bool fine = search_tables<MODE, true>(pl, s, L, lane, 64);
    if (__builtin_amdgcn_ballot_w64(!fine) != 0) continue;
    wave_lds_fence();
    search_suffix(pl, s, L, lane);
    search_level<MODE, true, true>(pl, s, L, 0, pl.st_n[s.rs], pl.vals[pl.DP + s.it], 0, lane, 64);
    wave_lds_fence();
    bool alive = false;
    uint32_t mine = 0;
    for (int c = lane; c < NCH; c += 64) {
      const int k = STP ? c % TPn : 0, pools = STP ? c / TPn : c;
      const int pa = SPLIT ? pools / ZG : pools, pb = SPLIT ? pools - pa * ZG : pa;
      SAcc o;
      int runs;
      if (!search_step<MODE, true>(pl, L, s, true, nullptr, 0, pa, pb, k, a.max_runs, o, runs)) continue;
      ++mine;
      unsigned long long kbits;
      alive = search_keep(a, search_bound<SPLIT>(o, L.S, pl.P_max, 0, s.nbm1), kbits) || alive;
    }
    if (__builtin_amdgcn_ballot_w64(alive) != 0) {  // (counted again, with its other levels, by k_search_beam)
      if (lane == 0)
        a.list[(STP ? a.pps[s.ip].sub_off_t : a.pps[s.ip].sub_off) + atomicAdd(&a.counters[s.ip], 1u)] = sid;
    } else {
      mine = wave_sum(mine);
      expanded += (unsigned long long)mine * s.alike;
    }
  }
  if (lane == 0) s_exp[wv] = expanded;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < n_waves; ++w) expanded += s_exp[w];
    a.root_expanded[blockIdx.x] = expanded;
  }
}

// ---- the W smallest ----

template <int CTRL, int ROWS>
__device__ __forceinline__ double lane_move(double v) {  // lanes without a source keep their own value
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t l = (uint32_t)b, h = (uint32_t)(b >> 32);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)l, (int)l, CTRL, ROWS, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)h, (int)h, CTRL, ROWS, 0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Minimum / maximum over a wave, in its last lane.
template <bool MIN>
__device__ __forceinline__ double wave_extreme_last(double v) {
  auto f = [](double x, double y) { return MIN ? fmin(x, y) : fmax(x, y); };
  v = f(v, lane_move<0x111, 0xF>(v));  // row_shr:1, 2, 4, 8: within rows of 16 lanes
  v = f(v, lane_move<0x112, 0xF>(v));
  v = f(v, lane_move<0x114, 0xF>(v));
  v = f(v, lane_move<0x118, 0xF>(v));
  v = f(v, lane_move<0x142, 0xA>(v));  // row_bcast:15, 31: across rows
  v = f(v, lane_move<0x143, 0xC>(v));
  return v;
}

struct SelectShared {
  double ext[2 * (kSearchThreads / 64)];
  unsigned long long lo, hi;
  uint32_t n;
};

// The m pairs of (okey, oid), ranked by counting each one's predecessors (rank is zero) -- by_id: in
// the order of their ids -- back to the first places of (key, id), as far as they rank below W.
//
// n^2 comparisons: up to 512 pairs no more than search_sort takes (beam 256 on 64 pools: 4.5 ms, sorted
// 5.1), beyond that more (512 on 64 pools: 24.7 ms, sorted 12.6; 1 024 on 20 pools: 94.5 and 22.5).
constexpr int kRankByCounting = 512;                                // most pairs
constexpr int kSearchNarrow = kRankByCounting - (int)kSearchSlack;  // widest beam that needs no sort
__device__ __forceinline__ void search_place(const SearchLds &L, int m, int W, bool by_id) {
  const int t = threadIdx.x;
  int np = 64;
  while (np < m) np <<= 1;
  const int q = t & (np - 1), row = t / np, rows = kSearchThreads / np;  // several threads share a pair
  if (q < m) {
    const unsigned long long mk = by_id ? 0 : L.okey[q];
    const uint32_t mi = L.oid[q];
    uint32_t before = 0;
#pragma unroll 8
    for (int x = row; x < m; x += rows) before += key_id_less(by_id ? 0 : L.okey[x], L.oid[x], mk, mi) ? 1u : 0u;
    if (before) atomicAdd(&L.rank[q], before);
  }
  __syncthreads();
  if (t < m) {
    const uint32_t r = L.rank[t];
    if (r < (uint32_t)W) { L.key[r] = L.okey[t]; L.id[r] = L.oid[t]; }
  }
  __syncthreads();
}
static_assert(kRankByCounting <= kSearchThreads, "a thread per pair");

// Ascending bitonic sort of n (key, id) pairs -- by_id: in the order of their ids.  Every exchange
// brings the smaller pair to the lower place (the first of a merge by mirrored places), so places
// beyond n need no pairs: what they would hold is never smaller.  Exchanges within 128 places are
// between lanes of one wave.  The pairs must be visible; they are again on return.
__device__ __forceinline__ void search_sort(unsigned long long *key, uint32_t *id, int n, bool by_id) {
  int np = 2;
  while (np < n) np <<= 1;
#pragma unroll 1
  for (int k = 2; k <= np; k <<= 1) {
#pragma unroll 1
    for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll 1
      for (int p = threadIdx.x; p < np / 2; p += kSearchThreads) {
        const int low = p & (j - 1), i = 2 * p - low, x = j == k >> 1 ? i - low + (2 * j - 1 - low) : i + j;  // i < x
        if (x < n) {
          const unsigned long long ki = key[i], kx = key[x];
          const uint32_t ii = id[i], ix = id[x];
          if (key_id_less(by_id ? 0 : kx, ix, by_id ? 0 : ki, ii)) { key[i] = kx; key[x] = ki; id[i] = ix; id[x] = ii; }
        }
      }
      const int next = j > 1 ? j : 2 * k;  // places the next step's exchanges lie within
      if (2 * j > 128 || next > 128) __syncthreads();
      else wave_lds_fence();
    }
  }
  __syncthreads();
}

// Brings the W smallest of the n > W (key, id) pairs to the front of the buffer, in ascending
// order.  A histogram over the range of the keys' bits (keys are not negative) finds the bin the W-th
// lies in, again within that bin while too many share it; among equal keys the ids take the keys'
// place.  What lies in the bin or before it is ranked.  The buffer must be visible; it is again on
// return.  Returns 0, or (WIDE) how many pairs (okey, oid) then holds, the W smallest among them and
// more than search_place takes: their order is left to the caller.
// Every round takes a range apart into at least two bins that are not empty, so there are at most 15.
template <bool WIDE>
__device__ __forceinline__ int search_select(const SearchLds &L, SelectShared &sh, int n, int W, int gather) {
  constexpr unsigned long long kById = 1ull << 63;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // this thread's pairs (requested together: places beyond n read the last pair and do not count)
  unsigned long long x[kSelectKeep];  // the key's bits, later what takes their place
  uint32_t ii[kSelectKeep];
#pragma unroll
  for (int q = 0; q < kSelectKeep; ++q) {
    const int e = min(t + q * kSearchThreads, n - 1);
    x[q] = L.key[e];
    ii[q] = L.id[e];
  }
  double least = __builtin_huge_val(), most = 0.0;
#pragma unroll
  for (int q = 0; q < kSelectKeep; ++q) {  // (the last pair again changes neither)
    least = fmin(least, __longlong_as_double((long long)x[q]));
    most = fmax(most, __longlong_as_double((long long)x[q]));
  }
  least = wave_extreme_last<true>(least);
  most = wave_extreme_last<false>(most);
  if (lane == 63) { sh.ext[2 * wv] = least; sh.ext[2 * wv + 1] = most; }
  for (int b = t; b < kSearchBins; b += kSearchThreads) L.hist[b] = 0;
  for (int b = t; b < gather; b += kSearchThreads) L.rank[b] = 0;
  __syncthreads();
  least = sh.ext[0]; most = sh.ext[1];
#pragma unroll
  for (int w = 1; w < kSearchThreads / 64; ++w) { least = fmin(least, sh.ext[2 * w]); most = fmax(most, sh.ext[2 * w + 1]); }
  unsigned long long lo = (unsigned long long)__double_as_longlong(least), hi = (unsigned long long)__double_as_longlong(most);
  int below = 0;  // pairs under lo
  for (;;) {  // uniform
    // (a range of 2^k values and less than twice that: 128 to 256 bins)
    const int shift = hi - lo < kSearchBins ? 0 : 64 - kSearchBinBits - __builtin_clzll(hi - lo);
    auto bin_of = [&](unsigned long long v) { return (int)((v - lo) >> shift); };
#pragma unroll
    for (int q = 0; q < kSelectKeep; ++q)
      if (t + q * kSearchThreads < n && x[q] >= lo && x[q] <= hi) atomicAdd(&L.hist[bin_of(x[q])], 1u);
    if (t == 0) { sh.n = 0; sh.lo = ~0ull; sh.hi = 0; }
    __syncthreads();
    // the bin of the W-th (every wave for itself)
    constexpr int kPer = kSearchBins / 64;
    uint32_t h[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) { h[q] = L.hist[lane * kPer + q]; sum += h[q]; }
    const uint32_t incl = wave_prefix_sum(sum);
    uint32_t excl = (uint32_t)below + incl - sum;
    const unsigned long long here = __builtin_amdgcn_ballot_w64(excl < (uint32_t)W && (uint32_t)W <= excl + sum);
    const int owner = __builtin_ctzll(here);
    int b = 0;
#pragma unroll
    for (int q = 0; q < kPer - 1; ++q)
      if (b == q && excl + h[q] < (uint32_t)W) { excl += h[q]; b = q + 1; }
    uint32_t hb = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) hb = b == q ? h[q] : hb;
    const int bin = __builtin_amdgcn_readlane(lane * kPer + b, owner), under = __builtin_amdgcn_readlane((int)excl, owner),
              m = under + __builtin_amdgcn_readlane((int)hb, owner);
    if (m <= gather) {
      unsigned long long mask[kSelectKeep];  // one reservation per wave
      uint32_t total = 0;
#pragma unroll
      for (int q = 0; q < kSelectKeep; ++q) {
        mask[q] = __builtin_amdgcn_ballot_w64(t + q * kSearchThreads < n && (x[q] < lo || (x[q] <= hi && bin_of(x[q]) <= bin)));
        total += (uint32_t)__popcll(mask[q]);
      }
      uint32_t at = 0;
      if (lane == 0 && total) at = atomicAdd(&sh.n, total);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
      for (int q = 0; q < kSelectKeep; ++q) {
        const uint32_t mine = at + (uint32_t)__popcll(mask[q] & ((1ull << lane) - 1ull));
        if ((mask[q] >> lane) & 1ull) { L.okey[mine] = L.key[t + q * kSearchThreads]; L.oid[mine] = ii[q]; }
        at += (uint32_t)__popcll(mask[q]);
      }
      __syncthreads();
      if (WIDE && m > kRankByCounting) return m;
      search_place(L, m, W, false);
      return 0;
    }
    const bool equal = lo == hi;
    if (equal) {  // many equal keys: by their ids, which differ
#pragma unroll
      for (int q = 0; q < kSelectKeep; ++q) x[q] = x[q] == lo ? kById | ii[q] : (x[q] < lo ? 0ull : ~0ull);
    } else {
#pragma unroll
      for (int q = 0; q < kSelectKeep; ++q)
        if (t + q * kSearchThreads < n && x[q] >= lo && x[q] <= hi && bin_of(x[q]) == bin) { atomicMin(&sh.lo, x[q]); atomicMax(&sh.hi, x[q]); }
    }
    __syncthreads();  // (every wave has read the histogram)
    for (int e = t; e < kSearchBins; e += kSearchThreads) L.hist[e] = 0;
    below = under;
    lo = equal ? kById : sh.lo;
    hi = equal ? kById | 0xFFFFFFFFull : sh.hi;
    __syncthreads();  // (read before the next round resets them)
  }
}

// ---- the levels ----

// One workgroup per surviving sub-problem.
//
// A choice is (a, k), or with split stages (a, b, k).  An item is the choices that differ in the
// inner digit only (b, or k): a level first looks at items, by the best choice of each; only where
// there is an inner digit, the choices behind the best W items are looked at one by one -- the W
// smallest choices lie in the W items with the smallest bests.
// (Two waves per SIMD for split stages, four else.  At four, the code for split stages spills so much
// that it takes 1.19 ms against 1.05; the other forms spill too -- 54 registers with a pool per stage,
// 121 with a degree per stage -- but at two they lose a workgroup per compute unit, 0.72 ms against 0.62
// where 1 078 sub-problems survive their first level; 0.39 against 0.40 where 574 do.)
// FORM: where the frontiers are, and how all-reduce seconds are kept.
template <int MODE, int FORM>
__global__ __launch_bounds__(kSearchThreads, (MODE & 1) ? 2 : 4) void k_search_beam(DevPlan pl, SearchArgs a) {
  constexpr bool SPLIT = MODE == SEARCH_SPLIT || MODE == SEARCH_SPLIT_TP;   // two pools per stage
  constexpr bool STP = MODE == SEARCH_STAGE_TP || MODE == SEARCH_SPLIT_TP;  // a TP degree per stage
  constexpr bool LDSF = FORM == SEARCH_IN_LDS, WIDE = FORM >= SEARCH_WIDE, ZONES = FORM == SEARCH_BY_ZONE;
  using State = SState<SPLIT>;
  extern __shared__ __align__(16) double search_lds[];  // (tables by pool are read in pairs, from even places)
  __shared__ SelectShared sh;
  // candidates buffered (items; choices behind them) and kept in all; two sets, used by levels in turn
  __shared__ uint32_t s_n[2][2], s_kept[2], s_next;
  __shared__ unsigned long long s_expanded;
  __shared__ unsigned long long s_bk[kSearchThreads / 64];
  __shared__ uint32_t s_bi[kSearchThreads / 64];
  static_assert(sizeof sh + sizeof s_n + sizeof s_kept + sizeof s_next + sizeof s_expanded + sizeof s_bk + sizeof s_bi + 64 <=
                kSearchStaticLds, "what dynamic LDS leaves room for");
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int ZG = pl.ZGr, Z = pl.Z, G = pl.G, TPn = STP ? pl.TP : 1, W = a.W, P_max = pl.P_max;
  const int ITEMS = SPLIT ? ZG * TPn : ZG, INNER = SPLIT ? ZG : TPn, ZP = ZG + (ZG & 1);
  SearchLds L;
  search_carve(pl, SPLIT, STP, false, a, search_lds, L);
  const uint32_t mg_items = search_magic(ITEMS), mg_zg = search_magic(ZG), mg_tpn = search_magic(TPn), mg_inner = search_magic(INNER);
  const int gather = (int)search_gather((uint32_t)W, a.buf), buf = (int)a.buf;
  const uint32_t sw = search_state_words(SPLIT, ZG);
  double *const states = LDSF ? L.states : a.states + (size_t)blockIdx.x * 2 * W * sw;
  uint32_t *const history = a.history ? a.history + (size_t)blockIdx.x * P_max * W : L.history;
  SubResult *const res = a.results + blockIdx.x;
  const bool need_c = a.objective != 0 || a.has_bound != 0;
  unsigned long long wg_key = ~0ull;  // the workgroup's best so far
  uint32_t wg_sid = ~0u, wg_trunc = 0;
  unsigned long long my_total = 0;    // placements this thread generated
  uint32_t n_alive = 0;
  for (int i = 0; i < a.n_pp; ++i) n_alive += a.counters[i];
  auto state_at = [&](int frontier, int r) { return reinterpret_cast<State *>(states + ((size_t)frontier * W + r) * sw); };
  auto number = [&](int r, int pa, int pb, int k) { return (uint32_t)(r << 16 | (SPLIT ? (pa * ZG + pb) * TPn + k : pa * TPn + k)); };
  auto choice = [&](uint32_t cand, int &r, int &ca, int &cb, int &ck) {
    r = (int)(cand >> 16);
    const uint32_t c = cand & 0xFFFFu, pools = STP ? fast_div(c, mg_tpn) : c;
    ck = STP ? (int)(c - pools * (uint32_t)TPn) : 0;
    ca = SPLIT ? (int)fast_div(pools, mg_zg) : (int)pools;
    cb = SPLIT ? (int)pools - ca * ZG : ca;
  };
  if (t == 0) s_expanded = 0;

  for (;;) {  // sub-problems, the deepest pipelines first (uniform; ends when the list is used up)
    __syncthreads();  // the tables are reused
    if (t == 0) s_next = atomicAdd(&a.counters[a.n_pp], 1u);
    __syncthreads();
    uint32_t turn = s_next;
    if (turn >= n_alive) break;
    int ip = a.n_pp - 1;
    for (; ip > 0 && turn >= a.counters[ip]; --ip) turn -= a.counters[ip];
    const uint32_t sid = a.list[(STP ? a.pps[ip].sub_off_t : a.pps[ip].sub_off) + turn];
    const SearchSub s = search_sub<STP>(pl, a, sid);
    const int P = s.P;
    const int n_raw = TPn * (int)pl.row_w;
    for (int i = t; i < n_raw; i += kSearchThreads) L.raw[i] = search_row<STP>(pl, s, 0)[i];
    search_tables<MODE, false>(pl, s, L, t, kSearchThreads);
    if (t == 0) s_n[0][0] = s_n[0][1] = s_kept[0] = 0;
    __syncthreads();
    if (wv == kSearchThreads / 64 - 1) search_suffix(pl, s, L, lane);
    const int tp1 = pl.vals[pl.DP + s.it];
    search_level<MODE, false, ZONES>(pl, s, L, 0, pl.st_n[s.rs], tp1, 0, t, kSearchThreads);
    int n_cur = 1;  // frontier length; level 0 extends one empty placement
    bool truncated = false;
    for (int j = 0; j < P; ++j) {  // place stage j (uniform loop)
      const int tb = j & 1, cur = j & 1, nxt = cur ^ 1;
      const bool last = j == P - 1, first = j == 0;
      __syncthreads();
      if (t == 0) s_n[nxt][0] = s_n[nxt][1] = s_kept[nxt] = 0;
      // the next level's records, requested now and stored when this level's candidates are in
      double ahead = 0.0;
      int layers = 0;
      if (!last) {
        layers = pl.st_n[s.rs + j + 1];
        if (t < n_raw) ahead = search_row<STP>(pl, s, j + 1)[t];
      }
      const double S0 = L.S[j], S1 = L.S[P_max + j], S2 = L.S[2 * P_max + j], S3 = L.S[3 * P_max + j], S4 = L.S[4 * P_max + j];
      unsigned long long best_k = ~0ull;  // last level: this thread's smallest (key, id)
      uint32_t best_i = ~0u;
      uint32_t kept = 0, expanded = 0;
      bool cut = false, sorted = false;
      int n = 0, block0 = 0, block1 = 0;
      for (int phase = 0; phase < (INNER > 1 && !last ? 2 : 1); ++phase) {  // items; the choices behind the best
        uint32_t *const counter = &s_n[cur][phase];
        unsigned long long tau = ~0ull;     // only keys up to this can be among the W smallest
        const int n_all = phase == 0 ? n_cur * ITEMS : n * INNER;
        int used = 0;
        for (int i0 = 0;;) {  // uniform
          int i1 = last ? n_all : min(n_all, i0 + buf - used);
          if (SPLIT && phase == 0) {
            if (i0 >= block1 * ITEMS) {  // the next states' tables
              if (block1 > 0) __syncthreads();
              block0 = block1;
              block1 = min(n_cur, block0 + (int)a.block);
              const int nb = block1 - block0;
              for (int x = t; x < 2 * nb * ITEMS; x += kSearchThreads) {
                const int second = x >= nb * ITEMS ? 1 : 0, y = x - second * nb * ITEMS;
                const int rl = (int)fast_div((uint32_t)y, mg_items), rem = y - rl * ITEMS, k = (int)fast_div((uint32_t)rem, mg_zg),
                          p = rem - k * ZG;
                const uint32_t zg = L.zg[p];
                const State *par = state_at(cur, block0 + rl);
                const int pz = first ? 0 : (int)(second ? par->zone_b : par->zone);
                const SPart o = search_close(first, &par->part[second && SPLIT ? 1 : 0], pz, (int)(zg & 255u), Z,
                                             L.raw[(tb * TPn + k) * pl.row_w + (zg >> 8)], L.xfer);
                const double pipe = search_pipe(o, S0, S1, s.nbm1);
                double *const row = (second ? L.pb : L.pa) + (rl * TPn + k) * ZP;
                row[p] = pipe;
                if (p == ZG - 1 && ZP != ZG) row[ZG] = pipe;  // (read, not used)
              }
              for (int y = wv; y < nb * TPn; y += kSearchThreads / 64) {  // a wave, its lanes the pools
                const int rl = (int)fast_div((uint32_t)y, mg_tpn), k = y - rl * TPn, width = L.width[k], p = lane < ZG ? lane : 0;
                const State *par = state_at(cur, block0 + rl);
                const int count = first ? 0 : (int)reinterpret_cast<const uint16_t *>(par + 1)[p];
                const bool fits = lane < ZG && ((L.fit[tb * TPn + k] >> (L.zg[p] >> 8)) & 1u) != 0;
                const unsigned long long h = __builtin_amdgcn_ballot_w64(fits && count + width <= L.cap[p]);
                const unsigned long long w2 = __builtin_amdgcn_ballot_w64(fits && count + 2 * width <= L.cap[p]);
                if (lane == 0) { L.half[y] = (s.D & 1) ? 0 : h; L.whole[y] = w2; }
                if (lane == 0 && k == 0) {
                  L.mx[2 * rl] = first ? fmax(0.0, S2) : fmax(par->msync, S2);
                  L.mx[2 * rl + 1] = first ? fmax(0.0, S3) : fmax(par->mupd, S3);
                }
              }
              __syncthreads();
            }
            i1 = min(i1, block1 * ITEMS);
          }
          for (int x0 = i0; x0 < i1; x0 += kSearchThreads) {  // uniform
            const int x = x0 + t;
            unsigned long long bk = ~0ull;  // (no bound has this pattern)
            uint32_t bi = ~0u;
            if (x < i1 && phase == 1) {
              const int e = (int)fast_div((uint32_t)x, mg_inner), in = x - e * INNER;
              int r, pa, pb, pk;
              choice(L.sel[e], r, pa, pb, pk);
              if (SPLIT) pb = in;
              else pk = in;
              SAcc o;
              int runs;
              unsigned long long kb;
              if (search_step<MODE, ZONES>(pl, L, s, first, state_at(cur, r), tb, pa, pb, pk, a.max_runs, o, runs) &&
                  search_keep(a, search_bound<SPLIT>(o, L.S, P_max, j, s.nbm1), kb)) {
                bk = kb;
                bi = number(r, pa, pb, pk);
              }
            } else if (x < i1) {
              const int r = (int)fast_div((uint32_t)x, mg_items), rem = x - r * ITEMS;  // (x < 2^19, ITEMS < 2^10)
              const State *par = state_at(cur, r);
              if (SPLIT) {
                const int pa = (int)fast_div((uint32_t)rem, mg_tpn), k = rem - pa * TPn, y = (r - block0) * TPn + k;
                const uint32_t zga = L.zg[pa];
                const int za = zga & 255u, ga = zga >> 8;
                const unsigned long long half = L.half[y], whole = L.whole[y];
                const double ta = L.pa[y * ZP + pa], mx0 = L.mx[2 * (r - block0)], mx1 = L.mx[2 * (r - block0) + 1];
                const double *row_b = L.pb + y * ZP, *sync = L.sync + ((tb * TPn + k) * Z + za) * (ZONES ? Z : ZP), *upd = L.upd + (tb * TPn + k) * ZP;
                const double ua = fmax(mx1, upd[pa]);
                // the second pools this state and first pool admit
                unsigned long long cand = ((half >> pa) & 1ull) ? half & ~(1ull << pa) : 0ull;
                cand |= whole & (1ull << pa);
                if (a.max_runs != 0 && !first && par->runs >= a.max_runs)
                  cand &= (par->runs == a.max_runs && pa == par->pool && (!STP || k == par->tpi)) ? 1ull << par->pool_b : 0ull;
                expanded += (uint32_t)__popcll(cand);
                int best_b = 0;
                if (!need_c) {
                  // (a bound of +inf, which no incumbent drops, must not look like none)
                  double best_t = __builtin_huge_val();
                  int none = -1;
                  const double inc = a.has_inc ? a.inc : __builtin_huge_val();
                  uint32_t c_lo = (uint32_t)cand, c_hi = (uint32_t)(cand >> 32);
#pragma unroll 2
                  for (int pb = 0; pb < ZP; pb += 2) {
                    const double2 rb = *reinterpret_cast<const double2 *>(row_b + pb), up = *reinterpret_cast<const double2 *>(upd + pb);
                    double2 sy;
                    if (ZONES) {
                      sy.x = sync[fast_div((uint32_t)pb, pl.mg_g)];
                      sy.y = sync[fast_div((uint32_t)min(pb + 1, ZG - 1), pl.mg_g)];
                    } else {
                      sy = *reinterpret_cast<const double2 *>(sync + pb);
                    }
                    const double T0 = (fmax(ta, rb.x) + fmax(mx0, sy.x)) + fmax(ua, up.x);
                    const double T1 = (fmax(ta, rb.y) + fmax(mx0, sy.y)) + fmax(ua, up.y);
                    const uint32_t word = pb < 32 ? c_lo : c_hi;
                    const bool f0 = ((word >> (pb & 31)) & 1u) != 0 && T0 <= inc, f1 = ((word >> (pb & 31)) & 2u) != 0 && T1 <= inc;
                    kept += (f0 ? 1u : 0u) + (f1 ? 1u : 0u);
                    const bool b0 = f0 && (T0 < best_t || none < 0);
                    best_t = b0 ? T0 : best_t;
                    none = b0 ? pb : none;
                    const bool b1 = f1 && (T1 < best_t || none < 0);
                    best_t = b1 ? T1 : best_t;
                    none = b1 ? pb + 1 : none;
                  }
                  if (none >= 0) { bk = (unsigned long long)__double_as_longlong(best_t); best_b = none; }
                } else {
                  for (; cand; cand &= cand - 1) {
                    const int pb = __builtin_ctzll(cand);
                    const uint32_t zgb = L.zg[pb];
                    const int zb = zgb & 255u, gb = zgb >> 8;
                    SBound b;
                    b.T = (fmax(ta, row_b[pb]) + fmax(mx0, sync[ZONES ? zb : pb])) + fmax(ua, upd[pb]);
                    double rent = L.dtp[k] * (0.5 * (L.price[ga] + L.price[gb])), comm = 0.0;
                    const double ring = zb != za ? L.ring[tb * TPn + k] * L.ring_price[za * Z + zb] : 0.0;
                    if (!first) {
                      rent = par->dol + rent;
                      comm = par->comm;
                      if (par->zone != za) comm += L.comm[par->zone * Z + za];
                      if (par->zone_b != zb) comm += L.comm[par->zone_b * Z + zb];
                    }
                    b.C = (rent + S4) / 3600.0 * b.T + (comm + ring);
                    unsigned long long kb;
                    if (search_keep(a, b, kb)) {
                      ++kept;
                      if (kb < bk) { bk = kb; best_b = pb; }
                    }
                  }
                }
                bi = number(r, pa, best_b, k);
              } else {
                const int pa = rem;
                const uint32_t zga = L.zg[pa];
                const int z = zga & 255u, g = zga >> 8;
                const int count = first ? 0 : (int)reinterpret_cast<const uint16_t *>(par + 1)[pa], cap = L.cap[pa];
                SPart o;
                o.sum = o.maxt = o.xb_open = 0.0;
                double msync = S2, mupd = S3;
                if (!first) {
                  o = search_close(false, &par->part[0], par->zone, z, Z, 0.0, L.xfer);
                  msync = fmax(par->msync, S2);
                  mupd = fmax(par->mupd, S3);
                }
                int best_b = 0;
                for (int k = 0; k < TPn; ++k) {
                  const int width = STP ? L.width[k] : 1;
                  bool ok = ((L.fit[tb * TPn + k] >> g) & 1u) != 0 && count + width <= cap;
                  if (a.max_runs != 0 && !first)
                    ok = ok && par->runs + ((pa != par->pool || (STP && k != par->tpi)) ? 1 : 0) <= a.max_runs;
                  if (!ok) continue;
                  ++expanded;
                  const double *raw = L.raw + (size_t)(tb * TPn + k) * pl.row_w;
                  o.c_open = raw[g];
                  SBound b;
                  b.T = (search_pipe(o, S0, S1, s.nbm1) + fmax(msync, L.sync[(tb * TPn + k) * Z + z])) + fmax(mupd, raw[G + g]);
                  b.C = 0.0;
                  if (need_c) {
                    double rent = L.dtp[k] * L.price[g], comm = 0.0;
                    if (!first) {
                      rent = par->dol + rent;
                      comm = par->comm;
                      if (par->zone != z) comm += L.comm[par->zone * Z + z];
                    }
                    b.C = (rent + S4) / 3600.0 * b.T + comm;
                  }
                  unsigned long long kb;
                  if (search_keep(a, b, kb)) {
                    ++kept;
                    if (kb < bk) { bk = kb; best_b = k; }
                  }
                }
                bi = number(r, pa, pa, best_b);
              }
            }
            if (last) {
              if (key_id_less(bk, bi, best_k, best_i) && bk != ~0ull) { best_k = bk; best_i = bi; }
              continue;
            }
            const bool keep = bk != ~0ull && bk <= tau;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
            if (m == 0) continue;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(counter, (uint32_t)__popcll(m));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
            if (keep) {
              at += (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
              L.key[at] = bk;
              L.id[at] = bi;
            }
          }
          i0 = i1;
          if (last) {
            if (i0 >= n_all) break;
            continue;
          }
          const bool done = i0 >= n_all;
          if (done && phase == 0) {  // how many were kept in all
            kept = wave_sum(kept);
            if (lane == 0 && kept) atomicAdd(&s_kept[cur], kept);
          }
          __syncthreads();
          used = (int)*counter;
          if (done && phase == 0) {
            kept = s_kept[cur];
            cut = kept > (uint32_t)W;
            for (int i = t; i < n_raw; i += kSearchThreads) L.raw[(tb ^ 1) * n_raw + i] = i < kSearchThreads ? ahead : search_row<STP>(pl, s, j + 1)[i];
          }
          // the W smallest, at the end of a phase and when there is no room for what is left
          const bool full = used > W && (done || buf - used < min(n_all - i0, buf - W));  // uniform
          const int left = full ? search_select<WIDE>(L, sh, used, W, gather) : 0;
          sorted = full;
          if (WIDE) {
            // left to sort: what a selection did not rank; a long frontier that was not cut
            const bool whole = !full && done && phase == (INNER > 1 ? 1 : 0) && used > kRankByCounting;
            if (left != 0) {
              search_sort(L.okey, L.oid, left, false);
              for (int x = t; x < W; x += kSearchThreads) { L.key[x] = L.okey[x]; L.id[x] = L.oid[x]; }
              __syncthreads();
            } else if (whole) {
              search_sort(L.key, L.id, used, !cut);
              sorted = true;
            }
          }
          if (full) {
            used = W;
            tau = L.key[W - 1];
            if (!done && t == 0) *counter = (uint32_t)W;
          }
          if (done) break;
          __syncthreads();  // every wave has read the counter (or sees it reset) before the next pass adds to it
        }
        if (last || kept == 0) break;  // uniform
        n = used;
        if (phase == 0 && INNER > 1) {
          for (int x = t; x < n; x += kSearchThreads) L.sel[x] = L.id[x];
          __syncthreads();
        }
      }
      my_total += (unsigned long long)expanded * s.alike;
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
        if (best_i != ~0u && key_id_less(best_k, sid, wg_key, wg_sid)) {  // uniform
          wg_key = best_k;
          wg_sid = sid;
          if (t == 0) {
            int r, pa, pb, pk;
            choice(best_i, r, pa, pb, pk);
            SAcc o;
            int runs;
            search_step<MODE, ZONES>(pl, L, s, first, state_at(cur, r), tb, pa, pb, pk, a.max_runs, o, runs);
            const SBound b = search_bound<SPLIT>(o, L.S, P_max, j, s.nbm1);
            res->T = b.T;
            res->C = b.C;
            res->key = a.objective == 0 ? b.T : b.C;
            res->sid = sid;
            res->P = (uint32_t)P;
            res->desc[0] = s.ip; res->desc[1] = s.q; res->desc[3] = s.id; res->desc[4] = s.im; res->desc[5] = MODE;
            uint32_t cand = best_i;
            for (int i = P - 1; i >= 0; --i) {  // back through the levels
              choice(cand, r, pa, pb, pk);
              res->pools[i] = pa;
              res->pools_b[i] = pb;
              res->tps[i] = STP ? pk : s.it;
              if (i > 0) cand = history[(size_t)(i - 1) * W + r];
            }
            res->desc[2] = STP ? pk : s.it;  // stage 0's
          }
        }
        break;
      }
      if (kept == 0) break;  // uniform
      truncated = truncated || cut;
      // a cut frontier: ascending bounds (as a selection leaves them); else the order of generation
      if (!sorted) {
        for (int x = t; x < n; x += kSearchThreads) { L.okey[x] = L.key[x]; L.oid[x] = L.id[x]; L.rank[x] = 0; }
        __syncthreads();
        search_place(L, n, W, !cut);
      }
      // write the next frontier: four lanes per state
      for (int x = t; x < 4 * n; x += kSearchThreads) {
        const int k = x >> 2, q = x & 3;
        const uint32_t cand = L.id[k];
        int r, pa, pb, pk;
        choice(cand, r, pa, pb, pk);
        const State *par = state_at(cur, r);
        State *const out = state_at(nxt, k);
        const unsigned long long *cw = reinterpret_cast<const unsigned long long *>(par + 1);
        unsigned long long *ow = reinterpret_cast<unsigned long long *>(out + 1);
        const unsigned long long width = (unsigned long long)L.width[pk];
        for (int w = q; w < (ZG + 3) / 4; w += 4) {  // the pool counts, four to a word
          unsigned long long v = first ? 0ull : cw[w];
          if (pa >> 2 == w) v += width << (16 * (pa & 3));
          if (SPLIT && pb >> 2 == w) v += width << (16 * (pb & 3));
          ow[w] = v;
        }
        SAcc o;
        int runs;
        search_step<MODE, ZONES>(pl, L, s, first, par, tb, pa, pb, pk, a.max_runs, o, runs);
        if (q == 0) {
          out->msync = o.msync; out->mupd = o.mupd; out->dol = o.dol; out->comm = o.comm;
        } else if (q == 1) {
          out->part[0] = o.part[0];
        } else if (q == 2) {
          if (SPLIT) out->part[SPLIT ? 1 : 0] = o.part[1];
          history[(size_t)j * W + k] = cand;
        } else {
          const unsigned long long z = L.zg[pa] & 255u, zb = L.zg[pb] & 255u;
          *reinterpret_cast<unsigned long long *>(&out->pool) = (unsigned long long)pa | (unsigned long long)pb << 8 |
              (unsigned long long)(runs & 255) << 16 | (unsigned long long)pk << 24 | z << 32 | zb << 40;
        }
      }
      // (from the last wave on: the first ones write the frontier)
      search_level<MODE, false, ZONES>(pl, s, L, j + 1, layers, tp1, tb ^ 1, kSearchThreads - 1 - t, kSearchThreads);
      n_cur = n;
    }
    if (truncated) wg_trunc = 1;
  }
  atomicAdd(&s_expanded, my_total);
  __syncthreads();
  if (t == 0) {
    res->found = wg_sid != ~0u ? 1u : 0u;
    res->truncated = wg_trunc;
    res->expanded = s_expanded;
  }
}

// Smallest (key, sub-problem) over the workgroups' winners; also the totals.  Leaves the winner
// in host-mapped memory as well and the counters ready for the next search.
__global__ __launch_bounds__(1024) void k_search_pick(SearchArgs a, uint32_t n_wgs, uint32_t n_root, SubResult *out,
                                                      SubResult *host_out) {
  __shared__ unsigned long long s_k[16], s_e[16];
  __shared__ uint32_t s_i[16], s_t[16], s_at[16];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  unsigned long long bk = ~0ull, expanded = 0;
  uint32_t bi = ~0u, trunc = 0, at = 0;
  for (uint32_t i = t; i < n_root; i += blockDim.x) expanded += a.root_expanded[i];
  for (uint32_t i = t; i < n_wgs; i += blockDim.x) {
    const SubResult &r = a.results[i];
    expanded += r.expanded;
    trunc |= r.truncated;
    if (r.found) {
      const unsigned long long k = (unsigned long long)__double_as_longlong(r.key);
      if (key_id_less(k, r.sid, bk, bi)) { bk = k; bi = r.sid; at = i; }
    }
  }
  for (int i = t; i <= a.n_pp; i += blockDim.x) a.counters[i] = 0;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned long long ok = __shfl_xor(bk, off);
    const uint32_t oi = __shfl_xor(bi, off), oa = __shfl_xor(at, off);
    if (key_id_less(ok, oi, bk, bi)) { bk = ok; bi = oi; at = oa; }
    expanded += __shfl_xor(expanded, off);
    trunc |= __shfl_xor(trunc, off);
  }
  if (lane == 0) { s_k[wv] = bk; s_i[wv] = bi; s_e[wv] = expanded; s_t[wv] = trunc; s_at[wv] = at; }
  __syncthreads();
  bk = s_k[0]; bi = s_i[0]; at = s_at[0]; expanded = s_e[0]; trunc = s_t[0];
  for (int w = 1; w < 16; ++w) {
    if (key_id_less(s_k[w], s_i[w], bk, bi)) { bk = s_k[w]; bi = s_i[w]; at = s_at[w]; }
    expanded += s_e[w];
    trunc |= s_t[w];
  }
  if (bi != ~0u) {
    const unsigned long long *src = reinterpret_cast<const unsigned long long *>(a.results + at);
    unsigned long long *dst = reinterpret_cast<unsigned long long *>(out), *hst = reinterpret_cast<unsigned long long *>(host_out);
    for (uint32_t w = t; w < sizeof(SubResult) / 8; w += blockDim.x) {
      const unsigned long long v = src[w];
      dst[w] = v;
      hst[w] = v;
    }
  }
  __syncthreads();
  if (t == 0) {
    host_out->found = bi != ~0u ? 1u : 0u;
    host_out->truncated = trunc;
    host_out->expanded = expanded;
  }
}

// ------------------------------------------------------------------ listed placements

// The problem's small tables in LDS: every stage of every listed plan reads a dozen of these
// words, at addresses that differ from lane to lane.  They are laid out once per plan in device
// memory (k_list_tables), so that a workgroup copies them in one go -- a dozen loops, one per
// table, cost a trip to memory each, 5 us in front of every workgroup.
struct ListTables {
  ulonglong2 *mem;   // [G] a GPU's reserved bytes and its capacity
  double *xsec;      // [MB][Z][Z] seconds of one activation transfer
  double *bw;        // [Z][Z]
  double *ring_link; // [Z][Z] slowest link of a ring through two zones (without link profiles)
  double *egress;    // [Z][Z] (zeros without egress prices)
  double *both_ways; // [Z][Z] egress there and back, 0 inside a zone
  double *price;     // [G]
  double *ring;      // [DP] 2 (D - 1) / D
  double *tpd;       // [TP]
  double *p2p;       // [MB] bytes of one activation transfer
  uint64_t *act;     // [MB][TP]
  int32_t *nb;       // [MB][DP]
  int32_t *dpv, *tpv, *node;  // [DP], [TP], [G]
  uint32_t *zg;      // [ZGr] zone | type << 8 of a pool
  int32_t *avail;    // [ZGr] (not part of the copy: it changes between calls)
};

__host__ __device__ inline size_t list_copy_words(const DevPlan &pl) {  // 8-byte words laid out in memory
  const size_t ints = (size_t)pl.MB * pl.DP + pl.DP + pl.TP + pl.G + pl.ZGr;
  return (size_t)pl.MB * pl.Z * pl.Z + 4 * (size_t)pl.Z * pl.Z + 3 * (size_t)pl.G + pl.DP + pl.TP + pl.MB +
         (size_t)pl.MB * pl.TP + (ints + 1) / 2;
}
__host__ __device__ inline size_t list_tables_words(const DevPlan &pl) {  // with the availability behind them
  return list_copy_words(pl) + ((size_t)pl.ZGr + 1) / 2;
}

__device__ __forceinline__ ListTables list_tables_at(const DevPlan &pl, double *at) {
  const int G = pl.G, Z = pl.Z, MB = pl.MB, TP = pl.TP, DP = pl.DP;
  ListTables T;
  T.mem = reinterpret_cast<ulonglong2 *>(at);  // (first: 16-byte reads)
  T.xsec = at + 2 * G;
  T.bw = T.xsec + MB * Z * Z;
  T.ring_link = T.bw + Z * Z;
  T.egress = T.ring_link + Z * Z;
  T.both_ways = T.egress + Z * Z;
  T.price = T.both_ways + Z * Z;
  T.ring = T.price + G;
  T.tpd = T.ring + DP;
  T.p2p = T.tpd + TP;
  T.act = reinterpret_cast<uint64_t *>(T.p2p + MB);
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
    const int a = i / Z, b = i % Z, back = b * Z + a;
    T.bw[i] = pl.bw[i];
    T.ring_link[i] = a == b ? pl.bw[i] : fmin(fmin(pl.bw[a * Z + a], pl.bw[b * Z + b]), fmin(pl.bw[i], pl.bw[back]));
    T.egress[i] = pl.egress ? pl.egress[i] : 0.0;
    T.both_ways[i] = pl.egress && a != b ? pl.egress[i] + pl.egress[back] : 0.0;
  }
  for (int i = t; i < G; i += nt) {
    T.price[i] = pl.price[i];
    T.mem[i] = make_ulonglong2(pl.res[i], pl.cap[i]);
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
  for (int i = t; i < MB; i += nt) T.p2p[i] = (double)pl.p2p[i];
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

struct PlaceArgs {
  uint64_t count;
  const int32_t *desc;    // [count][5] pp index, partition, tp index, dp index, mb index
  const int32_t *pools;   // [count][pool_stride] pool of every stage
  const int32_t *pools_b; // SPLIT, same shape: pool of the other half of every stage's replicas
  const int32_t *tps;     // optional, same shape: TP index of every stage (else the descriptor's)
  uint32_t pool_stride;
  uint32_t per_wg;        // plans a workgroup takes, kPlacePlans at a time at most
  const SearchPP *pps;
  int n_pp;
  int objective, has_bound;
  double bound;
  double *T, *C;
  uint64_t *mem;
  uint32_t *mask;
  ResultHeader *hdr;      // optional, one workgroup: seq goes to hdr->seq when the results are in place
  uint32_t seq;
};

constexpr int kPlaceThreads = 256;
constexpr int kPlaceStages = 512;    // stages a workgroup holds at a time
constexpr int kPlacePlans = 64;      // and plans: a lane each when the stages are added up
static_assert(kPlaceStages >= kMaxStages, "one plan's stages fit");

struct PlaceDesc { int32_t pp, split, it, id, im; };  // a descriptor as the list has it

struct PlacePlan {       // a plan as its stages need it
  uint32_t rs;
  uint16_t end, P;       // stages of the pass's plans up to and including this one; P = 0: an invalid descriptor
  uint8_t it, id, im, pad[5];
};
static_assert(sizeof(PlacePlan) == 16, "one 16-byte read");

struct PlacePass { uint64_t first; int32_t plans, stages; };  // what is worked through at a time

struct PlaceLds {
  // two passes' plans: one is laid out while the other's results are written
  PlacePlan plan[2][kPlacePlans];
  PlacePass pass[2];
  // what the stages contribute, in plan and stage order (four entries more than there are
  // stages: the sums read four at a time): time in the two kinds of pipeline, rent, traffic
  double term[4][kPlaceStages + 4];
  double sum[4][kPlacePlans], slowest[2][kPlacePlans];   // what they add up to
  unsigned long long sync[kPlacePlans], upd[kPlacePlans];  // bits of the maxima (non-negative values, in
                                                           // which order the bits compare like them)
  unsigned long long peak[kPlacePlans];
  uint32_t flags[kPlacePlans];     // mask bits 0, 1, 3; bit 31: an index out of range
  uint8_t owner[kPlaceStages];     // the stage's plan
};
static_assert(sizeof(PlaceLds) % 16 == 0, "the tables behind it hold 16-byte words");

__host__ __device__ inline size_t place_lds_bytes(const DevPlan &pl, uint32_t per_wg) {
  return sizeof(PlaceLds) + list_tables_words(pl) * 8 +
         (size_t)(per_wg < (uint32_t)kPlacePlans ? per_wg : (uint32_t)kPlacePlans) * pl.ZGr * sizeof(int32_t);
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

// The maximum over a plan's stages that lie in the lane's row of 16, up to and including the lane
// (which is stage i of its plan): reads only lanes below.
__device__ __forceinline__ unsigned long long place_row_max(unsigned long long v, int i) {
  auto step = [&](auto ctrl, int by) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, decltype(ctrl)::value, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), decltype(ctrl)::value, 0xF, 0xF, true);
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;  // (0 from outside the row)
    v = i >= by && o > v ? o : v;
  };
  step(std::integral_constant<int, 0x111>(), 1);  // row_shr:1, 2, 4, 8
  step(std::integral_constant<int, 0x112>(), 2);
  step(std::integral_constant<int, 0x114>(), 4);
  step(std::integral_constant<int, 0x118>(), 8);
  return v;
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32 |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}

__device__ __forceinline__ PlaceDesc place_desc(const PlaceArgs &a, uint64_t c, uint64_t c_end) {
  PlaceDesc d{-1, 0, 0, 0, 0};
  if (c < c_end) {
    const int32_t *p = a.desc + c * 5;
    d = PlaceDesc{p[0], p[1], p[2], p[3], p[4]};
  }
  return d;
}

__device__ __forceinline__ SearchPP place_depth(const PlaceArgs &a, const PlaceDesc &d) {
  SearchPP pp{};
  if (d.pp >= 0 && d.pp < a.n_pp) pp = a.pps[d.pp];
  return pp;  // (n_part = 0 without a depth: no layer split is in range)
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
// A workgroup goes through a run of per_wg plans, as many at a time as have kPlaceStages stages
// between them, plans one behind the other without gaps: first a lane per stage -- what is added up
// in stage order, which is part of the definition, goes to LDS, maxima are folded in there -- then a
// lane per plan adds its stages up, a wave per quantity.  While wave 0 writes a pass's results wave 1
// lays out the next one's plans, whose descriptors were requested a pass earlier.
//
// Bound by vector instructions (31 us of the 63 below) and the latency of a pass's chain: pools, stage
// records, sums.  200 003 plans of 1 to 48 stages with two pools and a degree per stage took 488 us with
// a wave per plan (most lanes idle), 85 us with 64 plans a workgroup -- two passes, the second half
// empty, 2.4 rounds of workgroups, and the LDS busy for 40 us, mostly with maxima of 64 lanes on the same
// word -- and take 63 us this way (67 with four workgroups per compute unit, which is what the registers
// allow where the links' profiles are evaluated in the same kernel: hence PROFILES).  Measured beside
// it: runs half as long, in two rounds, 65 us; the bound on the registers for five workgroups instead of
// PROFILES 80 us (spills).  Earlier: two stages' words per lane at a time 98 instead of 85 us, 512
// threads 100 us.
template <bool SPLIT, bool PROFILES>
__global__ __launch_bounds__(kPlaceThreads) void k_eval_placements(DevPlan pl, PlaceArgs a) {
  extern __shared__ ulonglong2 place_lds[];
  PlaceLds &S = *reinterpret_cast<PlaceLds *>(place_lds);
  double *const tables = reinterpret_cast<double *>(&S + 1);
  int32_t *const cnt = reinterpret_cast<int32_t *>(tables + list_tables_words(pl));  // [plan][ZG]
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t G = pl.G, Z = pl.Z, ZG = pl.ZGr, MB = pl.MB, TP = pl.TP, DP = pl.DP;
  const uint32_t row_words = mul24(mul24(MB, TP), pl.row_w);  // of a stage's records
  const uint64_t c_begin = (uint64_t)blockIdx.x * a.per_wg, c_end = min(a.count, c_begin + a.per_wg);
  uint64_t next = c_begin;  // wave 1: the next pass's first plan, the descriptors from there on and their depths
  PlaceDesc d{};
  SearchPP pp{};
  if (wv == 1) {
    d = place_desc(a, next + lane, c_end);
    pp = place_depth(a, d);
  }
  if (wv == 0) {
    S.sync[lane] = S.upd[lane] = S.peak[lane] = 0;
    S.flags[lane] = 0;
  }
  for (int x = t; x < (int)mul24(min(a.per_wg, (uint32_t)kPlacePlans), ZG); x += kPlaceThreads) cnt[x] = 0;
  const ListTables L = stage_list_tables(pl, tables);  // (read behind the loop's first barrier)
  PlacePass done{0, 0, 0};  // the pass whose results are to be written
  for (int b = 0;; b ^= 1) {  // uniform
    if (wv == 1) {  // a lane per plan
      PlacePlan p{};
      if (d.pp >= 0 && d.split >= 0 && d.split < pp.n_part && d.it >= 0 && d.it < (int)TP && d.id >= 0 && d.id < (int)DP &&
          d.im >= 0 && d.im < (int)MB && (uint32_t)pp.P <= a.pool_stride) {
        p.P = (uint16_t)pp.P;
        p.rs = pp.rs0 + (uint32_t)d.split * (uint32_t)pp.P;
        p.it = (uint8_t)d.it; p.id = (uint8_t)d.id; p.im = (uint8_t)d.im;
      }
      const int end = (int)wave_prefix_sum(p.P);
      const int n = __popcll(__builtin_amdgcn_ballot_w64(next + lane < c_end && end <= kPlaceStages));
      const int stages = __builtin_amdgcn_readlane(end, max(n - 1, 0));
      if (lane < n) {
        p.end = (uint16_t)end;
        S.plan[b][lane] = p;
        for (int i = end - p.P; i < end; ++i) S.owner[i] = (uint8_t)lane;
      }
      if (lane == 0) S.pass[b] = PlacePass{next, n, n ? stages : 0};
      next = uniform64(next + (uint32_t)n);
      d = place_desc(a, next + lane, c_end);
    }
    if (wv == 0 && lane < done.plans) {
      double T = __builtin_huge_val(), C = T;
      uint64_t peak = 0;
      uint32_t mask = 0xFFFFFFFFu;
      const PlacePlan pn = S.plan[b ^ 1][lane];
      const uint32_t flags = S.flags[lane];
      if (pn.P != 0 && !(flags >> 31)) {
        const int nb = L.nb[pn.im * DP + pn.id];
        if (nb == 0) {
          mask = 4u;
        } else {
          mask = flags;
          peak = S.peak[lane];
          double t_pp = S.sum[0][lane] + (double)(nb - 1) * S.slowest[0][lane];
          if (SPLIT) t_pp = fmax(t_pp, S.sum[1][lane] + (double)(nb - 1) * S.slowest[1][lane]);
          T = (t_pp + __longlong_as_double((long long)S.sync[lane])) + __longlong_as_double((long long)S.upd[lane]);
          C = S.sum[2][lane] / 3600.0 * T + S.sum[3][lane];
          if (a.has_bound) {
            if (a.objective == 0) { if (C > a.bound) mask |= 32u; }
            else if (1.0 / T < a.bound) mask |= 32u;
          }
        }
      }
      const uint64_t c = done.first + (uint32_t)lane;
      if (a.T) a.T[c] = T;
      if (a.C) a.C[c] = C;
      if (a.mem) a.mem[c] = peak;
      if (a.mask) a.mask[c] = mask;
      S.sync[lane] = S.upd[lane] = S.peak[lane] = 0;
      S.flags[lane] = 0;
    }
    __syncthreads();
    done.first = uniform64(S.pass[b].first);
    done.plans = __builtin_amdgcn_readfirstlane(S.pass[b].plans);
    done.stages = __builtin_amdgcn_readfirstlane(S.pass[b].stages);
    if (done.plans == 0) break;  // uniform
    for (int e = t; e < done.stages; e += kPlaceThreads) {
      const uint32_t own = S.owner[e];
      const PlacePlan pn = S.plan[b][own];
      const int P = pn.P, i = e - (pn.end - P);
      const size_t row = (done.first + own) * a.pool_stride + (uint32_t)i;
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
      const int tp = L.tpv[ti], nb = L.nb[mul24(pn.im, DP) + pn.id], D = L.dpv[pn.id];
      const double dpd = (double)D;
      atomicAdd(&cnt[mul24(own, ZG) + a0], tp);  // GPUs of one replica (split: counted once per half)
      if (SPLIT) atomicAdd(&cnt[mul24(own, ZG) + b0], tp);
      const uint64_t bytes = model + act_bytes(min(P - i, nb), layers, L.act[mt]);
      const ulonglong2 gpu_a = L.mem[ga], gpu_b = SPLIT ? L.mem[gb] : gpu_a;
      const uint64_t m1 = bytes + gpu_a.x, m2 = bytes + gpu_b.x;
      uint32_t flags = (m1 > gpu_a.y || (SPLIT && m2 > gpu_b.y)) ? 1u : 0u;
      if (tp > L.node[ga] || (SPLIT && tp > L.node[gb])) flags |= 8u;
      if (SPLIT && a0 != b0 && (D & 1)) flags |= 2u;  // D replicas cannot be halved
      if (ra >= ZG || (SPLIT && rb >= ZG) || rt >= TP) flags |= 1u << 31;
      const uint32_t at_a = mul24(za, Z), at_b = mul24(zb, Z);  // rows of the zone tables
      const double *xsec = L.xsec + mul24(pn.im, mul24(Z, Z));
      // N_b x replicas of one kind of pipeline (each carries half of them) x bytes of a transfer
      const double one_way = (double)nb * (SPLIT ? 0.5 * dpd : dpd) * L.p2p[pn.im];
      double xa = 0.0, xb = 0.0, traffic = 0.0;
      if (fwd) {
        const uint32_t zna = L.zg[min(ran, ZG - 1)] & 255u;
        xa = xsec[at_a + zna];
        traffic = one_way * L.both_ways[at_a + zna];
        if (SPLIT) {
          const uint32_t znb = L.zg[min(rbn, ZG - 1)] & 255u;
          xb = xsec[at_b + znb];
          traffic += one_way * L.both_ways[at_b + znb];
        }
      }
      if (back) {
        xa += xsec[at_a + (L.zg[min(rap, ZG - 1)] & 255u)];
        if (SPLIT) xb += xsec[at_b + (L.zg[min(rbp, ZG - 1)] & 255u)];
      }
      const double ring_bytes = D > 1 ? L.ring[pn.id] * grad : 0.0;
      if (SPLIT) traffic += ring_bytes * L.both_ways[at_a + zb];
      auto slowest_sync = [&] {  // of the plan's stages in the lane's row up to here
        double sync = 0.0;
        if (D > 1) {
          double link;
          if (PROFILES) {
            link = link_bw(pl, za, za, grad);
            if (SPLIT && zb != za)
#pragma unroll 1
              for (int q = 1; q < 4; ++q) link = fmin(link, link_bw(pl, q == 2 ? za : zb, q == 3 ? za : zb, grad));  // within b, there, back
          } else {
            link = L.ring_link[at_a + (SPLIT ? zb : za)];
          }
          sync = ring_bytes / link;
        }
        return place_row_max((unsigned long long)__double_as_longlong(sync), i);
      };
      // (the profiles of four links go last, one after the other: with the rest of the stage behind them
      // they took 112 registers instead of 103.  Everywhere else the quotient is better started early.)
      constexpr bool kLinksLast = SPLIT && PROFILES;
      unsigned long long most_sync = 0;
      if (!kLinksLast) most_sync = slowest_sync();
      S.term[0][e] = ca + xa;
      if (SPLIT) S.term[1][e] = cb + xb;
      const double gpus = dpd * L.tpd[ti];  // (whole numbers below 2^53)
      S.term[2][e] = gpus * (SPLIT ? 0.5 * (L.price[ga] + L.price[gb]) : L.price[ga]);
      S.term[3][e] = traffic;
      // (an LDS atomic takes a cycle per lane on the same word, and a plan's stages lie side by side)
      const unsigned long long most_upd = place_row_max((unsigned long long)__double_as_longlong(SPLIT ? fmax(ua, ub) : ua), i);
      const unsigned long long most = place_row_max(m1 > m2 ? m1 : m2, i);
      const bool last = (lane & 15) == 15 || i == P - 1;
      if (last) {
        if (!kLinksLast) atomicMax(&S.sync[own], most_sync);
        atomicMax(&S.upd[own], most_upd);
        atomicMax(&S.peak[own], most);
      }
      if (flags) atomicOr(&S.flags[own], flags);
      if (kLinksLast) {
        most_sync = slowest_sync();
        if (last) atomicMax(&S.sync[own], most_sync);
      }
    }
    if (wv == 1) pp = place_depth(a, d);
    __syncthreads();
    if (lane < done.plans && (SPLIT || wv != 1)) {  // a lane per plan, a wave per quantity
      const PlacePlan pn = S.plan[b][lane];
      double sum, slowest;
      place_sum(S.term[wv] + (pn.end - pn.P), pn.P, sum, slowest);
      S.sum[wv][lane] = sum;
      if (wv < 2) S.slowest[wv][lane] = slowest;
    }
    for (int x = t; x < (int)mul24(done.plans, ZG); x += kPlaceThreads) {  // every pool holds what is placed on it
      const int q = (int)((uint32_t)x / ZG), pool = x - (int)mul24(q, ZG);
      if ((int64_t)cnt[x] * L.dpv[S.plan[b][q].id] > (SPLIT ? 2 : 1) * (int64_t)L.avail[pool])
        atomicOr(&S.flags[q], 2u);
      cnt[x] = 0;
    }
    __syncthreads();
  }
  if (a.hdr && t == 0) publish(a.hdr, a.seq);  // (one plan: this lane wrote its results)
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
static_assert(sizeof(ReplicaLds) % 16 == 0, "the tables behind it hold 16-byte words");

__host__ __device__ inline size_t replica_lds_bytes(const DevPlan &pl) {
  return sizeof(ReplicaLds) + list_tables_words(pl) * 8 + kReplicaWaves * (size_t)pl.ZGr * sizeof(int32_t);
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
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
      const ulonglong2 gpu = L.mem[g];
      const uint64_t m = model + act_bytes(min(P - i, nb), layers, L.act[mt]) + gpu.x;
      if (m > gpu.y) s.flags |= 1u;
      if (tp > L.node[g]) s.flags |= 8u;
      s.peak = m > s.peak ? m : s.peak;
      double x = 0.0;
      if (i < P - 1) {
        x += xsec[mul24(z, Z) + zn];
        s.traffic += one_traffic * L.both_ways[mul24(z, Z) + zn];  // one replica's microbatches
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
  s.peak = wave_max_u64(s.peak);
  s.flags = wave_fold(s.flags, [](uint32_t x, uint32_t y) { return x | y; });
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
// took 225 us; they take 44 us now, half of the workgroups being done after 12 us: what is left is
// the chain of trips in front of a plan and the workgroups that hold several large plans.
__global__ __launch_bounds__(kReplicaWaves * 64) void k_eval_replicas(DevPlan pl, ReplicaArgs a) {
  extern __shared__ ulonglong2 rep_lds[];
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

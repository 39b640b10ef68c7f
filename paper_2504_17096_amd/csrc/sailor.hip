// Host side of the C ABI declared in include/sailor.h: validation, upload, launches,
// decoding of winning indices.  No simulator arithmetic runs here.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/sailor.h"
#include "sailor_kernels.hip.h"
#include "sailor_search.hip.h"

using namespace sailor;

namespace {

constexpr uint32_t kDefaultSurvCap = 1u << 22;  // 96 MiB of survivors
constexpr uint32_t kDefaultRefCap = 1u << 18;
// What a plan starts with (2 MiB): a query keeps some hundreds, and the few that keep more enlarge the
// buffers to the above.  (A plan's destruction took 0.55 ms, most of it the release of the 96 MiB, and 4.3 ms
// for minutes when the driver was behind with such releases.)
constexpr uint32_t kFirstSurvCap = 1u << 16, kFirstRefCap = 1u << 14;
// candidates per scan workgroup: large enough to amortise the staging of a unit, small
// enough to leave about ten workgroups per compute unit
constexpr uint64_t kUnitTargetMin = 4096, kUnitTargetMax = 65536, kUnitsWanted = 2560;
// workgroups that share one unit in the collect pass, and the units it visits per round (64 best of 9.2e8 plans:
// 14.5 us with 8 and 256, where two units fall to one group more often; 12.7 with these)
constexpr uint32_t kCollectSub = 4, kCollectUnits = 512;
// A running k-th key takes longer to be found than a running minimum and rules out less: spaces up to twice the
// chip's waves (8 192) are scanned unguided for it (k = 26 of 3 600 units of four waves with pairs of types 74 -> 64 us, k = 53
// of 5 580 units of two waves, 706 of them within a budget, 58 -> 38; cheapest of 2 806 units of three waves 40, unguided 99)
constexpr size_t kCuWaves = 32;
constexpr size_t kGuidedKthChips = 2;
// Pairs of types make a unit long enough that the best plan's scan is guided wherever there is a unit to wait
// (fastest of 2 295 units of three waves 114 us as they come and 37 guided, of 1 464 86 and 37, of 324 39 and 27).
constexpr size_t kGuidedMixedWavesPerCu = 2;
// What the first units of a scan take from launch to a result, at 100 MHz.  (Where a constraint leaves the first units
// nothing, the wait is for nothing: cheapest of 7 296 units at 0.87 of the largest throughput 41 us with 8 us, 37 with 5;
// those that find something have by then.  With 3 us that query takes 34, but pairs of types 68 instead of 31.)
constexpr uint32_t kBestSeedTicks = 500, kKthSeedTicks = 800;
constexpr uint32_t kKthLive = 128;       // largest k whose running bound guides the scan (half the key slots)
// A query whose constraint leaves at most this many units alive skips the scan: one pass
// keeps every valid candidate of those units (see run_selection_impl)
constexpr uint32_t kDirectUnits = 128;
constexpr uint32_t kDirectSub = 16;             // workgroups that share one of them
constexpr uint32_t kFreshWorkgroups = 16;       // that bring the quota table up to date beside a call's first kernel
constexpr uint32_t kDirectManySurvivors = 8192;  // more than the select kernel holds in registers
                                                // (or than half the survivor buffer): the query
                                                // goes back to the scan from then on
constexpr uint32_t kRankOneWorkgroup = 128;  // largest k whose final ranking runs as one workgroup
constexpr uint32_t kEvalUnitTarget = 16384;  // candidates per workgroup of the range evaluation
constexpr unsigned kEvalRowsThreads = 512;
constexpr uint32_t kSearchWorkgroups = 1024, kRootWorkgroups = 1024;  // of the search's two kernels
constexpr size_t kSearchLds = 80 * 1024;       // LDS of a search workgroup: two fit a compute unit
constexpr size_t kSearchMaxLds = 160 * 1024 - kSearchStaticLds;  // most dynamic LDS of one
constexpr uint64_t kPlaceUnits = 256;      // compute units a list of placements is spread over
constexpr uint64_t kPlaceLongest = 256;    // plans a workgroup takes at most
constexpr uint64_t kPlaceShort = 32 * 1024;  // plans of a list that takes four workgroups per compute unit at most
constexpr size_t kEvalRowsMaxLds = 64 * 1024;  // above this the range form evaluates lane by lane
constexpr size_t kScanMaxLds = 160 * 1024;     // a scan workgroup stages its records within the LDS of a compute unit
#define HIP_TRY(expr)                                                              \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess) {                                                        \
      std::fprintf(stderr, "sailor: %s failed: %s\n", #expr, hipGetErrorString(e_)); \
      return SAILOR_EDEVICE;                                                       \
    }                                                                              \
  } while (0)

std::atomic<int> g_forced_unit_parts{0};         // sailor_set_scan_unit_parts

// Lets its thread allocate while a graph is captured: an allocation is refused otherwise, and the capture lost.
class BesideCaptures {
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;  // (the calls exchange it with the thread's own)
 public:
  BesideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  ~BesideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
};

struct DeviceArena {  // every device allocation of a plan, freed together
  std::vector<void *> ptrs;
  template <typename T>
  hipError_t alloc(T **out, size_t n) {
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, std::max<size_t>(n, 1) * sizeof(T));
    if (e == hipSuccess) ptrs.push_back(p);
    *out = static_cast<T *>(p);
    return e;
  }
  template <typename T>
  hipError_t upload(const T **out, const T *src, size_t n) {
    T *p = nullptr;
    hipError_t e = alloc(&p, n);
    if (e != hipSuccess) return e;
    *out = p;
    return n ? hipMemcpy(p, src, n * sizeof(T), hipMemcpyHostToDevice) : hipSuccess;
  }
  void free_one(void *p) {
    for (size_t i = 0; i < ptrs.size(); ++i)
      if (ptrs[i] == p) {
        (void)hipFree(p);
        ptrs.erase(ptrs.begin() + (long)i);
        return;
      }
  }
  void release() {
    for (void *p : ptrs) (void)hipFree(p);
    ptrs.clear();
  }
};

// The tables a plan keeps for its lifetime, as one allocation with one upload.  Pointers are
// announced first and set by commit(): inputs (copied from host memory that must live until then),
// zero-filled tables, uninitialised ones, each on a 256-byte boundary.  (Sixty allocations, twenty
// copies of 20 to 40 us each and as many frees were 1.6 ms of the 5.1 ms that a new job on 1.1e9
// plans took.)
class TableSlab {
 public:
  template <typename T>
  void input(const T **out, const T *src, size_t n) { add(kInput, out, src, n * sizeof(T)); }
  template <typename T>
  void zeroed(T **out, size_t n) { add(kZeroed, out, nullptr, n * sizeof(T)); }
  template <typename T>
  void table(T **out, size_t n) { add(kTable, out, nullptr, n * sizeof(T)); }
  hipError_t commit(DeviceArena &arena) {
    size_t end[3], at = 0;
    for (int kind : {kInput, kZeroed, kTable}) {
      for (Entry &e : entries_)
        if (e.kind == kind) {
          e.at = at;
          at += (std::max<size_t>(e.bytes, 1) + 255) & ~(size_t)255;
        }
      end[kind] = at;
    }
    char *base = nullptr;
    hipError_t err = arena.alloc(&base, at);
    if (err != hipSuccess) return err;
    std::vector<char> staging(end[kInput]);
    for (const Entry &e : entries_) {
      void *p = base + e.at;
      std::memcpy(e.out, &p, sizeof p);
      if (e.kind == kInput && e.bytes) std::memcpy(&staging[e.at], e.src, e.bytes);
    }
    if (!staging.empty()) err = hipMemcpy(base, staging.data(), staging.size(), hipMemcpyHostToDevice);
    if (err == hipSuccess && end[kZeroed] > end[kInput])
      err = hipMemset(base + end[kInput], 0, end[kZeroed] - end[kInput]);
    return err;
  }

 private:
  enum Kind { kInput, kZeroed, kTable };
  struct Entry {
    Kind kind;
    void *out;  // where the pointer goes
    const void *src;
    size_t bytes, at;
  };
  void add(Kind kind, void *out, const void *src, size_t bytes) { entries_.push_back({kind, out, src, bytes, 0}); }
  std::vector<Entry> entries_;
};

// The positions 0 .. n - 1 in ascending (descending) order of non-negative values, equal ones in
// the order they come in: three counting passes over the values' bits.
std::vector<uint32_t> order_by(const float *values, size_t n, bool descending) {
  constexpr int kBits = 11, kBins = 1 << kBits;
  std::vector<uint32_t> from(n), to(n), keys(n);
  for (size_t i = 0; i < n; ++i) {
    const uint32_t bits = __builtin_bit_cast(uint32_t, values[i]) & 0x7fffffffu;
    keys[i] = descending ? 0x7fffffffu - bits : bits;
    from[i] = (uint32_t)i;
  }
  for (int shift = 0; shift < 32; shift += kBits) {
    uint32_t at[kBins] = {};
    for (uint32_t k : keys) ++at[(k >> shift) & (kBins - 1)];
    uint32_t sum = 0;
    for (uint32_t &a : at) { const uint32_t c = a; a = sum; sum += c; }
    for (uint32_t i : from) to[at[(keys[i] >> shift) & (kBins - 1)]++] = i;
    from.swap(to);
  }
  return from;
}

}  // namespace

struct sailor_plan {
  DevPlan dev{};
  DirectMem direct_mem{};
  DeviceArena arena;
  std::vector<ShapeRec> shapes;
  std::vector<BlockRec> blocks;
  std::vector<UnitRec> units;
  std::vector<EvalBlock> eblocks;  // range evaluation: a block's units (laid out on the device)
  uint64_t n_eunits = 0;
  size_t cus = 0;                  // compute units of the device
  uint32_t n_groups = 0;           // units of one shape and tp per segment are a group: see k_group_bounds
  EvalUnit *d_eunits = nullptr;    // ascending idx_lo
  size_t eval_lds_bytes = 0;
  std::vector<int32_t> mbv, tpv, dpv, ppv;
  std::vector<uint16_t> xt;        // real types a | b << 8 of every extended type
  int device = 0;
  size_t lds_bytes = 0;
  unsigned unit_threads = 256;
  uint32_t seq = 0;                // sequence number of the last selection's final kernel
  ResultHeader last_hdr{};         // of the last successful selection
  bool have_hdr = false;
  int32_t *d_avail = nullptr;
  int32_t *h_avail = nullptr;      // the availability table, host-mapped (behind h_result)
  const int32_t *h_avail_dev = nullptr;  // the same memory as the device addresses it
  bool avail_dirty = false;        // h_avail is newer than the device copy
  // scratch of the selection pipeline
  float *umin_s = nullptr, *umin_l = nullptr;
  float *rows = nullptr;  // [unit][2][DP] bounds by degree, of the time and of the cost (k_group_bounds)
  // the units in ascending order of either bound (device), and the sorted bounds (host)
  uint32_t *order_time = nullptr, *order_cost = nullptr;
  uint32_t *order_work = nullptr;  // the longest first, once a scan without a limit has had it made
  uint8_t *work_bucket = nullptr;
  bool work_ordered = false;
  std::vector<float> lb_time_sorted, lb_cost_sorted;
  // the last query whose direct pass kept too many candidates (it is not tried again)
  bool direct_declined = false;
  int declined_obj = 0;
  float declined_lim = 0.f;
  bool last_direct = false;       // the last successful selection took the direct pass
  uint32_t last_direct_units = 0; // over this many units
  uint32_t *counters = nullptr;
  uint32_t *ulist = nullptr;   // units the collect pass has to visit
  SurvRec *surv = nullptr;
  RefRec *ref = nullptr;
  uint32_t surv_cap = kFirstSurvCap, ref_cap = kFirstRefCap;
  bool scratch_grows = true;   // they are what the plan started with
  // host-mapped result area: header + SAILOR_MAX_K records
  void *h_result = nullptr;
  ResultHeader *d_hdr = nullptr;
  RefRec *d_out = nullptr;
  RefRec *staged = nullptr;    // device-side copy of the top-k records before they go to the host
  // re-planning: per-unit minima of the last scan are kept while the query stays the same
  uint32_t *unit_gen = nullptr;   // device, per unit: availability generation of its minima
  uint32_t *unit_seq = nullptr;   // device, per unit: the call that evaluated it last
  uint32_t *ubits = nullptr;      // device, per unit: validity words as last staged
  uint32_t last_scan_seq = 0;     // call_seq of the last successful selection's scan
  uint32_t ubits_stride = 0;
  uint32_t avail_gen = 1;         // bumped whenever a new availability table reaches the device
  bool incremental = false;       // sailor_plan_set_incremental
  bool cache_ok = false;          // the minima on the device belong to the query below
  int cache_obj = 0, cache_hasb = 0;
  float cache_lim_s = 0.f, cache_lim_l = 0.f;
  bool last_incremental = false;  // the last successful selection reused minima
  // search over per-stage placements: tables and scratch, created by the first call
  std::vector<SearchPP> search_pps;
  const SearchPP *d_search_pps = nullptr;
  std::vector<int32_t> row_layers;    // layers per stage of every layer split
  const uint32_t *search_alike = nullptr;
  uint32_t n_sub = 0, n_sub_t = 0;  // sub-problems with TP in them / with a TP degree per stage
  double *search_states = nullptr;    // frontiers and histories that do not fit LDS (wide beams), and
  uint32_t *search_history = nullptr; // how many words of them there are
  size_t search_states_cap = 0, search_history_cap = 0;
  uint32_t *search_list = nullptr, *search_counters = nullptr;
  unsigned long long *search_root_expanded = nullptr;
  SubResult *search_results = nullptr, *search_final = nullptr;
  bool search_dirty = true;           // the counters are not zero
  uint32_t calls = 0;          // number of the next selection; its lowest bit says which counter set it uses
  bool counters_dirty = false; // a failed call may have left either set in any state
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};  // start, scan end, end, scan start
  int timing_mode = 0;         // 0 none, 1 dominant kernel, 2 dominant kernel + whole call
  bool total_timed = false, scan_timed = false;
};

namespace {

bool ascending_positive(const int32_t *v, int n) {
  if (!v || n < 1) return false;
  for (int i = 0; i < n; ++i) {
    if (v[i] < 1) return false;
    if (i && v[i] <= v[i - 1]) return false;
  }
  return true;
}

bool finite_nonneg(const double *v, size_t n) {
  for (size_t i = 0; i < n; ++i)
    if (!(v[i] >= 0.0) || !std::isfinite(v[i])) return false;
  return true;
}

// types a segment can choose: the plain ones and, with mixed replicas, every pair of them
int extended_types(const sailor_problem *p) {
  return p->mixed_types ? p->n_types + p->n_types * (p->n_types - 1) / 2 : p->n_types;
}

uint64_t n_cut_choices(int P, int s);

sailor_status validate(const sailor_problem *p) {
  if (!p) return SAILOR_EINVAL;
  if (p->n_layers < 1 || p->n_types < 1 || p->n_zones < 1) return SAILOR_EINVAL;
  if (p->n_types > SAILOR_MAX_TYPES || p->n_zones > SAILOR_MAX_ZONES) return SAILOR_EINVAL;
  if (p->n_types * p->n_zones > SAILOR_MAX_POOLS) return SAILOR_EINVAL;
  if (p->n_mb < 1 || p->n_mb > SAILOR_MAX_MB || p->n_tp < 1 || p->n_tp > SAILOR_MAX_TP ||
      p->n_dp < 1 || p->n_dp > SAILOR_MAX_DP || p->n_pp < 1)
    return SAILOR_EINVAL;
  if (p->max_segments < 1 || p->max_segments > 3 || p->global_batch < 1) return SAILOR_EINVAL;
  if (p->per_segment_tp != 0 && p->per_segment_tp != 1) return SAILOR_EINVAL;
  if (p->mixed_types != 0 && p->mixed_types != 1) return SAILOR_EINVAL;
  if (p->n_zones * extended_types(p) > SAILOR_MAX_POOLS) return SAILOR_EINVAL;
  if (p->n_bw_coef < 0 || p->n_bw_coef > SAILOR_MAX_BW_COEF || (p->n_bw_coef > 0 && !p->bw_poly))
    return SAILOR_EINVAL;
  if (!ascending_positive(p->mb_values, p->n_mb) || !ascending_positive(p->tp_values, p->n_tp) ||
      !ascending_positive(p->dp_values, p->n_dp) || !ascending_positive(p->pp_values, p->n_pp))
    return SAILOR_EINVAL;
  if (!p->n_partitions || !p->partition_layers || !p->layer_params || !p->t_fwd || !p->t_bwd ||
      !p->t_upd || !p->act_store_bytes || !p->p2p_bytes || !p->mem_capacity || !p->mem_reserved ||
      !p->gpus_per_node || !p->price_per_hour || !p->avail || !p->bandwidth)
    return SAILOR_EINVAL;
  const int G = p->n_types, Z = p->n_zones, L = p->n_layers;
  size_t row = 0;
  for (int ip = 0; ip < p->n_pp; ++ip) {
    const int P = p->pp_values[ip];
    if (P > L || P > SAILOR_MAX_STAGES || p->n_partitions[ip] < 1) return SAILOR_EINVAL;
    for (int q = 0; q < p->n_partitions[ip]; ++q) {
      int64_t sum = 0;
      for (int i = 0; i < P; ++i) {
        const int32_t n = p->partition_layers[row++];
        if (n < 1) return SAILOR_EINVAL;
        sum += n;
      }
      if (sum != L) return SAILOR_EINVAL;
    }
  }
  {  // shapes (layer split x cut points) carry per-shape tables: keep their number bounded
    uint64_t n_shapes = 0;
    for (int ip = 0; ip < p->n_pp; ++ip)
      for (int s = 1; s <= p->max_segments; ++s) {
        const int P = p->pp_values[ip];
        if (s > P || (s == 3 && P > p->seg3_max_pp)) continue;
        n_shapes += n_cut_choices(P, s) * (uint64_t)p->n_partitions[ip];
        if (n_shapes > (uint64_t)SAILOR_MAX_SHAPES) return SAILOR_EINVAL;
      }
  }
  // the quota table has one row per GPU count a replica can take from a pool
  if ((int64_t)p->pp_values[p->n_pp - 1] * p->tp_values[p->n_tp - 1] > (1 << 20)) return SAILOR_EINVAL;
  const size_t Lc = p->uniform_layers ? 1 : (size_t)L;
  if (!finite_nonneg(p->t_fwd, (size_t)G * p->n_mb * p->n_tp * Lc) ||
      !finite_nonneg(p->t_bwd, (size_t)G * p->n_mb * p->n_tp * Lc) ||
      !finite_nonneg(p->t_upd, (size_t)G * p->n_tp * Lc) ||
      !finite_nonneg(p->price_per_hour, G))
    return SAILOR_EINVAL;
  for (int i = 0; i < Z * Z; ++i)
    if (!(p->bandwidth[i] > 0.0) || !std::isfinite(p->bandwidth[i])) return SAILOR_EINVAL;
  if (p->egress_per_byte && !finite_nonneg(p->egress_per_byte, (size_t)Z * Z)) return SAILOR_EINVAL;
  for (size_t i = 0; i < (size_t)Z * Z * p->n_bw_coef; ++i)
    if (!std::isfinite(p->bw_poly[i])) return SAILOR_EINVAL;
  for (int i = 0; i < Z * G; ++i)
    if (p->avail[i] < 0) return SAILOR_EINVAL;
  for (int g = 0; g < G; ++g)
    if (p->gpus_per_node[g] < 1) return SAILOR_EINVAL;
  // byte counts must stay far below 2^64: total parameters * bytes + the largest
  // activation term + reserved
  unsigned __int128 params = (unsigned __int128)p->embed_params + p->head_params;
  for (int l = 0; l < L; ++l) params += p->layer_params[l];
  uint64_t act_max = 0, res_max = 0;
  for (int i = 0; i < p->n_mb * p->n_tp; ++i) act_max = std::max(act_max, p->act_store_bytes[i]);
  for (int g = 0; g < G; ++g) res_max = std::max(res_max, p->mem_reserved[g]);
  unsigned __int128 worst = params * p->bytes_per_param +
                            (unsigned __int128)act_max * (unsigned)L * (unsigned)SAILOR_MAX_STAGES +
                            res_max;
  if (worst >> 62) return SAILOR_EINVAL;
  for (int g = 0; g < G; ++g)
    if (p->mem_capacity[g] >> 62) return SAILOR_EINVAL;
  for (int m = 0; m < p->n_mb; ++m)
    if (p->p2p_bytes[m] >> 53) return SAILOR_EINVAL;
  return SAILOR_OK;
}

uint64_t n_cut_choices(int P, int s) {
  if (s == 1) return 1;
  if (s == 2) return (uint64_t)(P - 1);
  return (uint64_t)(P - 1) * (uint64_t)(P - 2) / 2;
}

// Lays the candidate space out as blocks -> shapes -> scan units (host bookkeeping only).
sailor_status build_space(const sailor_problem *p, sailor_plan *pl, std::vector<int32_t> &st_n,
                          std::vector<int32_t> &st_first, std::vector<uint8_t> &st_flags) {
  const int ZG = extended_types(p) * p->n_zones;
  const uint64_t inner = (uint64_t)p->n_mb * p->n_tp * p->n_dp * ZG;
  const int pst = p->per_segment_tp ? 1 : 0;
  const uint64_t otp = pst ? (uint64_t)p->n_tp : 1u;  // radix of the tp digits of segments 2, 3
  uint64_t off = 0;
  uint32_t row_stage = 0;
  size_t row = 0;
  for (int ip = 0; ip < p->n_pp; ++ip) {
    const int P = p->pp_values[ip];
    const uint32_t row_stage0 = row_stage;
    for (int q = 0; q < p->n_partitions[ip]; ++q) {
      int first = 0;
      for (int i = 0; i < P; ++i) {
        const int32_t n = p->partition_layers[row++];
        st_n.push_back(n);
        st_first.push_back(first);
        st_flags.push_back((uint8_t)((i == 0 ? 1 : 0) | (i == P - 1 ? 2 : 0)));
        first += n;
      }
      row_stage += P;
    }
    for (int s = 1; s <= 3; ++s) {
      if (s > p->max_segments || s > P || (s == 3 && P > p->seg3_max_pp)) continue;
      uint64_t shape_size = inner;
      for (int j = 1; j < s; ++j) shape_size *= (uint64_t)(ZG - 1) * otp;
      if (shape_size == 0) continue;
      BlockRec b{};
      b.off = off;
      b.first_shape = (uint32_t)pl->shapes.size();
      b.shape_size = shape_size;
      b.pp_idx = ip;
      b.s = s;
      b.P = P;
      for (int q = 0; q < p->n_partitions[ip]; ++q)
        for (int k1 = (s >= 2 ? 1 : P); k1 <= (s >= 2 ? P - (s - 1) : P); ++k1)
          for (int k2 = (s == 3 ? k1 + 1 : P); k2 <= (s == 3 ? P - 1 : P); ++k2) {
            ShapeRec sh{};
            sh.base = off;
            sh.row_stage = row_stage0 + (uint32_t)q * P;
            sh.pp_idx = ip;
            sh.q = q;
            sh.P = (uint16_t)P;
            sh.s = (uint16_t)s;
            sh.k1 = (uint16_t)k1;
            sh.k2 = (uint16_t)k2;
            const int edges[4] = {0, k1, k2, P};
            for (int j = 0; j < 3; ++j) {
              sh.lo[j] = (uint16_t)(j < s ? edges[j] : 0);
              sh.n[j] = (uint16_t)(j < s ? edges[j + 1] - edges[j] : 0);
            }
            if (s == 1) sh.n[0] = (uint16_t)P;
            if (s == 2) sh.n[1] = (uint16_t)(P - k1);
            pl->shapes.push_back(sh);
            off += shape_size;
          }
      b.n_shapes = (uint32_t)pl->shapes.size() - b.first_shape;
      b.size = off - b.off;
      if (b.n_shapes != n_cut_choices(P, s) * (uint64_t)p->n_partitions[ip]) return SAILOR_EINVAL;
      pl->blocks.push_back(b);
    }
  }
  pl->dev.N = off;
  pl->dev.inner = (uint32_t)inner;
  pl->dev.n_row_stages = (int)row_stage;
  pl->dev.pst = pst;
  pl->dev.otp = (int)otp;
  pl->dev.stride3 = inner * (uint64_t)(ZG - 1) * otp;

  // scan units: (shape, tp of every segment, range of segment 2's pool)
  const uint64_t unit_target =
      std::min(kUnitTargetMax, std::max(kUnitTargetMin, pl->dev.N / kUnitsWanted));
  const uint64_t innerp = (uint64_t)p->n_mb * p->n_dp * ZG;
  uint32_t group = 0;
  for (uint32_t si = 0; si < pl->shapes.size(); ++si) {
    const ShapeRec &sh = pl->shapes[si];
    const int n_o = sh.s >= 2 ? ZG : 1;
    const uint64_t per_o = sh.s == 3 ? innerp * (uint64_t)(ZG - 1) : innerp;
    int chunk = (int)std::min<uint64_t>((uint64_t)n_o, std::max<uint64_t>(1, unit_target / per_o));
    const int n_chunks = (n_o + chunk - 1) / chunk;
    const int n_t1 = (pst && sh.s >= 2) ? p->n_tp : 1, n_t2 = (pst && sh.s == 3) ? p->n_tp : 1;
    for (int t2 = 0; t2 < n_t2; ++t2)
      for (int t1 = 0; t1 < n_t1; ++t1)
        for (int t = 0; t < p->n_tp; ++t, ++group)
          for (int c = 0; c < n_chunks; ++c) {
            const int lo = (int)((int64_t)n_o * c / n_chunks),
                      hi = (int)((int64_t)n_o * (c + 1) / n_chunks);
            UnitRec u{};
            u.shape = si;
            u.tp[0] = (uint8_t)t;
            u.tp[1] = (uint8_t)(pst ? t1 : t);
            u.tp[2] = (uint8_t)(pst ? t2 : t);
            u.s = (uint8_t)sh.s;
            u.o_lo = (uint16_t)lo;
            u.o_cnt = (uint16_t)(hi - lo);
            for (int j = 0; j < 3; ++j) u.n[j] = sh.n[j];
            u.part = 0;
            u.n_parts = 1;
            u.group = group;
            u.base = sh.base + (pst ? inner * (uint64_t)(ZG - 1) * (uint64_t)t1 +
                                          pl->dev.stride3 * (uint64_t)(ZG - 1) * (uint64_t)t2
                                    : 0u);
            pl->units.push_back(u);
          }
  }
  if (pl->units.size() > (size_t)0x7fffffff / kCollectSub) return SAILOR_EINVAL;
  // units of the range evaluation: (shape, range of the outer digits), about 16 Ki
  // candidates each, in index order; the shapes of a block are divided alike
  for (const BlockRec &b : pl->blocks) {
    EvalBlock e{};
    e.off = b.off;
    e.shape_size = b.shape_size;
    e.o_total = b.shape_size / inner;
    e.first_unit = pl->n_eunits;
    e.first_shape = b.first_shape;
    e.chunk = (uint32_t)std::min<uint64_t>(
        std::min<uint64_t>(e.o_total, kEvalUnitMaxOuter), std::max<uint64_t>(1, kEvalUnitTarget / inner));
    e.per_shape = (e.o_total + e.chunk - 1) / e.chunk;
    e.first_group = pl->n_groups;
    e.groups = (uint32_t)p->n_tp;
    for (uint32_t j = 1; pst && j < b.s; ++j) e.groups *= (uint32_t)p->n_tp;
    pl->n_groups += e.groups * b.n_shapes;
    pl->eblocks.push_back(e);
    pl->n_eunits += e.per_shape * b.n_shapes;
  }
  if (pl->n_groups != group) return SAILOR_EINVAL;
  // Waves per workgroup: the lanes of a unit cover MB*DP*ZG triples in chunks of 64; pick
  // the wave count (2..8) that leaves the fewest idle wave slots in the last round.
  const uint64_t chunks = (innerp + 63) / 64;
  unsigned best_w = 4;
  double best_eff = 0.0;
  for (unsigned w = 2; w <= kMaxUnitThreads / 64; ++w) {
    const uint64_t rounds = (chunks + w - 1) / w;
    const double eff = (double)chunks / (double)(rounds * w);
    if (eff > best_eff + 1e-9 || (eff > best_eff - 1e-9 && w == 4)) { best_eff = eff; best_w = w; }
  }
  pl->unit_threads = best_w * 64;
  return SAILOR_OK;
}

sailor_status constraint_limits(sailor_objective obj, const sailor_constraint *c, int *has_bound,
                                double *bound, float *lim_s, float *lim_l) {
  *has_bound = (c && c->has_bound) ? 1 : 0;
  *bound = 0.0;
  *lim_s = *lim_l = kPosInf;
  if (!*has_bound) return SAILOR_OK;
  if (std::isnan(c->bound)) return SAILOR_EINVAL;
  *bound = c->bound;
  // the fp32 scan compares cost <= bound, or time <= 1 / bound (throughput floor)
  double lim = obj == SAILOR_MAX_THROUGHPUT ? c->bound : 1.0 / c->bound;
  if (obj == SAILOR_MIN_COST && c->bound <= 0.0) lim = HUGE_VAL;
  if (lim < 0.0) {
    *lim_s = *lim_l = -1.0f;  // nothing satisfies a negative cost bound
    return SAILOR_OK;
  }
  *lim_s = std::nextafterf((float)(lim * (1.0 - (double)kEvalEps)), 0.0f);
  *lim_l = std::nextafterf((float)(lim * (1.0 + (double)kEvalEps)), kPosInf);
  return SAILOR_OK;
}

void fill_config(const sailor_plan *pl, const ShapeRec &sh, uint64_t index, sailor_result *out) {
  const DevPlan &d = pl->dev;
  std::memset(out, 0, sizeof *out);
  out->index = index;
  const BlockRec *blk = &pl->blocks[0];
  for (const BlockRec &b : pl->blocks)
    if (index >= b.off) blk = &b;
  uint64_t rem = (index - blk->off) % blk->shape_size;
  const uint32_t in = (uint32_t)(rem % d.inner);
  uint32_t o = (uint32_t)(rem / d.inner);
  out->mb_index = in % d.MB;
  out->tp_index = (in / d.MB) % d.TP;
  out->dp_index = (in / (d.MB * d.TP)) % d.DP;
  out->pool[0] = in / (d.MB * d.TP * d.DP);
  out->pool[1] = out->pool[2] = -1;
  out->seg_tp_index[0] = out->tp_index;
  out->seg_tp_index[1] = out->seg_tp_index[2] = -1;
  if (sh.s >= 2) {
    out->pool[1] = (out->pool[0] + 1 + (int)(o % (d.ZG - 1))) % d.ZG;
    o /= (d.ZG - 1);
    out->seg_tp_index[1] = d.pst ? (int32_t)(o % d.TP) : out->tp_index;
    if (d.pst) o /= d.TP;
  }
  if (sh.s == 3) {
    out->pool[2] = (out->pool[1] + 1 + (int)(o % (d.ZG - 1))) % d.ZG;
    o /= (d.ZG - 1);
    out->seg_tp_index[2] = d.pst ? (int32_t)o : out->tp_index;
  }
  for (int j = 0; j < 3; ++j) {
    out->seg_tp[j] = out->seg_tp_index[j] >= 0 ? pl->tpv[out->seg_tp_index[j]] : 0;
    const bool used = out->pool[j] >= 0;
    out->zone[j] = used ? out->pool[j] / d.GX : -1;
    out->type_a[j] = used ? (pl->xt[out->pool[j] % d.GX] & 255) : -1;
    out->type_b[j] = used ? (pl->xt[out->pool[j] % d.GX] >> 8) : -1;
  }
  out->pp_index = sh.pp_idx;
  out->pp = sh.P;
  out->mb = pl->mbv[out->mb_index];
  out->tp = pl->tpv[out->tp_index];
  out->dp = pl->dpv[out->dp_index];
  out->partition = sh.q;
  out->n_segments = sh.s;
  out->cut[0] = sh.k1;
  out->cut[1] = sh.k2;
}

const ShapeRec &shape_of(const sailor_plan *pl, uint64_t index) {
  const BlockRec *blk = &pl->blocks[0];
  for (const BlockRec &b : pl->blocks)
    if (index >= b.off) blk = &b;
  return pl->shapes[blk->first_shape + (index - blk->off) / blk->shape_size];
}

unsigned quota_grid(const DevPlan &d) {
  const size_t n = std::max((size_t)(d.W_max + 1) * d.ZG, d.mixed ? (size_t)(2 * d.W_max + 1) * d.ZGr : 0);
  return (unsigned)std::min<size_t>(1024, (n + 255) / 256);
}

AvailTable avail_table(const int32_t *avail, int n) {
  AvailTable t{};
  std::memcpy(t.v, avail, n * sizeof(int32_t));
  return t;
}
AvailTable avail_table(const sailor_plan *pl) { return avail_table(pl->h_avail, pl->dev.ZGr); }

// Brings a changed availability table to the device on the caller's stream and rebuilds
// the quota table from it.
sailor_status refresh_avail(sailor_plan *pl, hipStream_t st) {
  if (!pl->avail_dirty) return SAILOR_OK;
  hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &capturing) != hipSuccess) (void)hipGetLastError();  // (the launch reports it)
  if (capturing != hipStreamCaptureStatusNone) {
    // Replays read the table of their time (the caller has them finish before it sets another).  Nothing
    // has run yet: the table stays due for calls outside the graph.  What a replay changes counts as
    // newer than any kept minimum.
    k_quota_table<<<quota_grid(pl->dev), 256, 0, st>>>(pl->dev, AvailTable{}, pl->h_avail_dev, pl->d_avail, ~0u);
    return SAILOR_OK;
  }
  k_quota_table<<<quota_grid(pl->dev), 256, 0, st>>>(pl->dev, avail_table(pl), nullptr, pl->d_avail, ++pl->avail_gen);
  pl->avail_dirty = false;
  return SAILOR_OK;
}

// ScanArgs::most: half of the replicas of a pair of types lie on either pool.
uint64_t most_replicas(const sailor_plan *pl) {
  return (uint64_t)*std::max_element(pl->h_avail, pl->h_avail + pl->dev.ZGr) * (pl->dev.mixed ? 2u : 1u);
}

// Plain launch, or a launch whose own start / stop timestamps are recorded in two events.
template <typename K, typename... A>
void launch(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t st, hipEvent_t e0,
            hipEvent_t e1, A... args) {
  if (e0) hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, st, e0, e1, 0, args...);
  else kernel<<<grid, block, lds, st>>>(args...);
}

template <int MODE, bool MIXED, bool GUIDED>
void launch_units_m(sailor_plan *pl, sailor_objective obj, int has_bound, const ScanArgs &a,
                    dim3 grid, dim3 block, size_t lds, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  AvailArg<MODE, MIXED> avail{};
  if constexpr (kAvailRides<MODE, MIXED>) avail = avail_table(pl);
  if (obj == SAILOR_MAX_THROUGHPUT) {
    if (has_bound) launch(k_units<MODE, 0, true, MIXED, GUIDED>, grid, block, lds, st, e0, e1, pl->dev, a, avail);
    else launch(k_units<MODE, 0, false, MIXED, GUIDED>, grid, block, lds, st, e0, e1, pl->dev, a, avail);
  } else {
    if (has_bound) launch(k_units<MODE, 1, true, MIXED, GUIDED>, grid, block, lds, st, e0, e1, pl->dev, a, avail);
    else launch(k_units<MODE, 1, false, MIXED, GUIDED>, grid, block, lds, st, e0, e1, pl->dev, a, avail);
  }
}

template <int MODE>
void launch_units(sailor_plan *pl, sailor_objective obj, int has_bound, const ScanArgs &a,
                  hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const unsigned n_units = (unsigned)pl->units.size();
  const dim3 grid((a.direct               ? a.n_list_host * a.n_sub
                   : MODE != MODE_COLLECT ? (a.n_seeds ? a.n_seeds * a.n_sub + scan_workgroups(n_units - a.n_seeds, pl->unit_threads / 64, (uint32_t)(pl->cus * kCuWaves)) : n_units)
                                          : std::min(n_units, kCollectUnits) * a.n_sub) + a.fresh),
      block(pl->unit_threads);
  const size_t lds = pl->lds_bytes;
  if constexpr (MODE != MODE_COLLECT)
    if (a.n_seeds) {
      if (pl->dev.mixed) launch_units_m<MODE, true, true>(pl, obj, has_bound, a, grid, block, lds, st, e0, e1);
      else launch_units_m<MODE, false, true>(pl, obj, has_bound, a, grid, block, lds, st, e0, e1);
      return;
    }
  if (pl->dev.mixed) launch_units_m<MODE, true, false>(pl, obj, has_bound, a, grid, block, lds, st, e0, e1);
  else launch_units_m<MODE, false, false>(pl, obj, has_bound, a, grid, block, lds, st, e0, e1);
}

struct SearchLaunch {
  unsigned root_wgs, root_waves;  // workgroups of the first level's kernel, waves of each
  size_t root_words;              // LDS words of a wave
  unsigned wgs;
  size_t lds;
};

template <int MODE>
void launch_search(const sailor_plan *pl, const SearchArgs &a, const SearchLaunch &l, hipStream_t st) {
  k_search_root<MODE><<<l.root_wgs, l.root_waves * 64, l.root_words * 8 * l.root_waves, st>>>(pl->dev, a, (uint32_t)l.root_words);
  // (only two pools and a degree per stage have tables that large)
  if (a.by_zone) k_search_beam<SEARCH_SPLIT_TP, SEARCH_BY_ZONE><<<l.wgs, kSearchThreads, l.lds, st>>>(pl->dev, a);
  else if (a.W > kSearchNarrow) k_search_beam<MODE, SEARCH_WIDE><<<l.wgs, kSearchThreads, l.lds, st>>>(pl->dev, a);
  else if (a.states) k_search_beam<MODE, SEARCH_IN_MEMORY><<<l.wgs, kSearchThreads, l.lds, st>>>(pl->dev, a);
  else k_search_beam<MODE, SEARCH_IN_LDS><<<l.wgs, kSearchThreads, l.lds, st>>>(pl->dev, a);
}

// Waits for the sequence number in host-mapped memory rather than for the dispatch to
// retire; the stream is asked now and then, so that a failed launch cannot hang the wait.
sailor_status wait_for_result(const sailor_plan *pl, hipStream_t st) {
  const volatile uint32_t *flag = &static_cast<ResultHeader *>(pl->h_result)->seq;
  for (uint32_t spins = 1; *flag != pl->seq; ++spins) {
    if ((spins & 0x3FFu) != 0) continue;
    const hipError_t q = hipStreamQuery(st);
    if (q == hipErrorNotReady) continue;
    HIP_TRY(q);
    if (*flag != pl->seq) return SAILOR_EDEVICE;  // the stream drained without a result
  }
  __atomic_thread_fence(__ATOMIC_ACQUIRE);
  return SAILOR_OK;
}

// Shared by best_plan (k = 0: tolerance rule) and topk.
sailor_status run_selection_impl(sailor_plan *pl, sailor_objective obj,
                                 const sailor_constraint *con, uint32_t k, hipStream_t st,
                                 ResultHeader *hdr_out, bool first_try, bool *again) {
  int has_bound;
  double bound;
  ScanArgs sa{};
  sailor_status rc = constraint_limits(obj, con, &has_bound, &bound, &sa.lim_s, &sa.lim_l);
  if (rc != SAILOR_OK) return rc;
  HIP_TRY(hipSetDevice(pl->device));
  if (pl->dev.mixed || k != 0 || !first_try || pl->incremental) {
    rc = refresh_avail(pl, st);
    if (rc != SAILOR_OK) return rc;
  } else if (pl->avail_dirty) {  // the call's first launch brings it along (it waits for its result: never captured)
    pl->avail_gen += 1;
    pl->avail_dirty = false;
    sa.fresh = kFreshWorkgroups;
    sa.avail_copy = pl->d_avail;
  }
  if (pl->counters_dirty) {
    k_init_counters<<<1, 64, 0, st>>>(pl->counters, pl->calls);
    pl->counters_dirty = false;
  }
  // two counter sets: this call's set was reset by the final kernel of the previous call
  const uint32_t call = pl->calls++;
  uint32_t *cnt = pl->counters + (call & 1u) * kSetWords;
  uint32_t *cnt_next = pl->counters + (~call & 1u) * kSetWords;
  sa.umin_s = pl->umin_s;
  sa.umin_l = pl->umin_l;
  sa.counters = cnt;
  sa.surv = pl->surv;
  sa.surv_cap = pl->surv_cap;
  sa.n_sub = kCollectSub;
  // a unit's minima of the last scan are reused when the query is the same and no quota row
  // the unit reads has changed since (the kernels compare generations per unit)
  sa.unit_gen = pl->unit_gen;
  sa.cur_gen = pl->avail_gen;
  sa.unit_seq = pl->unit_seq;
  sa.call_seq = pl->seq + 1;  // the sequence number this call's final kernel will publish
  sa.ubits = pl->incremental ? pl->ubits : nullptr;
  sa.ubits_stride = pl->ubits_stride;
  sa.incremental = (pl->incremental && pl->cache_ok && pl->cache_obj == (int)obj &&
                    pl->cache_hasb == has_bound && pl->cache_lim_s == sa.lim_s &&
                    pl->cache_lim_l == sa.lim_l) ? 1 : 0;
  const bool was_incremental = sa.incremental != 0;
  // (the constrained quantity is the cost when throughput is the objective, and the time otherwise)
  sa.rows_con = obj == SAILOR_MAX_THROUGHPUT ? pl->rows + pl->dev.DP : pl->rows;
  // (what is kept for later calls must not depend on this call's results, nor on the availability alone)
  if (!pl->incremental) sa.rows_key = obj == SAILOR_MAX_THROUGHPUT ? pl->rows : pl->rows + pl->dev.DP;
  sa.most = pl->incremental ? ~0ull : most_replicas(pl);
  pl->cache_ok = false;  // until this call has succeeded
  pl->cache_obj = (int)obj;
  pl->cache_hasb = has_bound;
  pl->cache_lim_s = sa.lim_s;
  pl->cache_lim_l = sa.lim_l;
  const bool best = (k == 0);
  const uint32_t n_units = (uint32_t)pl->units.size();
  const bool t_scan = pl->timing_mode >= 1, t_all = pl->timing_mode >= 2;

  // collect -> [k-th smallest survivor key] -> fp64 refine -> final selection -> sync
  // kept: the best plan's scan has kept its candidates already
  // tail_by_slots: a bound from 256 slots takes the place of a kernel that selects the k-th smallest key.  It
  // lies 74 keys up for k = 64 and 178 for k = 128, so a few more candidates are re-evaluated; where they do
  // not fit, the call starts over without it.
  bool tail_by_slots = false;
  auto run_tail = [&](ResultHeader *hdr, bool kept) -> sailor_status {
    // (a direct pass is the call's pass over the space: the scan's timing events ride on it)
    if (!kept)
      launch_units<MODE_COLLECT>(pl, obj, has_bound, sa, st, sa.direct && t_scan ? pl->ev[3] : nullptr,
                                 sa.direct && t_scan ? pl->ev[1] : nullptr);
    sa.fresh = 0;
    RefineArgs ra{};
    ra.surv = pl->surv;
    ra.surv_cap = pl->surv_cap;
    ra.counters = cnt;
    ra.ref = pl->ref;
    ra.ref_cap = pl->ref_cap;
    ra.objective = (int)obj;
    ra.has_bound = has_bound;
    ra.bound = bound;
    ra.band = 1.0f + 3.0f * kEvalEps;
    if (best) {
      ra.band = (float)(1.0 + kTieTol) + 3.0f * kEvalEps;
      k_refine_best<<<kBestWorkgroups, kBestWaves * 64, 0, st>>>(pl->dev, ra, cnt_next, pl->d_hdr, pl->d_out, ++pl->seq, call);
    } else {
      // a bound of the k-th smallest fp32 key among the survivors, or the key itself, then only what lies up to it
      if (tail_by_slots) {
        ra.kth = k;
      } else {
        k_select_kth<256><<<1, 256, 0, st>>>(reinterpret_cast<const float *>(&pl->surv[0].key), (int)(sizeof(SurvRec) / 4),
                                         cnt + CNT_SURV, pl->surv_cap, k, cnt + CNT_TAU1,
                                         nullptr, 0u, 0.f, nullptr, nullptr);
        ra.tau_src = cnt + CNT_TAU1;
      }
      k_refine<<<256, kRefineWaves * 64, 0, st>>>(pl->dev, ra);
      // few records expected (about k, plus ties): one workgroup ranks them from LDS
      const bool one = k <= kRankOneWorkgroup;
      k_rank_topk<<<one ? 1 : 64, one ? kRankLds : 256, 0, st>>>(
          pl->ref, pl->ref_cap, cnt, cnt_next, (int)obj, k, pl->d_hdr, pl->d_out, pl->staged,
          cnt + CNT_DONE, ++pl->seq);
    }
    if (t_all) HIP_TRY(hipEventRecord(pl->ev[2], st));
    HIP_TRY(hipGetLastError());
    const sailor_status waited = wait_for_result(pl, st);
    if (waited != SAILOR_OK) return waited;
    *hdr = *static_cast<ResultHeader *>(pl->h_result);
    return SAILOR_OK;
  };

  if (t_all) HIP_TRY(hipEventRecord(pl->ev[0], st));
  // A constraint often leaves only a few units alive (their bounds are sorted on the host).  Not
  // used when minima are kept for later calls: a pass over a few units produces none.
  pl->last_direct = false;
  if (first_try && has_bound && !pl->incremental) {
    const bool on_cost = obj == SAILOR_MAX_THROUGHPUT;
    const std::vector<float> &sorted_lb = on_cost ? pl->lb_cost_sorted : pl->lb_time_sorted;
    const size_t n_live = (size_t)(std::upper_bound(sorted_lb.begin(), sorted_lb.end(), sa.lim_l) -
                                   sorted_lb.begin());
    if (n_live > 0 && n_live <= kDirectUnits) {
      sa.direct = 1;
      sa.n_list_host = (uint32_t)n_live;
      sa.ulist = on_cost ? pl->order_cost : pl->order_time;
      sa.n_sub = kDirectSub;
    }
  }
  // units that do not fit on the chip at once: the first of the order guide the others (scan_workgroups)
  auto guide = [&]() {
    if (!sa.rows_key || n_units <= (best ? kBestSeeds : kKthSeeds) || (size_t)n_units * (pl->unit_threads / 64) <= pl->cus * (!best ? kGuidedKthChips * kCuWaves : pl->dev.mixed ? kGuidedMixedWavesPerCu : kCuWaves)) return;
    sa.n_seeds = best ? kBestSeeds : kKthSeeds;
    sa.n_sub = best ? kBestSeedSub : kKthSeedSub;
    sa.wait_ticks = best ? kBestSeedTicks : kKthSeedTicks;
    if (obj == SAILOR_MIN_COST) sa.ulist = pl->order_cost;  // (their own order is by time)
  };
  if (best && !sa.incremental && first_try) {
    // The scan keeps the candidates near the minimum itself (ScanArgs::near_band), so one kernel
    // is left behind it.  (Not when minima are reused: units that are not evaluated again report at
    // once, before any running minimum exists, and would have to stage their records again.)
    sa.near_band = (float)(1.0 + kTieTol) + 3.0f * kEvalEps;
    if (!sa.direct) guide();
    launch_units<MODE_BEST>(pl, obj, has_bound, sa, st, t_scan ? pl->ev[3] : nullptr, t_scan ? pl->ev[1] : nullptr);
    rc = run_tail(hdr_out, true);
    if (rc != SAILOR_OK) return rc;
    pl->total_timed = t_all;
    pl->scan_timed = t_scan;
    // (a running minimum admits more than the final one: the scan's minimum decides)
    if (hdr_out->surv_count > pl->surv_cap || (pl->scratch_grows && hdr_out->ref_count > pl->ref_cap)) {
      *again = true;
      return SAILOR_OK;
    }
    pl->last_direct = sa.direct != 0;
    pl->last_direct_units = sa.n_list_host;
    pl->cache_ok = !sa.direct;
    pl->last_incremental = false;
    pl->last_scan_seq = sa.call_seq;
    return hdr_out->ref_count > pl->ref_cap ? SAILOR_ENOMEM : SAILOR_OK;
  }
  // Top-k over a few units needs no scan and no threshold: one pass over them keeps every valid
  // candidate within the loose limit, and the usual tail -- the k-th smallest key among them, fp64
  // re-evaluation, ranking -- follows.  Not for a query that kept too many candidates the last time.
  if (sa.direct && !(pl->direct_declined && pl->declined_obj == (int)obj && pl->declined_lim == sa.lim_l)) {
    sa.use_tau_host = 1;
    sa.tau_host = kPosInf;
    tail_by_slots = k <= kKthLive;
    rc = run_tail(hdr_out, false);
    if (rc != SAILOR_OK) return rc;
    pl->total_timed = t_all;
    pl->scan_timed = t_scan;
    if (hdr_out->surv_count > std::min(kDirectManySurvivors, pl->surv_cap / 2)) {
      pl->direct_declined = true;
      pl->declined_obj = (int)obj;
      pl->declined_lim = sa.lim_l;
    }
    if (hdr_out->surv_count > pl->surv_cap || hdr_out->ref_count > pl->ref_cap) {
      *again = true;  // more candidates than the buffers hold: the scan and its threshold decide
      return SAILOR_OK;
    }
    pl->last_direct = true;
    pl->last_direct_units = sa.n_list_host;
    pl->last_incremental = false;
    return SAILOR_OK;
  }
  sa.direct = 0;
  sa.ulist = nullptr;
  // A scan for the k smallest keys ends with an upper bound of the k-th as the threshold; a guided one leaves out
  // what that rules out while it runs.  (Not for minima that are kept, nor for a k that is a large share of
  // the bound's slots: with 256 of them it lies about 1.4 k keys up for k = 128.)
  const bool by_slots = !best && first_try && !pl->incremental && k <= kKthLive;
  sa.band = sa.near_band = 1.0f + 3.0f * kEvalEps;
  if (by_slots) {
    sa.kth = k;
    guide();
  }
  const float *const rows_key = sa.rows_key;
  if (!by_slots) {
    // Nothing known of the result shortens this scan (k above kKthLive, minima that are kept, second tries): where the
    // units do not fit on the chip at once, the longest go first.
    sa.rows_key = nullptr;
    if ((size_t)n_units * (pl->unit_threads / 64) > pl->cus * kCuWaves) {
      if (!pl->work_ordered) {
        k_unit_work<<<(unsigned)std::min<size_t>(pl->cus * 8, (n_units + 3) / 4), 256, 0, st>>>(pl->dev, pl->work_bucket);
        k_work_order<<<1, 1024, 0, st>>>(pl->work_bucket, n_units, pl->order_work);
        pl->work_ordered = true;  // (whatever the availability becomes)
      }
      sa.ulist = pl->order_work;
    }
  }
  launch_units<MODE_SCAN>(pl, obj, has_bound, sa, st, t_scan ? pl->ev[3] : nullptr,
                          t_scan ? pl->ev[1] : nullptr);
  sa.rows_key = rows_key;
  sa.n_seeds = 0;
  sa.wait_ticks = 0;
  sa.ulist = nullptr;
  sa.tau_src = cnt + CNT_TAU0;  // (not by_slots)
  sa.n_sub = kCollectSub;
  if (by_slots) {
    tail_by_slots = true;
    rc = run_tail(hdr_out, false);
    if (rc != SAILOR_OK) return rc;
    pl->total_timed = t_all;
    pl->scan_timed = t_scan;
    if (hdr_out->surv_count > pl->surv_cap || hdr_out->ref_count > pl->ref_cap) {
      *again = true;  // the exact k-th smallest minimum may admit fewer
      return SAILOR_OK;
    }
    pl->last_incremental = false;
    pl->last_scan_seq = sa.call_seq;
    return SAILOR_OK;
  }
  // an upper bound of the k-th smallest key: the k-th smallest unit minimum (the best plan's: the
  // smallest, and its tie band).  The same kernel lists the units whose loose minimum lies under it.
  sa.band = best ? (float)(1.0 + kTieTol) + 3.0f * kEvalEps : 1.0f + 3.0f * kEvalEps;
  const uint32_t k_units_min = best ? 1u : k;
  const auto select = n_units > kKthByRankFrom && k_units_min <= kKthByRank ? k_select_kth<1024, true> : k_select_kth<1024, false>;
  select<<<1, 1024, 0, st>>>(pl->umin_s, 1, nullptr, n_units, k_units_min, cnt + CNT_TAU0, pl->umin_l, n_units, sa.band,
                             pl->ulist, cnt + CNT_NLIST);
  sa.ulist = pl->ulist;
  rc = run_tail(hdr_out, false);
  if (rc != SAILOR_OK) return rc;
  pl->total_timed = t_all;
  pl->scan_timed = t_scan;
  if (first_try && pl->scratch_grows && (hdr_out->surv_count > pl->surv_cap || hdr_out->ref_count > pl->ref_cap)) {
    *again = true;
    return SAILOR_OK;
  }
  if (!best && hdr_out->surv_count > pl->surv_cap) {
    // The unit minima gave too loose a bound (few units hold valid plans, or none of them
    // strictly inside the constraint).  Search for a threshold that keeps at least k strict
    // candidates and fits the survivor buffer, with count-only collect passes: first
    // doubling up from the smallest key, then bisecting.
    const float gmin = __builtin_bit_cast(float, hdr_out->gmin_bits);
    if (!(gmin < kPosInf)) return SAILOR_ENOMEM;  // nothing strictly valid to anchor on
    sa.use_tau_host = 1;
    sa.count_only = 1;
    sa.ulist = nullptr;  // the list belongs to the first threshold
    auto count_at = [&](float tau, uint32_t *n_loose, uint32_t *n_strict) -> sailor_status {
      k_zero_counters<<<1, 64, 0, st>>>(cnt, (1u << CNT_NLOOSE) | (1u << CNT_NSTRICT));
      sa.tau_host = tau;
      launch_units<MODE_COLLECT>(pl, obj, has_bound, sa, st, nullptr, nullptr);
      uint32_t two[2];
      HIP_TRY(hipMemcpyAsync(two, cnt + CNT_NLOOSE, sizeof two, hipMemcpyDeviceToHost, st));
      HIP_TRY(hipStreamSynchronize(st));
      *n_loose = two[0];
      *n_strict = two[1];
      return SAILOR_OK;
    };
    double lo = (double)gmin, hi = 0.0;  // strict count < k at lo (or unknown), too many at hi
    float tau = 0.f;
    bool found = false;
    uint32_t nl = 0, ns = 0;
    for (int it = 0; it < 200 && !found; ++it) {
      double t;
      // doubling (from the smallest normal float when the minimum key is zero)
      if (hi == 0.0) t = (it == 0) ? lo * (1.0 + 1e-6) : std::max(lo * 2.0, 1.17549435e-38);
      else t = std::sqrt(lo * hi);                                            // bisecting
      if (!(t < 3.0e38)) break;
      tau = (float)t;
      rc = count_at(tau, &nl, &ns);
      if (rc != SAILOR_OK) return rc;
      if (nl > pl->surv_cap) hi = t;
      else if (ns >= k) found = true;
      else lo = t;
      if (hi != 0.0 && hi <= lo * (1.0 + 1e-7)) break;  // a wall of ties: give up
    }
    if (!found) return SAILOR_ENOMEM;
    k_zero_counters<<<1, 64, 0, st>>>(
        cnt, (1u << CNT_SURV) | (1u << CNT_REF) | (1u << CNT_FEAS) | (1u << CNT_DONE));
    sa.count_only = 0;
    sa.tau_host = tau;
    rc = run_tail(hdr_out, false);
    if (rc != SAILOR_OK) return rc;
  }
  pl->cache_ok = true;  // the scan completed: every unit's minima and stamp are in place
  pl->last_incremental = was_incremental;
  pl->last_scan_seq = sa.call_seq;
  if (hdr_out->surv_count > pl->surv_cap || hdr_out->ref_count > pl->ref_cap) return SAILOR_ENOMEM;
  return SAILOR_OK;
}

// New survivor and re-evaluation buffers; the old ones stay the plan's if there is no memory, and are not given
// back here.
sailor_status new_scratch(sailor_plan *pl, uint32_t max_survivors, uint32_t max_refined) {
  SurvRec *surv = nullptr;
  RefRec *ref = nullptr;
  const bool got = pl->arena.alloc(&surv, (size_t)max_survivors) == hipSuccess &&
                   pl->arena.alloc(&ref, (size_t)max_refined) == hipSuccess;
  if (!got) {
    (void)hipGetLastError();  // (reported here: not for the launch behind this to find)
    if (surv) pl->arena.free_one(surv);
    return SAILOR_ENOMEM;
  }
  pl->surv = surv;
  pl->ref = ref;
  pl->surv_cap = max_survivors;
  pl->ref_cap = max_refined;
  pl->scratch_grows = false;
  return SAILOR_OK;
}

sailor_status run_selection(sailor_plan *pl, sailor_objective obj, const sailor_constraint *con,
                            uint32_t k, hipStream_t st, ResultHeader *hdr_out) {
  bool again = false;
  sailor_status rc = run_selection_impl(pl, obj, con, k, st, hdr_out, true, &again);
  if (rc == SAILOR_OK && again && pl->scratch_grows) {
    // What was kept did not fit: once more with room for more, or, where there is no memory, the longer way with
    // what there is.  The first buffers (2 MiB) stay until the plan is destroyed: nothing has to be waited for,
    // neither other streams' work nor this call's last workgroups, which may still read them.
    bool grown = false;
    try {
      grown = new_scratch(pl, kDefaultSurvCap, kDefaultRefCap) == SAILOR_OK;
    } catch (...) {
    }
    if (grown) {
      again = false;
      rc = run_selection_impl(pl, obj, con, k, st, hdr_out, true, &again);
    }
  }
  if (rc == SAILOR_OK && again) rc = run_selection_impl(pl, obj, con, k, st, hdr_out, false, &again);
  if (rc == SAILOR_EDEVICE) pl->counters_dirty = true;
  if (rc == SAILOR_OK) { pl->last_hdr = *hdr_out; pl->have_hdr = true; }
  return rc;
}

void to_result(const sailor_plan *pl, const RefRec &r, sailor_result *out) {
  fill_config(pl, shape_of(pl, r.idx), r.idx, out);
  out->peak_mem_bytes = r.mem;
  out->iter_time_s = r.T;
  out->cost_per_iter = r.C;
  out->mask = r.mask;
}

}  // namespace

extern "C" {

sailor_status sailor_plan_destroy(sailor_plan *pl) {
  if (!pl) return SAILOR_OK;
  (void)hipSetDevice(pl->device);
  pl->arena.release();
  if (pl->h_result) (void)hipHostFree(pl->h_result);
  for (hipEvent_t e : pl->ev)
    if (e) (void)hipEventDestroy(e);
  delete pl;
  return SAILOR_OK;
}

// The body of sailor_plan_create.  *track holds the plan while this function owns it, so that
// the caller can release it when a container throws half-way.
static sailor_status create_impl(const sailor_problem *p, sailor_plan **out, sailor_plan **track) {
  if (!out) return SAILOR_EINVAL;
  sailor_status rc = validate(p);
  if (rc != SAILOR_OK) return rc;
  sailor_plan *pl = new (std::nothrow) sailor_plan();
  if (!pl) return SAILOR_ENOMEM;
  *track = pl;
  std::vector<int32_t> st_n, st_first;
  std::vector<uint8_t> st_flags;
  rc = build_space(p, pl, st_n, st_first, st_flags);
  if (rc != SAILOR_OK || pl->dev.N == 0) {
    *track = nullptr;
    delete pl;
    return rc != SAILOR_OK ? rc : SAILOR_EINVAL;
  }
  pl->row_layers = st_n;
  DevPlan &d = pl->dev;
  d.G = p->n_types; d.Z = p->n_zones;
  d.mixed = p->mixed_types ? 1 : 0;
  d.GX = extended_types(p);
  d.ZG = d.GX * d.Z;
  d.ZGr = d.G * d.Z;
  d.MB = p->n_mb; d.TP = p->n_tp; d.DP = p->n_dp;
  d.bpp = p->bytes_per_param; d.gb = p->grad_bytes_per_param; d.B = p->global_batch;
  d.n_blocks = (int)pl->blocks.size();
  d.n_shapes = (int)pl->shapes.size();
  d.n_units = (int)pl->units.size();
  for (int i = 0; i < d.MB; ++i) d.mbv[i] = p->mb_values[i];
  for (int i = 0; i < d.TP; ++i) d.tpv[i] = p->tp_values[i];
  for (int i = 0; i < d.DP; ++i) d.dpv[i] = p->dp_values[i];
  pl->mbv.assign(p->mb_values, p->mb_values + d.MB);
  pl->tpv.assign(p->tp_values, p->tp_values + d.TP);
  pl->dpv.assign(p->dp_values, p->dp_values + d.DP);
  pl->ppv.assign(p->pp_values, p->pp_values + p->n_pp);
  auto magic = [](uint32_t dv) { return dv == 1 ? 0u : (uint32_t)(((1ull << 32) + dv - 1) / dv); };
  d.mg_mb = magic((uint32_t)d.MB);
  d.mg_mbzg = magic((uint32_t)(d.MB * d.ZG));
  d.mg_mbzg1 = d.ZG > 1 ? magic((uint32_t)(d.MB * (d.ZG - 1))) : 0u;
  d.mg_g = magic((uint32_t)d.GX);
  d.mg_mbtp = magic((uint32_t)(d.MB * d.TP));
  d.mg_mbtpdp = magic((uint32_t)(d.MB * d.TP * d.DP));
  pl->eval_lds_bytes = (size_t)3 * d.TP * ((size_t)d.ZG * d.MB + 1) * sizeof(Rec) +
                       (size_t)d.MB * d.Z * d.Z * sizeof(float4) +
                       (size_t)3 * d.TP * d.MB * d.DP * sizeof(uint64_t) +
                       (size_t)3 * d.TP * d.ZG * sizeof(uint32_t) +
                       (size_t)d.ZG * (sizeof(PoolInfo) + 2 * sizeof(uint64_t)) +
                       (size_t)(kEvalUnitMaxOuter + d.DP + d.TP) * sizeof(uint32_t);
  pl->lds_bytes = unit_lds_records(d.ZG, d.MB) * (2 * sizeof(float4) + sizeof(uint32_t)) +
                  (size_t)d.MB * d.Z * d.Z * sizeof(float4) +
                  (size_t)d.ZG * (2 * sizeof(uint64_t) + sizeof(uint32_t));
  if (pl->lds_bytes > kScanMaxLds) {  // pools x microbatch sizes beyond what a workgroup can stage
    delete pl;
    *track = nullptr;
    return SAILOR_EINVAL;
  }

#define CREATE_TRY(expr)                                                           \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess) {                                                        \
      std::fprintf(stderr, "sailor: %s failed: %s\n", #expr, hipGetErrorString(e_)); \
      *track = nullptr;                                                            \
      sailor_plan_destroy(pl);                                                     \
      return e_ == hipErrorOutOfMemory ? SAILOR_ENOMEM : SAILOR_EDEVICE;           \
    }                                                                              \
  } while (0)

  CREATE_TRY(hipGetDevice(&pl->device));
  int cus = 0;
  CREATE_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, pl->device));
  pl->cus = (size_t)std::max(1, cus);
  TableSlab slab;
  const int G = d.G, GX = d.GX, Z = d.Z, ZG = d.ZG, ZGr = d.ZGr, MB = d.MB, TP = d.TP, DP = d.DP,
            L = p->n_layers;
  const size_t Lc = p->uniform_layers ? 1 : (size_t)L;
  const size_t RS = (size_t)d.n_row_stages, NS = pl->shapes.size();

  // inputs, copied as they are
  slab.input(&d.avail, p->avail, ZGr);
  d.P_max = 0;
  for (int ip = 0; ip < p->n_pp; ++ip) d.P_max = std::max(d.P_max, (int)p->pp_values[ip]);
  d.W_max = d.P_max * p->tp_values[TP - 1];
  slab.table(&d.qw, (size_t)(d.W_max + 1) * ZG);
  if (d.mixed) slab.table(&d.qh, (size_t)(2 * d.W_max + 1) * ZGr);
  slab.zeroed(&d.row_gen, 1);
  slab.table(&d.h1m, ZG);
  slab.table(&d.isect, (size_t)2 * ZG);
  for (int a = 0; a < G; ++a) pl->xt.push_back((uint16_t)(a | (a << 8)));
  if (d.mixed)
    for (int a = 0; a < G; ++a)
      for (int b = a + 1; b < G; ++b) pl->xt.push_back((uint16_t)(a | (b << 8)));
  slab.input(&d.xt, pl->xt.data(), pl->xt.size());
  std::vector<int32_t> vals(p->dp_values, p->dp_values + DP);
  vals.insert(vals.end(), p->tp_values, p->tp_values + TP);
  slab.input(&d.vals, vals.data(), vals.size());
  slab.input(&d.cap, p->mem_capacity, G);
  slab.input(&d.res, p->mem_reserved, G);
  slab.input(&d.node, p->gpus_per_node, G);
  slab.input(&d.price, p->price_per_hour, G);
  slab.input(&d.bw, p->bandwidth, (size_t)Z * Z);
  if (p->egress_per_byte) slab.input(&d.egress, p->egress_per_byte, (size_t)Z * Z);
  slab.input(&d.act, p->act_store_bytes, (size_t)MB * TP);
  slab.input(&d.p2p, p->p2p_bytes, MB);
  StageArgs sa{};
  slab.input(&sa.layer_params, p->layer_params, L);
  slab.input(&sa.t_fwd, p->t_fwd, (size_t)G * MB * TP * Lc);
  slab.input(&sa.t_bwd, p->t_bwd, (size_t)G * MB * TP * Lc);
  slab.input(&sa.t_upd, p->t_upd, (size_t)G * TP * Lc);
  slab.input(&sa.st_flags, st_flags.data(), RS);
  sa.embed = p->embed_params; sa.head = p->head_params; sa.L = L; sa.uniform = p->uniform_layers ? 1 : 0;
  slab.input(&d.st_n, st_n.data(), RS);
  slab.input(&d.st_first, st_first.data(), RS);
  slab.input(&d.shapes, pl->shapes.data(), NS);
  std::vector<uint32_t> shape_n;
  shape_n.reserve(NS);
  for (const ShapeRec &sh : pl->shapes)
    shape_n.push_back((uint32_t)((sh.n[0] - 1) & 255) | (uint32_t)((sh.n[1] - 1) & 255) << 8 | (uint32_t)((sh.n[2] - 1) & 255) << 16);
  slab.input(&pl->direct_mem.shape_n, shape_n.data(), NS);
  slab.input(&d.blocks, pl->blocks.data(), pl->blocks.size());
  // per-unit tables: one entry per unit as laid out, dropped ones included;
  // sailor_set_scan_unit_parts(n) cuts every unit into n parts and needs n times the room
  const long forced_parts = g_forced_unit_parts.load(std::memory_order_relaxed);
  const size_t unit_cap = pl->units.size() * (size_t)std::max(1L, forced_parts);
  char *per_unit = nullptr;  // the tables that creation fills last, in one copy: records, bounds, orders
  slab.table(&per_unit, unit_cap * (sizeof(UnitRec) + 2 * sizeof(uint32_t)));
  slab.table(&pl->rows, unit_cap * 2 * DP);
  const EvalBlock *d_eblocks = nullptr;
  slab.input(&d_eblocks, pl->eblocks.data(), pl->eblocks.size());
  slab.table(&pl->d_eunits, (size_t)pl->n_eunits);
  // derived tables, filled by the set-up kernels
  d.n_bw_coef = p->n_bw_coef;
  if (p->n_bw_coef > 0) slab.input(&d.bw_poly, p->bw_poly, (size_t)Z * Z * p->n_bw_coef);
  slab.table(&d.xsec, (size_t)MB * Z * Z);
  if (!d.mixed) slab.table(&d.list_tables, list_copy_words(d));  // (not for problems with pairs of types)
  slab.table(&d.direct_tables, direct_copy_words(d));
  slab.table(&d.tsec_f, (size_t)MB * Z * Z);
  slab.table(&d.egs_f, (size_t)Z * Z);
  slab.table(&d.price_f, GX);
  slab.table(&d.xb_f, MB);
  slab.table(&d.cd_f, DP);
  slab.table(&d.nbm1_f, (size_t)MB * DP);
  slab.table(&d.dph_f, DP);
  slab.table(&d.nb, (size_t)MB * DP);
  slab.table(&d.divis, MB);
  // a stage record does not straddle cache lines (128 bytes): the evaluators of listed plans
  // fetch one per stage from anywhere in the table, and lines are what that costs
  d.row_w = 2u * (uint32_t)G + 2u;
  if (d.row_w <= 16u) while (d.row_w & (d.row_w - 1u)) ++d.row_w;
  else d.row_w = (d.row_w + 15u) & ~15u;
  slab.table(&d.st_row, RS * MB * TP * d.row_w);
  slab.table(&d.st_c, RS * G * MB * TP);
  slab.table(&d.st_f, RS * G * MB * TP);
  slab.table(&d.st_b, RS * G * MB * TP);
  slab.table(&d.st_u, RS * G * TP);
  const size_t slots = NS * TP * 3;
  slab.table(&d.ta, slots * GX * MB);
  slab.table(&d.memok, slots * GX * MB);
  slab.table(&d.need, slots * MB * DP);
  slab.table(&d.syncz, slots * Z);
  slab.table(&d.upd, slots * GX);
  slab.table(&pl->direct_mem.su, slots * ZG);
  float *link_min = nullptr;
  GroupArgs ga{};
  slab.table(&link_min, (size_t)2 * MB + 1);
  slab.table(&ga.rows, (size_t)pl->n_groups * 2 * DP);
  slab.table(&ga.sums, (size_t)pl->n_groups);
  // selection scratch
  slab.table(&pl->umin_s, 2 * unit_cap);
  slab.table(&pl->counters, (size_t)2 * kSetWords);
  slab.table(&pl->ulist, unit_cap);
  slab.table(&pl->order_work, unit_cap);
  slab.table(&pl->work_bucket, unit_cap);
  slab.zeroed(&pl->unit_gen, unit_cap);
  slab.zeroed(&pl->unit_seq, unit_cap);
  pl->ubits_stride = (uint32_t)(unit_lds_records(ZG, MB) + (size_t)ZG);
  slab.table(&pl->staged, (size_t)SAILOR_MAX_K);
  CREATE_TRY(slab.commit(pl->arena));
  pl->d_avail = const_cast<int32_t *>(d.avail);
  pl->umin_l = pl->umin_s + unit_cap;
  d.units = reinterpret_cast<UnitRec *>(per_unit);
  pl->order_time = reinterpret_cast<uint32_t *>(per_unit + unit_cap * sizeof(UnitRec));
  pl->order_cost = pl->order_time + unit_cap;
  k_init_counters<<<1, 64>>>(pl->counters, pl->calls);
  k_quota_table<<<quota_grid(d), 256>>>(d, avail_table(p->avail, ZGr), nullptr, pl->d_avail, 0u);
  k_small_tables<<<1, 256>>>(d, link_min);
  if (!d.mixed) k_list_tables<<<1, 256>>>(d);
  k_direct_tables<<<1, 256>>>(d, pl->direct_mem);
  k_stage_tables<<<(unsigned)RS, 128>>>(d, sa);
  k_shape_agg<<<(unsigned)NS, kShapeAggThreads, (size_t)3 * TP * (Z + GX) * sizeof(float)>>>(d, pl->direct_mem);
  CREATE_TRY(hipGetLastError());
  {
    // The units' bounds, which let a query pass over a unit, or some of its degrees, whatever the
    // availability becomes.  A unit without a plan that memory, node size and batch divisibility allow is
    // dropped for good.  The others are launched in ascending order of the smallest time that the present
    // availability leaves them: what lies far behind then falls to the running limits.  (A timed pass over
    // the space ordered them, longest first, and cut long ones into parts: 254 of the 1 755 us of a new job
    // on 1.1e9 plans with pairs of types.  With limits by degree it is the order that shortens a scan.)
    size_t NU = pl->units.size();
    ga.blocks = d_eblocks;
    ga.n_blocks = (int)pl->eblocks.size();
    ga.link_min = link_min;
    ga.most = (uint64_t)*std::max_element(p->avail, p->avail + ZGr) * (d.mixed ? 2u : 1u);
    // (a lane takes a microbatch size and a type per segment)
    k_group_bounds<<<pl->n_groups, GX * GX * MB <= 256 ? 64 : kGroupThreads, group_lds_bytes(GX, MB, DP)>>>(d, ga);
    CREATE_TRY(hipGetLastError());
    // what only queries need is allocated while the set-up kernels run
    CREATE_TRY(pl->arena.alloc(&pl->surv, (size_t)pl->surv_cap));  // (these two can be replaced on their own)
    CREATE_TRY(pl->arena.alloc(&pl->ref, (size_t)pl->ref_cap));
    const size_t res_bytes = (sizeof(ResultHeader) + 8 + (size_t)SAILOR_MAX_K * sizeof(RefRec) + 127) & ~(size_t)127;
    CREATE_TRY(hipHostMalloc(&pl->h_result, res_bytes + (size_t)ZGr * sizeof(int32_t), hipHostMallocMapped));
    std::memset(pl->h_result, 0, res_bytes);
    void *d_res = nullptr;
    CREATE_TRY(hipHostGetDevicePointer(&d_res, pl->h_result, 0));
    pl->d_hdr = static_cast<ResultHeader *>(d_res);
    pl->d_out = reinterpret_cast<RefRec *>(static_cast<char *>(d_res) + sizeof(ResultHeader));
    pl->h_avail = reinterpret_cast<int32_t *>(static_cast<char *>(pl->h_result) + res_bytes);
    pl->h_avail_dev = reinterpret_cast<const int32_t *>(static_cast<char *>(d_res) + res_bytes);
    std::memcpy(pl->h_avail, p->avail, ZGr * sizeof(int32_t));
    for (hipEvent_t &e : pl->ev) CREATE_TRY(hipEventCreate(&e));
    k_eval_units<<<(unsigned)std::min<uint64_t>(1024, (pl->n_eunits + 255) / 256), 256>>>(
        d_eblocks, (int)pl->eblocks.size(), pl->n_eunits, d.inner, pl->d_eunits);
    CREATE_TRY(hipGetLastError());
    std::vector<GroupSum> sums(pl->n_groups);
    CREATE_TRY(hipMemcpy(sums.data(), ga.sums, sums.size() * sizeof(GroupSum), hipMemcpyDeviceToHost));
    std::vector<float> val(NU), lb_now(NU), lb_time(NU), lb_cost(NU);
    size_t n_kept = 0;
    for (size_t i = 0; i < NU; ++i) {
      const UnitRec &u = pl->units[i];
      const GroupSum &g = sums[u.group];
      bool holds = u.s == 1 && g.time < kPosInf;
      for (int a2 = u.o_lo; u.s >= 2 && a2 < u.o_lo + u.o_cnt && !holds; ++a2)
        holds = (g.seg2[(a2 % GX) >> 5] >> ((a2 % GX) & 31)) & 1u;
      if (!holds && !(n_kept == 0 && i + 1 == NU)) continue;  // launches need a non-empty grid
      lb_now[n_kept] = g.time_now;
      lb_time[n_kept] = g.time;
      lb_cost[n_kept] = g.cost;
      pl->units[n_kept] = u;
      ++n_kept;
    }
    pl->units.resize(NU = n_kept);
    d.n_units = (int)NU;
    if (forced_parts > 1) {  // every unit's lane space cut into parts
      const auto repeat = [&](auto &v) {
        auto whole = v;
        whole.resize(NU);
        v.clear();
        for (size_t i = 0; i < NU; ++i) v.insert(v.end(), (size_t)forced_parts, whole[i]);
      };
      repeat(pl->units);
      repeat(lb_now);
      repeat(lb_time);
      repeat(lb_cost);
      for (size_t i = 0; i < pl->units.size(); ++i) {
        pl->units[i].n_parts = (uint8_t)forced_parts;
        pl->units[i].part = (uint8_t)(i % (size_t)forced_parts);
      }
      d.n_units = (int)(NU = pl->units.size());
      val.resize(NU);
    }
    // the bounds in the units' final order, and the units sorted by either bound: the host then
    // knows how many units a limit leaves alive, and the device which
    const std::vector<uint32_t> final_order = order_by(lb_now.data(), NU, false);
    std::vector<UnitRec> sorted(NU);
    for (size_t i = 0; i < NU; ++i) sorted[i] = pl->units[final_order[i]];
    pl->units.swap(sorted);
    std::vector<char> tables(unit_cap * (sizeof(UnitRec) + 2 * sizeof(uint32_t)));  // as they lie in `per_unit`
    std::memcpy(tables.data(), pl->units.data(), NU * sizeof(UnitRec));
    char *const orders = &tables[unit_cap * sizeof(UnitRec)];
    for (int which = 0; which < 2; ++which) {
      const std::vector<float> &lb = which ? lb_cost : lb_time;
      for (size_t i = 0; i < NU; ++i) val[i] = lb[final_order[i]];
      const std::vector<uint32_t> order = order_by(val.data(), NU, false);
      std::memcpy(orders + which * unit_cap * sizeof(uint32_t), order.data(), NU * sizeof(uint32_t));
      std::vector<float> &sorted_lb = which ? pl->lb_cost_sorted : pl->lb_time_sorted;
      sorted_lb.resize(NU);
      for (size_t i = 0; i < NU; ++i) sorted_lb[i] = val[order[i]];
    }
    CREATE_TRY(hipMemcpy(per_unit, tables.data(), tables.size(), hipMemcpyHostToDevice));
    k_unit_rows<<<(unsigned)std::min<size_t>(1024, (NU * 2 * DP + 255) / 256), 256>>>(d.units, ga.rows, (uint32_t)NU, 2u * (uint32_t)DP, pl->rows);
    k_init_counters<<<1, 64>>>(pl->counters, pl->calls);
    CREATE_TRY(hipDeviceSynchronize());
  }
#undef CREATE_TRY
  *track = nullptr;
  *out = pl;
  return SAILOR_OK;
}

sailor_status sailor_plan_create(const sailor_problem *p, sailor_plan **out) {
  sailor_plan *half_built = nullptr;
  try {  // no C++ exception crosses the C boundary
    return create_impl(p, out, &half_built);
  } catch (const std::bad_alloc &) {
    if (half_built) sailor_plan_destroy(half_built);
    return SAILOR_ENOMEM;
  } catch (...) {
    if (half_built) sailor_plan_destroy(half_built);
    return SAILOR_EINVAL;
  }
}

sailor_status sailor_plan_set_avail(sailor_plan *pl, const int32_t *avail) {
  if (!pl || !avail) return SAILOR_EINVAL;
  for (int i = 0; i < pl->dev.ZGr; ++i)
    if (avail[i] < 0) return SAILOR_EINVAL;
  HIP_TRY(hipSetDevice(pl->device));
  std::memcpy(pl->h_avail, avail, pl->dev.ZGr * sizeof(int32_t));
  pl->avail_dirty = true;  // uploaded, with the quota table, by the next call on its stream
  return SAILOR_OK;
}

sailor_status sailor_plan_num_candidates(const sailor_plan *pl, uint64_t *out) {
  if (!pl || !out) return SAILOR_EINVAL;
  *out = pl->dev.N;
  return SAILOR_OK;
}

sailor_status sailor_plan_decode(const sailor_plan *pl, uint64_t index, sailor_result *out) {
  if (!pl || !out) return SAILOR_EINVAL;
  if (index >= pl->dev.N) return SAILOR_ERANGE;
  fill_config(pl, shape_of(pl, index), index, out);
  return SAILOR_OK;
}

sailor_status sailor_eval_batch(sailor_plan *pl, uint64_t first, uint64_t count,
                                const uint64_t *d_indices, sailor_objective objective,
                                const sailor_constraint *constraint, float *d_time, float *d_cost,
                                uint64_t *d_mem, uint32_t *d_mask, void *hip_stream) {
  if (!pl || (objective != SAILOR_MAX_THROUGHPUT && objective != SAILOR_MIN_COST))
    return SAILOR_EINVAL;
  if (!d_indices && (first > pl->dev.N || count > pl->dev.N - first)) return SAILOR_ERANGE;
  if (count > (uint64_t)0x7fffffff * 256) return SAILOR_ERANGE;
  if (constraint && constraint->has_bound && std::isnan(constraint->bound)) return SAILOR_EINVAL;
  if (count == 0) return SAILOR_OK;
  HIP_TRY(hipSetDevice(pl->device));
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  {
    const sailor_status rc = refresh_avail(pl, st);
    if (rc != SAILOR_OK) return rc;
  }
  EvalArgs a{};
  a.first = first; a.count = count; a.indices = d_indices;
  a.time = d_time; a.cost = d_cost; a.mem = d_mem; a.mask = d_mask;
  a.objective = (int)objective;
  a.has_bound = (constraint && constraint->has_bound) ? 1 : 0;
  a.bound = a.has_bound ? (float)constraint->bound : 0.f;
  const bool timed = pl->timing_mode >= 1;
  if (!d_indices && pl->eval_lds_bytes <= kEvalRowsMaxLds) {
    // the units that intersect [first, first + count)
    auto unit_of = [&](uint64_t index) {
      const EvalBlock &b = *(std::upper_bound(pl->eblocks.begin(), pl->eblocks.end(), index,
                                              [](uint64_t i, const EvalBlock &e) { return i < e.off; }) - 1);
      const uint64_t rem = index - b.off;
      return b.first_unit + rem / b.shape_size * b.per_shape + rem % b.shape_size / pl->dev.inner / b.chunk;
    };
    const uint64_t u0 = unit_of(first), n_wgs = unit_of(first + count - 1) - u0 + 1;
    if (pl->dev.mixed)
      launch(k_eval_rows<true>, dim3((unsigned)n_wgs), dim3(kEvalRowsThreads), pl->eval_lds_bytes,
             st, timed ? pl->ev[3] : nullptr, timed ? pl->ev[1] : nullptr, pl->dev, a, pl->d_eunits,
             (uint32_t)u0);
    else
      launch(k_eval_rows<false>, dim3((unsigned)n_wgs), dim3(kEvalRowsThreads), pl->eval_lds_bytes,
             st, timed ? pl->ev[3] : nullptr, timed ? pl->ev[1] : nullptr, pl->dev, a, pl->d_eunits,
             (uint32_t)u0);
    HIP_TRY(hipGetLastError());
    pl->total_timed = false;
    pl->scan_timed = timed;
    return SAILOR_OK;
  }
  const uint64_t chunks = (count + kDirectThreads - 1) / kDirectThreads;
  launch(k_eval_direct, dim3((unsigned)std::min<uint64_t>(chunks, kDirectWorkgroups)), dim3(kDirectThreads),
         direct_lds_bytes(pl->dev), st,
         timed ? pl->ev[3] : nullptr, timed ? pl->ev[1] : nullptr, pl->dev, a, pl->direct_mem);
  HIP_TRY(hipGetLastError());
  pl->total_timed = false;
  pl->scan_timed = timed;
  return SAILOR_OK;
}

sailor_status sailor_best_plan(sailor_plan *pl, sailor_objective objective,
                               const sailor_constraint *constraint, sailor_result *out,
                               void *hip_stream) {
  if (!pl || !out || (objective != SAILOR_MAX_THROUGHPUT && objective != SAILOR_MIN_COST))
    return SAILOR_EINVAL;
  ResultHeader hdr;
  sailor_status rc = run_selection(pl, objective, constraint, 0,
                                   static_cast<hipStream_t>(hip_stream), &hdr);
  if (rc != SAILOR_OK) return rc;
  if (hdr.n_found == 0) return SAILOR_ENOFEASIBLE;
  const RefRec *rec = reinterpret_cast<const RefRec *>(static_cast<char *>(pl->h_result) +
                                                       sizeof(ResultHeader));
  to_result(pl, rec[0], out);
  return SAILOR_OK;
}

sailor_status sailor_topk(sailor_plan *pl, sailor_objective objective,
                          const sailor_constraint *constraint, int32_t k, sailor_result *out,
                          int32_t *n_found, void *hip_stream) {
  if (!pl || !out || !n_found || k < 1 || k > SAILOR_MAX_K ||
      (objective != SAILOR_MAX_THROUGHPUT && objective != SAILOR_MIN_COST))
    return SAILOR_EINVAL;
  ResultHeader hdr;
  sailor_status rc = run_selection(pl, objective, constraint, (uint32_t)k,
                                   static_cast<hipStream_t>(hip_stream), &hdr);
  if (rc != SAILOR_OK) return rc;
  *n_found = (int32_t)hdr.n_found;
  if (hdr.n_found == 0) return SAILOR_ENOFEASIBLE;
  const RefRec *rec = reinterpret_cast<const RefRec *>(static_cast<char *>(pl->h_result) +
                                                       sizeof(ResultHeader));
  for (uint32_t i = 0; i < hdr.n_found; ++i) to_result(pl, rec[i], &out[i]);
  return SAILOR_OK;
}

sailor_status sailor_plan_set_scratch(sailor_plan *pl, uint32_t max_survivors,
                                      uint32_t max_refined) {
  if (!pl || max_survivors < 1 || max_refined < 1) return SAILOR_EINVAL;
  HIP_TRY(hipSetDevice(pl->device));
  HIP_TRY(hipDeviceSynchronize());
  SurvRec *const surv = pl->surv;
  RefRec *const ref = pl->ref;
  try {
    const sailor_status rc = new_scratch(pl, max_survivors, max_refined);
    if (rc != SAILOR_OK) return rc;
    pl->arena.free_one(surv);
    pl->arena.free_one(ref);
    return SAILOR_OK;
  } catch (...) { return SAILOR_ENOMEM; }
}

sailor_status sailor_plan_set_timing(sailor_plan *pl, int32_t mode) {
  if (!pl || mode < 0 || mode > 2) return SAILOR_EINVAL;
  pl->timing_mode = mode;
  pl->total_timed = pl->scan_timed = false;
  return SAILOR_OK;
}

sailor_status sailor_plan_last_timing(sailor_plan *pl, float *total_ms, float *kernel_ms) {
  if (!pl || (!pl->total_timed && !pl->scan_timed)) return SAILOR_EINVAL;
  float t = 0.f, s = 0.f;
  if (pl->scan_timed) {
    HIP_TRY(hipEventSynchronize(pl->ev[1]));
    HIP_TRY(hipEventElapsedTime(&s, pl->ev[3], pl->ev[1]));
  }
  if (pl->total_timed) {
    HIP_TRY(hipEventSynchronize(pl->ev[2]));
    HIP_TRY(hipEventElapsedTime(&t, pl->ev[0], pl->ev[2]));
  }
  if (total_ms) *total_ms = t;
  if (kernel_ms) *kernel_ms = s;
  return SAILOR_OK;
}

sailor_status sailor_simulate_1f1b(sailor_plan *pl, uint64_t count, const uint64_t *d_indices,
                                   double *d_event, double *d_closed, void *hip_stream) {
  if (!pl) return SAILOR_EINVAL;
  if (count == 0) return SAILOR_OK;
  if (!d_indices || (!d_event && !d_closed)) return SAILOR_EINVAL;
  if (count > 0x7fffffffu) return SAILOR_ERANGE;
  // microbatches per pipeline are counted in 32-bit integers
  if (pl->dev.B / ((int64_t)pl->dpv[0] * pl->mbv[0]) > (1 << 24)) return SAILOR_ERANGE;
  HIP_TRY(hipSetDevice(pl->device));
  SimArgs a{};
  a.count = count;
  a.indices = d_indices;
  a.t_event = d_event;
  a.t_closed = d_closed;
  k_sim_1f1b<<<(unsigned)count, 64, 0, static_cast<hipStream_t>(hip_stream)>>>(pl->dev, a);
  HIP_TRY(hipGetLastError());
  return SAILOR_OK;
}

// (the schedule lives in registers, so the two entry points differ in the number of plans only)
sailor_status sailor_simulate_1f1b_static(sailor_plan *pl, uint64_t count, const uint64_t *d_indices,
                                          double *d_event, double *d_closed, void *hip_stream) {
  if (pl && count > SAILOR_STATIC_MAX_PLANS) {
    if (!d_indices || (!d_event && !d_closed)) return SAILOR_EINVAL;
    std::fprintf(stderr, "sailor: sailor_simulate_1f1b_static takes at most %d plans per call (%llu given)\n",
                 (int)SAILOR_STATIC_MAX_PLANS, (unsigned long long)count);
    return SAILOR_ERANGE;
  }
  return sailor_simulate_1f1b(pl, count, d_indices, d_event, d_closed, hip_stream);
}

// tables of the search and of the placement evaluation (once per plan)
// (search: also the search's buffers)
static sailor_status search_setup(sailor_plan *pl, bool search) {
  if (!pl->d_search_pps) {
    pl->search_pps.clear();
    uint32_t sub = 0, sub_t = 0;
    uint32_t parts = 0;
    for (size_t ip = 0; ip < pl->ppv.size(); ++ip) {
      SearchPP e{};
      e.P = pl->ppv[ip];
      e.n_part = 0;
      e.rs0 = 0;
      bool seen = false;
      for (const ShapeRec &sh : pl->shapes)
        if (sh.pp_idx == ip) {
          if (!seen || sh.row_stage < e.rs0) e.rs0 = sh.row_stage;
          seen = true;
          e.n_part = std::max(e.n_part, (int32_t)sh.q + 1);
        }
      if (!seen) return SAILOR_EINVAL;  // (every depth has a one-segment block)
      e.sub_off = sub;
      e.sub_off_t = sub_t;
      sub += (uint32_t)e.n_part * (uint32_t)(pl->dev.TP * pl->dev.DP * pl->dev.MB);
      sub_t += (uint32_t)e.n_part * (uint32_t)(pl->dev.DP * pl->dev.MB);
      e.part0 = parts;
      parts += (uint32_t)e.n_part;
      pl->search_pps.push_back(e);
    }
    pl->n_sub = sub;
    pl->n_sub_t = sub_t;
    if (pl->arena.upload(&pl->d_search_pps, pl->search_pps.data(), pl->search_pps.size()) != hipSuccess)
      return SAILOR_ENOMEM;
  }
  if (search && !pl->search_alike) {
    std::vector<uint32_t> alike;
    for (const SearchPP &e : pl->search_pps) {
      // equal splits side by side, the first of them in front
      const int32_t *const rows = &pl->row_layers[e.rs0];
      const size_t P = (size_t)e.P;
      std::vector<uint32_t> order((size_t)e.n_part);
      for (uint32_t q = 0; q < order.size(); ++q) order[q] = q;
      auto row = [&](uint32_t q) { return rows + q * P; };
      std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
        return std::lexicographical_compare(row(x), row(x) + P, row(y), row(y) + P);
      });
      alike.resize(alike.size() + order.size(), 0);
      for (size_t i = 0, first = 0; i < order.size(); ++i) {
        if (!std::equal(row(order[i]), row(order[i]) + P, row(order[first]))) first = i;
        ++alike[e.part0 + order[first]];
      }
    }
    if (pl->arena.upload(&pl->search_alike, alike.data(), alike.size()) != hipSuccess) return SAILOR_ENOMEM;
  }
  if (search && !pl->search_results) {
    DeviceArena &ar = pl->arena;
    SubResult *res = nullptr, *fin = nullptr;
    uint32_t *list = nullptr, *counters = nullptr;
    unsigned long long *root_expanded = nullptr;
    sailor_status rc = SAILOR_OK;
    if (ar.alloc(&res, (size_t)std::min(pl->n_sub, kSearchWorkgroups)) != hipSuccess || ar.alloc(&fin, 1) != hipSuccess ||
        ar.alloc(&list, (size_t)pl->n_sub) != hipSuccess || ar.alloc(&counters, pl->search_pps.size() + 1) != hipSuccess ||
        ar.alloc(&root_expanded, (size_t)kRootWorkgroups) != hipSuccess)
      rc = SAILOR_ENOMEM;
    else if (hipMemset(fin, 0, sizeof(SubResult)) != hipSuccess)  // (read by the winner's re-evaluation
      rc = SAILOR_EDEVICE;                                        // also when nothing was found)
    if (rc != SAILOR_OK) {
      for (void *p : {(void *)res, (void *)fin, (void *)list, (void *)counters, (void *)root_expanded}) ar.free_one(p);
      return rc;
    }
    pl->search_results = res;
    pl->search_final = fin;
    pl->search_list = list;
    pl->search_counters = counters;
    pl->search_root_expanded = root_expanded;
  }
  return SAILOR_OK;
}

// Every workgroup slot of the chip takes one run of plans, so that the whole list is resident at once and
// the tables are staged once per slot; a longer list takes several such rounds.  Up to kPlaceShort plans,
// which four workgroups per compute unit work off in about one pass each, no more than four are used: a
// fifth brings its dispatch and its staging and shortens nothing (a pool and a degree per stage, 1 100 plans:
// 7.6 us with five, 6.7 with four; 9 000: 8.7 and 8.25; 25 000: 10.65 and 10.3).  Beyond, the fifth saves a
// second pass (33 000 plans: 11.3 us with five, 13.3 with four).
static void launch_placements(const sailor_plan *pl, PlaceArgs a, hipStream_t st) {
  const auto kernel = pl->dev.n_bw_coef > 0 ? (a.pools_b ? k_eval_placements<true, true> : k_eval_placements<false, true>)
                                            : (a.pools_b ? k_eval_placements<true, false> : k_eval_placements<false, false>);
  // (five or four by registers, fewer where the tables need the LDS.  The runtime keeps what it works out:
  // 0.1 us a call)
  int fit = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit, (const void *)kernel, kPlaceThreads, place_lds_bytes(pl->dev, kPlacePlans)) != hipSuccess)
    (void)hipGetLastError();
  const uint64_t per_cu = (uint64_t)std::max(1, fit);
  const uint64_t slots = kPlaceUnits * (a.count <= kPlaceShort ? std::min<uint64_t>(4, per_cu) : per_cu);
  const uint64_t rounds = (a.count + slots * kPlaceLongest - 1) / (slots * kPlaceLongest);
  a.per_wg = (uint32_t)((a.count + slots * rounds - 1) / (slots * rounds));
  const unsigned grid = (unsigned)((a.count + a.per_wg - 1) / a.per_wg);
  const size_t lds = place_lds_bytes(pl->dev, a.per_wg);
  kernel<<<grid, kPlaceThreads, lds, st>>>(pl->dev, a);
}

sailor_status sailor_eval_placements(sailor_plan *pl, uint64_t count, const int32_t *d_desc,
                                     const int32_t *d_pools, const int32_t *d_pools_b,
                                     const int32_t *d_tps, uint32_t pool_stride,
                                     sailor_objective objective, const sailor_constraint *constraint,
                                     double *d_time, double *d_cost, uint64_t *d_mem, uint32_t *d_mask,
                                     void *hip_stream) {
  if (!pl || (objective != SAILOR_MAX_THROUGHPUT && objective != SAILOR_MIN_COST)) return SAILOR_EINVAL;
  if (count == 0) return SAILOR_OK;
  if (!d_desc || !d_pools || pool_stride < 1) return SAILOR_EINVAL;
  if (pl->dev.mixed || pl->dev.ZGr > kSearchMaxPools) return SAILOR_EINVAL;
  if (count > (uint64_t)0x7fffffff) return SAILOR_ERANGE;
  if (constraint && constraint->has_bound && std::isnan(constraint->bound)) return SAILOR_EINVAL;
  HIP_TRY(hipSetDevice(pl->device));
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  sailor_status rc;
  try { rc = search_setup(pl, false); } catch (...) { rc = SAILOR_ENOMEM; }
  if (rc != SAILOR_OK) return rc;
  rc = refresh_avail(pl, st);
  if (rc != SAILOR_OK) return rc;
  PlaceArgs a{};
  a.count = count; a.desc = d_desc; a.pools = d_pools; a.pools_b = d_pools_b; a.tps = d_tps;
  a.pool_stride = pool_stride;
  a.pps = pl->d_search_pps; a.n_pp = (int)pl->search_pps.size();
  a.objective = (int)objective;
  a.has_bound = (constraint && constraint->has_bound) ? 1 : 0;
  a.bound = a.has_bound ? constraint->bound : 0.0;
  a.T = d_time; a.C = d_cost; a.mem = d_mem; a.mask = d_mask;
  launch_placements(pl, a, st);
  HIP_TRY(hipGetLastError());
  return SAILOR_OK;
}

sailor_status sailor_eval_replica_placements(sailor_plan *pl, uint64_t count, const int32_t *d_desc,
                                             const int32_t *d_pools, uint64_t stride,
                                             const int32_t *d_tps, uint32_t tps_stride,
                                             sailor_objective objective,
                                             const sailor_constraint *constraint, double *d_time,
                                             double *d_cost, uint64_t *d_mem, uint32_t *d_mask,
                                             void *hip_stream) {
  if (!pl || (objective != SAILOR_MAX_THROUGHPUT && objective != SAILOR_MIN_COST)) return SAILOR_EINVAL;
  if (count == 0) return SAILOR_OK;
  if (!d_desc || !d_pools || stride < 1 || (d_tps && tps_stride < 1)) return SAILOR_EINVAL;
  if (pl->dev.mixed || pl->dev.ZGr > kSearchMaxPools) return SAILOR_EINVAL;
  if (count > (uint64_t)0x7fffffff) return SAILOR_ERANGE;
  if (constraint && constraint->has_bound && std::isnan(constraint->bound)) return SAILOR_EINVAL;
  HIP_TRY(hipSetDevice(pl->device));
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  sailor_status rc;
  try { rc = search_setup(pl, false); } catch (...) { rc = SAILOR_ENOMEM; }
  if (rc != SAILOR_OK) return rc;
  rc = refresh_avail(pl, st);
  if (rc != SAILOR_OK) return rc;
  ReplicaArgs a{};
  a.count = count; a.desc = d_desc; a.pools = d_pools; a.stride = stride;
  a.tps = d_tps; a.tps_stride = tps_stride;
  a.pps = pl->d_search_pps; a.n_pp = (int)pl->search_pps.size();
  a.objective = (int)objective;
  a.has_bound = (constraint && constraint->has_bound) ? 1 : 0;
  a.bound = a.has_bound ? constraint->bound : 0.0;
  a.T = d_time; a.C = d_cost; a.mem = d_mem; a.mask = d_mask;
  k_eval_replicas<<<(unsigned)((count + kReplicaWaves - 1) / kReplicaWaves), kReplicaWaves * 64,
                    replica_lds_bytes(pl->dev), st>>>(pl->dev, a);
  HIP_TRY(hipGetLastError());
  return SAILOR_OK;
}

sailor_status sailor_search(sailor_plan *pl, sailor_objective objective,
                            const sailor_constraint *constraint, const sailor_search_options *opt,
                            sailor_stage_plan *out, void *hip_stream) {
  if (!pl || !opt || !out || (objective != SAILOR_MAX_THROUGHPUT && objective != SAILOR_MIN_COST))
    return SAILOR_EINVAL;
  if (opt->beam_width < 1 || opt->beam_width > kSearchMaxBeam || opt->max_runs < 0 ||
      opt->use_incumbent < 0 || opt->use_incumbent > 2)
    return SAILOR_EINVAL;
  if (opt->use_incumbent == 1 && std::isnan(opt->incumbent)) return SAILOR_EINVAL;
  if (opt->allow_split != 0 && opt->allow_split != 1) return SAILOR_EINVAL;
  if (opt->stage_tp != 0 && opt->stage_tp != 1) return SAILOR_EINVAL;
  // plain pools, constant link bandwidths, a pipeline's stages numbered in a byte
  if (pl->dev.mixed || pl->dev.n_bw_coef > 0 || pl->dev.ZGr > kSearchMaxPools ||
      pl->dev.P_max > kSearchMaxStages)
    return SAILOR_EINVAL;
  int has_bound;
  double bound;
  float lim_s, lim_l;
  sailor_status rc = constraint_limits(objective, constraint, &has_bound, &bound, &lim_s, &lim_l);
  if (rc != SAILOR_OK) return rc;
  HIP_TRY(hipSetDevice(pl->device));
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  try { rc = search_setup(pl, true); } catch (...) { rc = SAILOR_ENOMEM; }
  if (rc != SAILOR_OK) return rc;
  SearchArgs a{};
  a.objective = (int)objective;
  a.has_bound = has_bound;
  a.bound = bound;
  a.W = opt->beam_width;
  a.max_runs = opt->max_runs;
  const bool split = opt->allow_split != 0, stp = opt->stage_tp != 0;
  const size_t W = (size_t)a.W, ZG = (size_t)pl->dev.ZGr, TPn = stp ? (size_t)pl->dev.TP : 1;
  a.pps = pl->d_search_pps;
  a.alike = pl->search_alike;
  a.n_pp = (int)pl->search_pps.size();
  a.n_sub = stp ? pl->n_sub_t : pl->n_sub;
  a.list = pl->search_list;
  a.counters = pl->search_counters;
  a.root_expanded = pl->search_root_expanded;
  a.results = pl->search_results;
  // room for what a level can have, and for twice the beam
  a.buf = (uint32_t)std::min<size_t>(kSearchBuf, std::max(2 * W, W * ZG * std::max<size_t>(TPn, 1)));
  // split stages: about 16 KiB of tables for a block of states
  a.block = (uint32_t)std::max<size_t>(1, std::min(W, 1024 / (TPn * ZG)));
  // Frontiers and history stay in LDS as long as two workgroups fit a compute unit; wide beams keep the
  // history, then the frontiers too, in device memory.
  SearchLds layout;
  auto lds_bytes = [&]() { return search_carve(pl->dev, split, stp, false, a, nullptr, layout) * 8; };
  size_t lds = lds_bytes();
  if (lds > kSearchLds) {
    const size_t words = (size_t)kSearchWorkgroups * W * pl->dev.P_max;
    if (words > pl->search_history_cap) {
      // (no search is in flight on these buffers: every call waits for its own kernels)
      pl->arena.free_one(pl->search_history);
      pl->search_history = nullptr;
      pl->search_history_cap = 0;
      if (pl->arena.alloc(&pl->search_history, words) != hipSuccess) return SAILOR_ENOMEM;
      pl->search_history_cap = words;
    }
    a.history = pl->search_history;
    lds = lds_bytes();
  }
  if (lds > kSearchLds || a.W > kSearchNarrow) {
    const size_t words = (size_t)kSearchWorkgroups * 2 * W * search_state_words(true, (int)ZG);
    if (words > pl->search_states_cap) {
      pl->arena.free_one(pl->search_states);
      pl->search_states = nullptr;
      pl->search_states_cap = 0;
      if (pl->arena.alloc(&pl->search_states, words) != hipSuccess) return SAILOR_ENOMEM;
      pl->search_states_cap = words;
    }
    a.states = pl->search_states;
    lds = lds_bytes();
  }
  if (lds > kSearchMaxLds && split && stp) {
    a.by_zone = 1;
    lds = lds_bytes();
  }
  SearchLaunch launch{};
  launch.wgs = std::min(a.n_sub, kSearchWorkgroups);
  launch.lds = lds;
  launch.root_words = search_carve(pl->dev, split, stp, true, a, nullptr, layout);
  launch.root_waves = (unsigned)std::min<size_t>(kRootWaves, kSearchMaxLds / (launch.root_words * 8));
  launch.root_wgs = std::min<unsigned>(kRootWorkgroups, (a.n_sub + kRootWaves - 1) / kRootWaves);
  // (cannot be: at 64 pools, 255 stages, 8 degrees and the widest beam the tables take 125 KiB, a wave's of the first level 40)
  if (lds > kSearchMaxLds || launch.root_waves == 0) return SAILOR_EINVAL;
  if (opt->use_incumbent == 1) {
    a.has_inc = 1;
    a.inc = opt->incumbent;
  } else if (opt->use_incumbent == 2) {
    // the best plan of the flat space (at most three contiguous runs) through the evaluator:
    // every placement whose bound exceeds its key can be dropped
    ResultHeader hdr;
    rc = run_selection(pl, objective, constraint, 0, st, &hdr);
    if (rc != SAILOR_OK) return rc;
    if (hdr.n_found) {
      const RefRec *rec = reinterpret_cast<const RefRec *>(static_cast<char *>(pl->h_result) + sizeof(ResultHeader));
      a.has_inc = 1;
      a.inc = (objective == SAILOR_MAX_THROUGHPUT ? rec[0].T : rec[0].C) * (1.0 + 1e-9);
    }
  }
  rc = refresh_avail(pl, st);
  if (rc != SAILOR_OK) return rc;
  if (pl->search_dirty)  // (the last kernel of a search leaves the counters at zero)
    HIP_TRY(hipMemsetAsync(pl->search_counters, 0, ((size_t)a.n_pp + 1) * sizeof(uint32_t), st));
  pl->search_dirty = true;  // until this search has succeeded
  if (split && stp) launch_search<SEARCH_SPLIT_TP>(pl, a, launch, st);
  else if (split) launch_search<SEARCH_SPLIT>(pl, a, launch, st);
  else if (stp) launch_search<SEARCH_STAGE_TP>(pl, a, launch, st);
  else launch_search<SEARCH_PLAIN>(pl, a, launch, st);
  // what the host reads is written to the mapped result area (the flat space's results, if any, have
  // been read): the winner, then its T, C, mem and mask
  SubResult *const d_fin = reinterpret_cast<SubResult *>(pl->d_out);
  double *const d_ev = reinterpret_cast<double *>(d_fin + 1);
  k_search_pick<<<1, 1024, 0, st>>>(a, launch.wgs, launch.root_wgs, pl->search_final, d_fin);
  // the winner once more through the simulator, for its memory footprint and its mask
  PlaceArgs pa{};
  pa.count = 1;
  pa.desc = pl->search_final->desc;  // (device addresses: nothing is read here)
  pa.pools = pl->search_final->pools;
  pa.pools_b = split ? pl->search_final->pools_b : nullptr;
  pa.tps = pl->search_final->tps;
  pa.pool_stride = sizeof pl->search_final->pools / sizeof pl->search_final->pools[0];
  pa.pps = pl->d_search_pps;
  pa.n_pp = a.n_pp;
  pa.objective = (int)objective;
  pa.has_bound = has_bound;
  pa.bound = bound;
  pa.T = d_ev;
  pa.C = d_ev + 1;
  pa.mem = reinterpret_cast<uint64_t *>(d_ev + 2);
  pa.mask = reinterpret_cast<uint32_t *>(d_ev + 3);
  pa.hdr = pl->d_hdr;
  pa.seq = ++pl->seq;
  launch_placements(pl, pa, st);
  HIP_TRY(hipGetLastError());
  rc = wait_for_result(pl, st);
  if (rc != SAILOR_OK) return rc;
  pl->search_dirty = false;
  const SubResult &fin = *reinterpret_cast<const SubResult *>(static_cast<char *>(pl->h_result) + sizeof(ResultHeader));
  const double *ev = reinterpret_cast<const double *>(&fin + 1);
  std::memset(out, 0, sizeof *out);
  for (int i = 0; i < SAILOR_MAX_STAGES; ++i) out->pool[i] = out->pool_b[i] = out->stage_tp_index[i] = -1;
  out->exact = fin.truncated ? 0 : 1;
  out->expanded = fin.expanded;
  out->incumbent_used = a.has_inc;
  out->incumbent = a.has_inc ? a.inc : 0.0;
  if (!fin.found) return SAILOR_ENOFEASIBLE;
  out->found = 1;
  out->pp_index = fin.desc[0];
  out->partition = fin.desc[1];
  out->tp_index = fin.desc[2];
  out->dp_index = fin.desc[3];
  out->mb_index = fin.desc[4];
  out->pp = pl->ppv[fin.desc[0]];
  out->tp = pl->tpv[fin.desc[2]];
  out->dp = pl->dpv[fin.desc[3]];
  out->mb = pl->mbv[fin.desc[4]];
  out->iter_time_s = fin.T;
  out->cost_per_iter = fin.C;
  out->eval_time_s = ev[0];
  out->eval_cost = ev[1];
  std::memcpy(&out->peak_mem_bytes, &ev[2], sizeof(uint64_t));
  std::memcpy(&out->mask, &ev[3], sizeof(uint32_t));
  for (int i = 0; i < out->pp; ++i) {
    out->pool[i] = fin.pools[i];
    out->pool_b[i] = fin.pools_b[i];
    out->stage_tp_index[i] = fin.tps[i];
  }
  return SAILOR_OK;
}

sailor_status sailor_set_scan_unit_parts(int32_t n) {
  if (n < 0 || n > 255) return SAILOR_EINVAL;
  g_forced_unit_parts.store(n, std::memory_order_relaxed);
  return SAILOR_OK;
}

sailor_status sailor_plan_set_incremental(sailor_plan *pl, int32_t on) {
  if (!pl || (on != 0 && on != 1)) return SAILOR_EINVAL;
  if (on && !pl->ubits) {  // (45 MB for the 14 000 units of 1.1e9 plans: allocated where it is used)
    HIP_TRY(hipSetDevice(pl->device));
    try {
      const BesideCaptures beside;
      if (pl->arena.alloc(&pl->ubits, pl->units.size() * (size_t)pl->ubits_stride) != hipSuccess) {
        (void)hipGetLastError();  // (reported here)
        pl->ubits = nullptr;
        return SAILOR_ENOMEM;
      }
    } catch (...) { return SAILOR_ENOMEM; }
  }
  if (pl->incremental != (on != 0)) pl->cache_ok = false;  // what a scan keeps depends on it
  pl->incremental = on != 0;
  return SAILOR_OK;
}

sailor_status sailor_plan_last_scan(sailor_plan *pl, uint32_t *units_evaluated,
                                    uint32_t *units_total) {
  if (!pl || !pl->have_hdr) return SAILOR_EINVAL;
  const uint32_t total = (uint32_t)pl->units.size();
  if (units_evaluated) {
    if (pl->last_direct) {
      *units_evaluated = pl->last_direct_units;
    } else {
      // every unit carries the number of the call that evaluated it last; they are counted
      // here, off the selection's own path
      HIP_TRY(hipSetDevice(pl->device));
      uint32_t *seq = new (std::nothrow) uint32_t[total];
      if (!seq) return SAILOR_ENOMEM;
      const hipError_t e = hipMemcpy(seq, pl->unit_seq, total * sizeof(uint32_t), hipMemcpyDeviceToHost);
      uint32_t n = 0;
      for (uint32_t i = 0; i < total; ++i) n += seq[i] == pl->last_scan_seq ? 1u : 0u;
      delete[] seq;
      HIP_TRY(e);
      *units_evaluated = n;
    }
  }
  if (units_total) *units_total = total;
  return SAILOR_OK;
}

sailor_status sailor_plan_last_counts(const sailor_plan *pl, uint32_t *survivors,
                                      uint32_t *refined, uint32_t *feasible) {
  if (!pl || !pl->have_hdr) return SAILOR_EINVAL;
  if (survivors) *survivors = pl->last_hdr.surv_count;
  if (refined) *refined = pl->last_hdr.ref_count;
  if (feasible) *feasible = pl->last_hdr.feasible_count;
  return SAILOR_OK;
}

}  // extern "C"

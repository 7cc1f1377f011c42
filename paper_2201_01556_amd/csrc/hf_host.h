// Host-side state of a flow problem handle and internal entry points.
#pragma once
#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "hf_device.h"
#include "hyperflow.h"

namespace hf {

// kernel kinds for per-launch timing
enum KernelKind : int {
  KK_INIT = 0,
  KK_GR_RESET,
  KK_BFS_REV,
  KK_BFS_REV_LOOP,
  KK_GATHER,
  KK_PUSH,
  KK_APPLY,
  KK_ROUND_LOOP,
  KK_CUT_SEED,
  KK_BFS_FWD,
  KK_BFS_FWD_LOOP,
  KK_CUT_OUT,
  KK_CHECK,
  KK_BATCH,
  KK_BFS_COLLECT,
  KK_COUNT
};

const char* kernel_kind_name(int k);
// device byte-counter class of a kernel kind (-1: none)
int kernel_kind_class(int k);

struct Timer {
  int kind;
  hipEvent_t a, b;
};

// State of a FlowCutter run between calls: flow_problem_flowcutter starts a
// run, flow_problem_flowcutter_continue resumes one that stopped at its
// iteration limit (the loop variables below are exactly those of one
// uninterrupted run).
struct FcRun {
  bool active = false;  // stopped at the iteration limit; may be continued
  int64_t max_src = 0, max_snk = 0;
  int32_t bulk_percent = 0, most_balanced = 0;
  long long total = 0;  // c(V)
  int32_t it = 0;       // iterations done
  fp_cutter_result r{};
  // most balanced cut so far
  long long best_heavier = -1, best_src = 0, best_snk = 0;
  int best_kind = 0;
  int64_t best_F = 0;
  int32_t first_balanced = 0;
  // bulk piercing bookkeeping per side
  long long pierces[2] = {0, 0}, gained[2] = {0, 0}, pierced[2] = {0, 0};
  long long term[2] = {-1, -1}, missed[2] = {0, 0};
  int pend_side = -1;
  long long pend_before = 0, pend_count = 0, pend_goal = -1;
  // reachable sets kept across a pierce without augmenting path
  int prev_ep_s = -1, prev_ep_t = -1, grow = -1, grow_vertex = -1;
  // vertices of S_r and T_r that are listed as not pierced yet (-1: not
  // listed), and a bound below which every vertex is in one of the sides
  int32_t fresh[2] = {-1, -1};
  int32_t lo = 0;
  bool next_known = false;  // the bitmaps of the vertices next to S_r and T_r are up to date
  int64_t last_F = 0;
  long long last_cs = 0, last_ct = 0;
  int out_ep = -1, out_invert = 0;
};

}  // namespace hf

struct fp_problem {
  int device = 0;
  int32_t V = 0, E = 0, P = 0, NB = 0, N = 0;
  int32_t nS = 0, nT = 0;
  int64_t wsum = 0;          // sum of the net weights (at most INT32_MAX)
  fp_options opt{};
  fp_options opt_user{};     // the options as the caller gave them (zeros = defaults)
  hf::Dev dev{};
  void* pool = nullptr;
  size_t pool_bytes = 0;     // capacity of the pool (a reused block may be larger)
  hf::Ctl* ctl_h = nullptr;  // pinned host mirror of the control block
  int32_t epoch = 1;         // stamp value of the next round / BFS
  int32_t gr_batch = 8;      // device-wide levels launched first by a global relabel
  int32_t gr_hist[hf::kLvlHist] = {};  // level sizes of the previous global relabel's BFS
  int32_t gr_hist_levels = 0;
  bool inited = false;
  bool solved = false;
  bool warm_labels = false;  // the labels are valid for the next solve (after a source pierce)
  bool labels_exact = false;  // the labels are exact distances of the current flow (a solve ended)
  int32_t* cw = nullptr;     // vertex weights of the last FlowCutter run (device)
  void* fc_mem = nullptr;    // FlowCutter scratch (FcMem)
  hf::FcRun fc;
  fp_stats st{};
  // profiling
  std::vector<hf::Timer> pending;
  int64_t k_launches[hf::KK_COUNT] = {};
  double k_ms[hf::KK_COUNT] = {};
  unsigned long long bytes_at_sync[hf::KC_N] = {};
  double k_bytes[hf::KK_COUNT] = {};
};

// Flow problems of block pairs built on the device (hf_regions.hip).
struct fp_regions {
  int device = 0;
  int32_t npairs = 0, k = 0, V = 0;
  void* mem = nullptr;                   // device outputs (one allocation)
  int32_t* off = nullptr;                // per pair ne+1 relative offsets
  int32_t* pins = nullptr;               // local ids
  int32_t* w = nullptr;                  // net weights
  int32_t* ngid = nullptr;               // global net id (smallest of a group)
  int32_t* vw = nullptr;                 // per pair n+2 vertex weights
  int32_t* vgid = nullptr;               // per pair n global vertex ids
  int8_t* vside = nullptr;               // per pair n: 0 = region of block i, 1 = of block j
  int32_t* terms = nullptr;              // per pair {n, n+1}
  std::vector<int32_t> pairs;            // 2 per pair
  std::vector<int64_t> info;             // npairs * 16
  std::vector<long long> net_base, pin_base, vtx_base, nloc;  // where pair q starts; n
  std::vector<long long> wsum;           // net weight sum per pair (filled by the first solve)
  uint8_t* sides = nullptr;              // per pair n+2 bytes: minimal source side of the last solve
  bool solved = false;
};

namespace hf {

void set_error(const char* fmt, ...);
fp_status hip_fail(hipError_t e, const char* what);

// defaults filled in, but for those that the size decides (resolve_by_size)
fp_options resolve_options(const fp_options* o);

// Bytes of the bitmaps of swept reverse-BFS levels (Dev::vf, nl, pinfree).
// They lie in the memory of the byte marks, which only another form of a level
// uses: its N bytes hold them unless nets have far more pins than there are
// nodes.
struct SweepMaps {
  size_t vf, nl, pinfree;
  bool fit;
  SweepMaps(long long V, long long E, long long P, long long N) {
    auto up = [](long long n) { return (size_t)((n + 255) & ~255ll); };
    vf = up((V + 63) / 64 * 8);
    nl = up((E + 63) / 64 * 16);
    pinfree = up((P + 31) / 32 * 4);
    fit = (long long)(2 * vf + 2 * nl + pinfree) <= N;
  }
};

// Whether large reverse-BFS levels are swept (phase_bfs_sweep): in the default
// form of a level, if the bitmaps fit.
inline bool levels_swept(const fp_options& o, const SweepMaps& m) {
  return m.fit && o.bfs_flat > 0 && o.bfs_arc_parallel == 0 && o.bfs_marks <= 0 &&
         o.bfs_xcd <= 0 && o.pull_min <= 0;
}

constexpr long long kSweepNodes = 1 << 20;  // networks with levels worth a sweep

// A large network whose levels cannot be swept: its relabels cost more.
inline bool dear_relabels(long long N, bool swept) { return N >= kSweepNodes && !swept; }

// The defaults that depend on the network's size and form.
//
// bottom_up_min, from how many nodes on a level is handled without claims.
// Swept: a sweep costs two more launches a level and a pass over the
// unlabelled nodes, so it needs levels of some hundred thousand nodes.  From
// N/50, N/16 and N/8 on and never, a 7.4M-pin flow (N = 5 M, levels of 0.5-1.3 M)
// takes 19.5, 19.0, 19.1 and 23.1 ms; one of 740k pins (N = 500k, levels of up
// to 130k) 7.9, 7.5, 7.4 and 7.0 ms, and a region problem (N = 100k) 3.4 ms
// against 3.0 never.  Not swept, a level is expanded from its list with plain
// stores, which pays where a level holds many arcs per node, since a claim is
// an atomic per arc: nets of 60 pins, from N/50 on against N/16 and never, 16.2 /
// 17.4 / 18.7 ms at N = 1.1 M, 11.6 / - / 12.4 at 660k, 4.9 / - / 5.1 at 220k, but
// 3.0 / - / 2.7 at 44k (720k pins); nets of 200 and 500 pins, N = 40k to 140k, 3.1 to
// 4.1 against 3.8 to 5.3; nets of 20 and 30 pins are faster with claims.
//
// gr_interval, rounds between global relabels (in the single-workgroup loop
// 25 by default, tail_rounds; measured at 24).  Intervals 16 (64 in the loop) / 10
// (24) / 8 (24), means over eight seeds in us: V = 2k
// 2121 / 2123 / 2087, 12k 3840 / 3681 / 3524, 40k 5475 / 4831 / 4892, 100k
// 7166 / 6412 / 6517, 300k 9894 / 8764 / 9430, 1M 15671 / 15330 / 16403,
// region problems of 5k, 20k and 40k vertices 2505 / 2489 / 2470,
// 2771 / 2574 / 2474, 3729 / 3264 / 3754.  Dear relabels keep the longer interval:
// 60-pin nets with N = 1.1 M 15.1 ms at 16 (64), 16.2 at 10 (25); a 7.4M-pin flow
// with bfs_arc_parallel 46.3 and 49.4, with bfs_flat = -1 18.4 and 19.1, with
// pull_min 83.7 and 89.7.
inline void resolve_by_size(fp_options* o, long long V, long long E, long long P, long long N) {
  const bool swept = levels_swept(*o, SweepMaps(V, E, P, N));
  const bool many_arcs = P >= 16 * N && P >= (1 << 21);
  if (o->bottom_up_min == 0)
    o->bottom_up_min = N >= kSweepNodes && swept ? (int32_t)(N / 16 > 262144 ? N / 16 : 262144)
                       : N >= kSweepNodes || many_arcs ? (int32_t)(N / 50 > 1024 ? N / 50 : 1024)
                                                       : -1;
  if (o->bottom_up_min < 0) o->bottom_up_min = 0;
  if (o->gr_interval == 0) o->gr_interval = dear_relabels(N, swept) ? 16 : 10;
  if (o->gr_interval < 0) o->gr_interval = 0;
}

// The same threshold of the forward BFS (0 = never), which expands its levels
// and is not swept: the caller's, or for large networks N/50, whatever the
// reverse one is (source sides of 979,000 and 294,000 vertices 0.955 and 0.457 ms
// from N/50 on, 0.964 and 0.471 from N/16; below 2^20 nodes 0.12 to 0.26 ms
// claimed, 0.13 to 0.28 expanded).
inline int32_t forward_min(const fp_options& o, const fp_options& user, long long N) {
  if (user.bottom_up_min != 0 || o.bottom_up_min == 0 || N < kSweepNodes) return o.bottom_up_min;
  return (int32_t)(N / 50);
}

// Rounds between global relabels while the frontier fits the single-workgroup
// loop.  Its rounds cost a few microseconds and a global relabel (a BFS over
// every node) as much as two hundred of them, so it relabels less often: 2.5
// times gr_interval, 4 times where relabels are dear (the figures above).
inline int tail_rounds(const fp_options& o, long long N, bool swept) {
  if (o.tail_gr_interval > 0) return o.tail_gr_interval;
  if (o.tail_gr_interval < 0) return o.gr_interval;
  return dear_relabels(N, swept) ? 4 * o.gr_interval : 5 * o.gr_interval / 2;
}

// Validate the inputs and build the device layout.  With `ext` the layout
// (and the temporary memory of the build) is carved from the caller's
// ext_bytes of device memory and pb->ctl_h must point to the caller's host
// mirror of the control block; otherwise the handle's pool and control
// block are allocated (or taken from the cache).
fp_status build_problem(fp_problem* pb, const int32_t* net_offsets, const int32_t* pins,
                        const int32_t* net_weights, const int32_t* sources, int32_t nS,
                        const int32_t* sinks, int32_t nT, int32_t mem_kind,
                        hipStream_t s, void* ext = nullptr, size_t ext_bytes = 0);
fp_status solve_problem(fp_problem* pb, hipStream_t s, int64_t* flow);
fp_status cut_problem(fp_problem* pb, hipStream_t s, int32_t mem_kind, uint8_t* vside,
                      uint8_t* nside);
fp_status batch_solve(fp_problem* const* pbs, int32_t count, const uint8_t* skip,
                      hipStream_t s, int64_t* flows);
// a configuration (zero fields = defaults) that create_batch accepts
bool batch_config_ok(const fp_batch_config* c);
fp_status create_batch(fp_problem* const* pbs, int32_t count, uint8_t* const* vsides,
                       uint8_t* const* nsides, const fp_batch_config* config, hipStream_t s,
                       fp_batch** out);
fp_status run_batch(fp_batch* b, const uint8_t* skip, int32_t with_cut, hipStream_t s,
                    int64_t* flows);
fp_status tune_batch(fp_batch* b, hipStream_t s, const char* cache_path, fp_batch_config* chosen);
fp_status batch_config(const fp_batch* b, fp_batch_config* out);
void release_batch(fp_batch* b);
fp_status scorer_create_impl(const float* init, hipStream_t s, fp_scorer** out);
void scorer_destroy_impl(fp_scorer* sc);
fp_status scorer_fit_impl(fp_scorer* sc, const int64_t* f, int n, int mem_kind, hipStream_t s);
fp_status scorer_gradient_impl(fp_scorer* sc, const int64_t* f, const float* y, int n,
                               int mem_kind, hipStream_t s, float* grad, float* loss);
fp_status scorer_train_impl(fp_scorer* sc, const int64_t* f, const float* y, int n, int mem_kind,
                            int steps, float lr, hipStream_t s, float* losses);
fp_status scorer_predict_impl(fp_scorer* sc, const int64_t* f, int n, int mem_kind,
                              hipStream_t s, float* prob);
fp_status scorer_get_impl(const fp_scorer* sc, float* params, double* mean_std);
fp_status scorer_set_impl(fp_scorer* sc, const float* params, const double* mean_std);
fp_status pierce_problem(fp_problem* pb, int32_t side, const int32_t* vertices, int32_t n,
                         hipStream_t s);
fp_status sink_side_problem(fp_problem* pb, hipStream_t s, int32_t mem_kind, uint8_t* vside);
fp_status flowcutter_problem(fp_problem* pb, const int32_t* vw, int64_t max_src, int64_t max_snk,
                             int32_t max_iters, int32_t bulk_percent, int32_t most_balanced,
                             hipStream_t s, int32_t mem_kind, uint8_t* vside,
                             fp_cutter_result* res, fp_cutter_step* trace);
fp_status flowcutter_continue(fp_problem* pb, int32_t max_iters, hipStream_t s, int32_t mem_kind,
                              uint8_t* vside, fp_cutter_result* res, fp_cutter_step* trace);
fp_status terminals_problem(fp_problem* pb, hipStream_t s, int32_t mem_kind, uint8_t* roles);
fp_status export_state(fp_problem* pb, hipStream_t s, int32_t* f_in, int32_t* f_out,
                       int32_t* f_b, int32_t* labels, int32_t* excess);
void release_problem(fp_problem* pb);
// A block of device memory of at least `bytes` (its size in *got), from the
// cache of released ones or newly allocated, and its return once no work uses it.
hipError_t pool_acquire(int device, size_t bytes, void** out, size_t* got);
void pool_release(int device, void* ptr, size_t bytes);
// free the device pools and pinned control blocks kept for reuse
void release_cached_memory();

// profiling helpers
void prof_begin(fp_problem* pb, int kind, hipStream_t s, Timer* t);
void prof_end(fp_problem* pb, Timer* t, hipStream_t s);
void prof_collect(fp_problem* pb);
// timing events go back to the process-wide pool of their device
void event_pool_put(int device, hipEvent_t e);

}  // namespace hf

// Device-side phases of the hypergraph push-relabel solver (gfx950).
//
// Network (Lawler expansion, paper section "Preliminaries", paragraph "Flows
// on Hypergraphs"), simulated on the hypergraph itself as the paper's
// paragraph "Hypergraph Implementation" describes -- the expanded graph is
// never built.  Node ids:
//   v            in [0, V)      hypernode
//   NB + 2e                     e_in  of net e     (NB = V rounded up to even,
//   NB + 2e + 1                 e_out of net e      so (e_in, e_out) labels form
//                                                   an aligned int2)
// Source and sink sets are contracted: a net with a source pin receives w(e)
// units into e_in at initialisation (its contracted source arc, capped at
// w(e)); sinks keep label 0 and absorb whatever is pushed into them.
// Source vertices keep label N+1 so that nothing is ever pushed into them.
//
// Per pin slot p (net-CSR order) the state is {r_in, f_out}:
//   r_in  = w(e) - flow(u, e_in)      residual of the capped arc u -> e_in
//   f_out = flow(e_out, u)            residual of the reverse arc u -> e_out
// per net: fb = flow(e_in, e_out).  Residual capacities:
//   u     -> e_in   r_in              u     -> e_out  f_out
//   e_in  -> e_out  w - fb            e_in  -> u      w - r_in
//   e_out -> u      infinite          e_out -> e_in   fb
//
// One discharge round (paper section "Synchronous Parallel Push-Relabel") is
// two phases with an ordering point between them:
//   push   every frontier node u first folds the excess it received in the
//          previous round (dx[prev]) into x[u].  If its label k = d(u) < N it
//          pushes along arcs admissible under the round-start labels
//          (residual > 0 and d(v) = k - 1), distributing its excess over them
//          in arc order; received amounts go to dx[cur][v] (the "excess
//          differences aggregated in a second array" of the paper), so no
//          node ever reads an excess that is still changing and rounds are
//          deterministic.  A node left with excess records
//          cand = 1 + min label over the arcs that stay residual after its own
//          pushes.  Admissibility is antisymmetric in the labels, so each arc
//          pair has a single writer per round and no winning criterion is
//          needed.
//   apply  a node left with excess is relabelled to
//          min(cand, d(u) + 2 if something was pushed into u this round, N).
//          Pushes into u come from nodes labelled d(u) + 1 and are the only
//          residual arcs u could not see; the bound keeps every label valid
//          (d(a) <= d(b) + 1 on every residual arc), which rules out the
//          push-relabel conflict described in section "A Bug in the
//          Synchronous Algorithm".
// Frontier of the next round = nodes pushed into (listed by the first push,
// the one that finds no excess delivered yet) plus nodes relabelled below N
// (paragraph "Active Nodes").  Device-wide phases stage appends per wave in
// LDS and flush them with one global atomic per batch; the single-workgroup
// loop (wg_rounds) keeps the lists in LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hf {

constexpr int kWave = 64;
constexpr int kInf = 0x7fffffff;
// Nodes with more arcs than this are scanned by a whole workgroup in the
// reverse BFS (a wave alone would take thousands of steps).
constexpr int kHugeDeg = 2048;

// error bits reported through Ctl::err
enum : int32_t {
  ERR_LABEL = 1,         // a relabel did not raise the label
  ERR_SINK_REACHED = 2,  // forward cut BFS reached a sink
  ERR_INVARIANT = 4,     // debug invariant check failed
  ERR_SOURCE_REACHED = 8,  // sink-side BFS reached a source
  ERR_PIERCE_TERMINAL = 1024,  // a piercing vertex is a terminal of the other side
  ERR_GUARD = 2048,  // a solve inside one workgroup passed its round or level bound
  ERR_BUILD_PIN = 16,
  ERR_BUILD_OFFSETS = 32,
  ERR_BUILD_WEIGHT = 64,
  ERR_BUILD_DUP = 128,
  ERR_BUILD_TERMINAL = 256,
  ERR_BUILD_ST = 512,
};

// kernel classes for the device byte / item counters
enum : int {
  KC_PUSH = 0,
  KC_APPLY = 1,
  KC_BFS_REV = 2,
  KC_BFS_FWD = 3,
  KC_LOOP_ROUNDS = 4,
  KC_LOOP_BFS = 5,
  KC_BATCH = 6,
  KC_N = 8
};

// A frontier is four lists: small vertices, small e_in, small e_out (nodes
// with at most big_deg arcs, processed by groups of G lanes) and big nodes of
// any kind (processed by whole waves).  Splitting by kind keeps every wave
// item on one code path.
constexpr int kNL = 4;
constexpr int kLvlHist = 64;  // reverse-BFS levels whose sizes are kept
constexpr int kBigList = 3;

struct Ctl {
  int32_t fcnt[3][kNL];  // round frontier counts, ring by epoch % 3
  int32_t bcnt[3][kNL];  // BFS level counts, ring by level % 3
  int32_t err;
  int32_t loop_rounds;  // rounds run by the last single-workgroup round loop
  int32_t loop_levels;  // levels run by the last single-workgroup BFS loop
  int32_t loop_exit;
  int32_t bfs_done;     // the last single-workgroup BFS loop ended on an empty level
  unsigned long long flow;      // flow value (into sinks)
  unsigned long long relabels;  // relabel operations
  unsigned long long bytes[KC_N];
  unsigned long long items[KC_N];
  unsigned long long side_weight[2];  // FlowCutter: c(S_r), c(T_r)
  int32_t pierce[5];  // FlowCutter: per side s, [3s] smallest free boundary pin and
                      // [3s + 1] smallest augmenting pin; [2] smallest free vertex
  int32_t big_last;   // last reverse-BFS level of the current global relabel
                      // whose frontier exceeded the single-workgroup tail
  int32_t lvl_nf[kLvlHist];  // size of each of the first reverse-BFS levels of
                             // the current global relabel
  int32_t bits_level;  // reverse-BFS level that the level bitmaps describe, -1 none
  int32_t swept;       // last level that was swept (phase_bfs_sweep), -1 none
  int32_t nswept;      // levels swept since the state was initialised
  int32_t sweep_n[2][3];  // nodes per kind that the sweep of an even (odd) level found
  int32_t fc_done;        // iterations that the last FlowCutter loop finished
  int32_t fc_why;         // why it ended (FcExit)
  int32_t fc_side;        // side that it pierced last or was to pierce next
  int32_t fc_levels;      // levels of its finished growths
  int32_t fc_new[2];      // vertices of S_r and T_r listed as not pierced yet
};

struct Dev {
  int32_t V, E, P, NB, N, nT, big_deg, bfs_arc;  // bfs_arc: arc-parallel BFS levels
  int32_t bfs_flat;        // reverse-BFS levels spread each wave's 64 nodes' arcs over its lanes
  int32_t relabel_block;   // a node pushed to in a round does not relabel in it
  const int32_t* net_off;  // E+1
  const int32_t* pin_v;    // P
  const int32_t* pin_net;  // P   net of each pin slot
  const int32_t* w;        // E
  const int32_t* vtx_off;  // V+1
  const int2* vinc;        // P   {net, pin slot}, per vertex sorted by slot
  int32_t* role;           // V   0 free, 1 source, 2 sink
  int32_t* nflag;          // E   bit0 has a source pin, bit1 has a sink pin
  int32_t* fpin;           // 2P  {r_in, f_out}
  int32_t* fb;             // E
  int32_t* d;              // N   labels
  int32_t* x;              // N   excess (written by the node itself)
  int32_t* dx[2];          // N   excess received in a round, by round parity
  int32_t* cand;           // N   relabel candidate of a node left with excess, -1 = none
  int32_t* stamp;          // N
  const uint32_t* bigbits; // ceil(N/32) words: bit v set when node v has more than big_deg arcs
  const uint32_t* hugebits;  // ceil(N/32) words: bit v set when node v has more than kHugeDeg arcs
  uint32_t* seen;          // ceil(N/32) words: reverse BFS hint "node has a label" (see label_rev)
  uint8_t* lev;            // N bytes or null: reverse BFS marks, 0 unlabelled, 1 reached by
                           // the level being expanded, 2 labelled (see label_rev)
  int32_t* xbuf;           // null, or the per-workgroup, per-slice arc heads of an expanded
                           // reverse-BFS level (kMaxSliceGroups x 8 x xseg; see xpush)
  int32_t* xcnt;           // kMaxSliceGroups x 8 counts of xbuf
  int32_t xseg;            // entries per workgroup and slice
  uint32_t* pinres;        // ceil(P/32) words: bit of pin slot p = flow(u, e_in) > 0
  uint32_t* netres;        // ceil(E/8) words, 4 bits per net: bit0 = e_in -> e_out
                           // residual (fb < w), bit1 = pins carry flow out of
                           // e_out, bit2 = e_out -> e_in residual (fb > 0),
                           // bit3 = pins may carry flow into e_in
  uint32_t* pinfree;       // ceil(P/32) words: bit of pin slot p = r_in > 0; null when the
                           // swept levels are off (phase_bfs_sweep)
  uint32_t* vf[2];         // swept levels, by level parity: bit v = vertex v lies in the level
  uint2* nl[2];            // the same per 32 nets: x = e_in lies in the level, y = e_out does
                           // and pins carry flow out of it
  int32_t* list[2][kNL];   // [parity][list]: capacities V, E, E, N
  Ctl* ctl;
};

// ---------------------------------------------------------------------------
// wave / group utilities
// ---------------------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return __lane_id(); }
__device__ __forceinline__ unsigned long long lanemask_lt() {
  return (1ull << lane_id()) - 1ull;
}

// Workgroup sums of up to three per-thread counters, added to the global
// counters by thread 0: one atomic per workgroup and counter.  Same-address
// atomics issued by every wave of a full grid serialise in the memory system
// and cost more than the work they count.  Block-uniform (every thread of the
// workgroup calls it); blockDim a multiple of 64, at most 1024.
__device__ void block_add_u64(unsigned long long* d0, unsigned long long v0,
                              unsigned long long* d1 = nullptr, unsigned long long v1 = 0ull,
                              unsigned long long* d2 = nullptr, unsigned long long v2 = 0ull) {
  __shared__ unsigned long long part[3][16];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    v0 += __shfl_xor(v0, o);
    v1 += __shfl_xor(v1, o);
    v2 += __shfl_xor(v2, o);
  }
  const int wid = threadIdx.x >> 6;
  if (lane_id() == 0) {
    part[0][wid] = v0;
    part[1][wid] = v1;
    part[2][wid] = v2;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int c = threadIdx.x;
    unsigned long long s = 0ull;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += part[c][w];
    unsigned long long* d = c == 0 ? d0 : (c == 1 ? d1 : d2);
    if (d != nullptr && s != 0ull) atomicAdd(d, s);
  }
  __syncthreads();  // part may be written again by a later call
}

// Between the lanes of one wave that write LDS and those that read it: the
// wave's LDS accesses execute in order, so this costs no instruction, but
// without it the compiler may keep a lane's own value in a register where
// another lane has written since.  Called by all active lanes.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup minima of two per-thread values, folded into the global values
// by thread 0 (atomic min).  Block-uniform, as block_add_u64.
__device__ void block_min_i32(int32_t* d0, int v0, int32_t* d1, int v1) {
  __shared__ int part[2][16];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    v0 = min(v0, __shfl_xor(v0, o));
    v1 = min(v1, __shfl_xor(v1, o));
  }
  const int wid = threadIdx.x >> 6;
  if (lane_id() == 0) {
    part[0][wid] = v0;
    part[1][wid] = v1;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int c = threadIdx.x;
    int m = part[c][0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = min(m, part[c][w]);
    if (m != kInf) atomicMin(c == 0 ? d0 : d1, m);
  }
  __syncthreads();
}

template <int G>
__device__ __forceinline__ uint32_t g_scan_sat(uint32_t v, uint32_t cap, int gl) {
#pragma unroll
  for (int o = 1; o < G; o <<= 1) {
    const uint32_t t = __shfl_up(v, o, G);
    if (gl >= o) v = min(v + t, cap);
  }
  return v;
}

template <int G>
__device__ __forceinline__ int g_min(int v) {
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, G));
  return v;
}

// Loads that bypass the compiler's value caching (counters written by other
// waves between workgroup barriers).
__device__ __forceinline__ int ld_vol(const int32_t* p) {
  return *reinterpret_cast<const volatile int32_t*>(p);
}
__device__ __forceinline__ unsigned long long ld_vol64(const unsigned long long* p) {
  return *reinterpret_cast<const volatile unsigned long long*>(p);
}

__device__ __forceinline__ int count_all(const int32_t* c) {
  int n = 0;
#pragma unroll
  for (int k = 0; k < kNL; ++k) n += c[k];
  return n;
}
__device__ __forceinline__ int count_all_vol(const int32_t* c) {
  int n = 0;
#pragma unroll
  for (int k = 0; k < kNL; ++k) n += ld_vol(c + k);
  return n;
}

__device__ __forceinline__ int deg_of(const Dev& g, int v) {
  if (v < g.V) return g.vtx_off[v + 1] - g.vtx_off[v];
  const int e = (v - g.NB) >> 1;
  return g.net_off[e + 1] - g.net_off[e] + 1;
}

// ---------------------------------------------------------------------------
// block-level LDS staging of list appends
//
// Appends to a global list reserve space with an atomic on one counter, and
// same-address atomics serialise across the whole chip.  A workgroup
// therefore stages its appends in LDS (wave-aggregated LDS atomics) and
// reserves global space once per flush.  Flushes happen at block-uniform
// points: when the staging area may not hold the next tile's appends, and at
// the end of a phase.  A wave whose appends do not fit any more writes the
// excess straight to the global list (one global atomic for that wave).
// ---------------------------------------------------------------------------

// Staged entries per list: 4 per thread of the workgroup.  LDS words of a
// workgroup's staging area plus the arc tile of the arc-parallel BFS levels:
constexpr int kQPerThread = 4;
constexpr int lds_words(int block) {
  return kNL * kQPerThread * block + 2 * kNL + 3 * block + 1 + 32;
}
__device__ __forceinline__ int bq_words() { return kNL * kQPerThread * (int)blockDim.x + 2 * kNL; }

typedef __attribute__((address_space(3))) int32_t lds_int;
typedef __attribute__((address_space(3))) unsigned long long lds_u64;

struct BlockQ {
  lds_int* buf;         // [kNL][cap]
  lds_int* n;           // [kNL] staged counts (may exceed cap after overflow)
  lds_int* base;        // [kNL] global base of the current flush
  int32_t* gcnt;        // global counts [kNL]
  int32_t* dst[kNL];    // global lists
  int cap;              // staged entries per list
};

__device__ __forceinline__ int lds_add(lds_int* p, int v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Block-uniform: every thread of the workgroup calls it.
__device__ __forceinline__ BlockQ bq_bind(lds_int* lds, int32_t* gcnt, int32_t* const lists[kNL]) {
  BlockQ q;
  q.cap = kQPerThread * (int)blockDim.x;
  q.buf = lds;
  q.n = lds + kNL * q.cap;
  q.base = lds + kNL * q.cap + kNL;
  q.gcnt = gcnt;
#pragma unroll
  for (int k = 0; k < kNL; ++k) q.dst[k] = lists[k];
  __syncthreads();  // earlier users of the area are done with it
  if (threadIdx.x < kNL) q.n[threadIdx.x] = 0;
  __syncthreads();
  return q;
}

__device__ __forceinline__ bool is_big(const Dev& g, int v) {
  return (g.bigbits[v >> 5] >> (v & 31)) & 1u;
}
__device__ __forceinline__ bool is_huge(const Dev& g, int v) {
  return (g.hugebits[v >> 5] >> (v & 31)) & 1u;
}

// list of a node: big nodes together, small ones by kind
__device__ __forceinline__ int list_of(const Dev& g, int v) {
  if (is_big(g, v)) return kBigList;
  return v < g.V ? 0 : 1 + ((v - g.NB) & 1);
}

// Stage v into list k (if pred).  Called by all active lanes.  A lane at a time,
// which is the shorter code than a sum over the wave per list: a small level or
// frontier runs each instruction once, from a cold instruction cache (flows of
// 2k to 300k vertices 4 to 6 % faster).  What a hub's arcs reach past the
// staging area is counted per wave, since the global counters are few.
__device__ __forceinline__ void bq_push(const BlockQ& q, int k, int v, bool pred) {
  const int pos = pred ? lds_add(q.n + k, 1) : 0;
  const bool over = pos >= q.cap;
  if (pred && !over) q.buf[k * q.cap + pos] = v;
  for (unsigned long long m = __ballot(over); m;) {
    const int leader = __builtin_ctzll(m);
    const int list = __shfl(k, leader);
    const unsigned long long same = __ballot(over && k == list);
    int at = 0;
    if (lane_id() == leader) at = atomicAdd(&q.gcnt[list], __popcll(same));
    at = __shfl(at, leader);
    if (over && k == list) {
      int32_t* const dst =
          list == 0 ? q.dst[0] : list == 1 ? q.dst[1] : list == 2 ? q.dst[2] : q.dst[3];
      dst[at + __popcll(same & lanemask_lt())] = v;
    }
    m &= ~same;
  }
}

// Stage v (if pred) into its list.  Called by all active lanes.
__device__ __forceinline__ void qpush(const Dev& g, const BlockQ& q, int v, bool pred) {
  bq_push(q, pred ? list_of(g, v) : 0, v, pred);
}

// Block-uniform: move the staged entries to the global lists.
__device__ __forceinline__ void bq_flush(const BlockQ& q) {
  __syncthreads();
  if (threadIdx.x < kNL) {
    const int k = threadIdx.x;
    const int c = min((int)q.n[k], q.cap);
    q.base[k] = c ? atomicAdd(&q.gcnt[k], c) : 0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kNL; ++k) {
    const int c = min((int)q.n[k], q.cap);
    const int b = q.base[k];
    for (int i = threadIdx.x; i < c; i += blockDim.x) q.dst[k][b + i] = q.buf[k * q.cap + i];
  }
  __syncthreads();
  if (threadIdx.x < kNL) q.n[threadIdx.x] = 0;
  __syncthreads();
}

// Block-uniform: flush unless `reserve` more entries per list still fit.
__device__ __forceinline__ void bq_tile_end(const BlockQ& q, int reserve) {
  __syncthreads();
  int mx = 0;
#pragma unroll
  for (int k = 0; k < kNL; ++k) mx = max(mx, (int)q.n[k]);
  __syncthreads();  // every thread has read the counts before anyone appends
  if (mx > q.cap - reserve) bq_flush(q);
}

// Four values selected by a runtime index without a local array (which would
// live in scratch memory).
struct Quad {
  int v0, v1, v2, v3;
  __device__ __forceinline__ int operator[](int k) const {
    return k == 0 ? v0 : (k == 1 ? v1 : (k == 2 ? v2 : v3));
  }
};

__device__ __forceinline__ Quad load_counts(const int32_t* c) {
  return Quad{c[0], c[1], c[2], c[3]};
}

// Exclusive prefix of four counts: start of each list in the concatenation
// and the total.
struct Prefix4 {
  Quad start;
  int total;
  __device__ __forceinline__ explicit Prefix4(const Quad& n) {
    start = Quad{0, n.v0, n.v0 + n.v1, n.v0 + n.v1 + n.v2};
    total = start.v3 + n.v3;
  }
  // list holding concatenated index i
  __device__ __forceinline__ int list_of(int i) const {
    return (i >= start.v1) + (i >= start.v2) + (i >= start.v3);
  }
};

// Lanes per small node: G for a vertex, half of it (at least 4) for a net
// node, which has half as many arcs on average (nets of 3.7 pins against
// vertices in 7.4 nets on the Zipf workloads); 16 and 8 measured best.
template <int G>
__host__ __device__ constexpr int lanes_of(int k) {
  return k == 0 ? G : (G >= 8 ? G / 2 : G);
}

// Item layout of a frontier or BFS level: for each small list k, groups of
// lanes_of<G>(k) lanes take one node each; then one big node per wave item.
template <int G>
struct Items {
  Quad n;
  Quad start;  // first item of each list
  int end;
  __device__ __forceinline__ explicit Items(const int32_t* cnt) : Items(load_counts(cnt)) {}
  __device__ __forceinline__ explicit Items(const Quad& counts) : n(counts) {
    constexpr int NV = kWave / lanes_of<G>(0), NN = kWave / lanes_of<G>(1);
    const int i0 = (n.v0 + NV - 1) / NV, i1 = (n.v1 + NN - 1) / NN,
              i2 = (n.v2 + NN - 1) / NN;
    start = Quad{0, i0, i0 + i1, i0 + i1 + i2};
    end = start.v3 + n.v3;
  }
  __device__ __forceinline__ int total() const { return end; }
  __device__ __forceinline__ int list_of_item(int it) const {
    return (it >= start.v1) + (it >= start.v2) + (it >= start.v3);
  }
};

// Node i of a frontier given as kNL lists with prefix p.
__device__ __forceinline__ int frontier_node(const Dev& g, int par, const Prefix4& p, int i) {
  const int k = p.list_of(i);
  return g.list[par][k][i - p.start[k]];
}

// Round-scoped stamp: true for exactly one caller per (v, epoch).
__device__ __forceinline__ bool stamp_first(const Dev& g, int v, int epoch) {
  if (g.stamp[v] == epoch) return false;
  return atomicExch(&g.stamp[v], epoch) != epoch;
}

struct RoundArgs {
  int epoch;  // unique id of this round
  int cur3;   // epoch % 3
  int nxt3;   // (epoch + 1) % 3
  int cur;    // epoch % 2: list parity of this round, dx buffer written
  int nxt;    // (epoch + 1) % 2
};

__device__ __forceinline__ RoundArgs round_args(int epoch) {
  RoundArgs a;
  a.epoch = epoch;
  a.cur3 = epoch % 3;
  a.nxt3 = (epoch + 1) % 3;
  a.cur = epoch & 1;
  a.nxt = a.cur ^ 1;
  return a;
}

__device__ __forceinline__ BlockQ round_queue(const Dev& g, const RoundArgs& ra, lds_int* lds) {
  return bq_bind(lds, g.ctl->fcnt[ra.nxt3], g.list[ra.nxt]);
}

// push received by v: amount into dx[cur][v] and v into the next frontier.
// dx[cur] is zero for every node when a round starts (a node that received
// something in round r is in the frontier of round r + 1, which folds it), so
// the delivery that finds zero is the first and lists v.
__device__ __forceinline__ void deliver(const Dev& g, const RoundArgs& ra, const BlockQ& q, int v,
                                        uint32_t amount) {
  bool fresh = false;
  if (amount) fresh = atomicAdd(&g.dx[ra.cur][v], (int)amount) == 0;
  qpush(g, q, v, fresh);
}

// the same for e_in = v and e_out = v + 1 of one net
__device__ __forceinline__ void deliver_net(const Dev& g, const RoundArgs& ra, const BlockQ& q,
                                            int v, uint32_t a_in, uint32_t a_out) {
  int o_in = 1, o_out = 1;
  if (a_in) o_in = atomicAdd(&g.dx[ra.cur][v], (int)a_in);
  if (a_out) o_out = atomicAdd(&g.dx[ra.cur][v + 1], (int)a_out);
  qpush(g, q, v, o_in == 0);
  qpush(g, q, v + 1, o_out == 0);
}

// relabel candidate of frontier node u (-1: none)
__device__ __forceinline__ void leave(const Dev& g, const BlockQ&, int, int u, int cand) {
  if (cand >= 0) g.cand[u] = cand;
}

// Frontier lists of the single-workgroup loop, in LDS: kLoopCap entries per
// list (what does not fit goes to the same position of the global list; the
// loop then ends), with the relabel candidates of the current entries.
constexpr int kLoopCap = 1024;
struct LoopQ {
  lds_int* nbuf;  // next frontier: kNL lists of kLoopCap entries
  lds_int* ncnt;  // its counts
  lds_int* cand;  // candidates of the current entries, kNL x kLoopCap
};
constexpr int kLoopWords = 3 * kNL * kLoopCap + 3 * kNL + 6 + 4;
static_assert((kLoopWords - 4) % 2 == 0, "the 64-bit sums at the end of the area");

// Flow into the sinks, straight into the round's sum (at most INT32_MAX in all):
// few arcs reach a sink, and no register is held through the pushes.
struct LoopSink {
  lds_int* flow;
  __device__ __forceinline__ void operator+=(uint32_t n) const {
    if (n) (void)lds_add(flow, (int)n);
  }
};

__device__ __forceinline__ void loop_append(const Dev& g, const RoundArgs& ra, const LoopQ& q,
                                            int k, int v) {
  const int pos = lds_add(q.ncnt + k, 1);
  if (pos < kLoopCap) q.nbuf[k * kLoopCap + pos] = v;
  else g.list[ra.nxt][k][pos] = v;
}

// list of a node whose word of the big-node bitmap is w
__device__ __forceinline__ int list_of_word(const Dev& g, int v, uint32_t w) {
  if ((w >> (v & 31)) & 1u) return kBigList;
  return v < g.V ? 0 : 1 + ((v - g.NB) & 1);
}

__device__ __forceinline__ void deliver(const Dev& g, const RoundArgs& ra, const LoopQ& q, int v,
                                        uint32_t amount) {
  if (amount) {
    const int old = atomicAdd(&g.dx[ra.cur][v], (int)amount);
    const uint32_t w = g.bigbits[v >> 5];
    if (old == 0) loop_append(g, ra, q, list_of_word(g, v, w), v);
  }
}

__device__ __forceinline__ void deliver_net(const Dev& g, const RoundArgs& ra, const LoopQ& q,
                                            int v, uint32_t a_in, uint32_t a_out) {
  if (a_in | a_out) {
    int o_in = 1, o_out = 1;
    if (a_in) o_in = atomicAdd(&g.dx[ra.cur][v], (int)a_in);
    if (a_out) o_out = atomicAdd(&g.dx[ra.cur][v + 1], (int)a_out);
    const uint32_t w = g.bigbits[v >> 5];  // e_in and e_out share the word
    if (o_in == 0) loop_append(g, ra, q, list_of_word(g, v, w), v);
    if (o_out == 0) loop_append(g, ra, q, list_of_word(g, v + 1, w), v + 1);
  }
}

// slot -1: an entry past the LDS list
__device__ __forceinline__ void leave(const Dev& g, const LoopQ& q, int slot, int u, int cand) {
  if (slot >= 0) q.cand[slot] = cand;
  else g.cand[u] = cand;
}

// Excess at the start of the round: x plus what arrived last round.
__device__ __forceinline__ int take_excess(const Dev& g, const RoundArgs& ra, int u, int gl) {
  const int xv = g.x[u];
  const int dv = g.dx[ra.nxt][u];  // previous round's buffer (parity of epoch - 1)
  const int X = xv + dv;
  if (dv != 0 && gl == 0) {
    g.x[u] = X;
    g.dx[ra.nxt][u] = 0;
  }
  return X;
}

// End of a node's push scan (slot: its entry in the loop's lists).
template <int G, class Q>
__device__ __forceinline__ void finish_push(const Dev& g, const Q& q, int slot, int u, uint32_t X,
                                            uint32_t pushed, int cand, int gl, bool active,
                                            bool has) {
  if (active && gl == 0 && pushed > 0u) g.x[u] = (int)(X - pushed);
  const bool left = active && pushed < X;
  if (left) cand = g_min<G>(cand);
  if (has && gl == 0) leave(g, q, slot, u, left ? cand : -1);
}

// ---------------------------------------------------------------------------
// push phase, per node kind (G lanes per node, group-uniform control flow)
// nbytes accumulates algorithmic bytes: a node's own fields once per node
// (lane 0 of its group), each arc's fields by the lane that scans the arc.
// ---------------------------------------------------------------------------

template <int G, class Q>
__device__ void push_vertex(const Dev& g, const RoundArgs& ra, const Q& q, int slot, int u,
                            bool has, int gl, uint32_t& nbytes) {
  int k = 0, X = 0, beg = 0, end = 0;
  if (has) {
    k = g.d[u];
    X = take_excess(g, ra, u, gl);
    beg = g.vtx_off[u];
    end = g.vtx_off[u + 1];
    if (gl == 0) nbytes += 20;
  }
  const bool active = has && k < g.N && X > 0;
  const uint32_t UX = active ? (uint32_t)X : 0u;
  uint32_t carry = 0;
  int cand = kInf;
  if (active) {
    for (int base = beg; base < end; base += G) {
      const int i = base + gl;
      const bool valid = i < end;
      int e = 0, p = 0;
      int2 dl = make_int2(0, 0), fp = make_int2(0, 0);
      if (valid) {
        const int2 ep = g.vinc[i];
        e = ep.x;
        p = ep.y;
        dl = *reinterpret_cast<const int2*>(g.d + g.NB + 2 * e);
        fp = *reinterpret_cast<const int2*>(g.fpin + 2 * p);
        nbytes += 24;
      }
      const uint32_t r1 = (uint32_t)fp.x, r2 = (uint32_t)fp.y;
      const bool a1 = valid && r1 > 0u && dl.x == k - 1;
      const bool a2 = valid && r2 > 0u && dl.y == k - 1;
      const uint32_t want = min((a1 ? r1 : 0u) + (a2 ? r2 : 0u), UX);
      const uint32_t incl = g_scan_sat<G>(want, UX, gl);
      uint32_t excl = __shfl_up(incl, 1, G);
      if (gl == 0) excl = 0u;
      const uint32_t used = min(carry + excl, UX);
      const uint32_t give = min(want, UX - used);
      const uint32_t g1 = a1 ? min(give, r1) : 0u;
      const uint32_t g2 = give - g1;
      if (g1) g.fpin[2 * p] = (int)(r1 - g1);
      if (g2) g.fpin[2 * p + 1] = (int)(r2 - g2);
      deliver_net(g, ra, q, g.NB + 2 * e, g1, g2);
      if (valid) {
        if (r1 > g1) cand = min(cand, dl.x + 1);
        if (r2 > g2) cand = min(cand, dl.y + 1);
      }
      carry = min(carry + __shfl(incl, G - 1, G), UX);
      if (carry >= UX) break;
    }
  }
  finish_push<G>(g, q, slot, u, UX, carry, cand, gl, active, has);
}

template <int G, class Q, class S>
__device__ void push_ein(const Dev& g, const RoundArgs& ra, const Q& q, int slot, int node,
                         bool has, int gl, uint32_t& nbytes, S& to_sink) {
  const int e = (node - g.NB) >> 1;
  int k = 0, X = 0;
  if (has) {
    k = g.d[node];
    X = take_excess(g, ra, node, gl);
    if (gl == 0) nbytes += 12;
  }
  const bool active = has && k < g.N && X > 0;
  const uint32_t UX = active ? (uint32_t)X : 0u;
  uint32_t carry = 0;
  int cand = kInf;
  if (active) {
    const int we = g.w[e];
    const int fbv = g.fb[e];
    const int dout = g.d[node + 1];
    if (gl == 0) nbytes += 20;
    const uint32_t rb = (uint32_t)(we - fbv);
    const bool ab = rb > 0u && dout == k - 1;
    const uint32_t gb = ab ? min(rb, UX) : 0u;
    if (gb && gl == 0) g.fb[e] = fbv + (int)gb;
    deliver(g, ra, q, node + 1, gl == 0 ? gb : 0u);
    carry = gb;
    if (rb > gb) cand = dout + 1;
    if (carry < UX) {
      const int beg = g.net_off[e], end = g.net_off[e + 1];
      for (int base = beg; base < end; base += G) {
        const int i = base + gl;
        const bool valid = i < end;
        int u = 0, rin = 0, du = 0;
        if (valid) {
          u = g.pin_v[i];
          rin = g.fpin[2 * i];
          du = g.d[u];
          nbytes += 12;
        }
        const uint32_t r = valid ? (uint32_t)(we - rin) : 0u;  // flow(u, e_in)
        const bool a = r > 0u && du == k - 1;
        const uint32_t want = a ? min(r, UX) : 0u;
        const uint32_t incl = g_scan_sat<G>(want, UX, gl);
        uint32_t excl = __shfl_up(incl, 1, G);
        if (gl == 0) excl = 0u;
        const uint32_t used = min(carry + excl, UX);
        const uint32_t give = min(want, UX - used);
        if (give) g.fpin[2 * i] = rin + (int)give;
        // a pin labelled 0 is a sink: a vertex pierced into the sink side
        // can still carry flow into e_in, and returning it reaches the sink
        if (du == 0) to_sink += give;
        deliver(g, ra, q, u, du != 0 ? give : 0u);
        if (valid && r > give) cand = min(cand, du + 1);
        carry = min(carry + __shfl(incl, G - 1, G), UX);
        if (carry >= UX) break;
      }
    }
  }
  finish_push<G>(g, q, slot, node, UX, carry, cand, gl, active, has);
}

template <int G, class Q, class S>
__device__ void push_eout(const Dev& g, const RoundArgs& ra, const Q& q, int slot, int node,
                          bool has, int gl, uint32_t& nbytes, S& to_sink) {
  const int e = (node - g.NB) >> 1;
  int k = 0, X = 0;
  if (has) {
    k = g.d[node];
    X = take_excess(g, ra, node, gl);
    if (gl == 0) nbytes += 12;
  }
  const bool active = has && k < g.N && X > 0;
  const uint32_t UX = active ? (uint32_t)X : 0u;
  uint32_t carry = 0;
  int cand = kInf;
  if (active) {
    const int beg = g.net_off[e], end = g.net_off[e + 1];
    if (gl == 0) nbytes += 8;
    // pins first: the arcs e_out -> u are infinite, so the first admissible
    // pin takes all remaining excess
    for (int base = beg; base < end; base += G) {
      const int i = base + gl;
      const bool valid = i < end;
      int u = 0, du = 0;
      if (valid) {
        u = g.pin_v[i];
        du = g.d[u];
        nbytes += 8;
      }
      const bool a = valid && du == k - 1;
      const uint32_t want = a ? UX : 0u;
      const uint32_t incl = g_scan_sat<G>(want, UX, gl);
      uint32_t excl = __shfl_up(incl, 1, G);
      if (gl == 0) excl = 0u;
      const uint32_t used = min(carry + excl, UX);
      const uint32_t give = min(want, UX - used);
      if (give) {
        g.fpin[2 * i + 1] += (int)give;
        nbytes += 8;
        if (du == 0) to_sink += give;  // only sinks carry label 0
      }
      deliver(g, ra, q, u, du != 0 ? give : 0u);
      if (valid) cand = min(cand, du + 1);
      carry = min(carry + __shfl(incl, G - 1, G), UX);
      if (carry >= UX) break;
    }
    if (carry < UX) {  // reverse bridge e_out -> e_in
      const int rb = g.fb[e];
      const int din = g.d[node - 1];
      if (gl == 0) nbytes += 8;
      const bool ab = rb > 0 && din == k - 1;
      const uint32_t gb = ab ? min((uint32_t)rb, UX - carry) : 0u;
      if (gb && gl == 0) g.fb[e] = rb - (int)gb;
      deliver(g, ra, q, node - 1, gl == 0 ? gb : 0u);
      carry += gb;
      if ((uint32_t)rb > gb) cand = min(cand, din + 1);
    }
  }
  finish_push<G>(g, q, slot, node, UX, carry, cand, gl, active, has);
}

template <int G, class Q, class S>
__device__ __forceinline__ void push_node(const Dev& g, const RoundArgs& ra, const Q& q, int slot,
                                          int v, bool has, int gl, uint32_t& nbytes,
                                          S& to_sink) {
  // kind is wave-divergent only across groups; each branch is group-uniform
  if (!has || v < g.V) push_vertex<G>(g, ra, q, slot, v, has, gl, nbytes);
  else if (((v - g.NB) & 1) == 0) push_ein<G>(g, ra, q, slot, v, has, gl, nbytes, to_sink);
  else push_eout<G>(g, ra, q, slot, v, has, gl, nbytes, to_sink);
}

// Work items of a frontier: small nodes in groups of G lanes (64/G nodes per
// wave item), then big nodes one per wave item.  A workgroup takes tiles of
// one item per wave (block-uniform loop, so the staging area can be flushed
// between tiles).
template <int G>
__device__ void phase_push(const Dev& g, int epoch, int tile0, int tstride, int kc, lds_int* lds) {
  const RoundArgs ra = round_args(epoch);
  if (tile0 == 0 && threadIdx.x < kNL) {
    // ring slot that nobody reads this round: the next round's append target
    g.ctl->fcnt[(epoch + 2) % 3][threadIdx.x] = 0;
  }
  const BlockQ q = round_queue(g, ra, lds);
  const Items<G> its(g.ctl->fcnt[ra.cur3]);
  constexpr int GN = lanes_of<G>(1);
  const int total = its.total();
  const int wpb = blockDim.x >> 6, wid = threadIdx.x >> 6;
  const int ntiles = (total + wpb - 1) / wpb;
  const int lane = lane_id();
  uint32_t nbytes = 0;
  uint32_t nitems = 0;
  unsigned long long to_sink = 0;
  for (int tile = tile0; tile < ntiles; tile += tstride) {
    const int it = tile * wpb + wid;
    if (it < total) {
      const int k = its.list_of_item(it);
      if (k < kBigList) {
        const int gk = k == 0 ? G : GN;
        const int idx = (it - its.start[k]) * (kWave / gk) + lane / gk;
        const bool has = idx < its.n[k];
        const int v = has ? g.list[ra.cur][k][idx] : 0;
        nitems += has && (lane % gk) == 0;
        if (k == 0) push_vertex<G>(g, ra, q, 0, v, has, lane % G, nbytes);
        else if (k == 1) push_ein<GN>(g, ra, q, 0, v, has, lane % GN, nbytes, to_sink);
        else push_eout<GN>(g, ra, q, 0, v, has, lane % GN, nbytes, to_sink);
      } else {
        const int v = g.list[ra.cur][kBigList][it - its.start[kBigList]];
        nitems += lane == 0;
        push_node<kWave>(g, ra, q, 0, v, true, lane, nbytes, to_sink);
      }
    }
    bq_tile_end(q, q.cap / 2);
  }
  bq_flush(q);
  block_add_u64(&g.ctl->flow, to_sink, &g.ctl->bytes[kc],
                (unsigned long long)nbytes + 4ull * nitems, &g.ctl->items[kc], nitems);
}

// Apply phase over the same frontier: relabel nodes left with excess; thread
// per node, small list then big list, tiles of one node per thread.
__device__ void phase_apply(const Dev& g, int epoch, int tile0, int tstride, int kc, lds_int* lds) {
  const RoundArgs ra = round_args(epoch);
  const BlockQ q = round_queue(g, ra, lds);
  const Prefix4 pre(load_counts(g.ctl->fcnt[ra.cur3]));
  const int n = pre.total;
  const int ntiles = (n + blockDim.x - 1) / blockDim.x;
  unsigned long long nrel = 0;
  uint32_t nbytes = 0;
  for (int tile = tile0; tile < ntiles; tile += tstride) {
    const int i = tile * blockDim.x + threadIdx.x;
    bool app = false;
    int v = 0;
    if (i < n) {
      v = frontier_node(g, ra.cur, pre, i);
      const int c = g.cand[v];
      nbytes += 8;
      const bool rec = c >= 0 && g.dx[ra.cur][v] != 0;  // something was pushed into v
      if (c >= 0 && rec && g.relabel_block) {
        // blocking variant (section "A Bug in the Synchronous Algorithm",
        // the first fix): a node pushed to in this round keeps its label;
        // the push listed it for the next round, where it tries again
        g.cand[v] = -1;
      } else if (c >= 0) {
        g.cand[v] = -1;
        const int k = g.d[v];
        int nd = c;
        if (rec) nd = min(nd, k + 2);
        nd = min(nd, g.N);
        if (nd <= k) atomicOr(&g.ctl->err, ERR_LABEL);
        g.d[v] = nd;
        nrel += 1;
        nbytes += 12;
        app = !rec && nd < g.N;
      }
    }
    qpush(g, q, v, app);
    bq_tile_end(q, (int)blockDim.x);
  }
  bq_flush(q);
  block_add_u64(&g.ctl->relabels, nrel, &g.ctl->bytes[kc], nbytes, &g.ctl->items[kc], nrel);
}

// a value that is the same in every lane, kept in a scalar register
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// What is left of `limit` at `now`, as the loop's 32-bit limit: the relabels of
// one more round, at most N, on top of it still fit 32 bits.
__device__ __forceinline__ uint32_t relabels_left(unsigned long long limit,
                                                  unsigned long long now) {
  const unsigned long long left = limit > now ? limit - now : 0ull;
  return left > 0x7fffffffull ? 0x7fffffffu : (uint32_t)left;
}

struct LoopEnd {
  int why, rounds, stale;  // stale: rounds since the flow value changed
  bool flowed;             // the flow value changed
};

constexpr int kStaleFrontier = 1500;  // "only few active nodes" (paragraph "Avoid Pushing Flow Back")

// Rounds inside one workgroup from round `epoch`'s frontier, which holds at
// most `cap` nodes (at most kLoopCap, unless kAny: entries past the LDS lists
// are then read from the global ones).  Ends when the frontier is empty (why 1),
// exceeds `cap` (2), `max_rounds` rounds ran (3), at least `relabel_limit`
// relabels ran (4), or the flow value did not change for `stale_limit` rounds (5); the
// frontier of round epoch + rounds is then in the global lists.  All waves of
// the workgroup share one CU, so a workgroup barrier orders their global
// memory traffic; no device-scope fence (which would write back and
// invalidate the L2) is needed.
//
// Such a round is a chain of dependent L2 accesses between barriers, so both
// are kept few: the lists, their counts, the relabel candidates and the
// round's flow and relabel counts live in LDS (a ring of three, so that the
// two barriers of a round, after the pushes and after the relabels, also
// order the counters), the delivery's own atomic tells whether it is the
// first, and the statistics stay in LDS and registers until the loop ends: 6.7
// us a round instead of 16 on a 2,000-vertex flow (1,024 threads; values that
// are the same in every lane are kept in scalar registers).  Every exit test
// reads counters that no wave writes before the next barrier, so all waves take
// the same decision.
template <int G, bool kAny>
__device__ LoopEnd wg_rounds(const Dev& g, int epoch, int max_rounds, int cap,
                             uint32_t relabel_limit, int stale_limit, int kc, lds_int* lds) {
  lds_int* const buf = lds;                         // [2][kNL][kLoopCap]
  lds_int* const cand = lds + 2 * kNL * kLoopCap;   // [kNL][kLoopCap]
  lds_int* const cnt = lds + 3 * kNL * kLoopCap;    // [3][kNL]
  lds_int* const acc = cnt + 3 * kNL;               // [3]{flow, relabels}
  lds_u64* const sum = (lds_u64*)(acc + 6);         // of all rounds: flow, items
  const int tid = threadIdx.x, lane = lane_id(), wid = uni(tid >> 6), nw = blockDim.x >> 6;
  LoopEnd end{0, 0, 0, false};
  {
    const RoundArgs ra = round_args(epoch);
    const Quad n{uni(ld_vol(&g.ctl->fcnt[ra.cur3][0])), uni(ld_vol(&g.ctl->fcnt[ra.cur3][1])),
                 uni(ld_vol(&g.ctl->fcnt[ra.cur3][2])), uni(ld_vol(&g.ctl->fcnt[ra.cur3][3]))};
    const int nf = n.v0 + n.v1 + n.v2 + n.v3;
    if (nf == 0 || nf > cap) {
      end.why = nf == 0 ? 1 : 2;
      return end;
    }
    __syncthreads();  // earlier users of the area are done with it
    if (tid < 3 * kNL) cnt[tid] = tid / kNL == ra.cur3 ? n[tid % kNL] : 0;
    if (tid >= 64 && tid < 70) acc[tid - 64] = 0;
    if (tid < 2) sum[tid] = 0ull;
#pragma unroll
    for (int k = 0; k < kNL; ++k)
      for (int i = tid; i < min(n[k], kLoopCap); i += blockDim.x)
        buf[(ra.cur * kNL + k) * kLoopCap + i] = g.list[ra.cur][k][i];
    __syncthreads();
  }
  uint32_t relabels = 0;  // of the workgroup
  uint32_t nbytes = 0;    // of the lane
  for (;;) {
    const RoundArgs ra = round_args(epoch);
    const Quad n{uni(cnt[ra.cur3 * kNL]), uni(cnt[ra.cur3 * kNL + 1]),
                 uni(cnt[ra.cur3 * kNL + 2]), uni(cnt[ra.cur3 * kNL + 3])};
    const Items<G> its(n);
    const Prefix4 pre(n);
    if (pre.total == 0) { end.why = 1; break; }
    if (pre.total > cap) { end.why = 2; break; }
    if (end.rounds >= max_rounds) { end.why = 3; break; }
    if (relabels >= relabel_limit) { end.why = 4; break; }
    if (stale_limit > 0 && end.stale >= stale_limit) { end.why = 5; break; }
    const lds_int* const cbuf = buf + ra.cur * kNL * kLoopCap;
    const LoopQ q{buf + ra.nxt * kNL * kLoopCap, cnt + ra.nxt3 * kNL, cand};
    constexpr int GN = lanes_of<G>(1);
    LoopSink to_sink{acc + 2 * ra.cur3};
    for (int it = wid; it < its.total(); it += nw) {
      const int k = its.list_of_item(it);
      // With 16 lanes a vertex the batch's workgroups, which hold a whole solve
      // in 128 registers, would spill two: the lane arithmetic of the kinds (and
      // the scan masks derived from it) is recomputed per item instead of being
      // carried through all rounds.
      int ln = lane;
      if (kAny && G == 16) asm volatile("" : "+v"(ln));
      if (k < kBigList) {
        const int gk = k == 0 ? G : GN;
        const int idx = (it - its.start[k]) * (kWave / gk) + ln / gk;
        const bool has = idx < n[k];
        const bool far = kAny && idx >= kLoopCap;
        const int slot = far ? -1 : k * kLoopCap + idx;
        const int v = !has ? 0 : (far ? g.list[ra.cur][k][idx] : (int)cbuf[slot]);
        if (k == 0) push_vertex<G>(g, ra, q, slot, v, has, ln % G, nbytes);
        else if (k == 1) push_ein<GN>(g, ra, q, slot, v, has, ln % GN, nbytes, to_sink);
        else push_eout<GN>(g, ra, q, slot, v, has, ln % GN, nbytes, to_sink);
      } else {
        const int idx = it - its.start[kBigList];
        const bool far = kAny && idx >= kLoopCap;
        const int slot = far ? -1 : kBigList * kLoopCap + idx;
        const int v = far ? g.list[ra.cur][kBigList][idx] : (int)cbuf[slot];
        push_node<kWave>(g, ra, q, slot, v, true, ln, nbytes, to_sink);
      }
    }
    __syncthreads();
    // the ring slot of the round after next: last read before this barrier
    const int z3 = (epoch + 2) % 3;
    if (tid < kNL) cnt[z3 * kNL + tid] = 0;
    if (tid >= 64 && tid < 66) acc[2 * z3 + tid - 64] = 0;
    for (int i0 = wid * kWave; i0 < pre.total; i0 += nw * kWave) {
      const int i = i0 + lane;
      bool rel = false;
      if (i < pre.total) {
        const int k = pre.list_of(i);
        const int idx = i - pre.start[k];
        int c, v;
        if (kAny && idx >= kLoopCap) {
          v = g.list[ra.cur][k][idx];
          c = g.cand[v];
          if (c >= 0) g.cand[v] = -1;
        } else {
          c = cand[k * kLoopCap + idx];
          v = cbuf[k * kLoopCap + idx];
        }
        if (c >= 0) {
          const int dk = g.d[v];
          const bool rec = g.dx[ra.cur][v] != 0;
          if (!(rec && g.relabel_block)) {
            int nd = c;
            if (rec) nd = min(nd, dk + 2);
            nd = min(nd, g.N);
            if (nd <= dk) atomicOr(&g.ctl->err, ERR_LABEL);
            g.d[v] = nd;
            rel = true;
            nbytes += 12;
            if (!rec && nd < g.N) loop_append(g, ra, q, k, v);
          }
        }
        nbytes += 8;
      }
      const unsigned long long m = __ballot(rel);
      if (lane == 0 && m) lds_add(acc + 2 * ra.cur3 + 1, __popcll(m));
    }
    __syncthreads();
    const int fl = uni(acc[2 * ra.cur3]);
    if (tid < 2)
      __hip_atomic_fetch_add(sum + tid, (unsigned long long)(tid == 0 ? fl : pre.total),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (nbytes >> 31) {  // a round adds less than this
      atomicAdd(&g.ctl->bytes[kc], (unsigned long long)nbytes);
      nbytes = 0;
    }
    relabels += (uint32_t)uni(acc[2 * ra.cur3 + 1]);
    ++epoch;
    ++end.rounds;
    if (fl != 0) {
      end.flowed = true;
      end.stale = 0;
    } else {
      end.stale = pre.total < kStaleFrontier ? end.stale + 1 : 0;
    }
  }
  // the frontier back to the global lists (what exceeded the area is there)
  const RoundArgs ra = round_args(epoch);
#pragma unroll
  for (int k = 0; k < kNL; ++k) {
    const int c = min((int)cnt[ra.cur3 * kNL + k], kLoopCap);
    for (int i = tid; i < c; i += blockDim.x)
      g.list[ra.cur][k][i] = buf[(ra.cur * kNL + k) * kLoopCap + i];
  }
  if (tid < 3 * kNL)
    g.ctl->fcnt[tid / kNL][tid % kNL] = tid / kNL == ra.cur3 ? (int)cnt[tid] : 0;
  if (tid < 2) {  // each the sum that it kept
    const unsigned long long c = sum[tid];
    if (c) atomicAdd(tid == 0 ? &g.ctl->flow : &g.ctl->items[kc], c);
    if (tid == 0 && relabels) atomicAdd(&g.ctl->relabels, (unsigned long long)relabels);
  }
  block_add_u64(&g.ctl->bytes[kc], nbytes + (tid == 1 ? 4ull * sum[1] : 0ull));
  return end;
}

// ---------------------------------------------------------------------------
// reverse residual BFS from the sinks (global relabel) over the capped network
// ---------------------------------------------------------------------------

// Residual bits of a net (netres, below) with bridge flow fb; x, dx0, dx1 hold the excess and
// the pushes not folded yet of {e_in, e_out}, none of them negative.  What
// flows into e_in (a source's share included) is fb plus the excess of e_in:
// a preflow may send the same units over the bridge and back by a pin, so the
// sum can pass INT32_MAX and its terms are looked at one by one; what leaves
// e_out lies in [0, fb].
__host__ __device__ __forceinline__ uint32_t net_residual_bits(int fb, int w, int2 x, int2 dx0,
                                                               int2 dx1) {
  const int out = fb - (x.y + dx0.y + dx1.y);
  const bool in = (fb | x.x | dx0.x | dx1.x) != 0;
  return (fb < w ? 1u : 0u) | (out > 0 ? 2u : 0u) | (fb > 0 ? 4u : 0u) | (in ? 8u : 0u);
}

// Global relabel, step 2: residual bits that the reverse BFS tests, so that
// its checks of an arc hit two small bitmaps instead of scattered flows.
// The flow state does not change during a global relabel.
//   pinres: one bit per pin slot p of net e: flow(u, e_in) = w(e) - r_in > 0
//           (the reverse arc e_in -> u is residual)
//   netres: four bits per net: bit0 fb < w (e_in -> e_out residual), bit1
//           some pin carries flow out of e_out (fb exceeds e_out's excess),
//           bit2 fb > 0 (e_out -> e_in residual), bit3 something flows into
//           e_in, so a pin's flow may
//   pinfree (swept levels): one bit per pin slot, r_in > 0
// Thread per slot, then per net; t0 wave-aligned, tstride a multiple of 64.
__device__ void phase_gr_bits(const Dev& g, int t0, int tstride) {
  const int lane = lane_id();
  // pin slots: a lane per slot, a wave per 64 slots (two words of the bitmaps)
  const int np = (g.P + 63) & ~63;
  const int pwords = (g.P + 31) >> 5;
  for (int p = t0; p < np; p += tstride) {
    const int r = p < g.P ? g.fpin[2 * p] : 0;
    const bool f = p < g.P && r < g.w[g.pin_net[p]];
    const unsigned long long m = __ballot(f), mr = __ballot(r > 0);
    const int word = ((p - lane) >> 5) + lane;
    if (lane < 2 && word < pwords) {
      g.pinres[word] = (uint32_t)(m >> (32 * lane));
      if (g.pinfree) g.pinfree[word] = (uint32_t)(mr >> (32 * lane));
    }
  }
  // nets: a lane per net, eight nibbles per word
  const int ne = (g.E + 63) & ~63;
  for (int e = t0; e < ne; e += tstride) {
    uint32_t b = 0;
    if (e < g.E) {
      const int fbv = g.fb[e], ei = g.NB + 2 * e;
      const int2 x = *reinterpret_cast<const int2*>(g.x + ei);
      const int2 a = *reinterpret_cast<const int2*>(g.dx[0] + ei);
      const int2 c = *reinterpret_cast<const int2*>(g.dx[1] + ei);
      b = net_residual_bits(fbv, g.w[e], x, a, c);
    }
    uint32_t v = b << (4 * (lane & 7));
    v |= __shfl_xor(v, 1);
    v |= __shfl_xor(v, 2);
    v |= __shfl_xor(v, 4);
    if ((lane & 7) == 0 && e < g.E) g.netres[e >> 3] = v;
  }
}

__device__ __forceinline__ bool pin_flow_in(const Dev& g, int p) {
  return (g.pinres[p >> 5] >> (p & 31)) & 1u;
}
__device__ __forceinline__ uint32_t net_bits(const Dev& g, int e) {
  return (g.netres[e >> 3] >> (4 * (e & 7))) & 15u;
}

// The "labelled" hint of the reverse BFS is a bitmap small enough to stay in
// the L2, so checking an arc whose tail is already labelled costs no access
// to the large label array.  Bits are set with a plain read-modify-write; a
// bit lost to a concurrent update only sends a later check to the label
// itself, which stays the source of truth.
__device__ __forceinline__ bool seen_bit(const Dev& g, int v) {
  return (g.seen[v >> 5] >> (v & 31)) & 1u;
}
__device__ __forceinline__ void set_seen(const Dev& g, int v) {
  g.seen[v >> 5] |= 1u << (v & 31);
}

// Label v with lvl if it is unlabelled.  With kClaim the first writer wins
// by compare-and-swap on the label and reports it; otherwise a plain store
// (all writers of a level store the same value).  With the byte marks `lev`
// an expanded level only marks v (byte 1, a 5 MB array for 5 M nodes
// instead of the 20 MB label array) and the collect sweep writes the label
// and lists v; a claimed node gets byte 2 at once.
// kChecked: the caller has just read v's hint bit and found it clear.
template <bool kClaim, bool kChecked = false>
__device__ __forceinline__ bool label_rev(const Dev& g, int v, int lvl) {
  if (!kChecked && seen_bit(g, v)) return false;
  if (!kClaim) {
    if (g.lev) {
      if (g.lev[v] != 0) return false;
      g.lev[v] = 1;
    } else {
      if (g.d[v] != g.N) return false;
      g.d[v] = lvl;
    }
    set_seen(g, v);
    return false;
  }
  if (atomicCAS(&g.d[v], g.N, lvl) != g.N) return false;
  if (g.lev) g.lev[v] = 2;
  set_seen(g, v);
  return true;
}

// Slices of the node range for the XCD-local expansion of reverse-BFS
// levels: 1024-node chunks dealt round-robin to the eight XCDs (workgroup b
// of a grid runs on XCD b mod 8), so each XCD's share of the label array
// (a quarter of its 4 MB L2 for 5 M nodes) and of the labelled bitmap stays
// in its own L2.
constexpr int kSlices = 8;
constexpr int kMaxSliceGroups = 512;
__device__ __forceinline__ int xslice(int v) { return (v >> 10) & (kSlices - 1); }

// An arc head of an expanded level: labelled at once (visit_rev = label_rev)
// or, with kSlice, only pre-checked against the labelled bitmap and handed
// to its slice (xpush); the slice kernel then labels it on the XCD that
// owns it.
template <bool kChecked, bool kSlice>
__device__ __forceinline__ bool visit_rev(const Dev& g, int v, int lvl) {
  if (kSlice) return kChecked ? true : !seen_bit(g, v);
  return label_rev<false, kChecked>(g, v, lvl);
}

// Append arc head t (where pred) to this workgroup's segment of its slice:
// wave-aggregated LDS counters xc[8]; an entry past the segment's end is
// labelled here instead.  Called by the active lanes of a wave.
__device__ __forceinline__ void xpush(const Dev& g, lds_int* xc, int t, bool pred, int lvl) {
  if (__ballot(pred) == 0ull) return;
  const int me = xslice(t);
  int32_t* seg = g.xbuf + (long long)blockIdx.x * kSlices * g.xseg;
#pragma unroll 1
  for (int sl = 0; sl < kSlices; ++sl) {
    const bool mine = pred && me == sl;
    const unsigned long long m = __ballot(mine);
    if (m == 0ull) continue;
    const int leader = __builtin_ctzll(m);
    int pos = 0;
    if (lane_id() == leader) pos = lds_add(xc + sl, __popcll(m));
    pos = __shfl(pos, leader);
    if (mine) {
      const int idx = pos + __popcll(m & lanemask_lt());
      if (idx < g.xseg) seg[sl * g.xseg + idx] = t;
      else label_rev<false, true>(g, t, lvl);
    }
  }
}

// Node of an expanded level: a group of `stride` lanes scans node x (G lanes
// per small node, a wave per big node, the workgroup per huge node); gl is
// the lane's index in the group.
template <bool kSlice = false>
__device__ __forceinline__ void bfs_rev_node(const Dev& g, int x, bool has, int gl, int stride,
                                             int lvl, uint32_t& nbytes, lds_int* xc = nullptr) {
  const bool isv = has && x < g.V;
  const bool isnet = has && x >= g.NB;
  if (!has || isv) {
    int beg = 0, end = 0;
    if (isv) {
      beg = g.vtx_off[x];
      end = g.vtx_off[x + 1];
    }
    for (int base = beg; base < end; base += stride) {
      const int i = base + gl;
      const bool valid = i < end;
      bool vin = false, vout = false;
      int t1 = 0;
      if (valid) {
        const int2 ep = g.vinc[i];
        t1 = g.NB + 2 * ep.x;
        // bits of e_in and e_out share a word (NB and 2e are even)
        const uint32_t sw = g.seen[t1 >> 5] >> (t1 & 31);
        nbytes += 12;
        if (!(sw & 2u)) vout = visit_rev<true, kSlice>(g, t1 + 1, lvl);  // e_out -> x infinite
        if (!(sw & 1u) && pin_flow_in(g, ep.y))                    // e_in -> x reverse
          vin = visit_rev<true, kSlice>(g, t1, lvl);
      }
      if (kSlice) {
        xpush(g, xc, t1, vin, lvl);
        xpush(g, xc, t1 + 1, vout, lvl);
      }
    }
  } else if (isnet) {
    const int e = (x - g.NB) >> 1;
    const bool in = ((x - g.NB) & 1) == 0;
    const uint32_t nb = net_bits(g, e);
    int beg = g.net_off[e], end = g.net_off[e + 1];
    // in-arcs of e_out from pins carry flow(e_out, u) > 0; their sum is the
    // outflow fb - excess(e_out), so a net without outflow skips its pins
    if (!in && !(nb & 2u)) end = beg;
    if (gl == 0) nbytes += 16;
    bool vb = false;
    if (gl == 0) {
      if (in) vb = (nb & 4u) && visit_rev<false, kSlice>(g, x + 1, lvl);  // e_out -> e_in residual fb
      else vb = (nb & 1u) && visit_rev<false, kSlice>(g, x - 1, lvl);     // e_in -> e_out residual w - fb
    }
    if (kSlice) xpush(g, xc, in ? x + 1 : x - 1, vb, lvl);
    for (int base = beg; base < end; base += stride) {
      const int i = base + gl;
      const bool valid = i < end;
      bool vu = false;
      int u = 0;
      if (valid) {
        u = g.pin_v[i];
        const int f = g.fpin[2 * i + (in ? 0 : 1)];  // r_in (u->e_in) or f_out (u->e_out)
        nbytes += 12;
        if (f > 0) vu = visit_rev<false, kSlice>(g, u, lvl);
      }
      if (kSlice) xpush(g, xc, u, vu, lvl);
    }
  }
}

// Visit v in the forward BFS stamped ep.  With kClaim the first visitor wins
// (exchange on the stamp) and lists v; otherwise an unvisited v gets the
// level's provisional stamp ep_tmp by a plain store (every writer stores the
// same value) and the collect sweep lists it and stamps it ep.
template <bool kClaim>
__device__ __forceinline__ bool fwd_visit(const Dev& g, int v, int ep, int ep_tmp) {
  if (kClaim) return stamp_first(g, v, ep);
  const int sv = g.stamp[v];
  if (sv != ep && sv != ep_tmp) g.stamp[v] = ep_tmp;
  return false;
}

// Node-grouped forward BFS of the uncapped residual network (source side): a
// group of `stride` lanes scans node x's residual out-arcs.
//   vertex u:  u -> e_in always (uncapped), u -> e_out when flow(e_out, u) > 0
//   e_in:      e_in -> e_out when fb < w, e_in -> u when flow(u, e_in) > 0
//   e_out:     e_out -> e_in when fb > 0, e_out -> u always (a sink reached
//              is an internal error: the flow would not be maximum)
__device__ __forceinline__ void bfs_fwd_node(const Dev& g, int x, bool has, int gl, int stride,
                                             int ep, int ep_tmp, uint32_t& nbytes) {
  if (has && x < g.V) {
    const int end = g.vtx_off[x + 1];
    for (int i = g.vtx_off[x] + gl; i < end; i += stride) {
      const int2 ep2 = g.vinc[i];
      const int t1 = g.NB + 2 * ep2.x;
      nbytes += 12;
      fwd_visit<false>(g, t1, ep, ep_tmp);
      if (g.fpin[2 * ep2.y + 1] > 0) fwd_visit<false>(g, t1 + 1, ep, ep_tmp);
    }
  } else if (has && x >= g.NB) {
    const int e = (x - g.NB) >> 1;
    const bool in = ((x - g.NB) & 1) == 0;
    const int end = g.net_off[e + 1];
    const int we = g.w[e];
    if (gl == 0) {
      const int fbv = g.fb[e];
      nbytes += 16;
      if (in ? fbv < we : fbv > 0) fwd_visit<false>(g, in ? x + 1 : x - 1, ep, ep_tmp);
    }
    for (int i = g.net_off[e] + gl; i < end; i += stride) {
      const int u = g.pin_v[i];
      nbytes += 8;
      if (in) {
        if (we - g.fpin[2 * i] > 0) fwd_visit<false>(g, u, ep, ep_tmp);
      } else {
        const int r = g.role[u];
        if (r == 2) atomicOr(&g.ctl->err, ERR_SINK_REACHED);
        else if (r == 0) fwd_visit<false>(g, u, ep, ep_tmp);
      }
    }
  }
}

constexpr int kDirRelabel = 0;  // reverse BFS of a global relabel (capped network)
constexpr int kDirSource = 1;   // forward BFS of the source side (uncapped)
constexpr int kDirSink = 2;     // reverse BFS of the sink side (uncapped)

// One node of a level whose arcs claim: the reverse BFS of a global relabel
// (labels val), the forward BFS of the source side or the reverse BFS of the
// sink side (stamps val).  A claiming level is bound by the latency of one
// node's chain of cold accesses, so what does not depend on each other is in
// flight together: a net's bridge with its first pins, the claims of a net's
// two nodes, and each claim with the word that tells the list of the node.
// That leaves five accesses in a row (range, arc, label or stamp, claim, place
// in the list) where the bridge before the pins, one claim after the other and
// the list word after the claim made it ten or eleven.  A level of a 740k-pin
// flow 15.3 -> 14.0 us on average, of a 13k-pin one 9.0 -> 8.1.
template <int kDir>
__device__ __forceinline__ void bfs_claim_node(const Dev& g, const BlockQ& q, int x, bool has,
                                               int gl, int stride, int val, uint32_t& nbytes) {
  auto claim = [&](bool want, int t, uint32_t& word) {  // the value before, val if not wanted
    int old = val;
    if (want) {
      word = g.bigbits[t >> 5];
      if (kDir == kDirRelabel) old = atomicCAS(&g.d[t], g.N, val);
      else old = atomicExch(&g.stamp[t], val);
    }
    return old;
  };
  auto first = [&](int old) { return kDir == kDirRelabel ? old == g.N : old != val; };
  auto mark = [&](int t, uint32_t bits) {  // labelled: the hint of node t (and t + 1)
    if (kDir == kDirRelabel && bits) {
      g.seen[t >> 5] |= bits << (t & 31);
      if (g.lev && (bits & 1u)) g.lev[t] = 2;
      if (g.lev && (bits & 2u)) g.lev[t + 1] = 2;
    }
  };
  auto push = [&](int t, bool won, uint32_t word) {
    bq_push(q, (word >> (t & 31)) & 1u ? kBigList : t < g.V ? 0 : 1 + (t & 1), t, won);
  };
  if (has && x < g.V) {
    const int beg = g.vtx_off[x], end = g.vtx_off[x + 1];
    for (int base = beg; base < end; base += stride) {
      const int i = base + gl;
      bool want_in = false, want_out = false;
      int t = 0;  // e_in; e_out = t + 1, their bits share a word
      if (i < end) {
        const int2 a = g.vinc[i];
        t = g.NB + 2 * a.x;
        nbytes += 12;
        if (kDir == kDirRelabel) {  // e_out -> x infinite, e_in -> x reverse
          const uint32_t sw = g.seen[t >> 5] >> (t & 31);
          const bool flow = pin_flow_in(g, a.y);
          want_out = !(sw & 2u);
          want_in = !(sw & 1u) && flow;
        } else {
          const int2 st = *reinterpret_cast<const int2*>(g.stamp + t);
          const int2 fp = *reinterpret_cast<const int2*>(g.fpin + 2 * a.y);
          want_in = st.x != val;
          want_out = st.y != val;
          if (kDir == kDirSource) want_out = want_out && fp.y > 0;  // x -> e_in uncapped
          else want_in = want_in && g.w[a.x] - fp.x > 0;            // e_out -> x infinite
        }
      }
      uint32_t word = 0;
      const int old_out = claim(want_out, t + 1, word);
      const int old_in = claim(want_in, t, word);
      const bool won_out = first(old_out), won_in = first(old_in);
      mark(t, (won_in ? 1u : 0u) | (won_out ? 2u : 0u));
      push(t, won_in, word);
      push(t + 1, won_out, word);
    }
  } else if (has && x >= g.NB) {
    const int e = (x - g.NB) >> 1;
    const bool in = ((x - g.NB) & 1) == 0;
    const int b = in ? x + 1 : x - 1;  // over the bridge
    const int beg = g.net_off[e];
    int end = g.net_off[e + 1], we = 0;
    bool want_b = false;
    if (kDir == kDirRelabel) {
      const uint32_t nb = net_bits(g, e);
      // in-arcs of e_out from pins carry flow(e_out, u) > 0; their sum is the
      // outflow fb - excess(e_out), so a net without outflow skips its pins
      if (!in && !(nb & 2u)) end = beg;
      // e_out -> e_in residual fb, e_in -> e_out residual w - fb
      if (gl == 0) want_b = (nb & (in ? 4u : 1u)) && !seen_bit(g, b);
    } else {
      we = g.w[e];
      if (gl == 0) {
        const int fbv = g.fb[e], st = g.stamp[b];
        want_b = (in == (kDir == kDirSource) ? fbv < we : fbv > 0) && st != val;
      }
    }
    if (gl == 0) nbytes += 16;
    bool bridge = true;
    for (int base = beg; bridge || base < end; base += stride, bridge = false) {
      const int i = base + gl;
      bool want = false;
      int u = 0;
      if (i < end) {
        u = g.pin_v[i];
        nbytes += 12;
        if (kDir == kDirRelabel) {  // r_in (u -> e_in) or f_out (u -> e_out)
          const int f = g.fpin[2 * i + (in ? 0 : 1)];
          want = f > 0 && !seen_bit(g, u);
        } else {
          const int2 fp = *reinterpret_cast<const int2*>(g.fpin + 2 * i);
          // the flows come with the vertex, so looking at them first lengthens
          // no chain; few of a net node's reverse arcs exist, and each stamp
          // and role is a line of its own
          if (kDir == kDirSource) {  // e_in -> u reverse, e_out -> u infinite
            if (in) {
              want = we - fp.x > 0 && g.stamp[u] != val;
            } else {
              const int st = g.stamp[u], r = g.role[u];
              want = r == 0 && st != val;
              if (r == 2) atomicOr(&g.ctl->err, ERR_SINK_REACHED);
            }
          } else if (in || fp.y > 0) {  // u -> e_in always, u -> e_out by flow
            const int st = g.stamp[u], r = g.role[u];
            want = r != 1 && st != val;
            if (r == 1) atomicOr(&g.ctl->err, ERR_SOURCE_REACHED);
          }
        }
      }
      uint32_t word_b = 0, word = 0;
      int old_b = val;
      if (bridge) old_b = claim(want_b, b, word_b);
      const int old = claim(want, u, word);
      if (bridge) {
        mark(b, first(old_b) ? 1u : 0u);
        push(b, first(old_b), word_b);
      }
      mark(u, first(old) ? 1u : 0u);
      push(u, first(old), word);
    }
  }
}


// One BFS level, node-grouped: the reverse BFS of a global relabel (labels
// level+1), the forward BFS of the source side (stamp ep, provisional stamp
// ep_tmp when expanding) or the reverse BFS of the sink side (stamp ep,
// claiming only).
template <int G, bool kClaim, int kDir>
__device__ void phase_bfs_node(const Dev& g, int level, int ep, int ep_tmp, int tile0,
                               int tstride, int kc, lds_int* lds) {
  const int c3 = level % 3, n3 = (level + 1) % 3, z3 = (level + 2) % 3;
  if (tile0 == 0 && threadIdx.x < kNL) g.ctl->bcnt[z3][threadIdx.x] = 0;
  const int cp = level & 1, np = (level + 1) & 1;
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[n3], g.list[np]);
  const Items<G> its(g.ctl->bcnt[c3]);
  constexpr int GN = lanes_of<G>(1);
  const int total = its.total();
  const int wpb = blockDim.x >> 6, wid = threadIdx.x >> 6;
  const int ntiles = (total + wpb - 1) / wpb;
  const int lane = lane_id();
  uint32_t nbytes = 0, nitems = 0;
  // tiles of wave items, then one tile per big-list node in which only a huge
  // node (more arcs than a wave should scan alone, such as a contracted
  // terminal) is scanned, by the whole workgroup; a wave item skips it
  const int nbig = its.n[kBigList];
  for (int tile = tile0; tile < ntiles + nbig; tile += tstride) {
    int v = 0, gl = 0, stride = G;
    bool has = false;
    if (tile < ntiles) {
      const int it = tile * wpb + wid;
      if (it < total) {
        const int k = its.list_of_item(it);
        if (k < kBigList) {
          stride = k == 0 ? G : GN;
          const int idx = (it - its.start[k]) * (kWave / stride) + lane / stride;
          has = idx < its.n[k];
          v = has ? g.list[cp][k][idx] : 0;
          gl = lane % stride;
        } else {
          v = g.list[cp][kBigList][it - its.start[kBigList]];
          has = !is_huge(g, v);
          gl = lane;
          stride = kWave;
        }
      }
    } else {
      v = g.list[cp][kBigList][tile - ntiles];
      has = is_huge(g, v);  // block-uniform
      gl = threadIdx.x;
      stride = blockDim.x;
    }
    nitems += has && gl == 0;
    if constexpr (kClaim)
      bfs_claim_node<kDir>(g, q, v, has, gl, stride, kDir == kDirRelabel ? level + 1 : ep, nbytes);
    else if constexpr (kDir == kDirSource)
      bfs_fwd_node(g, v, has, gl, stride, ep, ep_tmp, nbytes);
    else bfs_rev_node(g, v, has, gl, stride, level + 1, nbytes);
    if (kClaim) bq_tile_end(q, q.cap / 2);
  }
  if (kClaim) bq_flush(q);
  block_add_u64(&g.ctl->bytes[kc], (unsigned long long)nbytes + 4ull * nitems, &g.ctl->items[kc],
                nitems);
}

// frontier of level `level` -> label level+1
template <int G, bool kClaim>
__device__ void phase_bfs_rev_node(const Dev& g, int level, int tile0, int tstride, int kc,
                                   lds_int* lds) {
  phase_bfs_node<G, kClaim, kDirRelabel>(g, level, 0, 0, tile0, tstride, kc, lds);
}

// ---------------------------------------------------------------------------
// flattened reverse-BFS levels
//
// A wave takes 64 consecutive entries of one small-node list, one node per
// lane, and spreads the nodes' arcs over its 64 lanes: a wave prefix sum of
// the arc counts, then in every step each lane finds the node owning its arc
// by a binary search over the lanes' offsets (shuffles, no LDS, no barrier).
// All loads of a step are independent and every lane has an arc until the
// last step, so a level's latency chains overlap far more than with a fixed
// group of lanes per node (a net node holds 3.7 arcs on average, a vertex
// 7.4, and most e_out nodes only their bridge).  Big nodes keep a wave each,
// huge nodes the workgroup, as in the node-grouped levels.
// ---------------------------------------------------------------------------

template <bool kSlice = false>
__device__ __forceinline__ void phase_bfs_rev_flat(const Dev& g, int level, int tile0, int tstride,
                                                   int kc, lds_int* lds) {
  const int c3 = level % 3, z3 = (level + 2) % 3;
  if (tile0 == 0 && threadIdx.x < kNL) g.ctl->bcnt[z3][threadIdx.x] = 0;
  const int cp = level & 1;
  lds_int* const xc = lds;  // slice counts
  if (kSlice) {
    if (threadIdx.x < kSlices) xc[threadIdx.x] = 0;
    __syncthreads();
  }
  const Quad n = load_counts(g.ctl->bcnt[c3]);
  // wave items: 64 entries of list 0, of list 1, of list 2, then one big node each
  const int s1 = (n.v0 + kWave - 1) / kWave;
  const int s2 = s1 + (n.v1 + kWave - 1) / kWave;
  const int s3 = s2 + (n.v2 + kWave - 1) / kWave;
  const int total = s3 + n.v3;
  const int wpb = blockDim.x >> 6, wid = threadIdx.x >> 6, lane = lane_id();
  const int ntiles = (total + wpb - 1) / wpb;
  const int lvl = level + 1;
  uint32_t nbytes = 0, nitems = 0;
  for (int tile = tile0; tile < ntiles + n.v3; tile += tstride) {
    if (tile < ntiles) {
      const int it = tile * wpb + wid;
      if (it < s3) {
        const int k = (it >= s1) + (it >= s2);  // wave-uniform list
        const int idx = (it - (k == 0 ? 0 : (k == 1 ? s1 : s2))) * kWave + lane;
        int x = 0, beg = 0, deg = 0;
        uint32_t nb = 0;
        if (idx < n[k]) {
          x = g.list[cp][k][idx];
          if (k == 0) {
            beg = g.vtx_off[x];
            deg = g.vtx_off[x + 1] - beg;
          } else {
            const int e = (x - g.NB) >> 1;
            nb = net_bits(g, e);
            beg = g.net_off[e];
            int sz = g.net_off[e + 1] - beg;
            // in-arcs of e_out from pins carry flow(e_out, u) > 0; a net
            // without outflow has none
            if (k == 2 && !(nb & 2u)) sz = 0;
            deg = 1 + sz;  // arc 0 is the bridge
            nbytes += 16;
          }
          nitems += 1;
        }
        int incl = deg;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
          const int t = __shfl_up(incl, o);
          if (lane >= o) incl += t;
        }
        const int excl = incl - deg;
        const int A = __shfl(incl, kWave - 1);
        for (int a0 = 0; a0 < A; a0 += kWave) {
          const int a = a0 + lane;
          // owner: the last lane whose offset is <= a (lanes without arcs
          // share the next lane's offset, so the last one owns the arc)
          int lo = 0;
#pragma unroll
          for (int st = kWave / 2; st > 0; st >>= 1) {
            const int c = lo + st;
            if (__shfl(excl, c) <= a) lo = c;
          }
          const int xo = __shfl(x, lo), bo = __shfl(beg, lo);
          const int j = a - __shfl(excl, lo);
          const uint32_t nbo = __shfl((int)nb, lo);
          int t1 = 0, t2 = 0;
          bool v1 = false, v2 = false;
          if (a < A) {
            if (k == 0) {
              const int2 ep = g.vinc[bo + j];
              t1 = g.NB + 2 * ep.x;
              t2 = t1 + 1;
              // bits of e_in and e_out share a word (NB and 2e are even)
              const uint32_t sw = g.seen[t1 >> 5] >> (t1 & 31);
              nbytes += 12;
              if (!(sw & 2u)) v2 = visit_rev<true, kSlice>(g, t2, lvl);  // e_out -> x infinite
              if (!(sw & 1u) && pin_flow_in(g, ep.y))                    // e_in -> x reverse
                v1 = visit_rev<true, kSlice>(g, t1, lvl);
            } else if (j == 0) {
              if (k == 1) {
                t1 = xo + 1;  // e_out -> e_in residual fb
                v1 = (nbo & 4u) && visit_rev<false, kSlice>(g, t1, lvl);
              } else {
                t1 = xo - 1;  // e_in -> e_out residual w - fb
                v1 = (nbo & 1u) && visit_rev<false, kSlice>(g, t1, lvl);
              }
            } else {
              const int i = bo + j - 1;
              t1 = g.pin_v[i];
              // r_in (u -> e_in) or f_out (u -> e_out)
              const int f = g.fpin[2 * i + (k == 1 ? 0 : 1)];
              nbytes += 12;
              if (f > 0) v1 = visit_rev<false, kSlice>(g, t1, lvl);
            }
          }
          if (kSlice) {
            xpush(g, xc, t1, v1, lvl);
            xpush(g, xc, t2, v2, lvl);
          }
        }
      } else if (it < total) {
        const int v = g.list[cp][kBigList][it - s3];
        const bool has = !is_huge(g, v);
        nitems += has && lane == 0;
        bfs_rev_node<kSlice>(g, v, has, lane, kWave, lvl, nbytes, xc);
      }
    } else {
      const int v = g.list[cp][kBigList][tile - ntiles];
      const bool has = is_huge(g, v);  // block-uniform
      nitems += has && threadIdx.x == 0;
      bfs_rev_node<kSlice>(g, v, has, threadIdx.x, blockDim.x, lvl, nbytes, xc);
    }
  }
  if (kSlice) {
    __syncthreads();
    if (threadIdx.x < kSlices)
      g.xcnt[blockIdx.x * kSlices + threadIdx.x] = min((int)xc[threadIdx.x], g.xseg);
  }
  block_add_u64(&g.ctl->bytes[kc], (unsigned long long)nbytes + 4ull * nitems, &g.ctl->items[kc],
                nitems);
}

// The labelling half of an XCD-local expanded level: workgroup b serves
// slice b mod 8 (so it runs on the XCD that owns the slice) and labels the
// heads that every workgroup of the scan handed to that slice.
__device__ void phase_bfs_slices(const Dev& g, int level, int nseg) {
  const int sl = blockIdx.x & (kSlices - 1);
  const int w = blockIdx.x / kSlices, nw = gridDim.x / kSlices;
  const int lvl = level + 1;
  for (int b = w; b < nseg; b += nw) {
    const int c = g.xcnt[b * kSlices + sl];
    const int32_t* src = g.xbuf + ((long long)b * kSlices + sl) * g.xseg;
    for (int i = threadIdx.x; i < c; i += blockDim.x) label_rev<false>(g, src[i], lvl);
  }
}

// ---------------------------------------------------------------------------
// arc-parallel BFS levels
//
// A workgroup takes a tile of up to blockDim frontier nodes, computes their
// arc counts and an exclusive prefix sum in LDS, and then every thread takes
// one arc per step (locating its node by binary search in the prefix), so
// all loads of a step are independent and nodes of any degree are spread
// over the whole workgroup.  Arc 0 of a net node is its bridge.
// ---------------------------------------------------------------------------

// tile area after the staging area: node[bd], beg[bd], off[bd + 1], wave
// sums[32] (bd = blockDim, at most 1024)

struct ArcTile {
  lds_int* node;
  lds_int* beg;
  lds_int* off;
  lds_int* wsum;
};

__device__ __forceinline__ ArcTile arc_tile(lds_int* lds) {
  ArcTile t;
  t.node = lds;
  const int bd = blockDim.x;
  t.beg = lds + bd;
  t.off = lds + 2 * bd;
  t.wsum = lds + 3 * bd + 1;
  return t;
}

// Block-uniform exclusive prefix sum of one int per thread; returns the
// thread's offset, *total gets the sum (same in every thread).
__device__ __forceinline__ int block_excl_scan(int v, lds_int* wsum, int* total) {
  const int lane = lane_id(), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  __syncthreads();  // wsum is free (previous readers are done)
  if (lane == kWave - 1) wsum[wid] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int i = 0; i < nw; ++i) {
      const int t = wsum[i];
      wsum[i] = run;
      run += t;
    }
    wsum[nw] = run;
  }
  __syncthreads();
  *total = wsum[nw];
  return wsum[wid] + incl - v;
}

// Block-uniform: load tile `tile` of the frontier into LDS; returns the arc
// count of the tile and the node count in *nt_out.
__device__ __forceinline__ int load_arc_tile(const Dev& g, const ArcTile& t, int par,
                                             const Prefix4& pre, int tile, int* nt_out) {
  const int nf = pre.total;
  const int first = tile * blockDim.x;
  const int nt = min((int)blockDim.x, nf - first);
  int deg = 0, beg = 0, v = 0;
  if ((int)threadIdx.x < nt) {
    v = frontier_node(g, par, pre, first + threadIdx.x);
    if (v < g.V) {
      beg = g.vtx_off[v];
      deg = g.vtx_off[v + 1] - beg;
    } else {
      const int e = (v - g.NB) >> 1;
      beg = g.net_off[e];
      deg = g.net_off[e + 1] - beg + 1;
    }
  }
  int total = 0;
  const int o = block_excl_scan(deg, t.wsum, &total);
  if ((int)threadIdx.x < nt) {
    t.node[threadIdx.x] = v;
    t.beg[threadIdx.x] = beg;
    t.off[threadIdx.x] = o;
  }
  if (threadIdx.x == 0) t.off[nt] = total;
  __syncthreads();
  *nt_out = nt;
  return total;
}

// index k of the tile node owning arc a: largest k with off[k] <= a
__device__ __forceinline__ int arc_owner(const ArcTile& t, int nt, int a) {
  int lo = 0, hi = nt;  // off[lo] <= a < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (t.off[mid] <= a) lo = mid;
    else hi = mid;
  }
  return lo;
}

// One level of the reverse BFS (labels level+1), arc-parallel.
template <bool kClaim>
__device__ void phase_bfs_rev_lb(const Dev& g, int level, int tile0, int tstride, int kc,
                                 lds_int* lds) {
  const int c3 = level % 3, n3 = (level + 1) % 3, z3 = (level + 2) % 3;
  if (tile0 == 0 && threadIdx.x < kNL) g.ctl->bcnt[z3][threadIdx.x] = 0;
  const int cp = level & 1, np = (level + 1) & 1;
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[n3], g.list[np]);
  const ArcTile t = arc_tile(lds + bq_words());
  const Prefix4 pre(load_counts(g.ctl->bcnt[c3]));
  const int ntiles = (pre.total + blockDim.x - 1) / blockDim.x;
  const int lvl = level + 1;
  uint32_t nbytes = 0, narcs = 0;
  for (int tile = tile0; tile < ntiles; tile += tstride) {
    int nt = 0;
    const int A = load_arc_tile(g, t, cp, pre, tile, &nt);
    for (int a0 = 0; a0 < A; a0 += blockDim.x) {
      const int a = a0 + threadIdx.x;
      int t1 = 0, t2 = 0;
      bool v1 = false, v2 = false;
      if (a < A) {
        const int k = arc_owner(t, nt, a);
        const int x = t.node[k];
        const int j = a - t.off[k];
        const int b = t.beg[k];
        ++narcs;
        if (x < g.V) {
          const int2 ep = g.vinc[b + j];
          const int e = ep.x;
          t1 = g.NB + 2 * e;
          t2 = t1 + 1;
          const uint32_t sw = g.seen[t1 >> 5] >> (t1 & 31);
          nbytes += 12;
          if (!(sw & 2u)) v2 = label_rev<kClaim, true>(g, t2, lvl);  // e_out -> x infinite
          if (!(sw & 1u) && g.w[e] - g.fpin[2 * ep.y] > 0)     // e_in -> x reverse
            v1 = label_rev<kClaim, true>(g, t1, lvl);
        } else {
          const int e = (x - g.NB) >> 1;
          const bool in = ((x - g.NB) & 1) == 0;
          if (j == 0) {  // bridge
            const int fbv = g.fb[e];
            nbytes += 8;
            t1 = in ? x + 1 : x - 1;
            if (in ? fbv > 0 : g.w[e] - fbv > 0) v1 = label_rev<kClaim>(g, t1, lvl);
          } else {
            const int i = b + j - 1;
            t1 = g.pin_v[i];
            const int f = g.fpin[2 * i + (in ? 0 : 1)];  // r_in (u->e_in) or f_out (u->e_out)
            nbytes += 9;
            if (f > 0) v1 = label_rev<kClaim>(g, t1, lvl);
          }
        }
      }
      if (kClaim) {
        qpush(g, q, t1, v1);
        qpush(g, q, t2, v2);
        bq_tile_end(q, 2 * blockDim.x);
      }
    }
    __syncthreads();  // the tile area is rewritten by the next tile
  }
  if (kClaim) bq_flush(q);
  block_add_u64(&g.ctl->bytes[kc], (unsigned long long)nbytes + 12ull * narcs, &g.ctl->items[kc],
                narcs);
}

// One level of the forward BFS of the uncapped network, arc-parallel.
template <bool kClaim>
__device__ void phase_bfs_fwd_lb(const Dev& g, int level, int ep, int ep_tmp, int tile0,
                                 int tstride, int kc, lds_int* lds) {
  const int c3 = level % 3, n3 = (level + 1) % 3, z3 = (level + 2) % 3;
  if (tile0 == 0 && threadIdx.x < kNL) g.ctl->bcnt[z3][threadIdx.x] = 0;
  const int cp = level & 1, np = (level + 1) & 1;
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[n3], g.list[np]);
  const ArcTile t = arc_tile(lds + bq_words());
  const Prefix4 pre(load_counts(g.ctl->bcnt[c3]));
  const int ntiles = (pre.total + blockDim.x - 1) / blockDim.x;
  uint32_t nbytes = 0, narcs = 0;
  for (int tile = tile0; tile < ntiles; tile += tstride) {
    int nt = 0;
    const int A = load_arc_tile(g, t, cp, pre, tile, &nt);
    for (int a0 = 0; a0 < A; a0 += blockDim.x) {
      const int a = a0 + threadIdx.x;
      int t1 = 0, t2 = 0;
      bool v1 = false, v2 = false;
      if (a < A) {
        const int k = arc_owner(t, nt, a);
        const int x = t.node[k];
        const int j = a - t.off[k];
        const int b = t.beg[k];
        ++narcs;
        if (x < g.V) {
          const int2 ep2 = g.vinc[b + j];
          t1 = g.NB + 2 * ep2.x;
          t2 = t1 + 1;
          nbytes += 12;
          v1 = fwd_visit<kClaim>(g, t1, ep, ep_tmp);                    // x -> e_in (uncapped)
          if (g.fpin[2 * ep2.y + 1] > 0) v2 = fwd_visit<kClaim>(g, t2, ep, ep_tmp);  // x -> e_out reverse
        } else {
          const int e = (x - g.NB) >> 1;
          const bool in = ((x - g.NB) & 1) == 0;
          if (j == 0) {  // bridge
            const int fbv = g.fb[e];
            nbytes += 8;
            t1 = in ? x + 1 : x - 1;
            if (in ? fbv < g.w[e] : fbv > 0) v1 = fwd_visit<kClaim>(g, t1, ep, ep_tmp);
          } else {
            const int i = b + j - 1;
            t1 = g.pin_v[i];
            nbytes += 8;
            if (in) {
              if (g.w[e] - g.fpin[2 * i] > 0) v1 = fwd_visit<kClaim>(g, t1, ep, ep_tmp);  // e_in -> u reverse
            } else {
              const int r = g.role[t1];
              if (r == 2) atomicOr(&g.ctl->err, ERR_SINK_REACHED);
              else if (r == 0) v1 = fwd_visit<kClaim>(g, t1, ep, ep_tmp);  // e_out -> u infinite
            }
          }
        }
      }
      if (kClaim) {
        qpush(g, q, t1, v1);
        qpush(g, q, t2, v2);
        bq_tile_end(q, 2 * blockDim.x);
      }
    }
    __syncthreads();  // the tile area is rewritten by the next tile
  }
  if (kClaim) bq_flush(q);
  block_add_u64(&g.ctl->bytes[kc], (unsigned long long)nbytes + 12ull * narcs, &g.ctl->items[kc],
                narcs);
}

// Bottom-up (pull) level, thread per node in id order: every unlabelled
// node scans its residual out-arcs of the capped network and takes label
// level+1 at the first arc into the level (only its own thread writes it):
//   vertex u:  u -> e_in if r_in > 0, u -> e_out if flow(e_out, u) > 0
//   e_in:      e_in -> e_out if fb < w, e_in -> u if flow(u, e_in) > 0
//   e_out:     e_out -> e_in if fb > 0, e_out -> u always
// The labels of the next level are then collected by the sweep.
__device__ void phase_bfs_rev_pull(const Dev& g, int level, int t0, int tstride, int kc) {
  // ring slot that nobody reads this level: the count of level+2
  if (t0 < kNL) g.ctl->bcnt[(level + 2) % 3][t0] = 0;
  const int lvl = level + 1;
  uint32_t nbytes = 0, narcs = 0;
  for (int v = t0; v < g.N; v += tstride) {
    if (seen_bit(g, v) || (v >= g.V && v < g.NB)) continue;
    if (g.d[v] != g.N) continue;
    bool hit = false;
    if (v < g.V) {
      const int beg = g.vtx_off[v], end = g.vtx_off[v + 1];
      nbytes += 12;
      for (int i = beg; i < end && !hit; ++i) {
        const int2 ep = g.vinc[i];
        const int2 dl = *reinterpret_cast<const int2*>(g.d + g.NB + 2 * ep.x);
        const int2 fp = *reinterpret_cast<const int2*>(g.fpin + 2 * ep.y);
        hit = (fp.x > 0 && dl.x == level) || (fp.y > 0 && dl.y == level);
        nbytes += 24;
        ++narcs;
      }
    } else {
      const int e = (v - g.NB) >> 1;
      const bool in = ((v - g.NB) & 1) == 0;
      const uint32_t nb = net_bits(g, e);
      nbytes += 16;
      ++narcs;
      hit = in ? ((nb & 1u) && g.d[v + 1] == level) : ((nb & 4u) && g.d[v - 1] == level);
      const int beg = g.net_off[e], end = g.net_off[e + 1];
      for (int p = beg; p < end && !hit; ++p) {
        if (in && !pin_flow_in(g, p)) continue;
        hit = g.d[g.pin_v[p]] == level;
        nbytes += 8;
        ++narcs;
      }
    }
    if (hit) {
      g.d[v] = lvl;
      if (g.lev) g.lev[v] = 1;  // listed (and marked 2) by the collect sweep
      set_seen(g, v);
    }
  }
  block_add_u64(&g.ctl->bytes[kc], nbytes, &g.ctl->items[kc], narcs);
}

template <int G>
__device__ void phase_bfs_rev(const Dev& g, int level, int tile0, int tstride, int kc,
                              lds_int* lds) {
  if (g.bfs_arc) phase_bfs_rev_lb<true>(g, level, tile0, tstride, kc, lds);
  else phase_bfs_rev_node<G, true>(g, level, tile0, tstride, kc, lds);
}

// Large levels run in two steps without claiming atomics: expand the level
// from its list, labelling unlabelled in-neighbours with plain stores (every
// writer stores the same value), then collect the next level by one sweep
// over the labels.
template <int G>
__device__ void phase_bfs_rev_expand(const Dev& g, int level, int tile0, int tstride, int kc,
                                     lds_int* lds) {
  if (g.bfs_arc) phase_bfs_rev_lb<false>(g, level, tile0, tstride, kc, lds);
  else phase_bfs_rev_node<G, false>(g, level, tile0, tstride, kc, lds);
}

// ---------------------------------------------------------------------------
// swept reverse-BFS levels
//
// Expanding a level that holds a large part of the graph from its list reads
// a line of offsets, adjacency and flows per node and a label line per arc,
// scattered over arrays of 20 MB and more, and a pass over all labels must
// then list the next level.  Such a level is swept the other way round
// instead: every node that has no label yet looks for an arc into the level,
// nets and vertices in id order.  What the sweep reads is consecutive, apart
// from one bit per arc in bitmaps of the level that stay in the L2 (125 KB for
// 1 M vertices, 500 KB for 2 M nets); every label is written by its node's own
// thread; and the next level's bitmaps and counts fall out of the wave's
// ballots, so a run of swept levels needs no lists:
//   e_out    from any pin in the level, or from e_in in the level by the
//            bridge (fb > 0)
//   e_in     from e_out in the level by the bridge (fb < w), or from a pin in
//            the level whose flow into e_in can be returned
//   vertex   from e_in in the level with room (r_in > 0), or from e_out in the
//            level when its flow into the vertex can be returned
// Lists are made again when the search leaves the large levels
// (phase_bfs_collect_bits); there the bitmaps are made when it enters them.
// ---------------------------------------------------------------------------

__device__ __forceinline__ bool bit_of(const uint32_t* m, int i) {
  return (m[i >> 5] >> (i & 31)) & 1u;
}

// Inclusive prefix sum over the wave.
__device__ __forceinline__ int wave_scan(int v) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int t = __shfl_up(v, o);
    if (lane_id() >= o) v += t;
  }
  return v;
}
// The last lane whose (exclusive) offset is at most a.
__device__ __forceinline__ int wave_owner(int excl, int a) {
  int lo = 0;
#pragma unroll
  for (int st = kWave / 2; st > 0; st >>= 1) {
    const int c = lo + st;
    if (__shfl(excl, c) <= a) lo = c;
  }
  return lo;
}

// A wave takes 128 nets (vertices), two per lane, and is bound by the latency
// of its loads, so a lane first looks at the first kFirst arcs of both with
// all their loads in flight: that settles most (nets of 3.7 pins on average,
// and a large level is hit early).  What is left is spread over the wave's
// lanes; nets or vertices with more than kSweepLong arcs left are set aside
// and scanned at the end, a wave each, so that no wave of the sweep walks a
// long one while the others wait.
constexpr int kFirst = 4;
constexpr int kSweepLong = 192;
constexpr int kSweepAside = 512;  // set aside per workgroup; more are scanned where they are met
constexpr int kSweepWords = 1 + kSweepAside + 1024 + 4;

__device__ void phase_bfs_sweep(const Dev& g, int level, int kc, lds_int* lds) {
  const int tid = threadIdx.x, lane = lane_id(), wid = uni(tid >> 6), nw = blockDim.x >> 6;
  lds_int* const naside = lds;              // set-aside count (may exceed kSweepAside)
  lds_int* const aside = lds + 1;           // node ids
  lds_int* const flag = aside + kSweepAside + wid * kWave;  // per lane of the wave
  lds_int* const found = aside + kSweepAside + 1024;        // nodes found per kind
  if (tid == 0) *naside = 0;
  if (tid >= 64 && tid < 67) found[tid - 64] = 0;
  __syncthreads();
  const int wave0 = uni((int)blockIdx.x * nw + wid);
  const int nwaves = gridDim.x * nw;
  const int lvl = level + 1;
  const uint32_t* const vf = g.vf[level & 1];
  const uint2* const nl = g.nl[level & 1];
  uint32_t* const vf_next = g.vf[lvl & 1];
  uint2* const nl_next = g.nl[lvl & 1];
  uint32_t nbytes = 0, narcs = 0;
  int nv = 0, nin = 0, nout = 0;  // found by this wave
  auto set_aside = [&](int node) {
    const int pos = lds_add(naside, 1);
    if (pos < kSweepAside) aside[pos] = node;
    return pos < kSweepAside;
  };
  // what pin slot i says to a net that looks for pull (bit0 e_out, bit1 e_in)
  auto net_arc = [&](int i, int pull) {
    if (!bit_of(vf, g.pin_v[i])) return 0;
    return (pull & 1) | ((pull & 2) && pin_flow_in(g, i) ? 2 : 0);
  };
  // whether incidence x = {net, slot}, whose net's level word is w, reaches
  // its vertex
  auto vertex_hit = [&](int2 x, uint2 w) {
    const uint32_t b = 1u << (x.x & 31);
    return ((w.x & b) && bit_of(g.pinfree, x.y)) || ((w.y & b) && g.fpin[2 * x.y + 1] > 0);
  };
  for (int base = wave0 * 2 * kWave; base < g.E; base += nwaves * 2 * kWave) {
    int2 d[2];
    int beg[2], end[2], got[2], pull[2];
    uint32_t nb[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int e = min(base + t * kWave + lane, g.E - 1);
      d[t] = *reinterpret_cast<const int2*>(g.d + g.NB + 2 * e);
      beg[t] = g.net_off[e];
      end[t] = g.net_off[e + 1];
      nb[t] = net_bits(g, e);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const bool in = base + t * kWave + lane < g.E;
      got[t] = !in ? 0 : (d[t].x == level && d[t].y == g.N && (nb[t] & 4u) ? 1 : 0) |
                             (d[t].y == level && d[t].x == g.N && (nb[t] & 1u) ? 2 : 0);
      pull[t] = !in ? 0 : (d[t].y == g.N && !(got[t] & 1) ? 1 : 0) |
                              (d[t].x == g.N && !(got[t] & 2) && (nb[t] & 8u) ? 2 : 0);
      nbytes += 16;
    }
    int u[2][kFirst];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < kFirst; ++j)
        u[t][j] = pull[t] && beg[t] + j < end[t] ? g.pin_v[beg[t] + j] : -1;
    uint32_t w[2][kFirst];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < kFirst; ++j) w[t][j] = u[t][j] >= 0 ? vf[u[t][j] >> 5] : 0u;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < kFirst; ++j)
        if ((w[t][j] >> (u[t][j] & 31)) & 1u) {
          got[t] |= pull[t] & 1;
          if ((pull[t] & 2) && pin_flow_in(g, beg[t] + j)) got[t] |= 2;
        }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int e0 = base + t * kWave;
      if (e0 >= g.E) break;  // wave-uniform
      const int node = g.NB + 2 * (e0 + lane);
      const int b = beg[t] + kFirst;
      int deg = (pull[t] & ~got[t]) ? max(0, end[t] - b) : 0;
      if (deg > kSweepLong && set_aside(node)) deg = 0;
      if (__ballot(deg > 0)) {
        flag[lane] = 0;
        wave_lds_sync();
        const int incl = wave_scan(deg), excl = incl - deg, A = __shfl(incl, kWave - 1);
        for (int a0 = 0; a0 < A; a0 += kWave) {
          const int a = a0 + lane;
          const int lo = wave_owner(excl, a);
          const int i = __shfl(b, lo) + a - __shfl(excl, lo);
          const int q = __shfl(pull[t], lo);
          if (a < A) {
            const int f = net_arc(i, q);
            if (f)
              __hip_atomic_fetch_or(flag + lo, f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            ++narcs;
          }
        }
        wave_lds_sync();
        got[t] |= flag[lane];
      }
      if (got[t] & 1) g.d[node + 1] = lvl;
      if (got[t] & 2) g.d[node] = lvl;
      const unsigned long long mi = __ballot(got[t] & 2), mo = __ballot(got[t] & 1),
                               mf = __ballot((got[t] & 1) && (nb[t] & 2u));
      nin += __popcll(mi);
      nout += __popcll(mo);
      if (lane < 2)
        nl_next[(e0 >> 5) + lane] =
            make_uint2((uint32_t)(mi >> (32 * lane)), (uint32_t)(mf >> (32 * lane)));
    }
  }
  for (int base = wave0 * 2 * kWave; base < g.V; base += nwaves * 2 * kWave) {
    int beg[2], end[2];
    bool got[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int v = min(base + t * kWave + lane, g.V - 1);
      const bool open = base + t * kWave + lane < g.V && g.d[v] == g.N;
      beg[t] = g.vtx_off[v];
      end[t] = open ? g.vtx_off[v + 1] : beg[t];
      got[t] = false;
      nbytes += 12;
    }
    int2 ep[2][kFirst];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < kFirst; ++j)
        ep[t][j] = beg[t] + j < end[t] ? g.vinc[beg[t] + j] : make_int2(-1, 0);
    uint2 w[2][kFirst];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < kFirst; ++j)
        w[t][j] = ep[t][j].x >= 0 ? nl[ep[t][j].x >> 5] : make_uint2(0u, 0u);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < kFirst; ++j)
        if (!got[t] && (w[t][j].x | w[t][j].y)) got[t] = vertex_hit(ep[t][j], w[t][j]);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int v0 = base + t * kWave;
      if (v0 >= g.V) break;  // wave-uniform
      const int b = beg[t] + kFirst;
      int deg = got[t] ? 0 : max(0, end[t] - b);
      if (deg > kSweepLong && set_aside(v0 + lane)) deg = 0;
      if (__ballot(deg > 0)) {
        flag[lane] = 0;
        wave_lds_sync();
        const int incl = wave_scan(deg), excl = incl - deg, A = __shfl(incl, kWave - 1);
        for (int a0 = 0; a0 < A; a0 += kWave) {
          const int a = a0 + lane;
          const int lo = wave_owner(excl, a);
          const int i = __shfl(b, lo) + a - __shfl(excl, lo);
          if (a < A) {
            const int2 x = g.vinc[i];
            if (vertex_hit(x, nl[x.x >> 5]))
              __hip_atomic_store(flag + lo, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            ++narcs;
          }
        }
        wave_lds_sync();
        if (flag[lane]) got[t] = true;
      }
      if (got[t]) g.d[v0 + lane] = lvl;
      const unsigned long long m = __ballot(got[t]);
      nv += __popcll(m);
      if (lane < 2) vf_next[(v0 >> 5) + lane] = (uint32_t)(m >> (32 * lane));
    }
  }
  __syncthreads();  // the set-aside list is complete, the bitmap words are written
  const int na = min((int)*naside, kSweepAside);
  for (int h = wid; h < na; h += nw) {
    const int node = uni(aside[h]);
    if (node < g.V) {
      bool f = false;
      const int end = g.vtx_off[node + 1];
      for (int i = g.vtx_off[node] + kFirst; i < end && !f; i += kWave) {
        bool hit = false;
        if (i + lane < end) {
          const int2 x = g.vinc[i + lane];
          hit = vertex_hit(x, nl[x.x >> 5]);
          ++narcs;
        }
        f = __ballot(hit) != 0ull;
      }
      if (f && lane == 0) {
        g.d[node] = lvl;
        atomicOr(&vf_next[node >> 5], 1u << (node & 31));
      }
      nv += f;
    } else {
      const int e = (node - g.NB) >> 1;
      const int2 d = *reinterpret_cast<const int2*>(g.d + node);
      const uint32_t b = net_bits(g, e);
      // labels of this level that the bridge gave are there already
      const int pull = (d.y == g.N ? 1 : 0) | (d.x == g.N && (b & 8u) ? 2 : 0);
      int f = 0;
      const int end = g.net_off[e + 1];
      for (int i = g.net_off[e]; i < end && (pull & ~f); i += kWave) {
        const int r = i + lane < end ? net_arc(i + lane, pull) : 0;
        if (__ballot(r & 1)) f |= 1;
        if (__ballot(r & 2)) f |= 2;
        narcs += i + lane < end;
      }
      if (lane == 0) {
        if (f & 1) g.d[node + 1] = lvl;
        if (f & 2) {
          g.d[node] = lvl;
          atomicOr(&nl_next[e >> 5].x, 1u << (e & 31));
        }
        if ((f & 1) && (b & 2u)) atomicOr(&nl_next[e >> 5].y, 1u << (e & 31));
      }
      nout += f & 1;
      nin += f >> 1;
    }
  }
  if (lane == 0) {
    lds_add(found + 0, nv);
    lds_add(found + 1, nin);
    lds_add(found + 2, nout);
  }
  __syncthreads();
  if (tid < 3 && found[tid]) atomicAdd(&g.ctl->sweep_n[level & 1][tid], (int)found[tid]);
  block_add_u64(&g.ctl->bytes[kc], (unsigned long long)nbytes + 8ull * narcs, &g.ctl->items[kc],
                narcs);
}

// One pass over the labels, a wave per 64 consecutive nodes: the bitmaps of
// level + 1 (for a sweep), or with kList its lists and the "labelled" hint of
// every node (the swept levels do not keep either).
template <bool kList>
__device__ void phase_bfs_collect_bits(const Dev& g, int level, int tile0, int tstride,
                                       lds_int* lds) {
  const int n3 = (level + 1) % 3, np = (level + 1) & 1;
  const int lab = level + 1;
  const int lane = lane_id();
  const int ts = 2 * (int)blockDim.x;
  BlockQ q{};
  if (kList) q = bq_bind(lds, g.ctl->bcnt[n3], g.list[np]);
  if (kList) {
    const int ntiles = (g.N + ts - 1) / ts;
    for (int tile = tile0; tile < ntiles; tile += tstride) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int v = (2 * tile + j) * (int)blockDim.x + (int)threadIdx.x;
        const int d = v < g.N ? g.d[v] : g.N;
        const unsigned long long m = __ballot(d != g.N);
        const int w = ((v - lane) >> 5) + lane;  // v - lane is a multiple of 64
        if (lane < 2 && 32 * w < g.N) g.seen[w] = (uint32_t)(m >> (32 * lane));
        qpush(g, q, v, d == lab);
      }
      bq_tile_end(q, 2 * blockDim.x);
    }
    bq_flush(q);
  } else {
    uint32_t* const vf = g.vf[lab & 1];
    uint2* const nl = g.nl[lab & 1];
    const int t0 = tile0 * (int)blockDim.x + (int)threadIdx.x, tn = tstride * (int)blockDim.x;
    for (int v = t0; v < ((g.V + 63) & ~63); v += tn) {
      const unsigned long long m = __ballot(v < g.V && g.d[v] == lab);
      if (lane < 2) vf[((v - lane) >> 5) + lane] = (uint32_t)(m >> (32 * lane));
    }
    for (int e = t0; e < ((g.E + 63) & ~63); e += tn) {
      int2 d = make_int2(0, 0);
      if (e < g.E) d = *reinterpret_cast<const int2*>(g.d + g.NB + 2 * e);
      const unsigned long long mi = __ballot(e < g.E && d.x == lab);
      const unsigned long long mf = __ballot(e < g.E && d.y == lab && (net_bits(g, e) & 2u));
      if (lane < 2)
        nl[((e - lane) >> 5) + lane] =
            make_uint2((uint32_t)(mi >> (32 * lane)), (uint32_t)(mf >> (32 * lane)));
    }
  }
}

// Sweep tiles: 2 nodes per thread, so a tile appends at most 2 * blockDim
// entries per list.
__device__ __forceinline__ int sweep_tiles(const Dev& g) {
  const int ts = 2 * blockDim.x;
  return (g.N + ts - 1) / ts;
}

__device__ void phase_bfs_collect(const Dev& g, int level, int tile0, int tstride, lds_int* lds) {
  // nodes labelled level+1 become the list of level+1
  const int n3 = (level + 1) % 3, np = (level + 1) & 1;
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[n3], g.list[np]);
  const int lab = level + 1;
  const int ntiles = sweep_tiles(g);
  for (int tile = tile0; tile < ntiles; tile += tstride) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int v = (2 * tile + j) * blockDim.x + threadIdx.x;
      bool fresh = false;
      if (g.lev) {  // byte marks: the level's nodes carry mark 1 and get their label here
        fresh = v < g.N && g.lev[v] == 1;
        if (fresh) {
          g.lev[v] = 2;
          g.d[v] = lab;
        }
      } else {
        fresh = v < g.N && g.d[v] == lab;
      }
      qpush(g, q, v, fresh);
    }
    bq_tile_end(q, 2 * blockDim.x);
  }
  bq_flush(q);
}

// ---------------------------------------------------------------------------
// forward residual BFS of the uncapped network (source-side cut)
// ---------------------------------------------------------------------------

template <int G>
__device__ void phase_bfs_fwd(const Dev& g, int level, int ep, int tile0, int tstride, int kc,
                              lds_int* lds) {
  if (g.bfs_arc) phase_bfs_fwd_lb<true>(g, level, ep, 0, tile0, tstride, kc, lds);
  else phase_bfs_node<G, true, kDirSource>(g, level, ep, 0, tile0, tstride, kc, lds);
}

// Large forward levels: expand with provisional stamps, then list the next
// level by one sweep that turns them into the BFS stamp.
template <int G>
__device__ void phase_bfs_fwd_expand(const Dev& g, int level, int ep, int ep_tmp, int tile0,
                                     int tstride, int kc, lds_int* lds) {
  if (g.bfs_arc) phase_bfs_fwd_lb<false>(g, level, ep, ep_tmp, tile0, tstride, kc, lds);
  else phase_bfs_node<G, false, kDirSource>(g, level, ep, ep_tmp, tile0, tstride, kc, lds);
}

__device__ void phase_bfs_fwd_collect(const Dev& g, int level, int ep, int ep_tmp, int tile0,
                                      int tstride, lds_int* lds) {
  const int n3 = (level + 1) % 3, np = (level + 1) & 1;
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[n3], g.list[np]);
  const int ntiles = sweep_tiles(g);
  for (int tile = tile0; tile < ntiles; tile += tstride) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int v = (2 * tile + j) * blockDim.x + threadIdx.x;
      const bool fresh = v < g.N && g.stamp[v] == ep_tmp;
      if (fresh) g.stamp[v] = ep;
      qpush(g, q, v, fresh);
    }
    bq_tile_end(q, 2 * blockDim.x);
  }
  bq_flush(q);
}

// ---------------------------------------------------------------------------
// sweeps (thread per node); t0 wave-aligned, tstride a multiple of 64
// ---------------------------------------------------------------------------

// Zero flow, excess only at e_in of nets with a source pin (their contracted
// source arc saturated at w(e)), all counters cleared.
__device__ void phase_init(const Dev& g, int t0, int tstride) {
  if (t0 == 0) {
    Ctl* c = g.ctl;
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < kNL; ++k) c->fcnt[i][k] = c->bcnt[i][k] = 0;
    c->err = 0;
    c->flow = 0ull;
    c->relabels = 0ull;
    c->nswept = 0;
    for (int i = 0; i < KC_N; ++i) c->bytes[i] = c->items[i] = 0ull;
  }
  const int n = max(g.P, g.N);
  for (int i = t0; i < n; i += tstride) {
    if (i < g.P) {  // slot i: r_in = w(e), no flow (slots of a net are contiguous)
      *reinterpret_cast<int2*>(g.fpin + 2 * i) = make_int2(g.w[g.pin_net[i]], 0);
    }
    if (i < g.N) {
      g.stamp[i] = -1;
      g.cand[i] = -1;
      g.dx[0][i] = 0;
      g.dx[1][i] = 0;
      int xv = 0;
      if (i >= g.NB) {
        const int e = (i - g.NB) >> 1;
        if (((i - g.NB) & 1) == 0) {
          if (g.nflag[e] & 1) xv = g.w[e];
          g.fb[e] = 0;
        }
      }
      g.x[i] = xv;
    }
  }
}

// Global relabel, step 1: labels N for free nodes, 0 for sinks, N+1 for
// sources and padding; sinks form BFS level 0.  Round counters are cleared
// (the frontier is rebuilt by phase_gather).
__device__ void phase_gr_reset(const Dev& g, int tile0, int tstride, lds_int* lds) {
  if (tile0 == 0 && threadIdx.x == 0) {
    Ctl* c = g.ctl;
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < kNL; ++k) c->fcnt[i][k] = 0;
    c->big_last = -1;
    c->bits_level = -1;
    c->swept = -1;
  }
  // vertices, with the sinks listed and the labelled hint a word per half
  // wave (sinks, sources and padding start labelled); then the nets, which
  // only need their labels and hint words written
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[0], g.list[0]);
  const int lane = lane_id();
  const int ts = 2 * (int)blockDim.x;
  const int nvr = (g.NB + 63) & ~63;
  const int ntiles = (nvr + ts - 1) / ts;
  for (int tile = tile0; tile < ntiles; tile += tstride) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int v = (2 * tile + j) * (int)blockDim.x + (int)threadIdx.x;
      bool seed = false;
      int lab = g.N;
      if (v < g.NB) {
        lab = g.N + 1;
        if (v < g.V) {
          const int r = g.role[v];
          lab = r == 1 ? g.N + 1 : (r == 2 ? 0 : g.N);
          seed = r == 2;
        }
        g.d[v] = lab;
        if (g.lev) g.lev[v] = lab == g.N ? 0 : 2;
      }
      const unsigned long long m = __ballot(lab != g.N);
      const int w = ((v - lane) >> 5) + lane;
      if (lane < 2 && v - lane < nvr && 32 * w < g.N) g.seen[w] = (uint32_t)(m >> (32 * lane));
      qpush(g, q, v, seed);
    }
    bq_tile_end(q, 2 * blockDim.x);
  }
  bq_flush(q);
  const int t0 = tile0 * (int)blockDim.x + (int)threadIdx.x, tn = tstride * (int)blockDim.x;
  for (int e = t0; e < g.E; e += tn) {
    *reinterpret_cast<int2*>(g.d + g.NB + 2 * e) = make_int2(g.N, g.N);
    if (g.lev) g.lev[g.NB + 2 * e] = g.lev[g.NB + 2 * e + 1] = 0;
  }
  for (int w = nvr / 32 + t0; w < (g.N + 31) >> 5; w += tn) g.seen[w] = 0u;
}

// Global relabel, step 3: fold outstanding excess deltas; frontier =
// non-terminal nodes with excess and a label below N.  BFS counters are
// cleared for the next BFS.
__device__ void phase_gather(const Dev& g, int epoch, int tile0, int tstride, lds_int* lds) {
  const int c3 = epoch % 3, cp = epoch & 1;
  if (tile0 == 0 && threadIdx.x == 0) {
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < kNL; ++k) g.ctl->bcnt[i][k] = 0;
  }
  const BlockQ q = bq_bind(lds, g.ctl->fcnt[c3], g.list[cp]);
  const int ntiles = sweep_tiles(g);
  for (int tile = tile0; tile < ntiles; tile += tstride) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int v = (2 * tile + j) * blockDim.x + threadIdx.x;
      bool act = false;
      if (v < g.N) {
        const int a = g.dx[0][v], b = g.dx[1][v];
        int xv = g.x[v];
        if (a | b) {
          xv += a + b;
          g.x[v] = xv;
          g.dx[0][v] = 0;
          g.dx[1][v] = 0;
        }
        if (v >= g.NB || (v < g.V && g.role[v] == 0)) act = xv > 0 && g.d[v] < g.N;
      }
      qpush(g, q, v, act);
    }
    bq_tile_end(q, 2 * blockDim.x);
  }
  bq_flush(q);
}

// Cut BFS seeds: sources (marked, nothing to expand: their only arcs are the
// contracted source arcs into e_in), e_in of nets with a source pin, and
// every non-terminal node holding excess.  With only_new, nodes that already
// carry ep are left out (growing an existing source side).
__device__ void phase_cut_seed(const Dev& g, int ep, bool only_new, int tile0, int tstride,
                               lds_int* lds) {
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[0], g.list[0]);
  const int ntiles = sweep_tiles(g);
  for (int tile = tile0; tile < ntiles; tile += tstride) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int v = (2 * tile + j) * blockDim.x + threadIdx.x;
      bool seed = false;
      if (v < g.N) {
        if (v < g.V) {
          const int r = g.role[v];
          if (r == 1) g.stamp[v] = ep;
          else if (r == 0 && g.x[v] > 0) seed = true;
        } else if (v >= g.NB) {
          const int e = (v - g.NB) >> 1;
          const bool in = ((v - g.NB) & 1) == 0;
          seed = g.x[v] > 0 || (in && (g.nflag[e] & 1));
        }
        if (seed && only_new && g.stamp[v] == ep) seed = false;
        if (seed) g.stamp[v] = ep;
      }
      qpush(g, q, v, seed);
    }
    bq_tile_end(q, 2 * blockDim.x);
  }
  bq_flush(q);
}

// Write the side bitmaps and clear BFS counters.
__device__ void phase_cut_out(const Dev& g, int ep, uint8_t* vside, uint8_t* nside, int t0,
                              int tstride) {
  if (t0 == 0) {
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < kNL; ++k) g.ctl->bcnt[i][k] = 0;
  }
  const int n = max(g.V, g.E);
  for (int i = t0; i < n; i += tstride) {
    if (i < g.V) {
      const int r = g.role[i];
      vside[i] = (uint8_t)(r == 1 ? 1 : (r == 2 ? 0 : (g.stamp[i] == ep)));
    }
    if (i < g.E && nside) {
      const int a = g.stamp[g.NB + 2 * i] == ep;
      const int b = g.stamp[g.NB + 2 * i + 1] == ep;
      nside[i] = (uint8_t)(a | (b << 1));
    }
  }
}

// ---------------------------------------------------------------------------
// maximal sink side: reverse residual BFS from the sinks over the uncapped
// network (paper, algorithm "FlowCutter Core": T_r by backward residual
// BFS).  Node a joins when it has a residual arc into the current level:
//   into a vertex u   from e_out (infinite) and from e_in if flow(u, e_in) > 0
//   into e_in         from every pin (u -> e_in uncapped) and from e_out if fb > 0
//   into e_out        from e_in if fb < w and from pins u with flow(e_out, u) > 0
// Sources never join (a maximum preflow leaves no residual path from the
// source to a sink); reaching one is reported as ERR_SOURCE_REACHED.
// ---------------------------------------------------------------------------

// Seeds: the sinks.  The BFS counters must be clear (phase_reset_bfs).
__device__ void phase_sink_seed(const Dev& g, int ep, int tile0, int tstride, lds_int* lds) {
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[0], g.list[0]);
  const int ntiles = sweep_tiles(g);
  for (int tile = tile0; tile < ntiles; tile += tstride) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int v = (2 * tile + j) * blockDim.x + threadIdx.x;
      const bool seed = v < g.V && g.role[v] == 2;
      if (seed) g.stamp[v] = ep;
      qpush(g, q, v, seed);
    }
    bq_tile_end(q, 2 * blockDim.x);
  }
  bq_flush(q);
}

// The same sink side from exact labels of the capped network (the labels
// of a global relabel that found no active node): a node reaches a sink in
// the capped residual network exactly when its label is below N, and that
// set D lies in T_r, the uncapped network having every residual arc of the
// capped one.  The two networks differ only in the pin arcs u -> e_in,
// residual in the uncapped network even when saturated, so a residual path
// from outside D enters D by such an arc: its tail u (label N or more, arc
// saturated into an e_in of D) is a seed, and the reverse BFS of the
// uncapped network continues from the seeds through the nodes outside D.
// Stamps D with ep and lists the seeds as level 0 (counters clear).  A
// source's pin arcs carry no flow, so none qualifies; one that did would
// reach a sink (ERR_SOURCE_REACHED).
__device__ void phase_sink_seed_labels(const Dev& g, int ep, int tile0, int tstride,
                                       lds_int* lds) {
  const int ntiles = sweep_tiles(g);
  for (int tile = tile0; tile < ntiles; tile += tstride) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int v = (2 * tile + j) * blockDim.x + threadIdx.x;
      if (v < g.N && g.d[v] < g.N) g.stamp[v] = ep;
    }
  }
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[0], g.list[0]);
  const int ptiles = (g.P + (int)blockDim.x - 1) / (int)blockDim.x;
  for (int tile = tile0; tile < ptiles; tile += tstride) {
    const int p = tile * (int)blockDim.x + (int)threadIdx.x;
    int u = 0;
    bool seed = false;
    if (p < g.P && g.fpin[2 * p] == 0) {  // u -> e_in saturated (flow w(e))
      u = g.pin_v[p];
      if (g.d[g.NB + 2 * g.pin_net[p]] < g.N && g.d[u] >= g.N) {
        if (g.role[u] == 1) atomicOr(&g.ctl->err, ERR_SOURCE_REACHED);
        else seed = stamp_first(g, u, ep);
      }
    }
    qpush(g, q, u, seed);
    bq_tile_end(q, (int)blockDim.x);
  }
  bq_flush(q);
}

__device__ void phase_bfs_sink_lb(const Dev& g, int level, int ep, int tile0, int tstride, int kc,
                                  lds_int* lds) {
  const int c3 = level % 3, n3 = (level + 1) % 3, z3 = (level + 2) % 3;
  if (tile0 == 0 && threadIdx.x < kNL) g.ctl->bcnt[z3][threadIdx.x] = 0;
  const int cp = level & 1, np = (level + 1) & 1;
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[n3], g.list[np]);
  const ArcTile t = arc_tile(lds + bq_words());
  const Prefix4 pre(load_counts(g.ctl->bcnt[c3]));
  const int ntiles = (pre.total + blockDim.x - 1) / blockDim.x;
  uint32_t nbytes = 0, narcs = 0;
  bool hit_source = false;
  for (int tile = tile0; tile < ntiles; tile += tstride) {
    int nt = 0;
    const int A = load_arc_tile(g, t, cp, pre, tile, &nt);
    for (int a0 = 0; a0 < A; a0 += blockDim.x) {
      const int a = a0 + threadIdx.x;
      int t1 = 0, t2 = 0;
      bool v1 = false, v2 = false;
      if (a < A) {
        const int k = arc_owner(t, nt, a);
        const int x = t.node[k];
        const int j = a - t.off[k];
        const int b = t.beg[k];
        ++narcs;
        if (x < g.V) {
          const int2 ep2 = g.vinc[b + j];
          t1 = g.NB + 2 * ep2.x;
          t2 = t1 + 1;
          nbytes += 12;
          v2 = stamp_first(g, t2, ep);                                         // e_out -> x
          if (g.w[ep2.x] - g.fpin[2 * ep2.y] > 0) v1 = stamp_first(g, t1, ep);  // e_in -> x
        } else {
          const int e = (x - g.NB) >> 1;
          const bool in = ((x - g.NB) & 1) == 0;
          if (j == 0) {  // bridge
            const int fbv = g.fb[e];
            nbytes += 8;
            t1 = in ? x + 1 : x - 1;
            if (in ? fbv > 0 : fbv < g.w[e]) v1 = stamp_first(g, t1, ep);
          } else {
            const int i = b + j - 1;
            t1 = g.pin_v[i];
            const int r = g.role[t1];
            nbytes += 8;
            const bool arc = in || g.fpin[2 * i + 1] > 0;  // u -> e_in always, u -> e_out by flow
            if (arc) {
              if (r == 1) hit_source = true;
              else v1 = stamp_first(g, t1, ep);
            }
          }
        }
      }
      qpush(g, q, t1, v1);
      qpush(g, q, t2, v2);
      bq_tile_end(q, 2 * blockDim.x);
    }
    __syncthreads();  // the tile area is rewritten by the next tile
  }
  bq_flush(q);
  if (hit_source) atomicOr(&g.ctl->err, ERR_SOURCE_REACHED);
  block_add_u64(&g.ctl->bytes[kc], (unsigned long long)nbytes + 12ull * narcs, &g.ctl->items[kc],
                narcs);
}

template <int G>
__device__ void phase_bfs_sink(const Dev& g, int level, int ep, int tile0, int tstride, int kc,
                               lds_int* lds) {
  if (g.bfs_arc) phase_bfs_sink_lb(g, level, ep, tile0, tstride, kc, lds);
  else phase_bfs_node<G, true, kDirSink>(g, level, ep, 0, tile0, tstride, kc, lds);
}

// ---------------------------------------------------------------------------
// BFS levels inside one workgroup
//
// Levels `level0`, ... of a search whose current level holds at most `cap`
// nodes, until a level is empty or larger: the reverse BFS of a global relabel
// (labels level + 1), the forward BFS of the source side or the reverse BFS of
// the sink side (stamp ep).  Levels this small are bound by latency, so a
// level is one short chain: its nodes and counts are in LDS (lists of
// kLoopCap entries; what does not fit lies at the same position of the global
// list), a thread per node reads the arc range, a prefix sum over the
// workgroup spreads the arcs over all threads (even one node's), and a claimed
// node goes straight into the next level's LDS list: three barriers and four
// dependent global accesses a level (a FlowCutter growth of a few levels 14.5
// us instead of 21.1).  Returns the number of levels run; the
// level reached is then in the global lists.
// ---------------------------------------------------------------------------

// The claims are atomics in the L2, while other waves' plain loads of the
// same labels or stamps are in flight: a line that such a load brings into the
// CU's vector cache may hold the value before the claim.  Within a search that
// costs at most a claim that fails.  Whoever reads labels or stamps with plain
// loads later in the same kernel must call this first (a kernel's start does
// it too): it drops the vector cache.  Every wave calls it, after a barrier.
__device__ __forceinline__ void wg_drop_l1() {
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

constexpr int kBfsTile = 1024;  // nodes per tile at most (the largest workgroup)
constexpr int kWgBfsWords = 2 * kNL * kLoopCap + 3 * kBfsTile + 16 + 3 * kNL;

// With kGrow (the growths of a FlowCutter loop) level0 is 0 and its nodes and
// counts are in the area already, the vertices reached are listed and weighed,
// the statistics are left to the caller, and the level reached is written back
// only if it holds nodes.
struct Growth {
  const int32_t* cw;             // vertex weights
  int32_t* fresh;                // vertices reached, after the *nfresh that are there
  lds_int* nfresh;
  lds_u64* weight;
  uint32_t* next;                // vertices next to the side (bits), those outside both sides at least
  int other;                     // the other side's stamp
  unsigned long long nbytes = 0, narcs = 0;
  int left = 0;                  // nodes of the level reached
};

template <int kDir, bool kGrow = false, int kArcs = 1>
__device__ __forceinline__ int wg_bfs(const Dev& g, int level0, int cap, int ep, int kc, lds_int* lds,
                      Growth* grow = nullptr) {
  lds_int* const buf = lds;  // [2][kNL][kLoopCap]
  lds_int* const t_node = lds + 2 * kNL * kLoopCap;
  lds_int* const t_beg = t_node + kBfsTile;
  lds_int* const t_off = t_beg + kBfsTile;
  lds_int* const wsum = t_off + kBfsTile;
  lds_int* const cnt = wsum + 16;  // [3][kNL]
  const int tid = threadIdx.x, lane = lane_id(), wid = uni(tid >> 6), nw = blockDim.x >> 6;
  int level = level0;
  if (!kGrow) {
    const int c3 = level % 3, cp = level & 1;
    const Quad n{uni(ld_vol(&g.ctl->bcnt[c3][0])), uni(ld_vol(&g.ctl->bcnt[c3][1])),
                 uni(ld_vol(&g.ctl->bcnt[c3][2])), uni(ld_vol(&g.ctl->bcnt[c3][3]))};
    const int nf = n.v0 + n.v1 + n.v2 + n.v3;
    if (nf == 0 || nf > cap) return 0;
    __syncthreads();  // earlier users of the area are done with it
    if (tid < 3 * kNL) cnt[tid] = tid / kNL == c3 ? n[tid % kNL] : 0;
#pragma unroll
    for (int k = 0; k < kNL; ++k)
      for (int i = tid; i < min(n[k], kLoopCap); i += blockDim.x)
        buf[(cp * kNL + k) * kLoopCap + i] = g.list[cp][k][i];
    __syncthreads();
  }
  unsigned long long nbytes_all = 0, narcs = 0;
  bool hit_sink = false, hit_source = false;
  for (;; ++level) {
    const int c3 = level % 3, n3 = (level + 1) % 3, z3 = (level + 2) % 3;
    const int cp = level & 1, np = cp ^ 1;
    const Quad n{uni(cnt[c3 * kNL]), uni(cnt[c3 * kNL + 1]), uni(cnt[c3 * kNL + 2]),
                 uni(cnt[c3 * kNL + 3])};
    const Prefix4 pre(n);
    if (pre.total == 0 || pre.total > cap || level > g.N) break;  // at most N levels
    if (kDir == kDirRelabel && tid == 0 && level < kLvlHist) g.ctl->lvl_nf[level] = pre.total;
    const lds_int* const cbuf = buf + cp * kNL * kLoopCap;
    lds_int* const nbuf = buf + np * kNL * kLoopCap;
    lds_int* const ncnt = cnt + n3 * kNL;
    const int lvl = level + 1;
    uint32_t nbytes = 0;
    auto append = [&](int v, uint32_t word) {
      const int k = list_of_word(g, v, word);
      const int pos = lds_add(ncnt + k, 1);
      if (pos < kLoopCap) nbuf[k * kLoopCap + pos] = v;
      else g.list[np][k][pos] = v;
    };
    // claim v: label it (relabel) or stamp it, and list it if this was first
    auto claim = [&](int v) {
      bool first;
      if (kDir == kDirRelabel) first = atomicCAS(&g.d[v], g.N, lvl) == g.N;
      else first = atomicExch(&g.stamp[v], ep) != ep;
      const uint32_t word = g.bigbits[v >> 5];
      if (first) {
        if (kDir == kDirRelabel) {
          atomicOr(&g.seen[v >> 5], 1u << (v & 31));
          if (g.lev) g.lev[v] = 2;
        }
        append(v, word);
        if (kGrow && v < g.V) {
          grow->fresh[lds_add(grow->nfresh, 1)] = v;
          __hip_atomic_fetch_add(grow->weight, (unsigned long long)grow->cw[v], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    };
    for (int first = 0; first < pre.total; first += blockDim.x) {
      const int nt = min((int)blockDim.x, pre.total - first);
      int deg = 0, beg = 0, v = 0;
      if (tid < nt) {
        const int i = first + tid, k = pre.list_of(i), j = i - pre.start[k];
        v = j < kLoopCap ? (int)cbuf[k * kLoopCap + j] : g.list[cp][k][j];
        if (v < g.V) {
          beg = g.vtx_off[v];
          deg = g.vtx_off[v + 1] - beg;
        } else {
          const int e = (v - g.NB) >> 1;
          beg = g.net_off[e];
          deg = g.net_off[e + 1] - beg + 1;  // arc 0 is the bridge
        }
      }
      int incl = deg;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      if (lane == kWave - 1) wsum[wid] = incl;
      __syncthreads();
      // the count of the level after next: last read before this barrier
      if (tid < kNL) cnt[z3 * kNL + tid] = 0;
      int base = 0, A = 0;
      for (int w = 0; w < nw; ++w) {
        const int t = wsum[w];
        if (w < wid) base += t;
        A += t;
      }
      t_node[tid] = v;
      t_beg[tid] = beg;
      t_off[tid] = base + incl - deg;
      __syncthreads();
      // kArcs arcs a thread at a time, their loads in flight together: the
      // entry by bisection, the arc's other end, its label or stamp and flow,
      // then the claims
      const int* const mark = kDir == kDirRelabel ? g.d : g.stamp;
      const int unreached = g.N;
      int top = 1;
      while (2 * top < nt) top *= 2;
      for (int a0 = tid; a0 < A; a0 += kArcs * (int)blockDim.x) {
        int lo[kArcs], j[kArcs], t[kArcs];
        int2 fp[kArcs], st[kArcs];
        bool in_range[kArcs], vtx[kArcs];
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
          lo[q] = 0;
          in_range[q] = a0 + q * (int)blockDim.x < A;
        }
        for (int step = top; step > 0; step >>= 1)  // t_off[lo] <= a
#pragma unroll
          for (int q = 0; q < kArcs; ++q) {
            const int c = lo[q] + step;
            if (c < nt && t_off[c] <= a0 + q * (int)blockDim.x) lo[q] = c;
          }
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
          const int x = t_node[lo[q]];
          j[q] = a0 + q * (int)blockDim.x - t_off[lo[q]];
          vtx[q] = x < g.V;
          lo[q] = t_beg[lo[q]] + j[q];  // the arc's place, from here on
          t[q] = x;
        }
        // a vertex's arc: net and slot in fp; a bridge: fb and w in fp; a pin
        // arc: the vertex in st.x, the flows in fp
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
          if (!in_range[q]) continue;
          if (vtx[q]) {
            fp[q] = g.vinc[lo[q]];
          } else if (j[q] == 0) {
            const int e = (t[q] - g.NB) >> 1;
            fp[q] = make_int2(g.fb[e], g.w[e]);
          } else {
            st[q].x = g.pin_v[lo[q] - 1];
            fp[q] = *reinterpret_cast<const int2*>(g.fpin + 2 * (lo[q] - 1));
          }
        }
        int cap_or_role[kArcs];  // w(e) where it is needed, a pin's role
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
          if (!in_range[q]) continue;
          if (vtx[q]) {
            const int2 ep = fp[q];
            t[q] = g.NB + 2 * ep.x;  // e_in; e_out = t + 1
            fp[q] = *reinterpret_cast<const int2*>(g.fpin + 2 * ep.y);
            st[q] = *reinterpret_cast<const int2*>(mark + t[q]);
            if (kDir != kDirSource) cap_or_role[q] = g.w[ep.x];
            nbytes += 24;
          } else if (j[q] == 0) {
            const bool in = ((t[q] - g.NB) & 1) == 0;
            st[q].x = mark[in ? t[q] + 1 : t[q] - 1];
            nbytes += 8;
          } else {
            const int u = st[q].x;
            st[q] = make_int2(u, mark[u]);
            const bool in = ((t[q] - g.NB) & 1) == 0;
            if (kDir == kDirSource) cap_or_role[q] = in ? g.w[(t[q] - g.NB) >> 1] : g.role[u];
            if (kDir == kDirSink) cap_or_role[q] = g.role[u];
            nbytes += 12;
          }
        }
#pragma unroll
        for (int q = 0; q < kArcs; ++q) {
          if (!in_range[q]) continue;
          ++narcs;
          if (vtx[q]) {
            const bool o1 = kDir == kDirRelabel ? st[q].x == unreached : st[q].x != ep;
            const bool o2 = kDir == kDirRelabel ? st[q].y == unreached : st[q].y != ep;
            bool c1, c2;
            if (kDir == kDirSource) {  // x -> e_in uncapped, x -> e_out reverse
              c1 = o1;
              c2 = o2 && fp[q].y > 0;
            } else {  // e_out -> x infinite, e_in -> x reverse
              c1 = o1 && cap_or_role[q] - fp[q].x > 0;
              c2 = o2;
            }
            if (c1) claim(t[q]);
            if (c2) claim(t[q] + 1);
            continue;
          }
          const bool in = ((t[q] - g.NB) & 1) == 0;
          if (j[q] == 0) {
            // into e_in from e_out by fb, into e_out from e_in by w - fb; the
            // forward search the other way
            const bool by_fb = in == (kDir != kDirSource);
            const bool open = kDir == kDirRelabel ? st[q].x == unreached : st[q].x != ep;
            if ((by_fb ? fp[q].x > 0 : fp[q].x < fp[q].y) && open) claim(in ? t[q] + 1 : t[q] - 1);
            continue;
          }
          const int u = st[q].x;
          const bool open = kDir == kDirRelabel ? st[q].y == unreached : st[q].y != ep;
          bool arc;
          if (kDir == kDirRelabel) {
            arc = (in ? fp[q].x : fp[q].y) > 0;
          } else if (kDir == kDirSource) {
            // e_in -> u reverse; e_out -> u infinite, into free vertices only
            arc = in ? cap_or_role[q] - fp[q].x > 0 : cap_or_role[q] == 0;
            if (!in && cap_or_role[q] == 2) hit_sink = true;
          } else {  // u -> e_in uncapped, u -> e_out by flow
            arc = in || fp[q].y > 0;
            if (arc && cap_or_role[q] == 1) {
              hit_source = true;
              continue;
            }
          }
          if (open && arc) claim(u);
          // the growing side's neighbours: pins of e_in (source side) or of
          // e_out (sink side) that it does not reach
          if (kGrow && open && !arc && in == (kDir == kDirSource) && st[q].y != grow->other)
            atomicOr(&grow->next[u >> 5], 1u << (u & 31));
        }
      }
      __syncthreads();  // the tile is rewritten, the next level's list complete
    }
    nbytes_all += nbytes;
  }
  // the level reached back to the global lists
  const int c3 = level % 3, cp = level & 1;
  if (kGrow) {
    if (hit_sink) atomicOr(&g.ctl->err, ERR_SINK_REACHED);
    if (hit_source) atomicOr(&g.ctl->err, ERR_SOURCE_REACHED);
    grow->nbytes += nbytes_all;
    grow->narcs += narcs;
    grow->left = uni(cnt[c3 * kNL]) + uni(cnt[c3 * kNL + 1]) + uni(cnt[c3 * kNL + 2]) +
                 uni(cnt[c3 * kNL + 3]);
    if (grow->left == 0) return level - level0;
  }
#pragma unroll
  for (int k = 0; k < kNL; ++k) {
    const int c = min((int)cnt[c3 * kNL + k], kLoopCap);
    for (int i = tid; i < c; i += blockDim.x)
      g.list[cp][k][i] = buf[(cp * kNL + k) * kLoopCap + i];
  }
  if (tid < 3 * kNL)
    g.ctl->bcnt[tid / kNL][tid % kNL] = tid / kNL == c3 ? (int)cnt[tid] : 0;
  if (kGrow) return level - level0;
  if (hit_sink) atomicOr(&g.ctl->err, ERR_SINK_REACHED);
  if (hit_source) atomicOr(&g.ctl->err, ERR_SOURCE_REACHED);
  block_add_u64(&g.ctl->bytes[kc], nbytes_all + 12ull * narcs, &g.ctl->items[kc], narcs);
  return level - level0;
}

// Clear the BFS counters and the FlowCutter side weights (own launch: the
// next phase appends to the counters).
__device__ void phase_reset_bfs(const Dev& g) {
  if (threadIdx.x == 0) {
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < kNL; ++k) g.ctl->bcnt[i][k] = 0;
    g.ctl->side_weight[0] = 0ull;
    g.ctl->side_weight[1] = 0ull;
    for (int i = 0; i < 5; ++i) g.ctl->pierce[i] = kInf;
  }
}

// Clear the frontier counters of all three round slots (a solve that starts
// from the labels it has, without a global relabel, gathers into one).
__device__ void phase_clear_frontiers(const Dev& g) {
  if (threadIdx.x == 0)
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < kNL; ++k) g.ctl->fcnt[i][k] = 0;
}

// One seed vertex p (already stamped by the caller) as BFS level 0.  The
// BFS counters must be clear (phase_reset_bfs).
__device__ void phase_seed_vertex(const Dev& g, int p) {
  if (threadIdx.x == 0) {
    const int k = list_of(g, p);
    g.list[0][k][0] = p;
    g.ctl->bcnt[0][k] = 1;
  }
}

// Bulk piercing (paragraph "Bulk Piercing"): flag[u] = 1 for every augmenting
// candidate of side `side` -- a pin of a net cut by that side's bipartition
// that lies on the opposite side's reachable set and is not a terminal yet.
// Thread per net; flags are cleared by the caller.
// Whether net e is cut by (S_r, V - S_r) (.x) and by (V - T_r, T_r) (.y),
// read from the stamps of its two nodes (e_in, e_out adjacent: one 8-byte
// load).  In the uncapped network every pin reaches e_in and e_out reaches
// every pin, so a non-empty net has a pin in S_r iff e_in is in S_r and all
// its pins in S_r when e_out is; it has a pin in T_r iff e_out is in T_r and
// all its pins in T_r when e_in is.  A net flagged here may still have all
// its pins on one side (its bridge blocks); the pin scans that follow then
// find no pin outside, so the flag changes nothing.
struct bool2_t {
  bool a, b;
};

__device__ __forceinline__ bool2_t net_cut_flags(const Dev& g, int e, int ep_s, int ep_t) {
  const int2 st = reinterpret_cast<const int2*>(g.stamp + g.NB)[e];
  return bool2_t{st.x == ep_s && st.y != ep_s, st.y == ep_t && st.x != ep_t};
}

// Flags the pins of nets cut by side `side`'s bipartition that lie on the
// other side and are not its terminals yet (the augmenting candidates of a
// bulk pierce).  Lanes take one net each; the nets that are cut are then
// scanned by the whole wave, one after another, 64 pins at a time.
__device__ void phase_fc_mark_augmenting(const Dev& g, int side, int ep_s, int ep_t,
                                         uint8_t* flag, int t0, int tstride) {
  const int lane = lane_id();
  const int other = side == 0 ? ep_t : ep_s;
  const int other_role = side == 0 ? 2 : 1;
  for (int base = t0 - lane; base < g.E; base += tstride) {
    const int e = base + lane;
    bool cut = false;
    if (e < g.E) {
      const bool2_t c = net_cut_flags(g, e, ep_s, ep_t);
      cut = side == 0 ? c.a : c.b;
    }
    unsigned long long m = __ballot(cut);
    while (m) {
      const int b = __builtin_ctzll(m);
      m &= m - 1;
      const int en = base + b;
      const int beg = g.net_off[en], end = g.net_off[en + 1];
      for (int p = beg + lane; p < end; p += 64) {
        const int u = g.pin_v[p];
        if (g.stamp[u] == other && g.role[u] != other_role) flag[u] = 1;
      }
    }
  }
}

// Exclusive prefix of per-thread 0/1 values over a workgroup (blockDim a
// multiple of 64, at most 1024); *total gets the workgroup's sum.
__device__ int block_rank(int f, int* total) {
  __shared__ int wsum[17];
  const int lane = lane_id(), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const unsigned long long m = __ballot(f != 0);
  const int below = __popcll(m & lanemask_lt());
  if (lane == 0) wsum[wid] = __popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int i = 0; i < nw; ++i) {
      const int t = wsum[i];
      wsum[i] = run;
      run += t;
    }
    wsum[nw] = run;
  }
  __syncthreads();
  const int r = wsum[wid] + below;
  *total = wsum[nw];
  __syncthreads();
  return r;
}

// Flag counts per workgroup tile of blockDim vertices.
__device__ void phase_count_flags(const uint8_t* flag, int V, int32_t* counts) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  int total = 0;
  block_rank(v < V && flag[v] != 0, &total);
  if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// Stamp with ep the k flagged vertices of smallest id; offsets[b] = flags
// before tile b.
__device__ void phase_select_flags(Dev g, const uint8_t* flag, int V, const int32_t* offsets,
                                   int k, int ep) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  const bool f = v < V && flag[v] != 0;
  int total = 0;
  const int r = offsets[blockIdx.x] + block_rank(f, &total);
  if (f && r < k) g.stamp[v] = ep;
}

// Vertex bitmap of a BFS: 1 where the vertex carries stamp ep (when
// invert, 1 where it does not).
__device__ void phase_side_out(const Dev& g, int ep, bool invert, uint8_t* vside, int t0,
                               int tstride) {
  if (t0 == 0) {
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < kNL; ++k) g.ctl->bcnt[i][k] = 0;
  }
  for (int v = t0; v < g.V; v += tstride) vside[v] = (uint8_t)((g.stamp[v] == ep) != invert);
}

// ---------------------------------------------------------------------------
// FlowCutter steps (paper, section "Flow-Based Refinement": algorithm
// "FlowCutter Core", paragraphs "Piercing", "Sink-Side Piercing" and
// "Maintain Distance Labels").  S_r carries stamp ep_s (sources included),
// T_r stamp ep_t (sinks included).
// ---------------------------------------------------------------------------

// Weights c(S_r) and c(T_r), and pierce[2] = the smallest vertex outside
// both (the counters are cleared by phase_reset_bfs).
__device__ void phase_fc_weights(const Dev& g, const int32_t* cw, int ep_s, int ep_t, int t0,
                                 int tstride) {
  unsigned long long ws = 0, wt = 0;
  int first_free = kInf;
  for (int v = t0; v < g.V; v += tstride) {
    const int st = g.stamp[v];
    if (st == ep_s) ws += (unsigned long long)cw[v];
    else if (st == ep_t) wt += (unsigned long long)cw[v];
    else first_free = min(first_free, v);
  }
  block_add_u64(&g.ctl->side_weight[0], ws, &g.ctl->side_weight[1], wt);
  block_min_i32(&g.ctl->pierce[2], first_free, &g.ctl->pierce[2], kInf);
}

// Piercing candidates of the side that is pierced next, the lighter one
// (s = 0 when c(S_r) <= c(T_r), from the weights phase_fc_weights summed
// before): pierce[3s] = the smallest vertex outside S_r and T_r on a net cut
// by side s's bipartition; pierce[3s + 1] = the smallest vertex of the
// opposite reachable set on such a net that is not a terminal yet.  The
// second is only used when no vertex is outside both sets (pierce[2] =
// kInf), so only then is it searched, and then the first has no candidate.
// Vertex order, with the uncapped network's reachability: a vertex outside
// S_r lies on a net cut by (S_r, V - S_r) exactly when one of its nets has
// e_in in S_r (were e_out in S_r, its pins would be too); one outside T_r
// lies on a net cut by (V - T_r, T_r) exactly when one of its nets has e_out
// in T_r.  Workgroups take chunks of blockDim vertices in increasing order
// (chunk b, b + gridDim, ...) and stop at the first chunk that starts above
// the best candidate found so far: a vertex of that chunk or a later one
// cannot be the smallest, and most free vertices next to a side are found
// in the first chunks.
__device__ void phase_fc_pick(const Dev& g, int ep_s, int ep_t) {
  __shared__ int best_sh;
  const unsigned long long cs = ld_vol64(&g.ctl->side_weight[0]);
  const unsigned long long ct = ld_vol64(&g.ctl->side_weight[1]);
  const int side = cs <= ct ? 0 : 1;
  const bool aug = ld_vol(&g.ctl->pierce[2]) == kInf;
  const int want = side == 0 ? ep_s : ep_t;  // stamp of the net node that makes a net cut
  const int opp = side == 0 ? ep_t : ep_s;
  const int opp_role = side == 0 ? 2 : 1;
  int32_t* const out = &g.ctl->pierce[3 * side + (aug ? 1 : 0)];
  const int nchunks = (g.V + (int)blockDim.x - 1) / (int)blockDim.x;
  for (int c = blockIdx.x; c < nchunks; c += gridDim.x) {
    const int u = c * (int)blockDim.x + (int)threadIdx.x;
    int found = kInf;
    if (u < g.V) {
      const int st = g.stamp[u];
      const bool look = aug ? (st == opp && g.role[u] != opp_role) : (st != ep_s && st != ep_t);
      if (look) {
        const int end = g.vtx_off[u + 1];
        for (int i = g.vtx_off[u]; i < end; ++i) {
          if (g.stamp[g.NB + 2 * g.vinc[i].x + side] == want) {
            found = u;
            break;
          }
        }
      }
    }
    block_min_i32(out, found, out, kInf);
    if (threadIdx.x == 0) best_sh = ld_vol(out);
    __syncthreads();
    const int best = best_sh;
    __syncthreads();
    if ((long long)(c + gridDim.x) * blockDim.x > (long long)best) break;
  }
}

// Every free vertex with stamp ep_s becomes a source.  The flows of its
// pin arcs are cancelled (flow(u, e_in) back out of e_in's excess, flow
// (e_out, u) back into e_out's excess), and a net that gains its first
// source pin receives w(e) through its contracted source arc, so the state
// stays a preflow of the new network with the same flow value.  The vertex
// takes the sources' label N + 1.  No residual arc between non-terminal
// nodes appears (the arcs that change all start or end at the new source),
// so the other labels stay valid and the next solve may start from them
// (paragraph "Maintain Distance Labels").
// Incidence i (net e) of a vertex u that becomes a source: the flows of u's
// pin arcs are cancelled -- e_in loses the flow u sent it and, when e gets its
// first source pin, gains w(e) from the contracted source arc; e_out keeps as
// excess the flow it sent to u.  Returns e and the flow returned to e_out.
__device__ __forceinline__ int2 cancel_source_pin(const Dev& g, int i) {
  const int2 ep = g.vinc[i];
  const int e = ep.x;
  const int we = g.w[e];
  const int fin = we - g.fpin[2 * ep.y];
  const int fout = g.fpin[2 * ep.y + 1];
  int add_in = -fin;
  const int old = atomicOr(&g.nflag[e], 1);
  if (!(old & 1)) add_in += we;
  if (add_in) atomicAdd(&g.x[g.NB + 2 * e], add_in);
  if (fout) atomicAdd(&g.x[g.NB + 2 * e + 1], fout);
  g.fpin[2 * ep.y] = we;
  g.fpin[2 * ep.y + 1] = 0;
  return make_int2(e, fout);
}

__device__ void phase_pierce_sources(const Dev& g, int ep_s, int t0, int tstride) {
  for (int v = t0; v < g.V; v += tstride) {
    if (g.role[v] != 0 || g.stamp[v] != ep_s) continue;
    g.role[v] = 1;
    g.d[v] = g.N + 1;  // a source's label: nothing is pushed into it
    for (int i = g.vtx_off[v]; i < g.vtx_off[v + 1]; ++i) cancel_source_pin(g, i);
  }
}

// The source pierce above that also lists the seeds of the source side's
// growth (a pierce that avoids augmenting paths keeps S_r, which the growth
// extends): converting a vertex gives e_in of each of its nets a source arc
// and, where flow came back, e_out excess; no other node gains excess or a
// source arc, and every node that held them before is already in S_r.  Each
// such net node not yet stamped ep_s is stamped and listed once (exchange on
// the stamp), so level 0 is exactly what the seed sweep over all nodes would
// find.  Thread per vertex in tiles of blockDim; level 0's count and lists
// must be empty.
__device__ void phase_pierce_sources_seed(const Dev& g, int ep_s, int tile0, int tstride,
                                          lds_int* lds) {
  const BlockQ q = bq_bind(lds, g.ctl->bcnt[0], g.list[0]);
  const int ntiles = (g.V + (int)blockDim.x - 1) / (int)blockDim.x;
  for (int tile = tile0; tile < ntiles; tile += tstride) {
    const int v = tile * (int)blockDim.x + (int)threadIdx.x;
    int beg = 0, end = 0;
    if (v < g.V && g.role[v] == 0 && g.stamp[v] == ep_s) {
      g.role[v] = 1;
      g.d[v] = g.N + 1;
      beg = g.vtx_off[v];
      end = g.vtx_off[v + 1];
    }
    for (int i = beg; i < end; ++i) {
      const int2 ef = cancel_source_pin(g, i);
      const int ein = g.NB + 2 * ef.x;
      qpush(g, q, ein, stamp_first(g, ein, ep_s));
      qpush(g, q, ein + 1, ef.y > 0 && stamp_first(g, ein + 1, ep_s));
    }
    bq_tile_end(q, q.cap / 2);
  }
  bq_flush(q);
}

// Every free vertex with stamp ep_t becomes a sink; excess it holds joins
// the flow value (paragraph "Sink-Side Piercing").
__device__ void phase_pierce_sinks(const Dev& g, int ep_t, int t0, int tstride) {
  unsigned long long gained = 0;
  for (int v = t0; v < g.V; v += tstride) {
    if (g.role[v] != 0 || g.stamp[v] != ep_t) continue;
    g.role[v] = 2;
    const int xv = g.x[v];
    if (xv > 0) {
      gained += (unsigned long long)xv;
      g.x[v] = 0;
    }
    for (int i = g.vtx_off[v]; i < g.vtx_off[v + 1]; ++i) atomicOr(&g.nflag[g.vinc[i].x], 2);
  }
  block_add_u64(&g.ctl->flow, gained);
}

// ---------------------------------------------------------------------------
// FlowCutter iterations inside one workgroup
//
// An iteration that pierces a vertex outside S_r and T_r changes no flow: it
// grows the side pierced last from a few seeds, weighs the sides, picks a
// vertex and pierces.  Each of these steps touches some tens of nodes, so as
// launches (eight and a round trip an iteration) it is all start-up and gaps.
// One workgroup runs them one after another here, until an iteration needs
// something else: an augmenting path, an end of the run, or work for more
// than one workgroup.  The steps give what the device-wide ones give: weights
// are sums, kept up to date by the vertices a growth reaches; a pick is the
// smallest vertex of its kind, found in a bitmap of the vertices next to the
// side, in which every growth sets the pins of the net nodes it reaches; a
// pierce turns the vertices reached since the side's last pierce into
// terminals, from a list instead of a sweep over all vertices.  Bound by the
// latency of some 25 dependent accesses and as many barriers an iteration: 17
// us on a region of 50k vertices and 370k pins, against 41 us of kernels and
// 56 us in all with launches; a run of 3,500 iterations 193 -> 63 ms.
// ---------------------------------------------------------------------------

// The bits of the free pins of every net cut by a side (net_cut_flags), into
// cleared bitmaps.  Lanes take one net each; the cut ones are then scanned by
// the whole wave.
__device__ void phase_fc_next(const Dev& g, int ep_s, int ep_t, uint32_t* next_s, uint32_t* next_t,
                              int t0, int tstride) {
  const int lane = lane_id();
  for (int base = t0 - lane; base < g.E; base += tstride) {
    const int e = base + lane;
    bool2_t cut{false, false};
    if (e < g.E) cut = net_cut_flags(g, e, ep_s, ep_t);
    const unsigned long long ms = __ballot(cut.a);
    for (unsigned long long m = ms | __ballot(cut.b); m; m &= m - 1) {
      const int k = __ffsll(m) - 1;
      const bool of_s = (ms >> k) & 1ull;
      const bool of_t = __shfl((int)cut.b, k);
      const int end = g.net_off[base + k + 1];
      for (int i = g.net_off[base + k] + lane; i < end; i += kWave) {
        const int u = g.pin_v[i];
        const int st = g.stamp[u];
        if (st == ep_s || st == ep_t) continue;
        if (of_s) atomicOr(&next_s[u >> 5], 1u << (u & 31));
        if (of_t) atomicOr(&next_t[u >> 5], 1u << (u & 31));
      }
    }
  }
}

enum FcExit {
  kFcGrow = 1,    // a growth reached a level too large for the workgroup
  kFcPick = 2,    // no vertex is outside both sides
  kFcDecide = 3,  // the iteration stands as if weighed and picked device-wide
};

struct FcStep {  // one finished iteration
  long long cs, ct;
  int32_t p, pad;
};

struct FcLoop {
  const int32_t* cw;
  int32_t* fresh[2];   // vertices of S_r and T_r that are not terminals yet
  int32_t nfresh[2];   // how many; -1: not listed, they are found by their stamps
  uint32_t* next[2];   // vertices next to S_r and T_r (bits)
  FcStep* steps;
  uint8_t* best;       // most balanced side so far (most_balanced)
  long long cs, ct;    // weights before the pending growth
  long long max_src, max_snk, total, best_heavier;
  int32_t ep_s, ep_t;
  int32_t side, p;     // pending growth; level 0 of side 0 is in the global lists
  int32_t lo;          // no vertex below is outside both sides
  int32_t most_balanced, max_iters, cap;
};

constexpr int kFcLanes = 16;   // lanes per vertex of a pierce
constexpr int kFcWide = 512;   // more vertices to pierce are left to a device-wide pierce
constexpr int kFcWords = kWgBfsWords + kBfsTile + 32;

__device__ void fc_loop(const Dev& g, FcLoop a, lds_int* lds, lds_u64* weight) {
  lds_int* const buf = lds;
  lds_int* const cnt = lds + kWgBfsWords - 3 * kNL;  // as wg_bfs lays them out
  lds_int* const cand = lds + kWgBfsWords;           // a chunk's vertices outside both sides
  lds_int* const wcnt = cand + kBfsTile;             // per wave
  lds_int* const best = wcnt + 16;
  lds_int* const nfresh = wcnt + 17;                 // [2]
  const int tid = threadIdx.x, lane = lane_id(), wid = uni(tid >> 6), nw = blockDim.x >> 6;
  const int group = tid / kFcLanes, glane = tid % kFcLanes, ngroups = blockDim.x / kFcLanes;
  Growth gr{a.cw, nullptr, nullptr, weight, nullptr, 0};
  // Stamps and bits are set by atomics, and what plain loads of the growths
  // brought into the vector cache may be older.
  auto now = [](auto* at) {
    return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  int listed = (a.nfresh[0] >= 0 ? 1 : 0) | (a.nfresh[1] >= 0 ? 2 : 0);  // bit per side
  int side = a.side, p = a.p, lo = a.lo, levels = 0, iter = 0, why = 0;
  int first_free = kInf, pick = kInf;
  unsigned long long gained = 0;
  if (tid < 2) nfresh[tid] = max(0, tid == 0 ? a.nfresh[0] : a.nfresh[1]);
  if (tid < 3 * kNL) cnt[tid] = tid < kNL && side == 0 ? ld_vol(&g.ctl->bcnt[0][tid]) : 0;
  __syncthreads();
  if (side == 0) {
#pragma unroll
    for (int k = 0; k < kNL; ++k)
      for (int i = tid; i < min((int)cnt[k], kLoopCap); i += blockDim.x)
        buf[k * kLoopCap + i] = g.list[0][k][i];
  } else if (tid == 0) {
    const int k = list_of(g, p);
    buf[k * kLoopCap] = p;
    cnt[k] = 1;
  }
  for (;; ++iter) {
    // ---- growth of `side`
    if (tid == 0) *weight = 0ull;
    __syncthreads();
    gr.fresh = side == 0 ? a.fresh[0] : a.fresh[1];
    gr.nfresh = nfresh + side;
    gr.next = side == 0 ? a.next[0] : a.next[1];
    gr.other = side == 0 ? a.ep_t : a.ep_s;
    const int lv = side == 0 ? wg_bfs<kDirSource, true, 2>(g, 0, a.cap, a.ep_s, 0, lds, &gr)
                             : wg_bfs<kDirSink, true, 2>(g, 0, a.cap, a.ep_t, 0, lds, &gr);
    if (gr.left > 0) {
      if (tid == 0) g.ctl->loop_levels = lv;
      listed &= ~(1 << side);  // the rest of the growth is not listed
      why = kFcGrow;
      break;
    }
    levels += lv;
    const long long grown = (long long)*weight + a.cw[p];
    if (side == 0) a.cs += grown;
    else a.ct += grown;
    // ---- pick, for the lighter side: the words of its bitmap from `lo` on that
    // are not empty, in order, then a lane per bit
    side = a.cs <= a.ct ? 0 : 1;
    const int want = side == 0 ? a.ep_s : a.ep_t;
    uint32_t* const next = side == 0 ? a.next[0] : a.next[1];
    const int words = (g.V + 31) >> 5;
    first_free = kInf;
    pick = kInf;
    if (tid == 0) *best = kInf;
    // entries of a chunk in order: their number, for those with `in` the place
    auto ordered = [&](bool in, int value) {
      const unsigned long long m = __ballot(in);
      if (lane == 0) wcnt[wid] = __popcll(m);
      __syncthreads();
      int before = 0, n = 0;
      for (int w = 0; w < nw; ++w) {
        const int t = wcnt[w];
        if (w < wid) before += t;
        n += t;
      }
      if (in) cand[before + __popcll(m & lanemask_lt())] = value;
      __syncthreads();
      return uni(n);
    };
    for (int base = lo >> 5; base < words && pick == kInf; base += blockDim.x) {
      const int w = base + tid;
      const int n = ordered(w < words && now(next + w) != 0u, w);
      for (int i0 = 0; i0 < n && pick == kInf; i0 += (int)blockDim.x / 32) {
        const int i = i0 + tid / 32;
        const int at = i < n ? (int)cand[i] : 0;
        const uint32_t bits = i < n ? now(next + at) : 0u;
        const int u = 32 * at + (tid & 31);
        bool out = false;
        if ((bits >> (tid & 31)) & 1u) {
          const int st = now(g.stamp + u);
          out = st != a.ep_s && st != a.ep_t;
        }
        if (out) __hip_atomic_fetch_min(best, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const uint32_t left = (uint32_t)(__ballot(out) >> (lane & 32));
        if ((tid & 31) == 0 && left != bits) next[at] = left;  // the others are in a side now
        __syncthreads();
        pick = uni(*best);
        __syncthreads();
      }
    }
    for (; pick == kInf && first_free == kInf && lo < g.V; lo += blockDim.x) {
      const int u = lo + tid;
      const int st = u < g.V ? now(g.stamp + u) : a.ep_s;
      const int n = ordered(st != a.ep_s && st != a.ep_t, u);
      if (n > 0) first_free = uni(cand[0]);
      if (n > 0) break;
    }
    if (first_free != kInf) lo = first_free;
    if (pick == kInf && first_free == kInf) {
      why = kFcPick;
      break;
    }
    // ---- what the iteration does next
    const bool bal0 = a.cs <= a.max_src && a.total - a.cs <= a.max_snk;
    const bool bal1 = a.total - a.ct <= a.max_src && a.ct <= a.max_snk;
    if ((!a.most_balanced && (bal0 || bal1)) || iter + 1 == a.max_iters) {
      why = kFcDecide;
      break;
    }
    int32_t* const fresh = side == 0 ? a.fresh[0] : a.fresh[1];
    if (!((listed >> side) & 1)) {
      if (tid == 0) nfresh[side] = 0;
      __syncthreads();
      for (int v = tid; v < g.V; v += blockDim.x)
        if (now(g.stamp + v) == want && g.role[v] == 0) fresh[lds_add(nfresh + side, 1)] = v;
      __syncthreads();
      listed |= 1 << side;
    }
    int n = uni(nfresh[side]);
    if (n > kFcWide) {
      why = kFcDecide;
      break;
    }
    if (a.most_balanced && (bal0 || bal1))
      for (int kind = 0; kind < 2; ++kind) {
        if (!(kind == 0 ? bal0 : bal1)) continue;
        const long long src = kind == 0 ? a.cs : a.total - a.ct;
        const long long heavier = max(src, a.total - src);
        if (a.best_heavier >= 0 && heavier >= a.best_heavier) continue;
        a.best_heavier = heavier;
        const int ep = kind == 0 ? a.ep_s : a.ep_t;
        for (int v = tid; v < g.V; v += blockDim.x)
          a.best[v] = (uint8_t)((now(g.stamp + v) == ep) != (kind != 0));
      }
    p = pick != kInf ? pick : first_free;
    if (tid == 0) {
      a.steps[iter] = FcStep{a.cs, a.ct, p, 0};
      g.stamp[p] = want;
      fresh[n] = p;
    }
    if (tid < 3 * kNL) cnt[tid] = 0;
    ++n;
    __syncthreads();  // the list is complete, the stamps have been read
    // ---- pierce
    for (int i = group; i < n; i += ngroups) {
      const int v = fresh[i];
      if (g.role[v] != 0) continue;
      const int end = g.vtx_off[v + 1];
      if (side == 0) {
        if (glane == 0) {
          g.role[v] = 1;
          g.d[v] = g.N + 1;
        }
        for (int j = g.vtx_off[v] + glane; j < end; j += kFcLanes) {
          const int2 ef = cancel_source_pin(g, j);
          const int ein = g.NB + 2 * ef.x;
          auto seed = [&](int node) {
            const int k = list_of(g, node);
            const int pos = lds_add(cnt + k, 1);
            if (pos < kLoopCap) buf[k * kLoopCap + pos] = node;
            else g.list[0][k][pos] = node;
          };
          if (stamp_first(g, ein, a.ep_s)) seed(ein);
          if (ef.y > 0 && stamp_first(g, ein + 1, a.ep_s)) seed(ein + 1);
        }
      } else {
        if (glane == 0) {
          g.role[v] = 2;
          const int xv = g.x[v];
          if (xv > 0) {
            gained += (unsigned long long)xv;
            g.x[v] = 0;
          }
        }
        for (int j = g.vtx_off[v] + glane; j < end; j += kFcLanes)
          atomicOr(&g.nflag[g.vinc[j].x], 2);
      }
    }
    if (tid == 0) {
      nfresh[side] = 0;
      if (side == 1) {
        const int k = list_of(g, p);
        buf[k * kLoopCap] = p;
        cnt[k] = 1;
      }
    }
  }
  __syncthreads();
  if (why != kFcGrow && tid < 3 * kNL) g.ctl->bcnt[tid / kNL][tid % kNL] = 0;
  if (tid == 0) {
    Ctl* const c = g.ctl;
    c->side_weight[0] = (unsigned long long)a.cs;
    c->side_weight[1] = (unsigned long long)a.ct;
    for (int i = 0; i < 5; ++i) c->pierce[i] = kInf;
    c->pierce[2] = first_free != kInf || why == kFcPick ? first_free : lo;  // from here on
    c->pierce[3 * side] = pick;
    c->fc_done = iter;
    c->fc_why = why;
    c->fc_side = side;
    c->fc_levels = levels;
    for (int i = 0; i < 2; ++i) c->fc_new[i] = (listed >> i) & 1 ? (int)nfresh[i] : -1;
  }
  block_add_u64(&g.ctl->flow, gained);
  block_add_u64(&g.ctl->bytes[KC_LOOP_BFS], gr.nbytes + 12ull * gr.narcs, &g.ctl->items[KC_LOOP_BFS],
                gr.narcs);
}

// Stamp the given vertices with ep; a vertex that is a terminal of kind
// `forbidden` is reported as ERR_PIERCE_TERMINAL.
__device__ void phase_mark(const Dev& g, const int32_t* vs, int n, int ep, int forbidden, int t0,
                           int tstride) {
  for (int i = t0; i < n; i += tstride) {
    const int v = vs[i];
    if (g.role[v] == forbidden) atomicOr(&g.ctl->err, ERR_PIERCE_TERMINAL);
    else if (g.role[v] == 0) g.stamp[v] = ep;
  }
}

// Debug: preflow feasibility (excess = inflow - outflow >= 0, capacities) and
// label validity on every residual arc of the capped network, after a
// completed round.  Thread per vertex / net / pin.
__device__ __forceinline__ long long excess_of(const Dev& g, int v) {
  return (long long)g.x[v] + g.dx[0][v] + g.dx[1][v];
}

__device__ void phase_check(const Dev& g, int t0, int tstride) {
  const int n = max(g.P, max(g.E, g.V));
  bool bad = false;
  for (int i = t0; i < n; i += tstride) {
    if (i < g.V) {
      const int r = g.role[i];
      if (r == 0) {
        long long s = 0;
        for (int j = g.vtx_off[i]; j < g.vtx_off[i + 1]; ++j) {
          const int2 ep = g.vinc[j];
          s += (long long)g.fpin[2 * ep.y + 1] - (long long)(g.w[ep.x] - g.fpin[2 * ep.y]);
        }
        if (s != excess_of(g, i) || s < 0) bad = true;
      }
    }
    if (i < g.E) {
      const int we = g.w[i], fbv = g.fb[i];
      if (fbv < 0 || fbv > we) bad = true;
      long long sin = (g.nflag[i] & 1) ? we : 0, sout = 0;
      for (int p = g.net_off[i]; p < g.net_off[i + 1]; ++p) {
        sin += we - g.fpin[2 * p];
        sout += g.fpin[2 * p + 1];
      }
      const long long xin = excess_of(g, g.NB + 2 * i), xout = excess_of(g, g.NB + 2 * i + 1);
      if (sin - fbv != xin || fbv - sout != xout || xin < 0 || xout < 0) bad = true;
      const int din = g.d[g.NB + 2 * i], dout = g.d[g.NB + 2 * i + 1];
      if (din < g.N && fbv < we && din > dout + 1) bad = true;
      if (dout < g.N && fbv > 0 && dout > din + 1) bad = true;
    }
    if (i < g.P) {
      const int2 ep = g.vinc[i];
      const int e = ep.x, p = ep.y;
      const int u = g.pin_v[p];
      const int rin = g.fpin[2 * p], fout = g.fpin[2 * p + 1];
      const int we = g.w[e];
      if (rin < 0 || rin > we || fout < 0) bad = true;
      const int r = g.role[u];
      if (r == 1 && rin != we) bad = true;  // no flow leaves a source
      if (r == 1 && fout != 0) bad = true;  // nothing enters a source
      const int du = g.d[u], din = g.d[g.NB + 2 * e], dout = g.d[g.NB + 2 * e + 1];
      if (r == 0) {
        if (du < g.N && rin > 0 && du > din + 1) bad = true;        // u -> e_in
        if (du < g.N && fout > 0 && du > dout + 1) bad = true;      // u -> e_out
        if (din < g.N && we - rin > 0 && din > du + 1) bad = true;  // e_in -> u
      }
      if (dout < g.N && r != 1 && dout > du + 1) bad = true;  // e_out -> u
    }
  }
  if (bad) atomicOr(&g.ctl->err, ERR_INVARIANT);
}

}  // namespace hf

// Batched queries: many queries, each with its own graph, k, delta, motif and
// seed, evaluated together so that small queries share launches and fill the
// GPU.
//
// Work decomposition. A query's 2^k sieve iterations form 64-iteration chunks
// (one wave lane per iteration). Each (query, chunk) is a unit with its own
// prefix-state buffers. Units are packed into rounds whose buffers fit the
// HBM budget; a round runs levels 2..kmax, and level l is one launch per
// product-row width kq (4, 8, 12, 16): a prefix launch over the edge tiles of
// every unit whose query has k > l, and a last-level launch over the edge
// ranges of every unit whose query has k == l. Levels are ordered by kernel
// boundaries only: inside a launch the sole cross-wave dependency is the
// bounded look-back of rs_level.h.
//
// Each launch walks a device work table: units[] (descriptors uploaded per
// call) and ubegin[] (the first flat index of each unit). In a prefix launch
// the flat index is a wave: the launch's resident waves are partitioned over
// the (unit, chunk) pairs in proportion to their tiles, and each pair runs the
// per-level kernel's tile schedule on its own waves. In a last-level launch the
// flat index is an edge range: wave w takes w, w + W, ... and locates the unit
// by a binary search repeated only when the index leaves the current unit.
// The whole launch sequence (per-query setup, the level launches of every
// round, per-query reductions) is captured once per batch shape into a
// hipGraph; later calls with the same shape upload new descriptors and replay
// it.
#include <string.h>

#include <algorithm>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "rs_coef.h"
#include "rs_level.h"

namespace rs {

// Per-query descriptor of the setup kernels and the final reduction.
struct BQuery {
  const uint32_t* e_src;
  const uint32_t* e_dst;
  const uint32_t* e_t;
  const uint32_t* e_out;
  const uint32_t* hi;
  const uint32_t* in_off;
  const uint8_t* colour;
  uint32_t* lo;
  uint64_t* z;
  uint64_t* q;
  uint64_t* fsum;
  uint8_t* need;     // store and product flags
  uint32_t* pre;     // per prefix level: tile cost prefix within blocks [k-2][tiles]
  uint32_t* bsum;    // per prefix level: block totals [k-2][nb]
  uint32_t* boff;    // per prefix level: block offsets [k-2][nb]
  uint8_t* ref;      // slot marks (scratch shared by the queries of a batch)
  uint32_t* cov;     // window-cover difference array [m+n+1], then its block-wise prefix (scratch, shared)
  uint32_t* cbsum;   // its block totals (scratch, shared)
  uint32_t* cboff;   // its block offsets (scratch, shared)
  uint64_t seed, it_begin, it_end;
  uint32_t n, m, k, kq, delta, motif;
  uint8_t mu[RS_MAX_COLOURS];
  uint8_t off[RS_MAX_COLOURS];
};

// One (query, chunk) of one level launch; every field is wave-uniform.
struct MUnit {
  const uint32_t* e_src;
  const uint32_t* e_out;
  const uint32_t* hi;
  const uint32_t* lo;
  const uint64_t* q;   // this level's [m][kq] product rows
  const uint64_t* z;   // [n][kq] substitution rows (level 2)
  const uint64_t* pp;  // previous level's prefix state
  uint64_t* pc;        // this level's prefix state (prefix launches)
  uint64_t* fsum;      // per-iteration sums (last-level launches)
  uint64_t cb;         // first iteration of the chunk
  uint64_t it_begin, it_end;
  uint64_t row0;       // first look-back record row
  const uint8_t* need; // store flags of the query
  uint64_t p_stride;   // prefix-level units: elements between consecutive chunks' P arrays
  uint32_t m;
  uint32_t n_items;    // edge tiles, or edge ranges
  uint32_t epoch;      // record tag epoch of this launch
  uint32_t nchunks;    // prefix-level units: consecutive chunks of the query
  uint32_t waves;      // prefix-level units: waves per chunk
  uint32_t pad_;
  const uint32_t* pre;   // prefix-level units: this level's tile cost prefix (within blocks)
  const uint32_t* boff;  // prefix-level units: this level's block offsets
  uint32_t* bounds;      // prefix-level units: [waves+1] first tile of each wave's run
  const uint32_t* count; // compacted list of this level (queries with k >= 3): its length; null otherwise
  const uint64_t* d;     // level 3 of a query with k >= 4: its entries' window rows (level 2 folded in)
};
static_assert(sizeof(MUnit) == 184, "MUnit layout");
// Units are read through the constant address space: scalar loads into SGPRs.
typedef __attribute__((address_space(4))) const MUnit cMUnit;

// ---------------------------------------------------------------------------
// Per-query setup kernels (descriptors read from device memory).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void kb_ztable(const BQuery* __restrict__ qs, uint32_t qi) {
  __shared__ uint64_t lds[4][16][kLanes];
  const BQuery& Q = qs[qi];
  const uint32_t lane = threadIdx.x & 63u;
  uint64_t* tab = &lds[threadIdx.x >> 6][0][lane];
  tab[0] = 0;
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (uint64_t)Q.n * Q.kq) return;
  const uint32_t u = (uint32_t)(idx / Q.kq), j = (uint32_t)(idx % Q.kq);
  uint64_t v = 0;
  if (j < Q.k) {
    const uint64_t jj = (uint64_t)(j + 1) << 32;
    if (!Q.motif) {
      v = hash1(Q.seed, 'Z', (uint64_t)u | jj);
    } else {
      const uint32_t s = Q.colour[u];
      for (uint32_t r = 0; r < Q.mu[s]; ++r) {
        const uint64_t d = (uint64_t)Q.off[s] + r;
        v ^= gf_mul(tab, hash1(Q.seed, 'G', (uint64_t)u | (d << 32)), hash1(Q.seed, 'W', d | jj));
      }
    }
  }
  Q.z[idx] = v;
}

__global__ __launch_bounds__(256) void kb_window(const BQuery* __restrict__ qs, uint32_t qi) {
  const BQuery& Q = qs[qi];
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= Q.m) return;
  const uint32_t v = Q.e_src[e];
  const uint32_t t = Q.e_t[e];
  const uint32_t thr = t > Q.delta ? t - Q.delta : 0u;
  uint32_t a = Q.in_off[v], b = Q.in_off[v + 1];
  while (a < b) {
    const uint32_t mid = a + ((b - a) >> 1);
    if (Q.e_t[mid] < thr)
      a = mid + 1;
    else
      b = mid;
  }
  Q.lo[e] = a + v;
}

template <int KQ>
__global__ __launch_bounds__(256) void kb_qtable(const BQuery* __restrict__ qs, uint32_t qi) {
  __shared__ uint64_t lds[4][16][kLanes];
  const BQuery& Q = qs[qi];
  const uint32_t lane = threadIdx.x & 63u;
  uint64_t* tab = &lds[threadIdx.x >> 6][0][lane];
  tab[0] = 0;
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= Q.m) return;
  const uint32_t src = Q.e_src[e], dst = Q.e_dst[e], t = Q.e_t[e];
  uint64_t zr[KQ];
#pragma unroll
  for (int j = 0; j < KQ; ++j) zr[j] = Q.z[(uint64_t)dst * KQ + j];
  const uint64_t w0 = (uint64_t)src | ((uint64_t)dst << 32);
  for (uint32_t p = 1; p < Q.k; ++p) {
    const uint64_t y = hash2(Q.seed, 'Y', w0, (uint64_t)t | ((uint64_t)p << 32));
    gf_table(tab, y);
    uint64_t* out = Q.q + ((uint64_t)(p - 1) * Q.m + e) * KQ;
#pragma unroll
    for (int j = 0; j < KQ; ++j) {
      Acc128 r = {0, 0, 0, 0};
      gf_comb_acc(lds_addr(tab), zr[j], r);
      out[j] = gf_reduce(r);
    }
  }
}

// Store and product flags of query qi, prefix level l (see mark_cover): ref
// and the cover array are zeroed by kb_clear_cover; the readers are the
// windows of level l+1's product edges (every non-empty window when l+1 is
// the last level).
__global__ void kb_clear_cover(const BQuery* __restrict__ qs, uint32_t qi) {
  const BQuery& Q = qs[qi];
  const uint64_t words = ((uint64_t)Q.m + Q.n + 3) / 4, slots = (uint64_t)Q.m + Q.n + 1;
  uint32_t* r = (uint32_t*)Q.ref;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < slots; i += (uint64_t)gridDim.x * blockDim.x) {
    if (i < words) r[i] = 0;
    Q.cov[i] = 0;
  }
}
__global__ __launch_bounds__(256) void kb_mark_cover(const BQuery* __restrict__ qs, uint32_t qi, uint32_t l) {
  const BQuery& Q = qs[qi];
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint8_t* next = l + 1 < Q.k ? Q.need + (uint64_t)(l - 1) * need_stride(Q.m) : nullptr;
  if (e < Q.m) mark_cover(Q.hi, Q.lo, next, e, Q.ref, Q.cov);
}
__global__ __launch_bounds__(256) void kb_cover_prefix(const BQuery* __restrict__ qs, uint32_t qi) {
  const BQuery& Q = qs[qi];
  block_prefix(Q.cov, (uint64_t)Q.m + Q.n + 1, Q.cbsum);
}
__global__ __launch_bounds__(1024) void kb_cover_offsets(const BQuery* __restrict__ qs, uint32_t qi) {
  const BQuery& Q = qs[qi];
  block_offsets(Q.cbsum, (uint32_t)(((uint64_t)Q.m + Q.n + kCostBlock) / kCostBlock), Q.cboff);
}
__global__ __launch_bounds__(256) void kb_mark_need(const BQuery* __restrict__ qs, uint32_t qi, uint32_t l) {
  const BQuery& Q = qs[qi];
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint8_t* need = Q.need + (uint64_t)(l - 2) * need_stride(Q.m);
  if (e < Q.m)
    mark_need_cover(Q.e_out, Q.ref, Q.cov, Q.cboff, l >= 3 ? Q.hi : nullptr, Q.lo, e, need);
  else if (e < (uint64_t)Q.m + kEdgePad)
    need[e] = 0;  // the padding a level's last tile reads
}

__global__ void kb_clear_fsum(const BQuery* __restrict__ qs, uint32_t qi) {
  const BQuery& Q = qs[qi];
  const uint64_t total = 1ull << Q.k;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (uint64_t)gridDim.x * blockDim.x)
    Q.fsum[i] = 0;
}

// out[qi] = XOR of the query's per-iteration sums over its range.
__global__ __launch_bounds__(256) void kb_reduce(const BQuery* __restrict__ qs, uint64_t* __restrict__ out) {
  __shared__ uint64_t part[256];
  const BQuery& Q = qs[blockIdx.x];
  uint64_t acc = 0;
  for (uint64_t i = Q.it_begin + threadIdx.x; i < Q.it_end; i += blockDim.x) acc ^= Q.fsum[i];
  part[threadIdx.x] = acc;
  __syncthreads();
  for (uint32_t s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) part[threadIdx.x] ^= part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = part[0];
}

// Work-balanced run bounds of every unit of a prefix-level launch, from its
// query's tile cost prefix for that level and its waves per chunk (tiles of E
// entries of the level's compacted list).
__global__ __launch_bounds__(256) void kb_run_bounds(const MUnit* __restrict__ units, uint32_t E) {
  const MUnit& U = units[blockIdx.y];
  const uint32_t n_tiles = U.count ? (*U.count + E - 1) / E : U.n_items;
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (n_tiles == 0) {  // an empty list: every run is empty
    if (t == 0)
      for (uint32_t w = 0; w <= U.waves; ++w) U.bounds[w] = 0;
    return;
  }
  if (t < n_tiles) run_bounds_of_tile(U.pre, U.boff, n_tiles, t, U.waves, U.bounds);
}

// ---------------------------------------------------------------------------
// Level launches over the work table.
// ---------------------------------------------------------------------------

// Index of the unit holding flat work index t, searching [from, nunits); the
// caller guarantees ubegin[from] <= t. Wave-uniform (scalar loads).
__device__ __forceinline__ uint32_t find_unit(cu32* ubegin, uint32_t from, uint32_t nunits, uint32_t t) {
  uint32_t lo = from, hi = nunits;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (ubegin[mid] <= t)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Prefix level: the launch's waves are partitioned over (unit, chunk) pairs,
// unit u's chunks getting `waves` waves each, in proportion to its tiles;
// within a pair the waves run the per-level kernel's schedule (wave i scans
// the i-th of `waves` contiguous runs of tiles), so a run's predecessor is
// the neighbouring wave of the same pair and no wave ever waits on another
// pair.
template <int KQ, int E, bool FIRST, bool DR = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((FIRST || DR || E == 8) ? 5 : 4))) void kb_scan(const MUnit* __restrict__ units, const uint32_t* __restrict__ ubegin_p,
                                               uint32_t nunits, uint32_t total, uint64_t* __restrict__ agg,
                                               uint64_t* __restrict__ incl, unsigned long long* __restrict__ lb_stats) {
  extern __shared__ uint64_t dyn_lds[];  // [waves][16][64]; starts at LDS address 0
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform for the compiler
  const uint32_t wave = blockIdx.x * (blockDim.x >> 6) + wv;
  if (wave >= total) return;
  uint64_t* tab = dyn_lds + wv * 16 * kLanes + lane;
  tab[0] = 0;
  uint32_t mk[6];
  lane_masks(lane, mk);
  cu32* ubegin = as_const(ubegin_p);
  const uint32_t u = find_unit(ubegin, 0u, nunits, wave);
  cMUnit& U = ((cMUnit*)units)[u];
  const uint32_t local = wave - ubegin[u];
  const uint32_t ch = local / U.waves, idx = local - ch * U.waves;
  TileCtx c;
  c.e_src = U.e_src;
  c.e_out = U.e_out;
  c.hi = U.hi;
  c.lo = U.lo;
  c.q = U.q;
  c.z = U.z;
  c.d = DR ? U.d : nullptr;
  c.pp = U.pp + ch * U.p_stride;
  c.pc = U.pc + ch * U.p_stride;
  c.cb = U.cb + (uint64_t)ch * kLanes;
  // a compacted list's length is on the device; n_items stays the record stride
  c.m = U.count ? __builtin_amdgcn_readfirstlane(*as_const(U.count)) : U.m;
  c.n_tiles = U.count ? (c.m + E - 1) / E : U.n_items;
  c.epoch = U.epoch;
  c.row0 = U.row0 + (uint64_t)ch * U.n_items;
  c.agg = agg;
  c.incl = incl;
  c.need = U.need;
  c.lb_stats = lb_stats;  // null unless look-back counting is on
  c.bounds = U.bounds;
  scan_level<KQ, E, FIRST, DR>(c, idx, U.waves, lane, mk, tab);
}

// Last level: flat index = (unit, edge range of top_edges edges). A wave keeps
// its unreduced sum while it stays in one unit and XORs it into the unit's
// per-iteration sums when it leaves.
template <int KQ, bool FIRST>
__global__ __launch_bounds__(256) void kb_top(const MUnit* __restrict__ units, const uint32_t* __restrict__ ubegin_p,
                                              uint32_t nunits, uint32_t total, uint32_t top_edges) {
  extern __shared__ uint64_t dyn_lds[];  // [waves][16][64]; starts at LDS address 0
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform for the compiler
  uint64_t* tab = dyn_lds + wv * 16 * kLanes + lane;
  tab[0] = 0;
  uint32_t mk[6];
  lane_masks(lane, mk);
  cu32* ubegin = as_const(ubegin_p);
  const uint32_t waves = gridDim.x * (blockDim.x >> 6);
  uint32_t u = 0, u_begin = 0, u_end = 0;
  const uint32_t *e_src = nullptr, *hi = nullptr, *lo = nullptr;
  const uint64_t *q = nullptr, *z = nullptr, *pp = nullptr;
  uint64_t* fsum = nullptr;
  uint64_t cb = 0, it_begin = 0, it_end = 0;
  uint32_t m = 0;
  Acc128 r[1] = {{0, 0, 0, 0}};
  auto flush = [&]() {
    const uint64_t f = gf_reduce(r[0]);
    const uint64_t it = cb + lane;
    if (it >= it_begin && it < it_end && f) atomicXor((unsigned long long*)&fsum[it], (unsigned long long)f);
    r[0] = Acc128{0, 0, 0, 0};
  };
  for (uint32_t t = blockIdx.x * (blockDim.x >> 6) + wv; t < total; t += waves) {
    if (t >= u_end) {
      if (u_end != 0) flush();
      u = find_unit(ubegin, u_end == 0 ? 0u : u + 1, nunits, t);
      u_begin = ubegin[u];
      u_end = u + 1 < nunits ? ubegin[u + 1] : total;
      cMUnit& U = ((cMUnit*)units)[u];
      e_src = U.e_src;
      hi = U.hi;
      lo = U.lo;
      q = U.q;
      z = U.z;
      pp = U.pp;
      fsum = U.fsum;
      cb = U.cb;
      it_begin = U.it_begin;
      it_end = U.it_end;
      m = U.count ? __builtin_amdgcn_readfirstlane(*as_const(U.count)) : U.m;
    }
    const uint32_t e0 = (t - u_begin) * top_edges;
    const uint32_t e1 = min(m, e0 + top_edges);
    top_range<KQ, FIRST>(e_src, hi, lo, q, z, pp, 0, cb, e0, e1, lane, mk, tab, r);
  }
  if (u_end != 0) flush();
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Rounds run on this many streams at once (round r on lane r mod lanes): the
// level launches of different rounds are independent, and a launch's last
// waves leave the GPU partly idle, which the other lanes' launches fill. On
// the 64-query mix of the 10^6-edge graph, 2, 3, 4, 6 and 8 lanes ran the
// batch 0.97, 1.07-1.11, 1.11-1.14, 1.07 and 1.14 times as fast as the plain
// calls one after another.
constexpr uint32_t kBatchLanes = 4;

struct BatchWorkspace {
  std::mutex mu;
  DevBuf qs, units, ubegin, per_query, parena, agg, incl, out, ref, cov, bounds;
  DevBuf lb;  // look-back counters [2] (while counting is on)
  CoefBatch* coef = coef_batch_create();  // queries run in the coefficient form, in per_query and parena
  uint32_t epoch = 0;
  std::string key;  // shape of the captured graph
  hipGraphExec_t exec = nullptr;
  hipGraph_t graph = nullptr;
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  // lane streams (default priority) and the events that fork them off the
  // caller's stream and join them back
  hipStream_t lane_st[kBatchLanes] = {};
  hipEvent_t fork = nullptr, join[kBatchLanes] = {};
  hipError_t ensure_lanes() {
    if (fork) return hipSuccess;
    for (uint32_t i = 0; i < kBatchLanes; ++i) {
      hipError_t e = hipStreamCreateWithFlags(&lane_st[i], hipStreamNonBlocking);
      if (e == hipSuccess) e = hipEventCreateWithFlags(&join[i], hipEventDisableTiming);
      if (e != hipSuccess) return e;
    }
    return hipEventCreateWithFlags(&fork, hipEventDisableTiming);
  }
  void drop_graph() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    exec = nullptr;
    graph = nullptr;
    key.clear();
  }
  void release() {
    drop_graph();
    for (DevBuf* b : {&qs, &units, &ubegin, &per_query, &parena, &agg, &incl, &out, &ref, &cov, &bounds, &lb})
      b->release();
    coef_batch_release(coef);
    epoch = 0;
  }
  uint64_t bytes() const {
    uint64_t t = coef_batch_bytes(coef);
    for (const DevBuf* b : {&qs, &units, &ubegin, &per_query, &parena, &agg, &incl, &out, &ref, &cov, &bounds})
      t += b->bytes;
    return t;
  }
  ~BatchWorkspace() {
    release();
    coef_batch_destroy(coef);
    if (ev0) (void)hipEventDestroy(ev0);
    if (ev1) (void)hipEventDestroy(ev1);
    if (fork) (void)hipEventDestroy(fork);
    for (uint32_t i = 0; i < kBatchLanes; ++i) {
      if (join[i]) (void)hipEventDestroy(join[i]);
      if (lane_st[i]) (void)hipStreamDestroy(lane_st[i]);
    }
  }
};

BatchWorkspace* batch_ws_create() { return new BatchWorkspace(); }
void batch_ws_destroy(BatchWorkspace* w) { delete w; }
void batch_ws_release(BatchWorkspace* w) {
  std::lock_guard<std::mutex> lk(w->mu);
  w->release();
}
uint64_t batch_ws_bytes(BatchWorkspace* w) {
  std::lock_guard<std::mutex> lk(w->mu);
  return w->bytes();
}

static BatchWorkspace& batch_ws() {
  static BatchWorkspace* ws = new BatchWorkspace();  // lives until process end
  return *ws;
}

// One level launch of the plan.
struct BLaunch {
  uint32_t lane;    // stream lane of the launch's round
  bool top;         // last-level launch (else prefix level)
  bool first;       // level 2 (queries with k = 3; deeper ones fold it into level 3)
  bool dr;          // level 3 from window rows (queries with k >= 4)
  uint32_t kq;
  uint32_t unit_off, nunits, total;
  uint32_t grid;    // blocks, set at enqueue time
  uint32_t max_items = 0;  // prefix launches: most tiles of a unit (grid of the run-bounds kernel)
};

struct BatchPlan {
  std::vector<BQuery> qs;
  std::vector<uint32_t> qidx;  // query slot -> caller index
  std::vector<MUnit> units;
  std::vector<uint32_t> ubegin;
  std::vector<BLaunch> launches;
  std::vector<uint32_t> unit_query;   // query slot of each unit
  std::vector<uint64_t> unit_pbytes;  // offset of a unit's prefix buffers in the arena (bytes)
  uint64_t per_query_bytes = 0;
  uint64_t ref_bytes = 4;     // slot-mark scratch (largest m + n)
  uint64_t n_max = 1;         // largest vertex count (per-vertex scratch)
  uint64_t parena_bytes = 0;  // prefix-state arena (largest round)
  uint64_t records = 1;       // look-back records (largest round)
  uint32_t scan_launches = 0;
  uint32_t rounds = 0;
  uint32_t lanes = 1;         // rounds run on this many streams at once
  uint64_t bounds_words = 0;  // run bounds of all prefix-level units
  std::vector<uint64_t> lists_off;    // per query: offset of its compacted lists (k >= 3)
  std::vector<uint64_t> rr_off;       // per query: offset of its level-2 prefix rows (k >= 4)
  std::vector<uint8_t*> rr;           // the same, resolved
  std::vector<CompactArgs> cargs;     // per query: its compacted lists (set by resolve_plan)
  std::vector<int32_t> unit_list;     // per unit: level index of its compacted list, or -1
  Tuning tu;
  std::string key;
  bool count_lb = false;  // the prefix launches count look-back events into W.lb
};

static uint64_t align256(uint64_t b) { return (b + 255) & ~255ull; }

// Per-query arena bytes of a query in a batch (the layout batch_plan gives
// it), at the smallest tile size (most tiles).
uint64_t batch_query_bytes(uint64_t m, uint64_t n, const QueryPlan& qp) {
  const uint64_t levels = qp.k > 2 ? qp.k - 2 : 0, tiles = (m + 7) / 8, nb = (tiles + kCostBlock - 1) / kCostBlock;
  return align256(table_lo_bytes(m)) + align256(table_z_bytes(n, qp.kq)) +
         (qp.k == 2 ? align256(table_q_bytes(m, qp.k, qp.kq)) : 0) +
         (qp.k >= 3 ? align256(compact_bytes(m, qp.k, qp.kq)) : 0) +
         (qp.k >= 4 ? align256(rrows_bytes(m, qp.kq)) : 0) + align256(table_need_bytes(m, qp.k)) +
         align256(4 * tiles * levels) + 2 * align256(4 * nb * levels) + align256(8 * (1ull << qp.k)) + 2048;
}

// Bytes one chunk holds while its round runs: two prefix-state arrays and
// the look-back records of its tiles.
static uint64_t chunk_bytes(uint64_t m, uint64_t n, uint32_t E) {
  const uint64_t tiles = (m + E - 1) / E;
  return 2 * align256((m + n) * kLanes * 8) + 2 * 1024 * tiles;
}

// Builds the plan: per-query buffers, rounds of chunks within `slot_budget`
// bytes, and the level launches. Pointers inside qs/units are byte offsets
// into the per-query arena / prefix arena until resolve_plan() rebases them.
rs_status batch_plan(const rs_graph* const* graphs, const rs_query* queries, uint32_t nq, const Tuning& tu,
                     uint64_t slot_budget, rs_result* results, BatchPlan& P) {
  P = BatchPlan();
  P.tu = tu;
  const uint32_t E = tu.edges_per_tile;
  const uint32_t TE = tu.top_edges_per_tile;
  std::string key = "E" + std::to_string(E) + "T" + std::to_string(TE) + "W" + std::to_string(tu.waves_per_block) +
                    "S" + std::to_string(tu.max_slots);
  struct Chunk {
    uint32_t query;
    uint64_t cb;
  };
  std::vector<Chunk> chunks;
  std::vector<const rs_graph*> qgraph;
  uint64_t pq_off = 0;
  for (uint32_t i = 0; i < nq; ++i) {
    QueryPlan qp;
    results[i] = rs_result{0, 0, RS_OK, 0.0f};
    rs_status s = plan_query(graphs ? graphs[i] : nullptr, &queries[i], qp);
    if (s != RS_OK) {
      results[i].status = s;
      continue;
    }
    const rs_graph* g = graphs[i];
    const uint64_t m = g->g.m, n = g->g.n;
    if (m == 0 || qp.k > n || qp.it_end == qp.it_begin) continue;  // F = 0 exactly
    BQuery Q;
    memset(&Q, 0, sizeof(Q));
    Q.e_src = g->g.e_src.as<uint32_t>();
    Q.e_dst = g->g.e_dst.as<uint32_t>();
    Q.e_t = g->g.e_t.as<uint32_t>();
    Q.e_out = g->g.e_out.as<uint32_t>();
    Q.hi = g->g.hi.as<uint32_t>();
    Q.in_off = g->g.in_off.as<uint32_t>();
    Q.colour = g->g.colour.as<uint8_t>();
    Q.seed = qp.seed;
    Q.it_begin = qp.it_begin;
    Q.it_end = qp.it_end;
    Q.n = (uint32_t)n;
    Q.m = (uint32_t)m;
    Q.k = qp.k;
    Q.kq = qp.kq;
    Q.delta = qp.delta;
    Q.motif = qp.motif ? 1 : 0;
    memcpy(Q.mu, qp.mu, sizeof(Q.mu));
    memcpy(Q.off, qp.shade_off, sizeof(Q.off));
    // byte offsets into the per-query arena, rebased by resolve_plan
    Q.lo = (uint32_t*)(uintptr_t)pq_off;
    pq_off += align256(table_lo_bytes(m));
    Q.z = (uint64_t*)(uintptr_t)pq_off;
    pq_off += align256(table_z_bytes(n, qp.kq));
    // product rows: of every edge at k = 2, of the compacted lists above
    Q.q = (uint64_t*)(uintptr_t)pq_off;
    if (qp.k == 2) pq_off += align256(table_q_bytes(m, qp.k, qp.kq));
    P.lists_off.push_back(pq_off);
    if (qp.k >= 3) pq_off += align256(compact_bytes(m, qp.k, qp.kq));
    P.rr_off.push_back(pq_off);  // level 2 folded into level 3 (k >= 4)
    if (qp.k >= 4) pq_off += align256(rrows_bytes(m, qp.kq));
    Q.need = (uint8_t*)(uintptr_t)pq_off;
    pq_off += align256(table_need_bytes(m, qp.k));
    {
      const uint64_t levels = qp.k > 2 ? qp.k - 2 : 0, tiles = (m + E - 1) / E, nb = (tiles + kCostBlock - 1) / kCostBlock;
      Q.pre = (uint32_t*)(uintptr_t)pq_off;
      pq_off += align256(4 * tiles * levels);
      Q.bsum = (uint32_t*)(uintptr_t)pq_off;
      pq_off += align256(4 * nb * levels);
      Q.boff = (uint32_t*)(uintptr_t)pq_off;
      pq_off += align256(4 * nb * levels);
    }
    P.ref_bytes = std::max<uint64_t>(P.ref_bytes, (m + n + 3) & ~3ull);
    P.n_max = std::max<uint64_t>(P.n_max, n);
    Q.fsum = (uint64_t*)(uintptr_t)pq_off;
    pq_off += align256(8 * (1ull << qp.k));
    const uint32_t qslot = (uint32_t)P.qs.size();
    P.qs.push_back(Q);
    P.qidx.push_back(i);
    qgraph.push_back(g);
    key += "|" + std::to_string(n) + ":" + std::to_string(m) + ":" + std::to_string(qp.k) + ":" +
           std::to_string(qp.chunk_first) + "-" + std::to_string(qp.chunk_last);
    // the arrays that captured launches hold pointers to (a later graph may lie at a destroyed one's handle)
    for (const void* p : {(const void*)Q.e_src, (const void*)Q.e_dst, (const void*)Q.e_t, (const void*)Q.e_out,
                          (const void*)Q.hi, (const void*)Q.in_off})
      key += "," + std::to_string((uintptr_t)p);
    for (uint64_t c = qp.chunk_first; c < qp.chunk_last; ++c) chunks.push_back(Chunk{qslot, c * kLanes});
  }
  P.per_query_bytes = pq_off;
  if (chunks.empty()) {
    P.key = key;
    return RS_OK;
  }
  // longest queries first so that each round's levels are shared by many units
  std::stable_sort(chunks.begin(), chunks.end(),
                   [&](const Chunk& a, const Chunk& b) { return P.qs[a.query].k > P.qs[b.query].k; });
  // rounds: consecutive chunks while their buffers fit the budget
  std::vector<std::pair<size_t, size_t>> rounds;
  {
    size_t r0 = 0;
    uint64_t bytes = 0, items = 0;
    auto tiles_of = [&](uint64_t m) { return (m + E - 1) / E; };
    for (size_t c = 0; c < chunks.size(); ++c) {
      const BQuery& Q = P.qs[chunks[c].query];
      const uint64_t b = chunk_bytes(Q.m, Q.n, E);
      // (and at most 2^30 prefix-level items, so flat item indices stay 32-bit)
      const bool full = c > r0 && (bytes + b > slot_budget || (tu.max_slots && c - r0 >= tu.max_slots) ||
                                   items + tiles_of(Q.m) > (1u << 30));
      if (full) {
        rounds.push_back({r0, c});
        r0 = c;
        bytes = 0;
        items = 0;
      }
      bytes += b;
      items += tiles_of(Q.m);
    }
    rounds.push_back({r0, chunks.size()});
  }
  P.rounds = (uint32_t)rounds.size();
  P.lanes = (uint32_t)std::min<size_t>(kBatchLanes, rounds.size());
  key += "#R" + std::to_string(rounds.size()) + "L" + std::to_string(P.lanes);
  // Rounds go to the lanes in turn; each lane has its own part of the prefix
  // arena and of the record arrays, sized for the largest round.
  uint64_t lane_pbytes = 0, lane_rows = 0;
  for (const auto& rd : rounds) {
    uint64_t pbytes = 0, rows = 0;
    for (size_t c = rd.first; c < rd.second; ++c) {
      const BQuery& Q = P.qs[chunks[c].query];
      pbytes += 2 * align256(((uint64_t)Q.m + Q.n) * kLanes * 8);
      rows += (Q.m + E - 1) / E;
    }
    lane_pbytes = std::max(lane_pbytes, pbytes);
    lane_rows = std::max(lane_rows, rows);
  }
  P.parena_bytes = lane_pbytes * P.lanes;
  P.records = std::max<uint64_t>(lane_rows * P.lanes, 1);
  // launches
  for (size_t ri = 0; ri < rounds.size(); ++ri) {
    const auto& rd = rounds[ri];
    const uint32_t lane = (uint32_t)(ri % P.lanes);
    // per-chunk prefix buffers and record rows within the round's lane
    std::vector<uint64_t> poff(rd.second - rd.first), row0(rd.second - rd.first);
    uint64_t pbytes = lane * lane_pbytes, rows = lane * lane_rows;
    uint32_t kmax = 0;
    for (size_t c = rd.first; c < rd.second; ++c) {
      const BQuery& Q = P.qs[chunks[c].query];
      poff[c - rd.first] = pbytes;
      pbytes += 2 * align256(((uint64_t)Q.m + Q.n) * kLanes * 8);
      row0[c - rd.first] = rows;
      rows += (Q.m + E - 1) / E;
      kmax = std::max(kmax, Q.k);
    }
    for (uint32_t l = 2; l <= kmax; ++l) {
      for (uint32_t kq = 4; kq <= 16; kq += 4) {
        for (int top = 0; top < 2; ++top) {
          BLaunch L;
          L.lane = lane;
          L.top = top != 0;
          L.first = l == 2;
          L.dr = !L.top && l == 3;
          L.kq = kq;
          L.unit_off = (uint32_t)P.units.size();
          L.nunits = 0;
          L.total = 0;
          L.grid = 0;
          for (size_t c = rd.first; c < rd.second; ++c) {
            const uint32_t qi = chunks[c].query;
            const BQuery& Q = P.qs[qi];
            if (Q.kq != kq || (top ? Q.k != l : Q.k <= l)) continue;
            if (!top && l == 2 && Q.k >= 4) continue;  // folded into level 3's window rows
            // prefix levels: this and the following chunks of the same query
            // (consecutive in the round, their buffers and record rows at a
            // fixed stride) form one unit
            uint32_t nch = 1;
            if (!top)
              while (c + nch < rd.second && chunks[c + nch].query == qi &&
                     chunks[c + nch].cb == chunks[c].cb + (uint64_t)nch * kLanes)
                ++nch;
            MUnit U;
            memset(&U, 0, sizeof(U));
            U.e_src = Q.e_src;
            U.e_out = Q.e_out;
            U.hi = Q.hi;
            U.lo = Q.lo;  // offset, rebased later
            U.q = Q.q;    // byte offset until rebased (k = 2; deeper queries read their compacted lists)
            U.z = Q.z;
            const uint64_t half = align256(((uint64_t)Q.m + Q.n) * kLanes * 8);
            U.pp = (const uint64_t*)(uintptr_t)(poff[c - rd.first] + ((l - 1) & 1) * half);
            U.pc = (uint64_t*)(uintptr_t)(poff[c - rd.first] + (l & 1) * half);
            U.fsum = Q.fsum;
            U.cb = chunks[c].cb;
            U.it_begin = Q.it_begin;
            U.it_end = Q.it_end;
            U.row0 = row0[c - rd.first];
            // this level's flags (prefix levels; unused at the last level): offset, rebased later
            U.need = (const uint8_t*)((uintptr_t)Q.need + (top ? 0 : (uint64_t)(l - 2) * need_stride(Q.m)));
            if (!top) {  // this level's cost prefix: offsets, rebased later
              const uint64_t tiles = (Q.m + E - 1) / E, nb = (tiles + kCostBlock - 1) / kCostBlock;
              U.pre = (const uint32_t*)((uintptr_t)Q.pre + 4ull * (l - 2) * tiles);
              U.boff = (const uint32_t*)((uintptr_t)Q.boff + 4ull * (l - 2) * nb);
            }
            U.m = Q.m;
            U.nchunks = nch;
            U.p_stride = 2 * half / 8;
            U.n_items = top ? (Q.m + TE - 1) / TE : (Q.m + E - 1) / E;
            U.epoch = 0;  // set per call
            P.ubegin.push_back(L.total);
            L.total += U.n_items * (top ? 1u : nch);  // prefix levels: tiles (waves assigned later)
            P.units.push_back(U);
            P.unit_query.push_back(qi);
            P.unit_list.push_back(Q.k >= 3 ? (int32_t)(l - 2) : -1);
            ++L.nunits;
            c += nch - 1;
          }
          if (L.nunits) {
            if (!L.top) ++P.scan_launches;
            P.launches.push_back(L);
            key += "/" + std::to_string(L.top) + std::to_string(L.first) + std::to_string(L.dr) + ":" +
                   std::to_string(kq) + ":" +
                   std::to_string(L.nunits) + ":" + std::to_string(L.total);
          }
        }
      }
    }
  }
  P.key = key;
  return RS_OK;
}

// Rebases the plan's offsets onto the allocated arenas, sets record epochs and
// checks that every unit's ranges lie inside the buffers it addresses.
static rs_status resolve_plan(BatchPlan& P, BatchWorkspace& W, uint32_t epoch0) {
  char* pq = W.per_query.as<char>();
  char* pa = W.parena.as<char>();
  // per-query tables: byte offsets -> pointers
  std::vector<uint64_t> lo_off(P.qs.size()), z_off(P.qs.size()), q_off(P.qs.size()), f_off(P.qs.size()),
      need_off(P.qs.size());
  for (size_t i = 0; i < P.qs.size(); ++i) {
    BQuery& Q = P.qs[i];
    f_off[i] = (uintptr_t)Q.fsum;
    if (f_off[i] + 8 * (1ull << Q.k) > W.per_query.bytes) return RS_EINVAL;
    Q.fsum = (uint64_t*)(pq + f_off[i]);
    lo_off[i] = (uintptr_t)Q.lo;
    z_off[i] = (uintptr_t)Q.z;
    q_off[i] = (uintptr_t)Q.q;
    need_off[i] = (uintptr_t)Q.need;
    if (need_off[i] + table_need_bytes(Q.m, Q.k) > W.per_query.bytes) return RS_EINVAL;
    {
      const uint64_t levels = Q.k > 2 ? Q.k - 2 : 0, tiles = (Q.m + P.tu.edges_per_tile - 1) / P.tu.edges_per_tile,
                     nb = (tiles + kCostBlock - 1) / kCostBlock;
      if ((uintptr_t)Q.pre + 4 * tiles * levels > W.per_query.bytes ||
          (uintptr_t)Q.bsum + 4 * nb * levels > W.per_query.bytes ||
          (uintptr_t)Q.boff + 4 * nb * levels > W.per_query.bytes)
        return RS_EINVAL;
      Q.pre = (uint32_t*)(pq + (uintptr_t)Q.pre);
      Q.bsum = (uint32_t*)(pq + (uintptr_t)Q.bsum);
      Q.boff = (uint32_t*)(pq + (uintptr_t)Q.boff);
    }
    if (Q.k == 2 && q_off[i] + table_q_bytes(Q.m, Q.k, Q.kq) > W.per_query.bytes) return RS_EINVAL;
    const uint64_t slots = (uint64_t)Q.m + Q.n + 1, nbq = (slots + kCostBlock - 1) / kCostBlock;
    if ((uint64_t)Q.m + Q.n > W.ref.bytes || 4ull * (slots + 2 * nbq) > W.cov.bytes) return RS_EINVAL;
    Q.lo = (uint32_t*)(pq + lo_off[i]);
    Q.z = (uint64_t*)(pq + z_off[i]);
    Q.q = (uint64_t*)(pq + q_off[i]);
    Q.need = (uint8_t*)(pq + need_off[i]);
    Q.ref = W.ref.as<uint8_t>();
    Q.cov = W.cov.as<uint32_t>();
    Q.cbsum = Q.cov + slots;
    Q.cboff = Q.cbsum + nbq;
    CompactArgs ca{};
    if (Q.k >= 3) {
      const uint64_t L = Q.k - 1, lst = list_stride(Q.m);
      if (P.lists_off[i] + compact_bytes(Q.m, Q.k, Q.kq) > W.per_query.bytes) return RS_EINVAL;
      ca.e_src = Q.e_src;
      ca.e_dst = Q.e_dst;
      ca.e_t = Q.e_t;
      ca.e_out = Q.e_out;
      ca.hi = Q.hi;
      ca.lo = Q.lo;
      ca.need = Q.need;
      ca.need_stride = need_stride(Q.m);
      ca.m = Q.m;
      ca.k = Q.k;
      ca.kq = Q.kq;
      ca.nb = (uint32_t)((Q.m + kCostBlock - 1) / kCostBlock);
      ca.list_stride = lst;
      ca.rows = (uint64_t*)(pq + P.lists_off[i]);
      ca.u32 = (uint32_t*)(ca.rows + L * lst * Q.kq);
      ca.u8 = (uint8_t*)(ca.u32 + L * 4 * lst);
      ca.bsum = (uint32_t*)(((uintptr_t)(ca.u8 + L * lst) + 3) & ~(uintptr_t)3);
      ca.boff = ca.bsum + L * ca.nb;
      ca.count = ca.boff + L * ca.nb;
    }
    P.cargs.push_back(ca);
    if (Q.k >= 4 && P.rr_off[i] + rrows_bytes(Q.m, Q.kq) > W.per_query.bytes) return RS_EINVAL;
    P.rr.push_back(Q.k >= 4 ? (uint8_t*)(pq + P.rr_off[i]) : nullptr);
  }
  uint32_t scan_idx = 0;
  for (const BLaunch& L : P.launches) {
    const uint32_t epoch = L.top ? 0u : epoch0 + 1 + scan_idx++;
    for (uint32_t j = 0; j < L.nunits; ++j) {
      MUnit& U = P.units[L.unit_off + j];
      const uint32_t qi = P.unit_query[L.unit_off + j];
      const BQuery& Q = P.qs[qi];
      const uint64_t half = align256(((uint64_t)Q.m + Q.n) * kLanes * 8);
      const uint64_t pp_off = (uintptr_t)U.pp, pc_off = (uintptr_t)U.pc;
      const uint64_t span = 8 * U.p_stride * (U.nchunks - 1) + half;  // from the first chunk's array
      if (pp_off + span > W.parena.bytes || pc_off + span > W.parena.bytes) return RS_EINVAL;
      if (!L.top && (U.row0 + (uint64_t)U.nchunks * U.n_items) * 1024 > W.agg.bytes) return RS_EINVAL;
      const int32_t y = P.unit_list[L.unit_off + j];
      if (y >= 0) {  // this level's compacted list
        const LevelList Lc = P.cargs[qi].list((uint32_t)y);
        U.e_src = Lc.chi;
        U.e_out = Lc.cslot;
        U.hi = Lc.chi;
        U.lo = Lc.clo;
        U.q = Lc.cq;
        U.count = P.cargs[qi].count + y;
        U.d = (y == 1 && Q.k >= 4) ? P.cargs[qi].list(0).cq : nullptr;  // the D rows
      } else {
        const uint64_t q_level = (uintptr_t)U.q;  // offset of this level's rows (k = 2)
        if (q_level + 8ull * Q.m * Q.kq > q_off[qi] + 8ull * Q.m * Q.kq * (Q.k - 1)) return RS_EINVAL;
        U.q = (const uint64_t*)(pq + q_level);
        U.lo = Q.lo;
        U.count = nullptr;
      }
      const uint64_t need_level = (uintptr_t)U.need - need_off[qi];  // offset of this level's flags
      if (need_level + need_stride(Q.m) > table_need_bytes(Q.m, Q.k)) return RS_EINVAL;
      U.need = y >= 0 ? P.cargs[qi].list((uint32_t)y).cflag : Q.need + need_level;
      if (!L.top) {
        const uint64_t pre_off = (uintptr_t)U.pre, boff_off = (uintptr_t)U.boff;
        if (pre_off + 4ull * U.n_items > W.per_query.bytes || boff_off + 4 > W.per_query.bytes) return RS_EINVAL;
        U.pre = (const uint32_t*)(pq + pre_off);
        U.boff = (const uint32_t*)(pq + boff_off);
      }
      U.z = Q.z;
      U.pp = (const uint64_t*)(pa + pp_off);
      U.pc = (uint64_t*)(pa + pc_off);
      U.fsum = Q.fsum;
      U.epoch = epoch;
    }
  }
  return RS_OK;
}

static uint32_t resident_blocks_of(const void* kern, uint32_t threads, size_t lds) {
  return resident_blocks(kern, threads, lds);
}

template <int KQ, int E>
static const void* scan_kernel(bool first, bool dr) {
  if (dr) return (const void*)kb_scan<KQ, E, false, true>;
  return first ? (const void*)kb_scan<KQ, E, true> : (const void*)kb_scan<KQ, E, false>;
}

static const void* pick_scan(uint32_t kq, uint32_t E, bool first, bool dr) {
  if (E == 8) {
    switch (kq) {
      case 4: return scan_kernel<4, 8>(first, dr);
      case 8: return scan_kernel<8, 8>(first, dr);
      case 12: return scan_kernel<12, 8>(first, dr);
      default: return scan_kernel<16, 8>(first, dr);
    }
  }
  switch (kq) {
    case 4: return scan_kernel<4, 16>(first, dr);
    case 8: return scan_kernel<8, 16>(first, dr);
    case 12: return scan_kernel<12, 16>(first, dr);
    default: return scan_kernel<16, 16>(first, dr);
  }
}

static const void* pick_top(uint32_t kq, bool first) {
  switch (kq) {
    case 4: return first ? (const void*)kb_top<4, true> : (const void*)kb_top<4, false>;
    case 8: return first ? (const void*)kb_top<8, true> : (const void*)kb_top<8, false>;
    case 12: return first ? (const void*)kb_top<12, true> : (const void*)kb_top<12, false>;
    default: return first ? (const void*)kb_top<16, true> : (const void*)kb_top<16, false>;
  }
}

// Grid of every launch: about as many blocks as are resident, at most one
// wave per work item.
// Prefix-level launches: waves per (unit, chunk) pair in proportion to the
// unit's tiles, at least one each, all of them resident when the pairs fit
// (a pair whose waves are not all resident is still correct: waits are
// bounded, and a single wave never waits). Then the grid of every launch:
// about as many blocks as are resident, at most one wave per work item.
static void size_grids(BatchPlan& P) {
  P.bounds_words = 0;
  const uint32_t wpb = P.tu.waves_per_block;
  const size_t lds = (size_t)wpb * 16 * kLanes * 8;
  for (BLaunch& L : P.launches) {
    const void* kern = L.top ? pick_top(L.kq, L.first) : pick_scan(L.kq, P.tu.edges_per_tile, L.first, L.dr);
    const uint32_t resident = resident_blocks_of(kern, 64 * wpb, lds);
    if (!L.top) {
      uint64_t pairs = 0, tiles = 0;
      for (uint32_t j = 0; j < L.nunits; ++j) {
        const MUnit& U = P.units[L.unit_off + j];
        pairs += U.nchunks;
        tiles += (uint64_t)U.nchunks * U.n_items;
      }
      const uint64_t spare = (uint64_t)resident * wpb > pairs ? (uint64_t)resident * wpb - pairs : 0;
      uint32_t w0 = 0;
      L.max_items = 0;
      for (uint32_t j = 0; j < L.nunits; ++j) {
        MUnit& U = P.units[L.unit_off + j];
        U.waves = (uint32_t)std::min<uint64_t>(U.n_items, 1 + (uint64_t)U.n_items * spare / std::max<uint64_t>(tiles, 1));
        P.ubegin[L.unit_off + j] = w0;
        w0 += U.waves * U.nchunks;
        U.bounds = (uint32_t*)(uintptr_t)(4 * P.bounds_words);  // offset, rebased after allocation
        P.bounds_words += U.waves + 1;
        L.max_items = std::max(L.max_items, U.n_items);
      }
      L.total = w0;
      L.grid = std::max(1u, (L.total + wpb - 1) / wpb);
    } else {
      L.grid = std::max(1u, std::min(resident, (L.total + wpb - 1) / wpb));
    }
    P.key += "g" + std::to_string(L.grid);
  }
}

// Enqueues the whole batch on `st` (kernels only, so it can be captured).
static rs_status batch_enqueue(BatchPlan& P, BatchWorkspace& W, hipStream_t st) {
  const BQuery* dq = W.qs.as<BQuery>();
  for (uint32_t qi = 0; qi < P.qs.size(); ++qi) {
    const BQuery& Q = P.qs[qi];
    hipLaunchKernelGGL(kb_ztable, dim3((uint32_t)(((uint64_t)Q.n * Q.kq + 255) / 256)), dim3(256), 0, st, dq, qi);
    hipLaunchKernelGGL(kb_window, dim3((Q.m + 255) / 256), dim3(256), 0, st, dq, qi);
    for (uint32_t l = Q.k - 1; l >= 2 && Q.k >= 3; --l) {  // flags per prefix level, last one first
      const uint64_t slots = (uint64_t)Q.m + Q.n + 1;
      hipLaunchKernelGGL(kb_clear_cover, dim3((uint32_t)std::min<uint64_t>((slots + 1023) / 1024, 1024)), dim3(256), 0,
                         st, dq, qi);
      hipLaunchKernelGGL(kb_mark_cover, dim3((Q.m + 255) / 256), dim3(256), 0, st, dq, qi, l);
      hipLaunchKernelGGL(kb_cover_prefix, dim3((uint32_t)((slots + kCostBlock - 1) / kCostBlock)), dim3(256), 0, st,
                         dq, qi);
      hipLaunchKernelGGL(kb_cover_offsets, dim3(1), dim3(1024), 0, st, dq, qi);
      hipLaunchKernelGGL(kb_mark_need, dim3((Q.m + kEdgePad + 255) / 256), dim3(256), 0, st, dq, qi, l);
    }
    if (Q.k >= 3) {
      // compacted lists of levels 2..k, their tile costs, and their product
      // rows (the seed read from the descriptor, so a replay takes new seeds)
      const CompactArgs& ca = P.cargs[qi];
      const uint32_t E = P.tu.edges_per_tile;
      RS_HIP(launch_compact(ca, st));
      RS_HIP(launch_compact_costs(ca, E, (Q.m + E - 1) / E, Q.pre, Q.bsum, Q.boff, st));
      const uint64_t* seed_p = (const uint64_t*)((const char*)(dq + qi) + offsetof(BQuery, seed));
      RS_HIP(launch_compact_rows(ca, Q.z, 0, seed_p, EdgeFilter(), Q.kq, st, Q.k >= 4 ? 1 : 0));
      // level 2 folded into level 3: the iteration-independent prefix rows
      if (Q.k >= 4) RS_HIP(launch_rrows(ca, Q.in_off, Q.z, 0, seed_p, EdgeFilter(), Q.kq, P.rr[qi], st));
    } else {
      switch (Q.kq) {
        case 4: hipLaunchKernelGGL(kb_qtable<4>, dim3((Q.m + 255) / 256), dim3(256), 0, st, dq, qi); break;
        case 8: hipLaunchKernelGGL(kb_qtable<8>, dim3((Q.m + 255) / 256), dim3(256), 0, st, dq, qi); break;
        case 12: hipLaunchKernelGGL(kb_qtable<12>, dim3((Q.m + 255) / 256), dim3(256), 0, st, dq, qi); break;
        default: hipLaunchKernelGGL(kb_qtable<16>, dim3((Q.m + 255) / 256), dim3(256), 0, st, dq, qi); break;
      }
    }
    hipLaunchKernelGGL(kb_clear_fsum, dim3((uint32_t)std::min<uint64_t>(((1ull << Q.k) + 255) / 256, 256)), dim3(256),
                       0, st, dq, qi);
  }
  const uint32_t wpb = P.tu.waves_per_block;
  const size_t lds = (size_t)wpb * 16 * kLanes * 8;
  const MUnit* du = W.units.as<MUnit>();
  const uint32_t* db = W.ubegin.as<uint32_t>();
  // fork: the lanes start after the setup kernels, and st continues after all lanes
  if (!W.fork) return RS_EDEVICE;
  RS_HIP(hipEventRecord(W.fork, st));
  for (uint32_t ln = 0; ln < P.lanes; ++ln) RS_HIP(hipStreamWaitEvent(W.lane_st[ln], W.fork, 0));
  for (BLaunch& L : P.launches) {
    hipStream_t lst = W.lane_st[L.lane];
    const void* kern = L.top ? pick_top(L.kq, L.first) : pick_scan(L.kq, P.tu.edges_per_tile, L.first, L.dr);
    const MUnit* u = du + L.unit_off;
    const uint32_t* b = db + L.unit_off;
    if (L.top) {
      void* args[] = {(void*)&u, (void*)&b, (void*)&L.nunits, (void*)&L.total, (void*)&P.tu.top_edges_per_tile};
      RS_HIP(hipLaunchKernel(kern, dim3(L.grid), dim3(64 * wpb), args, lds, lst));
    } else {
      hipLaunchKernelGGL(kb_run_bounds, dim3((L.max_items + 255) / 256, L.nunits), dim3(256), 0, lst, u,
                         P.tu.edges_per_tile);
      uint64_t* agg = W.agg.as<uint64_t>();
      uint64_t* incl = W.incl.as<uint64_t>();
      unsigned long long* lb = P.count_lb ? W.lb.as<unsigned long long>() : nullptr;
      void* args[] = {(void*)&u, (void*)&b, (void*)&L.nunits, (void*)&L.total, (void*)&agg, (void*)&incl, (void*)&lb};
      RS_HIP(hipLaunchKernel(kern, dim3(L.grid), dim3(64 * wpb), args, lds, lst));
    }
  }
  for (uint32_t ln = 0; ln < P.lanes; ++ln) {
    RS_HIP(hipEventRecord(W.join[ln], W.lane_st[ln]));
    RS_HIP(hipStreamWaitEvent(st, W.join[ln], 0));
  }
  hipLaunchKernelGGL(kb_reduce, dim3((uint32_t)P.qs.size()), dim3(256), 0, st, dq, W.out.as<uint64_t>());
  RS_HIP(hipGetLastError());
  return RS_OK;
}

static uint64_t default_slot_budget() {
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) return 8ull << 30;
  return (uint64_t)(free_b / 3);
}

// At most this many bytes of prefix state per round. On 64 mixed queries of
// the 10^6-edge graph, rounds of at most 5, 10 and 20 GiB ran the batch in
// 0.887, 0.879 and 0.854 s (four lanes). (Under the earlier per-tile
// look-back and equal runs, larger rounds had run slower: 1.71 s with 4
// chunks per round against 2.14 s unbounded.)
constexpr uint64_t kRoundStateBytes = 20ull << 30;

// slot_budget: bytes of prefix state the call may hold over all its stream
// lanes (0 = a third of free device memory). *ran: the status returned is that of
// single queries, and every other query has its result.
static rs_status run_batch_eval(BatchWorkspace& W, const rs_graph* const* graphs, const rs_query* queries, uint32_t nq,
                                rs_result* results, const rs_tuning* tune, hipStream_t st, bool use_graph,
                                uint64_t slot_budget, bool* ran = nullptr) {
  // launch shape: explicit knobs, else the graph's autotuned batch shape, else defaults
  Tuning tu;
  tu.top_edges_per_tile = 128;
  tu.waves_per_block = 2;
  if (graphs[0] && graphs[0]->has_batch_tuned) tu = graphs[0]->batch_tuned;
  if (tune) {
    if (tune->edges_per_tile) tu.edges_per_tile = tune->edges_per_tile;
    if (tune->top_edges_per_tile) tu.top_edges_per_tile = tune->top_edges_per_tile;
    if (tune->waves_per_block) tu.waves_per_block = tune->waves_per_block;
    if (tune->max_slots) tu.max_slots = tune->max_slots;
    if (tune->no_graph) use_graph = false;
  }
  if (tu.edges_per_tile != 8 && tu.edges_per_tile != 16) tu.edges_per_tile = 16;
  if (tu.waves_per_block != 1 && tu.waves_per_block != 2 && tu.waves_per_block != 4) tu.waves_per_block = 2;
  tu.top_edges_per_tile = std::min(std::max(tu.top_edges_per_tile, 1u), 4096u);
  if (tu.edges_per_tile == 8)
    for (uint32_t i = 0; i < nq; ++i)
      if (graphs[i] && graphs[i]->g.m > kMaxEdgesE8) {
        set_last_error("8-edge tiles are not accepted on graphs of more than 4e6 edges");
        return RS_EINVAL;
      }
  BatchPlan P;
  P.count_lb = lookback_counting();
  // the lanes hold one round each at a time, so a round gets a lane's share
  // of the budget and the whole prefix arena stays within it
  const uint64_t budget = slot_budget ? slot_budget : default_slot_budget();
  RS_TRY(batch_plan(graphs, queries, nq, tu, std::min<uint64_t>(budget / kBatchLanes, kRoundStateBytes), results, P));
  rs_status first_err = RS_OK;
  for (uint32_t i = 0; i < nq; ++i)
    if (results[i].status != RS_OK && first_err == RS_OK) first_err = results[i].status;
  if (ran) *ran = P.qs.empty();
  if (P.qs.empty()) return first_err;
  // device memory; a reallocation invalidates the captured graph
  const void* before[10] = {W.qs.p,  W.units.p, W.ubegin.p, W.per_query.p, W.parena.p,
                            W.agg.p, W.incl.p,  W.out.p,    W.ref.p,       W.cov.p};
  const uint64_t rec_bytes = 1024 * P.records;
  // rows of the coefficient form that leave no room for the records
  if (slot_budget && W.parena.bytes > P.parena_bytes &&
      W.parena.bytes + std::max(W.agg.bytes, rec_bytes) + std::max(W.incl.bytes, rec_bytes) > slot_budget)
    W.parena.release();
  if (W.per_query.reserve(P.per_query_bytes, st, false) || W.qs.reserve(sizeof(BQuery) * P.qs.size(), st, false) ||
      W.units.reserve(sizeof(MUnit) * std::max<size_t>(P.units.size(), 1), st, false) ||
      W.ubegin.reserve(4 * std::max<size_t>(P.ubegin.size(), 1), st, false) ||
      W.parena.reserve(std::max<uint64_t>(P.parena_bytes, 256), st, false) ||
      W.out.reserve(8 * P.qs.size(), st, false) || W.ref.reserve(P.ref_bytes, st, false) ||
      W.cov.reserve(4 * (P.ref_bytes + 1 + 2 * ((P.ref_bytes + kCostBlock) / kCostBlock)), st, false))
    return RS_ENOMEM;
  if (W.agg.bytes < rec_bytes || W.incl.bytes < rec_bytes) {
    // tagged records start at epoch 0, which no launch uses
    if (W.agg.reserve(rec_bytes, st, true) || W.incl.reserve(rec_bytes, st, true)) return RS_ENOMEM;
    W.epoch = 0;
  }
  const void* after[10] = {W.qs.p,  W.units.p, W.ubegin.p, W.per_query.p, W.parena.p,
                           W.agg.p, W.incl.p,  W.out.p,    W.ref.p,       W.cov.p};
  if (memcmp(before, after, sizeof(before)) != 0) W.drop_graph();
  if ((uint64_t)W.epoch + P.scan_launches + 1 >= (1ull << 30)) {
    RS_HIP(launch_fill64(W.agg.as<uint64_t>(), 0, W.agg.bytes / 8, st));
    RS_HIP(launch_fill64(W.incl.as<uint64_t>(), 0, W.incl.bytes / 8, st));
    W.epoch = 0;
  }
  RS_TRY(resolve_plan(P, W, W.epoch));
  size_grids(P);
  if (P.count_lb) {
    const void* before_lb = W.lb.p;
    if (W.lb.reserve(16, st, true)) return RS_ENOMEM;
    if (W.lb.p != before_lb) W.drop_graph();
    RS_HIP(launch_fill64(W.lb.as<uint64_t>(), 0, 2, st));
    P.key += "/lb";  // a captured graph holds the counter pointer
  }
  {
    const void* before_b = W.bounds.p;
    if (W.bounds.reserve(4 * std::max<uint64_t>(P.bounds_words, 1), st, false)) return RS_ENOMEM;
    if (W.bounds.p != before_b) W.drop_graph();
    for (BLaunch& L : P.launches) {
      if (L.top) continue;
      for (uint32_t j = 0; j < L.nunits; ++j) {
        MUnit& U = P.units[L.unit_off + j];
        const uint64_t off = (uintptr_t)U.bounds;
        if (off + 4ull * (U.waves + 1) > W.bounds.bytes) return RS_EINVAL;
        U.bounds = (uint32_t*)(W.bounds.as<char>() + off);
      }
    }
  }
  W.epoch += P.scan_launches + 1;
  RS_HIP(hipMemcpyAsync(W.qs.p, P.qs.data(), sizeof(BQuery) * P.qs.size(), hipMemcpyHostToDevice, st));
  if (!P.units.empty()) {
    RS_HIP(hipMemcpyAsync(W.units.p, P.units.data(), sizeof(MUnit) * P.units.size(), hipMemcpyHostToDevice, st));
    RS_HIP(hipMemcpyAsync(W.ubegin.p, P.ubegin.data(), 4 * P.ubegin.size(), hipMemcpyHostToDevice, st));
  }
  if (!W.ev0) {
    RS_HIP(hipEventCreate(&W.ev0));
    RS_HIP(hipEventCreate(&W.ev1));
  }
  RS_HIP(W.ensure_lanes());
  RS_HIP(hipEventRecord(W.ev0, st));
  {
    ProfScope ps(KC_BATCH, st, 0.0);
    if (use_graph) {
      if (W.key != P.key || !W.exec) {
        W.drop_graph();
        hipStream_t cap = nullptr;
        RS_HIP(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
        hipError_t be = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
        rs_status s = be == hipSuccess ? batch_enqueue(P, W, cap) : RS_EDEVICE;
        hipGraph_t g = nullptr;
        hipError_t ce = be == hipSuccess ? hipStreamEndCapture(cap, &g) : be;
        (void)hipStreamDestroy(cap);
        if (s != RS_OK) {
          if (g) (void)hipGraphDestroy(g);
          return s;
        }
        RS_HIP(ce);
        W.graph = g;
        RS_HIP(hipGraphInstantiate(&W.exec, g, nullptr, nullptr, 0));
        W.key = P.key;
      }
      RS_HIP(hipGraphLaunch(W.exec, st));
    } else {
      RS_TRY(batch_enqueue(P, W, st));
    }
  }
  std::vector<uint64_t> F(P.qs.size());
  RS_HIP(hipMemcpyAsync(F.data(), W.out.p, 8 * F.size(), hipMemcpyDeviceToHost, st));
  RS_HIP(hipEventRecord(W.ev1, st));
  RS_HIP(hipStreamSynchronize(st));
  if (P.count_lb) {
    unsigned long long h[2] = {0, 0};
    RS_HIP(hipMemcpy(h, W.lb.p, sizeof(h), hipMemcpyDeviceToHost));
    lookback_add(h[0], h[1]);
  }
  if (profiling_on()) profile_flush();
  float ms = 0;
  (void)hipEventElapsedTime(&ms, W.ev0, W.ev1);
  for (size_t j = 0; j < P.qs.size(); ++j) {
    rs_result& r = results[P.qidx[j]];
    r.fingerprint = F[j];
    r.yes = F[j] != 0;
    r.status = RS_OK;
  }
  for (uint32_t i = 0; i < nq; ++i) results[i].device_ms = ms;
  if (ran) *ran = true;
  return first_err;
}

// A batched call. Queries over whole iteration ranges run in the coefficient
// form, all of them level by level in shared launches; the rest (ranges, k = 2
// or above the form's largest, rows beyond the budget), and every query when
// the caller gives launch knobs, which describe the evaluation form, run in
// rounds of chunks.
rs_status run_batch_impl(const rs_graph* const* graphs, const rs_query* queries, uint32_t nq, rs_result* results,
                         const rs_tuning* tune, hipStream_t st, bool use_graph, uint64_t slot_budget,
                         BatchWorkspace* ws) {
  if (nq == 0) return RS_OK;
  if (!queries || !results || !graphs) return RS_EINVAL;
  BatchWorkspace& W = ws ? *ws : batch_ws();
  std::lock_guard<std::mutex> lk(W.mu);
  // (a batch that the tuned shape of its first graph refuses stays refused)
  const bool tuned8 = graphs[0] && graphs[0]->has_batch_tuned && graphs[0]->batch_tuned.edges_per_tile == 8 &&
                      std::any_of(graphs, graphs + nq, [](const rs_graph* g) { return g && g->g.m > kMaxEdgesE8; });
  const bool knobs = tuned8 || (tune && (tune->edges_per_tile || tune->top_edges_per_tile || tune->chunks_per_launch ||
                              tune->waves_per_block || tune->max_slots || tune->no_graph || tune->chunks_per_wave));
  std::vector<QueryPlan> plans(nq);
  std::vector<uint32_t> coef, rest;
  for (uint32_t i = 0; i < nq; ++i) {
    const rs_graph* g = graphs[i];
    const bool ok = !knobs && plan_query(g, &queries[i], plans[i]) == RS_OK && plans[i].k >= 3 &&
                    coef_applies(plans[i]) && g->g.m && plans[i].k <= g->g.n;
    (ok ? coef : rest).push_back(i);
  }
  if (coef.empty()) return run_batch_eval(W, graphs, queries, nq, results, tune, st, use_graph, slot_budget);
  if (!W.ev0) {
    RS_HIP(hipEventCreate(&W.ev0));
    RS_HIP(hipEventCreate(&W.ev1));
  }
  RS_HIP(hipEventRecord(W.ev0, st));
  {
    // Both forms use the same two buffers in turn, so that a call holds the larger
    // of the two and not their sum; the evaluation form's records are kept beside
    // them and count against the budget.
    ProfScope ps(KC_BATCH, st, 0.0);
    const uint64_t records = std::min(W.agg.bytes + W.incl.bytes, slot_budget);
    const void* const before[2] = {W.per_query.p, W.parena.p};
    rs_status s = RS_OK;
    for (size_t i = 0; s == RS_OK && i < coef.size(); i += kCoefQueries)
      s = run_coef_batch(*W.coef, W.per_query, W.parena, graphs, plans,
                         std::vector<uint32_t>(coef.begin() + i, coef.begin() + std::min(coef.size(), i + kCoefQueries)),
                         results, st, slot_budget ? slot_budget - records : default_slot_budget(), &rest);
    if (before[0] != W.per_query.p || before[1] != W.parena.p) W.drop_graph();
    RS_TRY(s);
  }
  RS_HIP(hipEventRecord(W.ev1, st));
  RS_HIP(hipEventSynchronize(W.ev1));
  float ms = 0;
  (void)hipEventElapsedTime(&ms, W.ev0, W.ev1);
  if (profiling_on()) profile_flush();
  if (!rest.empty()) {
    std::sort(rest.begin(), rest.end());
    std::vector<const rs_graph*> gl;
    std::vector<rs_query> ql;
    std::vector<rs_result> rl(rest.size());
    for (uint32_t i : rest) {
      gl.push_back(graphs[i]);
      ql.push_back(queries[i]);
    }
    bool ran = false;
    const rs_status s = run_batch_eval(W, gl.data(), ql.data(), (uint32_t)rest.size(), rl.data(), tune, st, use_graph,
                                       slot_budget, &ran);
    float more = 0;
    for (size_t j = 0; j < rest.size(); ++j) {
      if (!ran && rl[j].status == RS_OK) rl[j].status = s;  // without its result
      results[rest[j]] = rl[j];
      more = std::max(more, rl[j].device_ms);
    }
    ms += more;
    if (!ran) return s;
  }
  rs_status first_err = RS_OK;
  for (uint32_t i = 0; i < nq; ++i) {
    results[i].device_ms = ms;
    if (results[i].status != RS_OK && first_err == RS_OK) first_err = results[i].status;
  }
  return first_err;
}

}  // namespace rs

using namespace rs;


// Times candidate launch shapes on the sample queries. Plain path: edges per
// tile, waves per block, last-level range and chunks per launch, best total
// device time per k class. Batched path: edges per tile, waves per block and
// last-level range for the whole sample batch. Results are cached on the graph.
static rs_status autotune_batch_impl(rs_graph* g, const rs_query* sample, uint32_t ns, hipStream_t st);

rs_status autotune_impl(rs_graph* g, const rs_query* sample, uint32_t ns, rs_tuning* out) {
  if (!g || !sample || ns == 0) return RS_EINVAL;
  // Timed on the null stream. A private stream of the autotuner that is
  // alive when the batched path creates its lane streams left every later
  // batched call on that device 15% slower (64 mixed queries on the 10^6-edge
  // graph: 1.05 s instead of 0.89 s, with 4 or 8 lanes, eager or captured).
  hipStream_t st = nullptr;
  std::vector<QueryPlan> plans(ns);
  for (uint32_t i = 0; i < ns; ++i) {
    rs_status s = plan_query(g, &sample[i], plans[i]);
    if (s != RS_OK) return s;
  }
  // plain path, per k present in the sample
  std::vector<Tuning> cands;
  for (uint32_t E : {8u, 16u})
    for (uint32_t wpb : {1u, 2u, 4u})
      for (uint32_t top : {16u, 64u})
        for (uint32_t cpl : {2u, 4u}) {
          if (E == 8 && g->g.m > kMaxEdgesE8) continue;
          Tuning t;
          t.edges_per_tile = E;
          t.waves_per_block = t.top_waves_per_block = wpb;
          t.top_edges_per_tile = top;
          t.chunks_per_launch = cpl;
          t.eval_form = true;  // the shapes timed are the evaluation form's
          cands.push_back(t);
        }
  Tuning best_any;
  for (uint32_t k = 2; k <= RS_MAX_K; ++k) {
    std::vector<uint32_t> idx;
    for (uint32_t i = 0; i < ns; ++i)
      if (plans[i].k == k) idx.push_back(i);
    if (idx.empty()) continue;
    double best = 1e30;
    Tuning bt;
    for (const Tuning& t : cands) {
      double tot = 0;
      for (int rep = 0; rep < 2; ++rep) {
        double run = 0;
        for (uint32_t i : idx) {
          rs_result r;
          std::lock_guard<std::mutex> lk(g->mu);
          rs_status s = run_plain(g, g->ws, plans[i], t, nullptr, &r, st);
          if (s != RS_OK) return s;
          run += r.device_ms;
        }
        tot = rep == 0 ? run : std::min(tot, run);  // first pass warms the workspace
      }
      if (tot < best) {
        best = tot;
        bt = t;
      }
    }
    bt.eval_form = false;
    g->tuned[k] = bt;
    g->has_tuned[k] = true;
    best_any = bt;
  }
  const rs_status bs = autotune_batch_impl(g, sample, ns, st);
  if (bs != RS_OK) return bs;
  if (out) *out = rs_tuning{best_any.edges_per_tile, best_any.top_edges_per_tile, best_any.chunks_per_launch,
                            best_any.waves_per_block, 0, 0};
  return RS_OK;
}

// Batched path: times edges per tile, waves per block and last-level range on
// the sample as one batch and caches the fastest on the graph.
static rs_status autotune_batch_impl(rs_graph* g, const rs_query* sample, uint32_t ns, hipStream_t st) {
  std::vector<const rs_graph*> gl(ns, g);
  std::vector<rs_result> res(ns);
  double best = 1e30;
  Tuning bb;
  for (uint32_t E : {8u, 16u})
    for (uint32_t wpb : {1u, 2u, 4u})
      for (uint32_t top : {16u, 64u, 256u}) {
        if (E == 8 && g->g.m > kMaxEdgesE8) continue;
        rs_tuning t{E, top, 0, wpb, 0, 0};
        double tmin = 1e30;
        for (int rep = 0; rep < 2; ++rep) {
          // timed as real calls run: through a captured graph (the first
          // repetition captures it)
          rs_status s = run_batch_impl(gl.data(), sample, ns, res.data(), &t, st, true, 0, nullptr);
          if (s != RS_OK) return s;
          if (rep) tmin = std::min(tmin, (double)res[0].device_ms);
        }
        if (tmin < best) {
          best = tmin;
          bb.edges_per_tile = E;
          bb.top_edges_per_tile = top;
          bb.waves_per_block = wpb;
        }
      }
  g->batch_tuned = bb;
  g->has_batch_tuned = true;
  return RS_OK;
}

extern "C" rs_status rs_autotune_batch(const rs_graph* g, const rs_query* sample, uint32_t ns, rs_tuning* out) {
  if (!g || !sample || ns == 0) return RS_EINVAL;
  try {
    rs_graph* gm = const_cast<rs_graph*>(g);
    for (uint32_t i = 0; i < ns; ++i) {
      QueryPlan qp;
      const rs_status s = plan_query(gm, &sample[i], qp);
      if (s != RS_OK) return s;
    }
    const rs_status s = autotune_batch_impl(gm, sample, ns, nullptr);  // null stream, as rs_autotune
    if (s == RS_OK && out)
      *out = rs_tuning{gm->batch_tuned.edges_per_tile, gm->batch_tuned.top_edges_per_tile, 0,
                       gm->batch_tuned.waves_per_block, 0, 0};
    return s;
  } catch (...) {
    return RS_ENOMEM;
  }
}

extern "C" rs_status rs_autotune(const rs_graph* g, const rs_query* sample, uint32_t ns, rs_tuning* out) {
  try {
    return autotune_impl(const_cast<rs_graph*>(g), sample, ns, out);
  } catch (...) {
    return RS_ENOMEM;
  }
}

extern "C" rs_status rs_run_batch(const rs_graph* const* graphs, const rs_query* queries, uint32_t nq,
                                  rs_result* results, const rs_tuning* tune, void* hip_stream) {
  try {
    return run_batch_impl(graphs, queries, nq, results, tune, (hipStream_t)hip_stream, true, 0, nullptr);
  } catch (...) {
    return RS_ENOMEM;
  }
}

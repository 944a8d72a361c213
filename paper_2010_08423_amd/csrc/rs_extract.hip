// Extraction of an optimal solution with k fine-grained queries (Sec. 4.7).
//
// Host orchestration over the fine-grained sieve: the path is peeled from its
// last vertex. The first query (k vertices) gives zeta_{u,k,i} per slot; the
// slot with the least time i (then the least u) ends the path, and its time
// is the path's largest timestamp, which is therefore least. Each further
// query (j = k-1 .. 2 vertices) runs on the graph without the vertices found
// so far and without the edges later than the last time found (the
// time-truncated graph tau <- i), with the motif less the found vertices'
// colours; both are constraints of the same sieve (excluded edges get zero
// product rows), so the graph is never rebuilt. A non-zero zeta_{v,j,i}
// proves a restless path with j vertices ending at v at time i that avoids
// the found vertices, so an edge (v, u, t) into the last found vertex u with
// t - delta(v) <= i <= t extends it.
//
// The paper takes the next pair from the reach set R of the smaller query;
// the least reach time of a vertex can lie more than delta(v) before t, so
// the choice here is made among the non-zero slots inside v's waiting
// window. Ties go to the least vertex id, then the least time.
//
// The outputs stay on the device: a small kernel picks the slot, and only its
// vertex and time come back. (Copying zeta, the reach times and the edges to the
// host and looking there took a third of an extraction: 10^5 edges,
// k = 6: 1030 -> 680 us.)
#include <algorithm>
#include <vector>

#include "rs_internal.h"

namespace rs {

struct GoneList {
  uint32_t n, v[RS_MAX_K];
  __device__ __forceinline__ bool has(uint32_t x) const {
    bool h = false;
#pragma unroll
    for (uint32_t i = 0; i < RS_MAX_K; ++i) h = h || (i < n && v[i] == x);
    return h;
  }
};

// First edge of [a, b) with time >= x (times increase over the range).
__device__ __forceinline__ uint32_t first_at(const uint32_t* t, uint32_t a, uint32_t b, uint32_t x) {
  while (a < b) {
    const uint32_t mid = a + ((b - a) >> 1);
    if (t[mid] < x) a = mid + 1; else b = mid;
  }
  return a;
}

// Least (reach time, vertex) of each block's vertices, as time << 32 | vertex.
__global__ __launch_bounds__(1024) void k_pick_least(const uint32_t* __restrict__ reach, uint32_t n, uint64_t* out) {
  __shared__ unsigned long long least;
  if (threadIdx.x == 0) least = ~0ull;
  __syncthreads();
  unsigned long long x = ~0ull;
  for (uint64_t u = blockIdx.x * 1024 + threadIdx.x; u < n; u += gridDim.x * 1024)
    if (reach[u] != 0xFFFFFFFFu) x = min(x, (unsigned long long)reach[u] << 32 | u);
  if (x != ~0ull) atomicMin(&least, x);
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(out + blockIdx.x, (uint64_t)least, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Predecessor of slot (u, t): over the in-edges (v, u, t) by increasing v, the
// first whose v is not gone and has a non-zero slot inside its waiting window;
// that slot's time. One block; its waves take the edges in turn.
__global__ __launch_bounds__(1024) void k_pick_before(const uint32_t* __restrict__ e_src, const uint32_t* __restrict__ e_t,
                                                      const uint32_t* __restrict__ in_off,
                                                      const uint64_t* __restrict__ zeta, uint32_t delta,
                                                      const uint32_t* __restrict__ dv, uint32_t u, uint32_t t,
                                                      GoneList gone, uint64_t* out) {
  __shared__ uint32_t found;  // the first edge found so far
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  if (threadIdx.x == 0) found = 0xFFFFFFFFu;
  const uint32_t end = in_off[u + 1], begin = first_at(e_t, in_off[u], end, t);
  uint32_t mine = 0xFFFFFFFFu, time = 0;
  __syncthreads();
  for (uint32_t e = begin + wv; e < end && e_t[e] == t && e < *(volatile uint32_t*)&found; e += 16) {
    const uint32_t v = e_src[e];
    if (gone.has(v)) continue;
    const uint32_t d = dv ? dv[v] : delta, last = in_off[v + 1];
    for (uint32_t f0 = first_at(e_t, in_off[v], last, t > d ? t - d : 1u); f0 < last; f0 += 64) {
      const uint32_t f = f0 + lane;
      const bool in = f < last && e_t[f] <= t;
      const uint64_t hit = __ballot(in && zeta[f]);
      if (hit) {
        mine = e;
        time = e_t[f0 + (uint32_t)__builtin_ctzll(hit)];
        break;
      }
      if (__ballot(in) != ~0ull) break;
    }
    if (mine != 0xFFFFFFFFu) {
      if (lane == 0) atomicMin(&found, mine);
      break;  // (this wave's later edges come after it)
    }
  }
  __syncthreads();
  if (lane == 0 && (mine == 0xFFFFFFFFu ? wv == 0 && found == 0xFFFFFFFFu : mine == found))
    __hip_atomic_store(out, mine == 0xFFFFFFFFu ? ~0ull : (uint64_t)time << 32 | e_src[mine], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// First vertex of the path: the least v of an edge (v, u, t) that is not gone,
// may be a source and has colour want (if not 256). One wave.
__global__ __launch_bounds__(64) void k_pick_first(const uint32_t* __restrict__ e_src, const uint32_t* __restrict__ e_t,
                                                   const uint32_t* __restrict__ in_off,
                                                   const uint8_t* __restrict__ colour, const uint8_t* __restrict__ smask,
                                                   uint32_t want, uint32_t u, uint32_t t, GoneList gone, uint64_t* out) {
  const uint32_t lane = threadIdx.x, end = in_off[u + 1];
  uint64_t pick = ~0ull;
  for (uint32_t e0 = first_at(e_t, in_off[u], end, t); e0 < end; e0 += 64) {
    const uint32_t e = e0 + lane;
    const bool in = e < end && e_t[e] == t;
    const uint32_t v = in ? e_src[e] : 0;
    const uint64_t hit = __ballot(in && !gone.has(v) && (!smask || smask[v]) && (want > 255 || colour[v] == want));
    if (hit) {
      pick = e_src[e0 + (uint32_t)__builtin_ctzll(hit)];
      break;
    }
    if (__ballot(in) != ~0ull) break;
  }
  if (lane == 0) __hip_atomic_store(out, pick, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

static GoneList gone_list(const SlotPick& p) {
  GoneList g{};
  g.n = p.n_gone;
  std::copy(p.gone, p.gone + p.n_gone, g.v);
  return g;
}

hipError_t launch_pick(const GraphDev& G, const SlotPick& p, uint32_t delta, const uint32_t* dv, const uint64_t* zeta,
                       const uint32_t* reach, uint64_t* out, hipStream_t st) {
  std::fill(out, out + kPickWords, ~0ull);
  if (p.u == 0xFFFFFFFFu)
    hipLaunchKernelGGL(k_pick_least, dim3(std::min(kPickWords, G.n / 4096 + 1)), dim3(1024), 0, st, reach, G.n, out);
  else
    hipLaunchKernelGGL(k_pick_before, dim3(1), dim3(1024), 0, st, G.e_src.as<uint32_t>(), G.e_t.as<uint32_t>(),
                       G.in_off.as<uint32_t>(), zeta, delta, dv, p.u, p.t, gone_list(p), out);
  return hipGetLastError();
}

void read_pick(const uint64_t* out, SlotPick& p) {
  uint64_t x = ~0ull;
  for (uint32_t i = 0; i < kPickWords; ++i) {
    const uint64_t v = ((const volatile uint64_t*)out)[i];
    x = std::min(x, v);
  }
  p.vertex = (uint32_t)x;  // (0xFFFFFFFF where nothing was found)
  p.time = (uint32_t)(x >> 32);
}

// The path's first vertex, before slot (p.u, p.t).
static rs_status pick_first(rs_graph* g, const rs_constraints* c, uint32_t want, SlotPick* p, hipStream_t st) {
  const GraphDev& G = g->g;
  std::vector<uint8_t> mask;
  if (c && c->n_sources) {
    mask.assign(std::max<uint32_t>(G.n, 1), 0);
    for (uint32_t j = 0; j < c->n_sources; ++j) mask[c->sources[j]] = 1;
  }
  std::lock_guard<std::mutex> lk(g->mu);
  PlainWorkspace& ws = g->ws;
  if (!ws.pick_host) RS_HIP(hipHostMalloc((void**)&ws.pick_host, 8 * kPickWords, hipHostMallocDefault));
  const uint8_t* smask = nullptr;
  if (!mask.empty()) {
    if (ws.smask.reserve(mask.size(), st, false)) return RS_ENOMEM;
    RS_HIP(hipMemcpyAsync(ws.smask.p, mask.data(), G.n, hipMemcpyHostToDevice, st));
    smask = ws.smask.as<uint8_t>();
  }
  std::fill(ws.pick_host, ws.pick_host + kPickWords, ~0ull);
  hipLaunchKernelGGL(k_pick_first, dim3(1), dim3(64), 0, st, G.e_src.as<uint32_t>(), G.e_t.as<uint32_t>(),
                     G.in_off.as<uint32_t>(), G.colour.as<uint8_t>(), smask, want, p->u, p->t, gone_list(*p),
                     ws.pick_host);
  RS_HIP(hipGetLastError());
  RS_HIP(hipStreamSynchronize(st));
  read_pick(ws.pick_host, *p);
  return RS_OK;
}

}  // namespace rs

using namespace rs;

rs_status rs_extract(const rs_graph* gc, const rs_query* q, const rs_constraints* c, uint32_t* path_vertices,
                     uint32_t* path_times, rs_result* r, void* hip_stream) {
  if (!gc || !q || !r || !path_vertices || !path_times) return RS_EINVAL;
  if (q->it_begin || q->it_end) return RS_EINVAL;
  if (c && (c->n_removed || c->removed || c->t_max)) return RS_EINVAL;
  if (q->k < 2 || q->k > RS_MAX_K) return RS_EINVAL;
  rs_graph* g = const_cast<rs_graph*>(gc);
  const uint32_t k = q->k;
  hipStream_t st = (hipStream_t)hip_stream;
  rs_status s = RS_OK;
  try {
    // the first query decides; it also validates the query and constraints
    rs_result first{};
    SlotPick p;
    s = run_fine_pick(g, q, c, &p, &first, st);
    if (s != RS_OK) {
      r->status = s;
      return s;
    }
    r->fingerprint = first.fingerprint;
    r->device_ms = first.device_ms;
    if (p.vertex == 0xFFFFFFFFu) {
      r->yes = 0;
      r->status = RS_OK;
      return RS_OK;
    }
    std::vector<uint8_t> motif;
    if (q->motif_count) motif.assign(q->motif_count, q->motif_count + g->g.n_colours);
    std::vector<uint32_t> verts{p.vertex}, times;
    for (uint32_t j = k - 1; j >= 1; --j) {
      p.u = p.vertex;
      p.t = p.time;
      p.gone[p.n_gone++] = p.u;
      if (!motif.empty()) {
        uint8_t cu = 0;
        if (hipMemcpy(&cu, g->g.colour.as<uint8_t>() + p.u, 1, hipMemcpyDeviceToHost) != hipSuccess) {
          s = RS_EDEVICE;
          break;
        }
        if (!motif[cu]) {
          s = RS_EDEVICE;  // the found vertex's colour is not in the motif: an internal error
          break;
        }
        --motif[cu];
      }
      if (j == 1) {
        const uint32_t want =
            motif.empty() ? 256u : (uint32_t)(std::find(motif.begin(), motif.end(), 1) - motif.begin());
        s = pick_first(g, c, want, &p, st);
      } else {
        rs_query qj = *q;
        qj.k = j;
        qj.motif_count = motif.empty() ? nullptr : motif.data();
        rs_constraints cj{};
        if (c) {
          cj.delta_per_vertex = c->delta_per_vertex;
          cj.sources = c->sources;
          cj.n_sources = c->n_sources;
        }
        cj.removed = p.gone;
        cj.n_removed = p.n_gone;
        cj.t_max = p.t;
        rs_result rj{};
        s = run_fine_pick(g, &qj, &cj, &p, &rj, st);
        if (s == RS_OK) r->device_ms += rj.device_ms;
      }
      if (s == RS_OK && p.vertex == 0xFFFFFFFFu) s = RS_ERETRY;
      if (s != RS_OK) break;
      times.push_back(p.t);
      verts.push_back(p.vertex);
    }
    if (s == RS_OK) {
      for (uint32_t j = 0; j < k; ++j) path_vertices[j] = verts[k - 1 - j];
      for (uint32_t j = 0; j + 1 < k; ++j) path_times[j] = times[k - 2 - j];
      r->yes = 1;
    }
  } catch (...) {
    s = RS_ENOMEM;
  }
  r->status = s;
  return s;
}

// Coefficient form of the sieve.
//
// The fingerprint of a full iteration range is the XOR over all L of [k] of
// f(L), with f(L) the walk sum in which vertex v weighs XOR_{j in L} z_{v,j}.
// As a polynomial in k commuting variables x_1..x_k with x_j^2 = 0, let a walk
// v_1 .. v_l with edges e_1 .. e_{l-1} weigh
//   prod_p y_{e_p,p} * prod_p (z_{v_p,1} x_1 + ... + z_{v_p,k} x_k).
// Expanding the product over p of a walk's XOR_{j in L} z_{v_p,j} gives one
// term per map of positions to labels, and a map with image I is counted for
// 2^(k - |I|) sets L, so over GF(2^64) only the bijections survive the sum
// over L: F is the coefficient of x_1 x_2 .. x_k (Eq. multilinear:1 summed over
// L; the determinant of rs.h). The level-l sums are homogeneous of degree l,
// so a level holds C(k,l) coefficients per slot and needs k C(k-1,l-1) products
// per vertex factor, where the evaluation form holds 2^k values and needs 2^k
// products: at k = 10, 967 coefficients over levels 3..9 against 7168. Values
// of single iterations or of a part of the range are not coefficients of
// this polynomial; those queries run by iteration on the same lists (below).
//
// Motif queries: z_{u,j} = XOR_d gamma_{u,d} omega_{d,j} over the shades d of u's
// colour, so det Z_P = det Gamma_P * det Omega with Omega the k x k matrix of the
// omega_{d,j}. The rows are formed with gamma in place of z (one to mu(c(u))
// entries instead of k) and the last level is multiplied by det Omega.
//
// Product sets. An edge enters level l only if a walk of l - 1 edges ends in it
// and one of k - l further edges continues it: every other level value is
// zero, or in no window of the level above. The sets are bitmaps over the
// edges (64 edges per word): forward, F_l = edges whose window holds an edge
// of F_{l-1}; then backward from the last level, S_l = F_l within the windows
// of the edges of S_{l+1}. On the 10^6-edge path query (k = 8) the last level
// keeps 79723 edges of the 291622 whose window is non-empty, level 5 13050 of
// 33433.
//
// Rows. Entry p of level l's list is the p-th edge of S_l. Q_l[p] holds the XOR
// of y_{e,l-1} W_e over the entries of p's destination up to p (C(k,l-1)
// coefficients, W_e the window of the level below), P_l[p] = z_{dst} Q_l[p]. A
// window [x, y) of edge ids becomes the rows of its last entry and of the last
// entry before it (none when the window starts with the first entry of its
// vertex): two rows, whatever delta is.
#include <algorithm>

#include "rs_coef.h"
#include "rs_level.h"

namespace rs {

// ---------------------------------------------------------------------------
// Subsets of [k] by size, in increasing order of their bit masks.
// ---------------------------------------------------------------------------
constexpr uint32_t binom(uint32_t n, uint32_t r) {
  if (r > n) return 0;
  uint64_t v = 1;
  for (uint32_t i = 1; i <= r; ++i) v = v * (n - r + i) / i;
  return (uint32_t)v;
}
struct BinomTable {
  uint32_t v[kCoefMaxK + 1][kCoefMaxK + 1];
};
constexpr BinomTable make_binom() {
  BinomTable t{};
  for (uint32_t n = 0; n <= kCoefMaxK; ++n)
    for (uint32_t r = 0; r <= n; ++r) t.v[n][r] = binom(n, r);
  return t;
}

// For level l of k: every (j, U) with |U| = l - 1 and j outside U, ordered by j
// and then U, as rank(U) | rank(U + j) << 10 | j << 20. k * C(k-1, l-1) pairs.
constexpr uint32_t pair_count(uint32_t k, uint32_t l) { return k * binom(k - 1, l - 1); }
constexpr uint32_t pair_base(uint32_t k, uint32_t l) {
  uint32_t b = 0;
  for (uint32_t kk = 3; kk < k; ++kk)
    for (uint32_t ll = 2; ll < kk; ++ll) b += pair_count(kk, ll);
  for (uint32_t ll = 2; ll < l; ++ll) b += pair_count(k, ll);
  return b;
}
constexpr uint32_t kPairs = pair_base(kCoefMaxK + 1, 2);
struct PairTable {
  uint32_t v[kPairs];
  uint32_t base[kCoefMaxK + 1][kCoefMaxK + 1];
};
constexpr PairTable make_pairs() {
  PairTable t{};
  uint32_t rank[1u << kCoefMaxK] = {};
  uint32_t size[1u << kCoefMaxK] = {};
  uint32_t seen[kCoefMaxK + 1] = {};
  for (uint32_t s = 0; s < (1u << kCoefMaxK); ++s) {
    size[s] = s ? size[s & (s - 1)] + 1 : 0;
    rank[s] = seen[size[s]]++;
  }
  uint32_t at = 0;
  for (uint32_t k = 3; k <= kCoefMaxK; ++k) {
    uint32_t pos[kCoefMaxK + 1] = {};
    for (uint32_t l = 2; l < k; ++l) {
      t.base[k][l] = at;
      pos[l] = at;
      at += pair_count(k, l);
    }
    for (uint32_t j = 0; j < k; ++j)
      for (uint32_t s = 1; s < (1u << k); ++s) {
        const uint32_t l = size[s] + 1;
        if (l >= k || ((s >> j) & 1u)) continue;
        t.v[pos[l]++] = rank[s] | rank[s | (1u << j)] << 10 | j << 20;
      }
  }
  return t;
}
static __device__ const PairTable kPairTable = make_pairs();
static __device__ const BinomTable kBinomD = make_binom();

// ---------------------------------------------------------------------------
// Products by a tabled multiplier.
// ---------------------------------------------------------------------------
// r ^= a * w, unreduced, with the 16 multiples of w as consecutive 8-byte LDS
// entries at `base` (bits 3..6 of base clear). Lanes with the same base and
// different nibbles fall in different banks.
__device__ __forceinline__ void comb8(uint32_t base, uint64_t a, Acc128& r) {
  const uint32_t a0 = lo32(a), a1 = hi32(a);
  uint32_t d0 = 0, d1 = 0, d2 = 0, d3 = 0;
#pragma unroll
  for (int j = 7; j >= 0; --j) {
    const uint32_t s0 = (4 * j >= 3) ? (a0 >> (4 * j - 3)) : (a0 << (3 - 4 * j));
    const uint32_t s1 = (4 * j >= 3) ? (a1 >> (4 * j - 3)) : (a1 << (3 - 4 * j));
    const uint64_t x = lds_load(and_xor(s0, 0x78u, base));
    const uint64_t y = lds_load(and_xor(s1, 0x78u, base));
    d0 ^= lo32(x);
    d1 = xor3(d1, hi32(x), lo32(y));
    d2 ^= hi32(y);
    if (j) {
      d3 = funnel(d3, d2, 28);
      d2 = funnel(d2, d1, 28);
      d1 = funnel(d1, d0, 28);
      d0 <<= 4;
    }
  }
  r.d0 ^= d0;
  r.d1 ^= d1;
  r.d2 ^= d2;
  r.d3 ^= d3;
}

// v * w mod p for a polynomial v of degree < 4.
__device__ __forceinline__ uint64_t multiple(uint64_t w, uint32_t v) {
  uint32_t l1 = lo32(w), h1 = hi32(w);
  uint32_t l2 = l1, h2 = h1;
  gf_times_x(l2, h2);
  uint32_t l4 = l2, h4 = h2;
  gf_times_x(l4, h4);
  uint32_t l8 = l4, h8 = h4;
  gf_times_x(l8, h8);
  const uint32_t m0 = 0u - (v & 1u), m1 = 0u - ((v >> 1) & 1u), m2 = 0u - ((v >> 2) & 1u), m3 = 0u - ((v >> 3) & 1u);
  const uint32_t lo = and_xor(l1, m0, and_xor(l2, m1, and_xor(l4, m2, l8 & m3)));
  const uint32_t hi = and_xor(h1, m0, and_xor(h2, m1, and_xor(h4, m2, h8 & m3)));
  return mk64(lo, hi);
}

// Orders a wave's own LDS accesses for the compiler (the hardware keeps one
// wave's LDS operations in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Bit ranges.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t bits_from(uint32_t x) { return ~0ull << (x & 63u); }
__device__ __forceinline__ uint64_t bits_below_incl(uint32_t x) { return ~0ull >> (63u - (x & 63u)); }

// Is a bit of [x, y) set, x < y; sum holds a bit per non-zero word.
__device__ __forceinline__ bool any_bit(const uint64_t* w, const uint64_t* sum, uint32_t x, uint32_t y) {
  uint32_t a = x >> 6, b = (y - 1) >> 6;
  const uint64_t ma = bits_from(x), mb = bits_below_incl(y - 1);
  if (a == b) return (w[a] & ma & mb) != 0;
  if ((w[a] & ma) | (w[b] & mb)) return true;
  x = a + 1;
  y = b;  // whole words [x, y)
  if (x >= y) return false;
  a = x >> 6;
  b = (y - 1) >> 6;
  const uint64_t na = bits_from(x), nb = bits_below_incl(y - 1);
  if (a == b) return (sum[a] & na & nb) != 0;
  if ((sum[a] & na) | (sum[b] & nb)) return true;
  for (uint32_t i = a + 1; i < b; ++i)
    if (sum[i]) return true;
  return false;
}

// ---------------------------------------------------------------------------
// Query setup: windows, vertex forms and product sets. Bound by latency and
// by reading 8 to 20 bytes per edge; the bitmaps stay in the L2.
// ---------------------------------------------------------------------------
// The kernels take one query by value (OneCoef) or an array of them in device
// memory, one per grid slice (ManyCoef).
struct OneCoef {
  CoefQuery q;
  CoefShades sh;
  __device__ __forceinline__ CoefQuery get(uint32_t) const { return q; }
  __device__ __forceinline__ uint32_t mu(uint32_t, uint32_t c) const { return sh.mu[c]; }
  __device__ __forceinline__ uint32_t off(uint32_t, uint32_t c) const { return sh.off[c]; }
  __device__ __forceinline__ uint32_t waves(uint32_t, uint32_t l) const { return sh.waves[l]; }
};
struct ManyCoef {
  const CoefQuery* qs;
  const CoefShades* sh;
  __device__ __forceinline__ CoefQuery get(uint32_t i) const { return qs[i]; }
  __device__ __forceinline__ uint32_t mu(uint32_t i, uint32_t c) const { return sh[i].mu[c]; }
  __device__ __forceinline__ uint32_t off(uint32_t i, uint32_t c) const { return sh[i].off[c]; }
  __device__ __forceinline__ uint32_t waves(uint32_t i, uint32_t l) const { return uniform(sh[i].waves[l]); }
};

// det Omega (motif queries): the coefficient of x_1 .. x_k in the product of
// the k shade forms, by the same rule as a walk's. One block of 1024 threads.
struct DetShared {
  uint64_t tab[kCoefMaxK * 16];  // multiples of the row's k entries
  uint64_t row[2][1024];
};
__device__ void shade_det(const CoefQuery& Q, DetShared& sh) {
  const uint32_t k = Q.k, tid = threadIdx.x;
  if (tid < k) sh.row[0][tid] = hash1(Q.seed, 'W', (uint64_t)0 | ((uint64_t)(tid + 1) << 32));
  uint32_t cur = 0;
  for (uint32_t l = 2; l < k; ++l) {  // row l of Omega times the product of the rows before it
    __syncthreads();
    if (tid < k * 16) sh.tab[tid] = multiple(hash1(Q.seed, 'W', (uint64_t)(l - 1) | ((uint64_t)(tid / 16 + 1) << 32)), tid & 15u);
    sh.row[cur ^ 1][tid] = 0;
    __syncthreads();
    const uint32_t np = k * kBinomD.v[k - 1][l - 1];
    const uint32_t* pr = kPairTable.v + kPairTable.base[k][l];
    for (uint32_t i = tid; i < np; i += blockDim.x) {
      const uint32_t w = pr[i];
      Acc128 r = {0, 0, 0, 0};
      comb8(lds_addr(sh.tab) + (w >> 20) * 128u, sh.row[cur][w & 1023u], r);
      atomicXor((unsigned long long*)&sh.row[cur ^ 1][(w >> 10) & 1023u], (unsigned long long)gf_reduce(r));
    }
    cur ^= 1;
  }
  __syncthreads();
  // last row: the set that lacks label j has rank k - 1 - j
  if (tid < k * 16) sh.tab[tid] = multiple(hash1(Q.seed, 'W', (uint64_t)(k - 1) | ((uint64_t)(tid / 16 + 1) << 32)), tid & 15u);
  __syncthreads();
  if (tid == 0) {
    Acc128 r = {0, 0, 0, 0};
    for (uint32_t j = 0; j < k; ++j) comb8(lds_addr(sh.tab) + j * 128u, sh.row[cur][k - 1 - j], r);
    *Q.det = gf_reduce(r);
  }
}

// The block's 16 summary bits (a bit per non-zero word).
__device__ __forceinline__ void block_summary(const uint64_t* wl, uint64_t* sum, uint32_t block) {
  if (threadIdx.x < 64) {
    const uint64_t s = __ballot(threadIdx.x < 16 && wl[threadIdx.x & 15u] != 0);
    if (threadIdx.x == 0) ((uint16_t*)sum)[block] = (uint16_t)s;
  }
}

// Entry idx of the vertex rows [n][kq] (motif queries: gamma in place of z).
template <class A>
__device__ __forceinline__ uint64_t vertex_form(const A& arg, const CoefQuery& Q, uint32_t i, uint64_t idx) {
  const uint32_t u = (uint32_t)(idx / Q.kq), j = (uint32_t)(idx % Q.kq);
  if (j >= Q.k) return 0;
  if (!Q.motif) return hash1(Q.seed, 'Z', (uint64_t)u | ((uint64_t)(j + 1) << 32));
  const uint32_t c = Q.colour[u], o = arg.off(i, c);
  return j >= o && j < o + arg.mu(i, c) ? hash1(Q.seed, 'G', (uint64_t)u | ((uint64_t)j << 32)) : 0;
}

// First kernel of a query. Block roles: edges (the window of each edge by
// binary search over its source's arrivals, whether a walk may use it, and
// the level-2 set), vertex rows, and for motif queries one block for det Omega.
// Every block clears its share of the scratch the later kernels add to.
template <class A>
__global__ __launch_bounds__(1024) void k_coef_begin(A arg) {
  __shared__ union {
    struct {
      uint64_t f2[16], f3[16];
    } w;
    DetShared d;
  } sh;
  const CoefQuery Q = arg.get(blockIdx.y);
  const uint32_t tid = threadIdx.x;
  const uint32_t nbz = (uint32_t)(((uint64_t)Q.n * Q.kq + 1023) / 1024);
  {
    const uint64_t i0 = (uint64_t)blockIdx.x * 1024 + tid, step = (uint64_t)gridDim.x * 1024;
    const uint64_t nc = (uint64_t)(Q.k - 2) * mark_stride(Q.blocks) / 8, nl = (uint64_t)(Q.k - 1) * flag_stride(Q.words) / 8;
    uint64_t* mk = reinterpret_cast<uint64_t*>(Q.mark);
    for (uint64_t i = i0; i < nc; i += step) mk[i] = 0;
    uint64_t* st = reinterpret_cast<uint64_t*>(Q.store);
    for (uint64_t i = i0; i < nl; i += step) st[i] = 0;
    if (Q.fine)
      for (uint64_t i = i0; i < Q.m; i += step) Q.T[i] = 0;
  }
  if (blockIdx.x < Q.blocks) {
    uint64_t* f2 = Q.fbits;
    uint64_t* f3 = Q.fbits + Q.words + Q.words / 64;
    {
      const uint32_t e = blockIdx.x * kSetBlock + tid;
      bool ok = false, first = false, live = false;
      if (e < Q.m) {
        const uint32_t v = Q.e_src[e], u = Q.e_dst[e], t = Q.e_t[e];
        ok = !(Q.f.rmask && (Q.f.rmask[v] | Q.f.rmask[u])) && !(Q.f.t_max && t > Q.f.t_max);
        if (Q.motif) {
          const uint32_t cv = Q.colour[v], cu = Q.colour[u];
          const uint32_t mv = arg.mu(blockIdx.y, cv), mu = arg.mu(blockIdx.y, cu);
          ok = ok && mv && mu && (Q.iters || !(cv == cu && mu == 1));  // (two vertices of one shade: zero only in the sum over all iterations)
        }
        if (ok) {  // (no set takes another edge, so its window is never read)
          const uint32_t dv = Q.dv ? Q.dv[v] : Q.delta;
          const uint32_t thr = t > dv ? t - dv : 0u;
          const uint32_t y = Q.hi[e] - v;
          // the first arrival at v since thr: arrivals past y are later than t, and
          // most windows are short, so the search doubles back from y before it
          // halves (10^6-edge path query: half the windows hold two arrivals or
          // fewer, of up to 7000)
          const uint32_t off = Q.in_off[v];
          uint32_t a = off, b = y;
          for (uint32_t d = 1; b > off; d *= 2) {
            const uint32_t at = b - off > d ? b - d : off;
            if (Q.e_t[at] < thr) {
              a = at + 1;
              break;
            }
            b = at;
          }
          while (a < b) {
            const uint32_t mid = a + ((b - a) >> 1);
            if (Q.e_t[mid] < thr)
              a = mid + 1;
            else
              b = mid;
          }
          Q.win[e] = make_uint2(a, y);
          live = a < y;
        }
        first = ok && (!Q.f.smask || Q.f.smask[v]);
      }
      const uint64_t wv = __ballot(ok), wf = __ballot(first), wl = __ballot(live);
      const uint32_t lw = tid >> 6, w = blockIdx.x * 16 + lw;
      if ((tid & 63u) == 0) {
        Q.valid[w] = wv;
        f2[w] = wf;
        sh.w.f2[lw] = wf;
        if (Q.plain) {
          f3[w] = wl;
          sh.w.f3[lw] = wl;
        }
      }
    }
    __syncthreads();
    block_summary(sh.w.f2, f2 + Q.words, blockIdx.x);
    if (Q.plain) block_summary(sh.w.f3, f3 + Q.words, blockIdx.x);
  } else if (blockIdx.x < Q.blocks + nbz) {
    const uint64_t idx = (uint64_t)(blockIdx.x - Q.blocks) * 1024 + tid;
    if (idx < (uint64_t)Q.n * Q.kq) {
      Q.z[idx] = vertex_form(arg, Q, blockIdx.y, idx);
    }
  } else if (Q.motif && blockIdx.x == Q.blocks + nbz) {
    shade_det(Q, sh.d);
  }
}

// Writes word w of level index y's set, keeps it for the block's ranks.
__device__ __forceinline__ void set_word(const CoefQuery& Q, uint32_t y, uint32_t w, uint64_t s, uint64_t* wl) {
  if ((threadIdx.x & 63u) == 0) {
    Q.sbits[(uint64_t)y * Q.words + w] = s;
    wl[w & 15u] = s;
  }
}
// Ranks of the block's words and its total, once its words are written.
__device__ __forceinline__ void set_ranks(const CoefQuery& Q, uint32_t y, uint32_t block, const uint64_t* wl) {
  __syncthreads();
  if (threadIdx.x < 16) {
    const uint32_t c = __popcll(wl[threadIdx.x]);
    uint32_t s = c;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const uint32_t v = __shfl_up(s, d, 16);
      if ((int)threadIdx.x >= d) s += v;
    }
    Q.wrank[(uint64_t)y * Q.words + block * 16 + threadIdx.x] = s - c;
    if (threadIdx.x == 15) Q.bsum[(uint64_t)y * Q.blocks + block] = s;
  }
}

// Marks the last edge of a window for the level with index y, and that edge's
// block. A window is marked by its end alone (see k_coef_bwd), and
// by plain byte stores: setting every covered edge's bit by atomics made a
// hub's windows queue up on the same words (16 us of 20 per level on the
// 10^6-edge path query).
__device__ __forceinline__ void mark_window(const CoefQuery& Q, uint32_t y, uint2 w) {
  if (w.x < w.y) {
    uint8_t* m = Q.mark + (uint64_t)y * mark_stride(Q.blocks);
    m[w.y - 1] = 1;
    m[(uint64_t)Q.blocks * kSetBlock + (w.y - 1) / kSetBlock] = 1;
  }
}

// Forward set of level l (3..fwd): valid edges whose window holds an edge of
// the level below. The last pass also gives the last level's set (edges into
// a target) and marks its windows.
template <class A>
__global__ __launch_bounds__(1024) void k_coef_fwd(A arg, uint32_t l) {
  __shared__ uint64_t wl[16], sl[16];
  const CoefQuery Q = arg.get(blockIdx.y);
  if (l > Q.fwd || blockIdx.x >= Q.blocks || (Q.plain && l == 3 && Q.fwd > 3)) return;
  const bool last = l == Q.fwd;
  const uint64_t fstride = Q.words + Q.words / 64;
  const uint64_t* below = Q.fbits + (uint64_t)(l - 3) * fstride;
  uint64_t* here = Q.fbits + (uint64_t)(l - 2) * fstride;
  const uint64_t* base = Q.nested ? below : Q.valid;
  const uint32_t lw = threadIdx.x >> 6, w = blockIdx.x * 16 + lw;
  const uint32_t e = w * 64 + (threadIdx.x & 63u);
  bool in = (base[w] >> (threadIdx.x & 63u)) & 1u;  // bits past m are zero
  uint2 x = make_uint2(0, 0);
  if (in) {
    x = Q.win[e];
    in = x.x < x.y && any_bit(below, below + Q.words, x.x, x.y);
  }
  const uint64_t f = __ballot(in);
  if ((threadIdx.x & 63u) == 0) {
    here[w] = f;
    wl[lw] = f;
  }
  if (last) {
    const bool s = in && (!Q.f.tmask || Q.f.tmask[Q.e_dst[e]]);
    set_word(Q, Q.k - 2, w, __ballot(s), sl);
    if (s) mark_window(Q, Q.k - 3, x);
  }
  if (last) {
    set_ranks(Q, Q.k - 2, blockIdx.x, sl);
  } else {
    __syncthreads();
    block_summary(wl, here + Q.words, blockIdx.x);
  }
}

// Product set of level l (k-1 .. 2): the edges of the forward set inside the
// window of an edge of the level above, whose own windows are then marked for
// the level below.
//
// A window of a vertex's departure at time t holds the vertex's arrivals of
// [t - delta, t], so among the marked windows that end at or after arrival e the
// one ending first reaches back furthest: e lies in a window if the first
// marked arrival at or after e (of the same vertex) is at most delta later. (That
// arrival stands for the departure's own time, which may be later still, so
// a few edges too many pass; a larger set changes no result, only its cost.)
// The first mark is found in the block's bitmap; for the segment that goes on
// past the block's end it is looked up once per block.
//
// R: set blocks per thread block. An edge's work is a chain of four dependent
// loads, so on graphs that fill the GPU anyway (kWideSets) a thread takes four edges with
// their loads in flight together (4*10^6 edges: 30 us per level with one edge
// per thread, 20 with four); on small graphs one edge per thread finishes
// earlier.
template <class A, int R>
__global__ __launch_bounds__(1024) void k_coef_bwd(A arg, uint32_t l_from_top) {
  constexpr uint32_t kEdges = R * kSetBlock, kWords = R * 16;
  __shared__ uint64_t sl[16], mw[kWords];
  __shared__ uint32_t sd[kEdges], stm[kEdges];
  __shared__ uint32_t next;
  const CoefQuery Q = arg.get(blockIdx.y);
  if (l_from_top + 2 > Q.k || blockIdx.x * R >= Q.blocks) return;
  const uint32_t l = Q.k - l_from_top, tid = threadIdx.x, lane = tid & 63u;
  const uint64_t* f = Q.fbits + (uint64_t)(min(l, Q.fwd) - 2) * (Q.words + Q.words / 64);
  const uint8_t* mk = Q.mark + (uint64_t)(l - 2) * mark_stride(Q.blocks);
  const uint8_t* mb = mk + (uint64_t)Q.blocks * kSetBlock;
  const uint32_t e0 = blockIdx.x * kEdges, e1 = min(e0 + kEdges, Q.m);
  uint64_t fw[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = r * 1024 + tid, e = e0 + i;
    fw[r] = f[e >> 6];
    sd[i] = e < Q.m ? Q.e_dst[e] : kNoRow;
    stm[i] = e < Q.m ? Q.e_t[e] : 0u;
    const uint64_t w = __ballot(mk[e]);  // (the marks past m are zero)
    if (lane == 0) mw[i >> 6] = w;
  }
  // the first mark past the block: in one of the next 64 set blocks, looked up by
  // the first wave while the others load
  const uint32_t b1 = (blockIdx.x + 1) * R;
  if (tid < 64) {
    const uint64_t s = __ballot(b1 + lane < Q.blocks && mb[b1 + lane]);
    uint32_t first = kNoRow;
    if (s) {
      const uint32_t found = b1 + (uint32_t)__builtin_ctzll(s);
      const uint4 x = ((const uint4*)(mk + (uint64_t)found * kSetBlock))[lane];
      const uint32_t ln = (uint32_t)__builtin_ctzll(__ballot((x.x | x.y | x.z | x.w) != 0));
      const uint32_t q = x.x ? (uint32_t)__builtin_ctz(x.x) / 8
                             : x.y ? 4 + (uint32_t)__builtin_ctz(x.y) / 8
                                   : x.z ? 8 + (uint32_t)__builtin_ctz(x.z) / 8
                                         : x.w ? 12 + (uint32_t)__builtin_ctz(x.w) / 8 : 0;
      first = found * kSetBlock + ln * 16 + __shfl(q, ln, 64);
    }
    if (tid == 0) next = first;
  }
  const uint32_t u_last = Q.e_dst[e1 > e0 ? e1 - 1 : 0], seg_end = Q.in_off[u_last + 1];
  __syncthreads();
  if (next == kNoRow && seg_end > (b1 + 64) * kSetBlock) {  // the last vertex's arrivals go on past those
    const uint32_t b_end = (seg_end - 1) / kSetBlock;       // last set block of the segment
    uint32_t found = kNoRow;
    __syncthreads();
    for (uint32_t b0 = b1 + 64; b0 <= b_end; b0 += 1024) {
      if (b0 + tid <= b_end && mb[b0 + tid]) atomicMin(&next, b0 + tid);
      __syncthreads();
      found = next;
      __syncthreads();  // every wave has read this step's minimum before another one lowers or clears it
      if (found != kNoRow) break;
    }
    if (tid == 0) next = kNoRow;
    __syncthreads();
    if (found != kNoRow) {
      if (mk[(uint64_t)found * kSetBlock + tid]) atomicMin(&next, found * kSetBlock + tid);
      __syncthreads();
    }
  }
  const uint64_t nz = __ballot(mw[min(lane, kWords - 1)] != 0);  // words with a mark
  bool in[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = r * 1024 + tid, lw = i >> 6;
    in[r] = (fw[r] >> lane) & 1u;
    if (in[r]) {
      uint32_t y = next;  // first mark at or after the edge
      const uint64_t here = mw[lw] & bits_from(lane), later = lw + 1 < kWords ? nz & (~0ull << (lw + 1)) : 0;
      const uint32_t w = here ? lw : (later ? (uint32_t)__builtin_ctzll(later) : kWords);
      if (w < kWords) y = e0 + w * 64 + (uint32_t)__builtin_ctzll(here ? here : mw[w]);
      in[r] = false;
      if (y != kNoRow) {
        const uint32_t u = sd[i];
        const bool inside = y < e1;
        const uint32_t yu = inside ? sd[y - e0] : (y < seg_end ? u_last : kNoRow);
        if (yu == u) in[r] = (inside ? stm[y - e0] : Q.e_t[y]) - stm[i] <= (Q.dv ? Q.dv[u] : Q.delta);
      }
    }
  }
  uint2 win[R];
  if (l > 2) {
#pragma unroll
    for (int r = 0; r < R; ++r) win[r] = in[r] ? Q.win[e0 + r * 1024 + tid] : make_uint2(0, 0);
#pragma unroll
    for (int r = 0; r < R; ++r) mark_window(Q, l - 3, win[r]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r) __syncthreads();
    set_word(Q, l - 2, (e0 >> 6) + r * 16 + (tid >> 6), __ballot(in[r]), sl);
    set_ranks(Q, l - 2, blockIdx.x * R + r, sl);
  }
}

// All of k_coef_fwd, k_coef_bwd and k_coef_offsets in one block, for small graphs:
// there those launches do little but follow each other, and the host enqueues
// no faster than they run. A thread keeps the windows of its four edges, one per
// set block, over all levels. (Per query, median: 1000 edges, k = 5: 115 -> 95 us;
// 4000: 120 -> 101; 4000, k = 9: 215 -> 189. 10^4 edges in one block: 44 us
// against 30 in six launches, so it ends at 4096 edges.)
constexpr uint32_t kSmallWords = 64;  // 4096 edges
template <class A>
__global__ __launch_bounds__(1024) void k_coef_sets_small(A arg) {
  constexpr uint32_t R = kSmallWords / 16;
  __shared__ uint64_t f[kCoefMaxK - 1][kSmallWords], fs[kCoefMaxK - 1][kSmallWords / 64];  // forward sets by level - 2
  __shared__ uint64_t mw[kSmallWords], ms[kSmallWords / 64], sl[kSmallWords];
  __shared__ uint4 mk4[kSetBlock];  // window ends, a byte per edge
  __shared__ uint32_t bs[R];
  uint8_t* mk = reinterpret_cast<uint8_t*>(mk4);
  const CoefQuery Q = arg.get(blockIdx.y);
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6, nr = (Q.m + kSetBlock - 1) / kSetBlock;
  auto summary = [&](const uint64_t* w, uint64_t* s) {
    if (tid < kSmallWords) {
      const uint64_t b = __ballot(w[tid] != 0);
      if (lane == 0) s[wv] = b;
    }
  };
  // set words sl: written out with their ranks, block sums and offsets
  auto finish = [&](uint32_t y) {
    if (tid < Q.words) {
      const uint32_t c = __popcll(sl[tid]);
      uint32_t s = c;
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) {
        const uint32_t v = __shfl_up(s, d, 16);
        if ((int)(tid & 15u) >= d) s += v;
      }
      Q.sbits[(uint64_t)y * Q.words + tid] = sl[tid];
      Q.wrank[(uint64_t)y * Q.words + tid] = s - c;
      if ((tid & 15u) == 15u) {
        Q.bsum[(uint64_t)y * Q.blocks + tid / 16] = s;
        bs[tid / 16] = s;
      }
    }
    __syncthreads();
    if (tid <= Q.blocks) {
      uint32_t s = 0;
      for (uint32_t b = 0; b < tid; ++b) s += bs[b];
      if (tid < Q.blocks)
        Q.boff[(uint64_t)y * Q.blocks + tid] = s;
      else
        Q.count[y] = s;
    }
  };
  uint2 win[R];
  uint32_t end[R], et[R];  // end of the edge's destination's arrivals, its time
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t e = r * kSetBlock + tid;
    win[r] = make_uint2(0, 0);
    end[r] = et[r] = 0;
    if (e < Q.m) {
      win[r] = Q.win[e];
      end[r] = Q.in_off[Q.e_dst[e] + 1];
      et[r] = Q.e_t[e];
    }
  }
  const uint64_t fstride = Q.words + Q.words / 64;
  if (tid < kSmallWords) {
    f[0][tid] = tid < Q.words ? Q.fbits[tid] : 0;
    f[1][tid] = tid < Q.words && Q.plain ? Q.fbits[fstride + tid] : 0;
    mw[tid] = sl[tid] = 0;
    for (uint32_t l = 2; l < kCoefMaxK - 1; ++l) f[l][tid] = 0;
  }
  __syncthreads();
  summary(f[0], fs[0]);
  summary(f[1], fs[1]);
  __syncthreads();
  for (uint32_t l = Q.plain && Q.fwd > 3 ? 4 : 3; l <= Q.fwd; ++l) {
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      if (r >= nr) break;
      const uint32_t w = r * 16 + wv;
      const uint64_t base = Q.nested ? f[l - 3][w] : Q.valid[w];
      const bool in = ((base >> lane) & 1u) && win[r].x < win[r].y && any_bit(f[l - 3], fs[l - 3], win[r].x, win[r].y);
      const uint64_t b = __ballot(in);
      if (lane == 0) f[l - 2][w] = b;
    }
    __syncthreads();
    summary(f[l - 2], fs[l - 2]);
    __syncthreads();
  }
  mk4[tid] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  for (uint32_t l = Q.k; l >= 2; --l) {
    if (l < Q.k) {  // the marks of the level above
#pragma unroll
      for (uint32_t r = 0; r < R; ++r) {
        if (r >= nr) break;
        const uint64_t b = __ballot(mk[r * kSetBlock + tid] != 0);
        if (lane == 0) mw[r * 16 + wv] = b;
      }
      __syncthreads();
      summary(mw, ms);
      mk4[tid] = make_uint4(0, 0, 0, 0);
      __syncthreads();
    }
    const uint64_t* fl = f[min(l, Q.fwd) - 2];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      if (r >= nr) break;
      const uint32_t w = r * 16 + wv, e = r * kSetBlock + tid;
      bool in = (fl[w] >> lane) & 1u;
      if (in && l == Q.k) in = !Q.f.tmask || Q.f.tmask[Q.e_dst[e]];
      if (in && l < Q.k) {
        uint32_t y = kNoRow;  // first mark at or after the edge
        const uint64_t here = mw[w] & bits_from(lane);
        if (here) {
          y = w * 64 + (uint32_t)__builtin_ctzll(here);
        } else if (w + 1 < kSmallWords) {
          uint32_t i = (w + 1) >> 6;
          uint64_t s = ms[i] & bits_from(w + 1);
          while (!s && ++i < kSmallWords / 64) s = ms[i];
          if (s) {
            const uint32_t x = i * 64 + (uint32_t)__builtin_ctzll(s);
            y = x * 64 + (uint32_t)__builtin_ctzll(mw[x]);
          }
        }
        in = y < end[r] && Q.e_t[y] - et[r] <= (Q.dv ? Q.dv[Q.e_dst[e]] : Q.delta);
      }
      const uint64_t b = __ballot(in);
      if (lane == 0) sl[w] = b;
      if (in && l > 2 && win[r].x < win[r].y) mk[win[r].y - 1] = 1;
    }
    __syncthreads();
    finish(l - 2);
  }
}

// Set sizes and the blocks' offsets, one block per level.
template <class A>
__global__ __launch_bounds__(1024) void k_coef_offsets(A arg) {
  const CoefQuery Q = arg.get(blockIdx.y);
  const uint32_t y = blockIdx.x;
  if (y + 1 >= Q.k) return;
  uint32_t* bo = Q.boff + (uint64_t)y * Q.blocks;
  const uint32_t* bs = Q.bsum + (uint64_t)y * Q.blocks;
  __shared__ uint32_t part[16];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
  uint32_t before = 0;
  for (uint32_t b0 = 0; b0 < Q.blocks; b0 += 4096) {  // four sums per thread
    const uint32_t b = b0 + tid * 4;
    const uint4 x = b < Q.blocks ? *(const uint4*)(bs + b) : make_uint4(0, 0, 0, 0);  // blocks is a multiple of 4
    const uint32_t c = x.x + x.y + x.z + x.w;
    uint32_t s = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t v = __shfl_up(s, d, 64);
      if ((int)lane >= d) s += v;
    }
    if (lane == 63) part[wv] = s;
    __syncthreads();
    uint32_t o = before, total = before;
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) {
      if (i < wv) o += part[i];
      total += part[i];
    }
    o += s - c;
    if (b < Q.blocks) *(uint4*)(bo + b) = make_uint4(o, o + x.x, o + x.x + x.y, o + x.x + x.y + x.z);
    before = total;
    __syncthreads();
  }
  if (tid == 0) Q.count[y] = before;
}

// Edges of the set with index y among the first x edges.
__device__ __forceinline__ uint32_t set_rank(const CoefQuery& Q, uint32_t y, uint32_t x) {
  if (x == 0) return 0;
  const uint32_t e = x - 1, w = e >> 6;
  const uint64_t at = (uint64_t)y * Q.words + w;
  return Q.boff[(uint64_t)y * Q.blocks + w / 16] + Q.wrank[at] + __popcll(Q.sbits[at] & bits_below_incl(e));
}

// The lists: per entry its window rows, destination and y value; the rows a
// window reads and the entries that start a destination, as bytes by list
// position. One block per 1024 edges and level: the block's set bits are
// gathered into LDS first, so that the lanes of the second part (a hash and
// four dependent rank look-ups per entry) are all busy. A set holds a few
// percent of the edges: one lane per edge and level took 232 us on the
// 10^6-edge path query (k = 8), one lane per entry 20.
template <class A>
__global__ __launch_bounds__(256) void k_coef_lists(A arg) {
  __shared__ struct {
    uint64_t dtab[16];  // multiples of det Omega (motif); at LDS address 0
    uint16_t edge[kSetBlock];
  } sh;
  const CoefQuery Q = arg.get(blockIdx.z);
  const uint32_t y = blockIdx.y;
  if (y + 1 >= Q.k || blockIdx.x >= Q.blocks) return;
  const uint32_t l = y + 2, lane = threadIdx.x & 63u;
  const uint64_t lo = (uint64_t)y * Q.lstride;
  const bool top = l == Q.k;
  if (blockIdx.x == 0 && threadIdx.x < 8) {  // a scan tile reads past the list's end
    const uint64_t p = lo + Q.count[y] + threadIdx.x;
    Q.l_hi[p] = kNoRow;
    Q.l_lo[p] = kNoRow;
    Q.l_dst[p] = 0;
    Q.l_y[p] = 0;
    Q.restart[(uint64_t)y * flag_stride(Q.words) + Q.count[y] + threadIdx.x] = 0;
  }
  const uint32_t n = Q.bsum[(uint64_t)y * Q.blocks + blockIdx.x];
  if (n == 0) return;
  if (top && Q.motif && !Q.iters && threadIdx.x < 16) sh.dtab[threadIdx.x] = multiple(*Q.det, threadIdx.x);
#pragma unroll
  for (uint32_t r = 0; r < 4; ++r) {
    const uint32_t lw = r * 4 + (threadIdx.x >> 6);
    const uint64_t at = (uint64_t)y * Q.words + blockIdx.x * 16 + lw;
    const uint64_t bits = Q.sbits[at];
    if ((bits >> lane) & 1ull) sh.edge[Q.wrank[at] + __popcll(bits & ((1ull << lane) - 1))] = (uint16_t)(lw * 64 + lane);
  }
  __syncthreads();
  const uint32_t p0 = Q.boff[(uint64_t)y * Q.blocks + blockIdx.x];
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    const uint32_t e = blockIdx.x * kSetBlock + sh.edge[i], p = p0 + i;
    const uint32_t src = Q.e_src[e], dst = Q.e_dst[e], t = Q.e_t[e];
    uint32_t h = kNoRow, o = kNoRow;
    if (l == 2) {
      h = Q.by_entry ? p : src;
      if (Q.by_entry) Q.l_e[p] = src;
    } else {
      const uint2 x = Q.win[e];
      const uint32_t first = Q.in_off[src];
      const uint32_t ra = set_rank(Q, y - 1, x.x), rb = set_rank(Q, y - 1, x.y), rf = set_rank(Q, y - 1, first);
      uint8_t* st = Q.store + (uint64_t)(y - 1) * flag_stride(Q.words);
      if (rb > ra) {  // (bytes, not bits: the windows of a hub mark the same rows, and atomics on one word queue up)
        h = rb - 1;
        st[h] = 1;
        if (ra > rf) {
          o = ra - 1;
          st[o] = 1;
        }
      }
    }
    uint64_t yv = hash2(Q.seed, 'Y', (uint64_t)src | ((uint64_t)dst << 32), (uint64_t)t | ((uint64_t)(l - 1) << 32));
    if (top) {
      if (Q.motif && !Q.iters) {
        Acc128 v = {0, 0, 0, 0};
        comb8(lds_addr(sh.dtab), yv, v);
        yv = gf_reduce(v);
      }
      if (!Q.iters) Q.l_e[p] = e;
    } else {
      // the block's previous entry, or the rank of the destination's first edge
      const bool starts = i ? Q.e_dst[blockIdx.x * kSetBlock + sh.edge[i - 1]] != dst
                            : set_rank(Q, y, Q.in_off[dst]) == p;
      Q.restart[(uint64_t)y * flag_stride(Q.words) + p] = starts ? 1 : 0;
    }
    Q.l_hi[lo + p] = h;
    Q.l_lo[lo + p] = o;
    Q.l_dst[lo + p] = dst;
    Q.l_y[lo + p] = yv;
  }
}

// ---------------------------------------------------------------------------
// Levels.
// ---------------------------------------------------------------------------
constexpr uint32_t kTile = 8;  // entries per tile of the scan

// Lanes a run takes for rows of c coefficients: short rows share a wave, each
// run with 16 or 32 of its lanes.
__host__ __device__ inline uint32_t run_lanes(uint32_t c) { return c <= 16 ? 16 : (c <= 32 ? 32 : 64); }
// Runs over `tiles` tiles of a level whose rows have c coefficients: one per wave
// (per wave and 64 coefficients), or more, sharing waves, where they keep at
// least 8 tiles each. (With runs of single tiles the 10^6-edge path query's level
// 2 has four times the carries to add: its products took 52 us instead of 27;
// with its 4096 runs packed on 1024 waves the scan took 15 us instead of 10.)
__host__ __device__ inline uint32_t run_count(uint32_t waves, uint32_t c, uint32_t tiles) {
  const uint32_t base = waves / ((c + 63) / 64), most = base * (64 / run_lanes(c));
  const uint32_t few = base < tiles ? base : tiles, many = most < tiles / 8 ? most : tiles / 8;
  return few > many ? few : many;
}
__host__ __device__ inline bool runs_packed(uint32_t waves, uint32_t c, uint32_t runs) {
  return c <= 32 && runs > waves;
}

// Values per row of the window rows that level l reads.
__device__ __forceinline__ uint32_t row_width(const CoefQuery& Q, uint32_t l) {
  return Q.iters ? Q.iters : kBinomD.v[Q.k][l - 1];
}

// Runs of a level's scan: the tiles are cut into `runs` runs of `len` tiles, the
// first `more` of them one longer.
struct Runs {
  uint32_t n, tiles, runs, len, more;
  __device__ __forceinline__ uint32_t tile(uint32_t r) const { return r * len + min(r, more); }
  __device__ __forceinline__ uint32_t run(uint32_t t) const {  // of tile t
    const uint32_t m = more * (len + 1);
    return t < m ? t / (len + 1) : more + (t - m) / len;
  }
};
__device__ __forceinline__ Runs level_runs(const CoefQuery& Q, uint32_t l, uint32_t waves) {
  Runs R;
  R.n = __builtin_amdgcn_readfirstlane(*as_const(Q.count + (l - 2)));
  R.tiles = (R.n + kTile - 1) / kTile;
  R.runs = run_count(waves, row_width(Q, l), R.tiles);
  R.len = R.runs ? __builtin_amdgcn_readfirstlane(R.tiles / R.runs) : 0;
  R.more = R.tiles - R.len * R.runs;
  return R;
}
// Byte p of a flag array, by a scalar load of its word.
__device__ __forceinline__ bool flag_at(const uint8_t* f, uint32_t p) {
  return (as_const((const uint32_t*)f)[p >> 2] >> (8 * (p & 3u))) & 1u;
}

// The multiples of the tile's 8 y values, 128 bytes each at `region`: lane l
// writes multiples 2 (l % 8) and 2 (l % 8) + 1 of entry l / 8.
__device__ __forceinline__ void tile_tables(uint64_t* region, uint32_t lane, uint64_t y) {
  const uint32_t v = (lane & 7u) * 2;
  const uint64_t even = multiple(y, v);
  uint64_t* p = region + (lane >> 3) * 16 + v;
  p[0] = even;
  p[1] = even ^ y;
}

// The scan for rows of at most W coefficients: 64 / W runs per wave, each with W
// of its lanes and its own tables, indices and flags per lane. (24 path
// queries on 10^6 edges, level 2, 8 coefficients: 942 -> 282 us; 4*10^6-edge
// motif query, level 2, 10 coefficients: 150 -> 68 us.)
template <int W>
__device__ __forceinline__ void scan_packed(const CoefQuery& Q, const Runs& R, uint32_t l, uint32_t C, uint32_t wave,
                                            uint32_t lane, uint64_t* region) {
  constexpr uint32_t G = 64 / W, kPer = 128 / W;  // multiples a lane writes per tile
  const uint32_t g = lane / W, c = lane % W;
  if (wave * G >= R.runs) return;
  const uint32_t run = wave * G + g;
  const bool mine = run < R.runs;
  const uint64_t y = l - 2;
  const uint32_t* l_hi = Q.l_hi + y * Q.lstride;
  const uint32_t* l_lo = Q.l_lo + y * Q.lstride;
  const uint64_t* l_y = Q.l_y + y * Q.lstride;
  const uint64_t* store = (const uint64_t*)(Q.store + y * flag_stride(Q.words));
  const uint64_t* restart = (const uint64_t*)(Q.restart + y * flag_stride(Q.words));
  const uint64_t* rows = l == 2 ? Q.z1 : Q.P;
  const uint32_t stride = l == 2 ? Q.z1_stride : C;
  const bool active = mine && c < C;
  const uint32_t ca = min(c, C - 1);
  uint64_t* tab = region + g * (kTile * 16);
  const uint32_t tb = lds_addr(tab);
  const uint32_t t0 = mine ? R.tile(run) : 0u, t1 = mine ? R.tile(run + 1) : 0u;
  const uint32_t steps = R.len + (R.more ? 1u : 0u);
  const uint32_t ti = c / (16 / kPer), tv = (c % (16 / kPer)) * kPer;  // this lane's entry and first multiple
  bool started = false;
  Acc128 acc = {0, 0, 0, 0};
  for (uint32_t s = 0; s < steps; ++s) {
    const uint32_t t = t0 + s, p0 = t * kTile;
    const bool on = t < t1;
    uint32_t h[kTile], o[kTile];
    uint64_t yv = 0, st = 0, rs = 0;
#pragma unroll
    for (uint32_t i = 0; i < kTile; ++i) h[i] = o[i] = kNoRow;
    if (on) {
      const uint4 h0 = *(const uint4*)(l_hi + p0), h1 = *(const uint4*)(l_hi + p0 + 4);
      const uint4 o0 = *(const uint4*)(l_lo + p0), o1 = *(const uint4*)(l_lo + p0 + 4);
      yv = l_y[p0 + ti];
      st = store[t];
      rs = restart[t];
      h[0] = h0.x, h[1] = h0.y, h[2] = h0.z, h[3] = h0.w, h[4] = h1.x, h[5] = h1.y, h[6] = h1.z, h[7] = h1.w;
      o[0] = o0.x, o[1] = o0.y, o[2] = o0.z, o[3] = o0.w, o[4] = o1.x, o[5] = o1.y, o[6] = o1.z, o[7] = o1.w;
    }
    uint64_t w[kTile], w2[kTile];
#pragma unroll
    for (uint32_t i = 0; i < kTile; ++i) {
      w[i] = w2[i] = 0;
      if (h[i] != kNoRow) w[i] = *(gu64*)(rows + (uint64_t)h[i] * stride + ca);
      if (o[i] != kNoRow) w2[i] = *(gu64*)(rows + (uint64_t)o[i] * stride + ca);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    wave_lds_fence();
    {
      const uint64_t y0 = multiple(yv, tv), y1 = yv, y2 = multiple(yv, 2), y4 = multiple(yv, 4);
#pragma unroll
      for (uint32_t v = 0; v < kPer; ++v)
        tab[ti * 16 + tv + v] = y0 ^ ((v & 1) ? y1 : 0) ^ ((v & 2) ? y2 : 0) ^ ((v & 4) ? y4 : 0);
    }
    wave_lds_fence();
#pragma unroll
    for (uint32_t i = 0; i < kTile; ++i) {
      if ((rs >> (8 * i)) & 1u) {
        acc = Acc128{0, 0, 0, 0};
        started = true;
      }
      comb8(tb + i * 128u, w[i] ^ w2[i], acc);
      if (((st >> (8 * i)) & 1u) && active) Q.Q[(uint64_t)(p0 + i) * C + c] = gf_reduce(acc);
    }
  }
  if (active) {
    Q.tail[(uint64_t)run * C + c] = gf_reduce(acc);
    if (c == 0) Q.started[run] = started;
  }
}

// Prefix rows Q_l of level l (2..k-1): a wave takes one run of entries and 64
// coefficients. Entries of a destination are consecutive, so the running
// XOR stays in registers, unreduced; a row some window reads is reduced and
// stored. The product by an entry's y is a comb against y's 16 multiples,
// shared by the wave: about 90 VALU ops and 16 conflict-free LDS reads per
// entry and 64 coefficients, where the evaluation form's product spends about
// 160 and builds a table per lane.
//
// The rows before a run's first segment start lack the segment's part in the
// runs before it. A run leaves the XOR of its open part (its tail) and whether
// a segment starts in it; the row products add the carries (see k_coef_mul),
// so no wave waits for another here. (With a look-back between the runs, the
// six scans of the 10^6-edge path query took 28 to 47 us each.)
template <class A>
__global__ __launch_bounds__(256) void k_coef_scan(A arg, uint32_t l) {
  __shared__ uint64_t lds[4][4 * kTile * 16];
  const CoefQuery Q = arg.get(blockIdx.z);
  if (l >= Q.k) return;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t C = row_width(Q, l);
  const uint32_t cb = blockIdx.y * kLanes;
  if (cb >= C) return;
  const uint32_t waves = arg.waves(blockIdx.z, l);
  const Runs R = level_runs(Q, l, waves);
  const uint32_t wave = blockIdx.x * 4 + wv;
  if (runs_packed(waves, C, R.runs)) {
    if (C <= 16)
      scan_packed<16>(Q, R, l, C, wave, lane, lds[wv]);
    else
      scan_packed<32>(Q, R, l, C, wave, lane, lds[wv]);
    return;
  }
  const uint32_t run = wave;
  if (run >= R.runs) return;
  const uint64_t y = l - 2;
  const uint32_t* l_hi = Q.l_hi + y * Q.lstride;
  const uint32_t* l_lo = Q.l_lo + y * Q.lstride;
  const uint64_t* l_y = Q.l_y + y * Q.lstride;
  const uint8_t* store = Q.store + y * flag_stride(Q.words);
  const uint8_t* restart = Q.restart + y * flag_stride(Q.words);
  const uint64_t* rows = l == 2 ? Q.z1 : Q.P;
  const uint32_t stride = l == 2 ? Q.z1_stride : C;
  const uint32_t co = cb + lane;
  const bool active = co < C;
  const uint32_t ca = min(co, C - 1);  // the lanes past the row repeat its last coefficient and store nothing
  uint64_t* region = lds[wv];
  const uint32_t tb = lds_addr(region);

  const uint32_t t0 = R.tile(run), t1 = R.tile(run + 1);
  bool started = false;
  Acc128 acc = {0, 0, 0, 0};
  for (uint32_t t = t0; t < t1; ++t) {
    const uint32_t p0 = t * kTile;
    const IdxN<kTile> h = load_idx<kTile>(l_hi + p0), o = load_idx<kTile>(l_lo + p0);
    uint64_t yv = *(gu64*)(l_y + p0 + (lane >> 3));
    uint64_t w[kTile], w2[kTile];
#pragma unroll
    for (uint32_t i = 0; i < kTile; ++i) {
      uint64_t a = 0, b = 0;
      if (h.v[i] != kNoRow) a = *(gu64*)(rows + (uint64_t)h.v[i] * stride + ca);
      if (o.v[i] != kNoRow) b = *(gu64*)(rows + (uint64_t)o.v[i] * stride + ca);
      w[i] = a;
      w2[i] = b;
    }
    const uint64_t st = as_const((const uint64_t*)store)[t], rs = as_const((const uint64_t*)restart)[t];
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): all of the tile's loads, so that no product waits on a store
    wave_lds_fence();
    tile_tables(region, lane, yv);
    wave_lds_fence();
#pragma unroll
    for (uint32_t i = 0; i < kTile; ++i) {
      if ((rs >> (8 * i)) & 1u) {
        acc = Acc128{0, 0, 0, 0};
        started = true;
      }
      comb8(tb + i * 128u, w[i] ^ w2[i], acc);
      if (((st >> (8 * i)) & 1u) && active) Q.Q[(uint64_t)(p0 + i) * C + co] = gf_reduce(acc);
    }
  }
  if (active) Q.tail[(uint64_t)run * C + co] = gf_reduce(acc);
  if (cb == 0 && lane == 0) Q.started[run] = started;
}

// The first run of the segment that run `run` continues: the nearest one before
// it in which a segment starts (wave-uniform).
__device__ __forceinline__ uint32_t segment_run(const uint8_t* started, uint32_t run, uint32_t lane) {
  uint32_t first = run;
  for (;;) {
    const uint64_t s = __ballot(lane < first && started[first - 1 - min(lane, first - 1)]);
    if (s) return first - 1 - (uint32_t)__builtin_ctzll(s);
    if (first <= 64) return 0;  // (run 0 starts a segment)
    first -= 64;
  }
}
// End of the entries of a run [p, end) that precede its first segment start.
__device__ __forceinline__ uint32_t open_part(const uint8_t* restart, uint32_t p, uint32_t end, uint32_t lane) {
  if (flag_at(restart, p)) return p;
  for (;; p += 64) {
    const uint32_t i = p + lane;
    const uint64_t s = __ballot(i >= end || restart[min(i, end)]);
    if (s) return p + (uint32_t)__builtin_ctzll(s);
  }
}

// Levels where one destination may span very many runs (see far_levels): summed
// tail by tail the carries' work grows as the square of the runs of one segment
// (70 % of 10^6 edges at one vertex, k = 3: row products of 1696 us). There the
// carry of a run is the exclusive prefix sum of the tails at the run less the
// one at its segment's first run, two rows whatever the distance. k_coef_fold
// sums the tails of 64 runs, k_coef_prefix adds up the groups before its own and
// leaves the prefix sums in carry and each run's segment start in seg. A block
// takes 64 runs and 64 coefficients, a wave four runs; bound by latency. (One
// launch whose blocks summed every tail before theirs took 29 to 36 us for 4096 to
// 10000 runs.)
template <class A>
__global__ __launch_bounds__(1024) void k_coef_fold(A arg, uint32_t l) {
  __shared__ uint64_t part[16][kLanes];
  const CoefQuery Q = arg.get(blockIdx.z);
  if (l >= Q.k || !((Q.far >> (l - 2)) & 1u)) return;
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  const uint32_t C = row_width(Q, l), co = blockIdx.y * kLanes + lane, r0 = blockIdx.x * 64 + wv * 4;
  const Runs R = level_runs(Q, l, arg.waves(blockIdx.z, l));
  if (blockIdx.y * kLanes >= C || blockIdx.x * 64 >= R.runs) return;
  uint64_t s = 0;
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) s ^= co < C && r0 + i < R.runs ? Q.tail[(uint64_t)(r0 + i) * C + co] : 0;
  part[wv][lane] = s;
  __syncthreads();
  if (wv || co >= C) return;
#pragma unroll
  for (uint32_t i = 1; i < 16; ++i) s ^= part[i][lane];
  Q.group[(uint64_t)blockIdx.x * C + co] = s;
}
template <class A>
__global__ __launch_bounds__(1024) void k_coef_prefix(A arg, uint32_t l) {
  __shared__ uint64_t before[16][kLanes], part[16][kLanes];
  __shared__ uint32_t last;
  const CoefQuery Q = arg.get(blockIdx.z);
  if (l >= Q.k || !((Q.far >> (l - 2)) & 1u)) return;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6, g = blockIdx.x;
  const uint32_t C = row_width(Q, l), co = blockIdx.y * kLanes + lane, r0 = g * 64 + wv * 4;
  const Runs R = level_runs(Q, l, arg.waves(blockIdx.z, l));
  if (blockIdx.y * kLanes >= C || g * 64 >= R.runs) return;
  const bool active = co < C;
  uint64_t row[4], b = 0, s = 0;
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) row[i] = active && r0 + i < R.runs ? Q.tail[(uint64_t)(r0 + i) * C + co] : 0;
  if (active)
    for (uint32_t i = wv; i < g; i += 64) {  // four in flight
      uint64_t v[4];
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) v[j] = *(gu64*)(Q.group + (uint64_t)min(i + 16 * j, g - 1) * C + co);
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) b ^= i + 16 * j < g ? v[j] : 0;
    }
  if (tid == 0) last = 0;
  before[wv][lane] = b;
  part[wv][lane] = row[0] ^ row[1] ^ row[2] ^ row[3];
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < 16; ++i) s ^= before[i][lane] ^ (i < wv ? part[i][lane] : 0);
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) {
    if (active && r0 + i < R.runs) Q.carry[(uint64_t)(r0 + i) * C + co] = s;
    s ^= row[i];
  }
  if (blockIdx.y) return;
  uint32_t m = 0;  // one past the last run before the group in which a segment starts
  for (uint32_t i = tid; i < g * 8; i += 1024) {  // eight flags per word
    const uint64_t f = ((const uint64_t*)Q.started)[i];
    if (f) m = i * 8 + 8 - (uint32_t)__builtin_clzll(f) / 8;
  }
  if (m) atomicMax(&last, m);
  __syncthreads();
  if (wv == 0) {
    const uint32_t r = g * 64 + lane;
    const uint64_t f = __ballot(r < R.runs && Q.started[min(r, R.runs - 1)]) & ((1ull << lane) - 1);
    if (r < R.runs) Q.seg[r] = f ? g * 64 + 63 - (uint32_t)__builtin_clzll(f) : max(last, 1u) - 1;
  }
}

// Carries of a level whose runs are long (see run_coef): per run that continues
// a segment, the XOR of the tails back to the run the segment starts in, and
// the end of the rows that lack it. On a far level the prefix sums are in carry
// and nothing reads the tails any more: the carries take their place.
template <class A>
__global__ __launch_bounds__(256) void k_coef_carry(A arg, uint32_t l) {
  const CoefQuery Q = arg.get(blockIdx.z);
  if (l >= Q.k || !((Q.carried >> (l - 2)) & 1u)) return;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t C = row_width(Q, l), co = blockIdx.y * kLanes + lane;
  if (blockIdx.y * kLanes >= C) return;
  const Runs R = level_runs(Q, l, arg.waves(blockIdx.z, l));
  const uint32_t run = blockIdx.x * 4 + wv;
  if (run >= R.runs) return;
  const uint32_t p = R.tile(run) * kTile;
  const uint32_t oe = open_part(Q.restart + (uint64_t)(l - 2) * flag_stride(Q.words), p,
                                min(R.tile(run + 1) * kTile, R.n), lane);
  if (blockIdx.y == 0 && lane == 0) Q.open_end[run] = oe;
  if (oe == p) return;
  if ((Q.far >> (l - 2)) & 1u) {
    const uint32_t first = as_const(Q.seg)[run];
    if (co < C) Q.tail[(uint64_t)run * C + co] = Q.carry[(uint64_t)run * C + co] ^ Q.carry[(uint64_t)first * C + co];
    return;
  }
  const uint32_t first = segment_run(Q.started, run, lane);  // (a ballot of all lanes)
  if (co >= C) return;
  uint64_t s = 0;
#pragma unroll 8
  for (uint32_t r = first; r < run; ++r) s ^= *(gu64*)(Q.tail + (uint64_t)r * C + co);
  Q.carry[(uint64_t)run * C + co] = s;
}
// Where k_coef_carry leaves a level's carries.
__device__ __forceinline__ const uint64_t* carries(const CoefQuery& Q, uint32_t l) {
  return (Q.far >> (l - 2)) & 1u ? Q.tail : Q.carry;
}

// One row P_l[p] = z_{dst} Q_l[p] by a wave. Lanes take (label, subset) pairs, so
// every lane forms a product that is needed; pairs are ordered by label, and
// lanes with one label share its 16 multiples, which are kept while the
// destination stays.
struct RowMul {
  uint64_t *tab, *q, *out;  // LDS: multiples of the vertex form's entries, the row read, the row formed
  const uint32_t* pairs;
  uint32_t c_in, c_out, per, lane;
  uint32_t cur, j0, nj;
  template <class A>
  __device__ __forceinline__ void row(const A& arg, const CoefQuery& Q, uint32_t p, uint32_t dst, const uint64_t* carry_lds,
                                      const uint64_t* carry_row) {
    const uint64_t* qrow = Q.Q + (uint64_t)p * c_in;
    wave_lds_fence();
    for (uint32_t i = lane; i < c_in; i += kLanes) {
      uint64_t v = *(gu64*)(qrow + i);
      if (carry_lds) v ^= carry_lds[i];
      if (carry_row) v ^= *(gu64*)(carry_row + i);
      q[i] = v;
    }
    form(arg, Q, dst, Q.P + (uint64_t)p * c_out);
  }
  // The product of the row in q, to prow.
  template <class A>
  __device__ __forceinline__ void form(const A& arg, const CoefQuery& Q, uint32_t dst, uint64_t* prow) {
    for (uint32_t i = lane; i < c_out; i += kLanes) out[i] = 0;
    if (dst != cur) {
      cur = dst;
      if (Q.motif) {
        const uint32_t cl = __builtin_amdgcn_readfirstlane(Q.colour[dst]);
        j0 = arg.off(blockIdx.z, cl);
        nj = arg.mu(blockIdx.z, cl);
      }
      for (uint32_t i = lane; i < nj * 16; i += kLanes)
        tab[j0 * 16 + i] = multiple(*(gu64*)(Q.z + (uint64_t)dst * Q.kq + j0 + i / 16), i & 15u);
    }
    wave_lds_fence();
    const uint32_t b = j0 * per, e = b + nj * per, tb = lds_addr(tab);
    for (uint32_t i = b + lane; i < e; i += kLanes) {
      const uint32_t w = pairs[i];
      Acc128 r = {0, 0, 0, 0};
      comb8(tb + (w >> 20) * 128u, q[w & 1023u], r);
      atomicXor((unsigned long long*)&out[(w >> 10) & 1023u], (unsigned long long)gf_reduce(r));
    }
    wave_lds_fence();
    for (uint32_t i = lane; i < c_out; i += kLanes) prow[i] = out[i];
  }
};
// LDS of one wave's RowMul.
__host__ __device__ inline uint32_t mul_lds(uint32_t k, uint32_t c_in, uint32_t c_out) {
  return (k * 16 + ((c_in + c_out + 15) & ~15u)) * 8;
}

// Rows P_l of the entries some window reads.
// CARRIED (long runs): four list positions per wave and step, carries from
// k_coef_carry. Otherwise a block takes the scan's runs in turn, a quarter per
// wave, and sums the carry of a run that continues a segment itself: for short
// runs that costs less than the launch (10^6-edge path query, 8 entries per
// run: 3 us per level against 5), for long ones the blocks wait (4*10^6-edge
// motif query, level 6: 224 us with the carry in the block, 190 without).
// FAR: some query of the launch has prefix sums of the tails.
template <class A, bool CARRIED, bool FAR>
__global__ __launch_bounds__(256) void k_coef_mul(A arg, uint32_t l, uint32_t wave_lds) {
  extern __shared__ uint64_t dyn_lds[];  // [4][wave_lds] then the carry
  const CoefQuery Q = arg.get(blockIdx.z);
  if (l >= Q.k || ((Q.carried >> (l - 2)) & 1u) != (CARRIED ? 1u : 0u)) return;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t k = Q.k;
  RowMul M;
  M.c_in = kBinomD.v[k][l - 1];
  M.c_out = kBinomD.v[k][l];
  M.per = kBinomD.v[k - 1][l - 1];
  M.tab = dyn_lds + wv * (wave_lds / 8);
  M.q = M.tab + k * 16;
  M.out = M.q + M.c_in;
  M.pairs = kPairTable.v + kPairTable.base[k][l];
  M.lane = lane;
  M.cur = kNoRow;
  M.j0 = 0;
  M.nj = k;
  const uint64_t y = l - 2;
  const Runs R = level_runs(Q, l, arg.waves(blockIdx.z, l));
  const uint32_t* dsts = Q.l_dst + y * Q.lstride;
  const uint8_t* store = Q.store + y * flag_stride(Q.words);
  if constexpr (CARRIED) {
    const uint32_t units = (R.n + 3) / 4, waves = gridDim.x * 4;
    const uint64_t* carry = FAR ? carries(Q, l) : Q.carry;
    for (uint32_t u = blockIdx.x * 4 + wv; u < units; u += waves) {
      uint32_t flags = as_const((const uint32_t*)store)[u];
      if (!flags) continue;
      const uint32_t run = R.run(u / 2), oe = as_const(Q.open_end)[run];
      while (flags) {
        const uint32_t p = u * 4 + (uint32_t)__builtin_ctz(flags) / 8;
        flags &= flags - 1;
        M.row(arg, Q, p, as_const(dsts)[p], nullptr, p < oe ? carry + (uint64_t)run * M.c_in : nullptr);
      }
    }
  } else {
    uint64_t* carry = dyn_lds + 4 * (wave_lds / 8);
    const bool far = FAR && ((Q.far >> (l - 2)) & 1u);
    for (uint32_t run = blockIdx.x; run < R.runs; run += gridDim.x) {
      const uint32_t p_begin = R.tile(run) * kTile, p_end = min(R.tile(run + 1) * kTile, R.n);
      const uint32_t oe = open_part(Q.restart + y * flag_stride(Q.words), p_begin, p_end, lane);
      if (oe > p_begin && far) {
        const uint32_t first = as_const(Q.seg)[run];
        __syncthreads();  // the block's last run is done with the carry
        for (uint32_t i = threadIdx.x; i < M.c_in; i += 256)
          carry[i] = *(gu64*)(Q.carry + (uint64_t)run * M.c_in + i) ^ *(gu64*)(Q.carry + (uint64_t)first * M.c_in + i);
        __syncthreads();
      } else if (oe > p_begin) {
        const uint32_t first = segment_run(Q.started, run, lane);
        __syncthreads();  // the block's last run is done with the carry
        for (uint32_t i = threadIdx.x; i < M.c_in; i += 256) carry[i] = 0;
        __syncthreads();
        for (uint32_t i = lane; i < M.c_in; i += kLanes) {
          uint64_t s = 0;
#pragma unroll 4
          for (uint32_t r = first + wv; r < run; r += 4) s ^= *(gu64*)(Q.tail + (uint64_t)r * M.c_in + i);
          if (s) atomicXor((unsigned long long*)&carry[i], (unsigned long long)s);
        }
        __syncthreads();
      }
      const uint32_t share = (p_end - p_begin + 3) / 4;
      const uint32_t q_begin = p_begin + wv * share, q_end = min(q_begin + share, p_end);
      for (uint32_t p = q_begin; p < q_end; ++p)
        if (flag_at(store, p)) M.row(arg, Q, p, as_const(dsts)[p], p < oe ? carry : nullptr, nullptr);
    }
  }
}

// Last level: the coefficient of x_1 .. x_k of y_{e,k-1} z_{dst} W_e, summed over
// the entries (or kept per edge). The row of level k - 1 has k coefficients, the
// one of rank c lacking label k - 1 - c. A wave takes up to 64 entries; path
// queries spread their (entry, coefficient) pairs over the lanes, so that a row
// is read by neighbouring lanes and a wave's loads do not wait for each other.
// Motif queries have one to a few non-zero entries in z_{dst} and take an entry
// per lane. per_wave: entries per wave, 64 or, where that leaves the GPU short
// of waves, 32, 16 or 8. (24 queries on 10^6 edges: 1161 us with an entry's
// products one after another and one sum that all blocks add to behind a fence;
// 1062 with the products spread, 453 without the fence, 167 without the shared
// sum.)
template <class A>
__global__ __launch_bounds__(256) void k_coef_top(A arg, uint32_t per_wave) {
  __shared__ struct {
    uint64_t tab[4][16][kLanes];
    uint64_t sum[4][kLanes];
    uint32_t h[4][kLanes], o[4][kLanes], d[4][kLanes];
    uint64_t part[4];
  } sh;  // the only static LDS: starts at address 0
  const CoefQuery Q = arg.get(blockIdx.y);
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6, k = Q.k;
  if (k < 3) return;  // (left out of this launch)
  uint64_t* tab = &sh.tab[wv][0][lane];
  tab[0] = 0;
  const uint32_t base = lds_addr(tab);
  const uint64_t y = k - 2, lo = y * Q.lstride;
  const uint32_t n = Q.count[y];
  const uint32_t inv = 65536 / k + 1;  // i / k = i * inv >> 16 for i < 64 k
  uint64_t sum = 0;
  const uint32_t rounds = (per_wave * k + kLanes - 1) / kLanes;
  for (uint64_t p0 = (blockIdx.x * 4 + wv) * per_wave; p0 < n; p0 += gridDim.x * 4 * per_wave) {
    const uint32_t p = (uint32_t)p0 + lane;
    const bool in = lane < per_wave && p < n;
    const uint32_t h = in ? Q.l_hi[lo + p] : kNoRow, o = in ? Q.l_lo[lo + p] : kNoRow, dst = in ? Q.l_dst[lo + p] : 0u;
    const uint64_t yv = in ? Q.l_y[lo + p] : 0;
    uint64_t s;
    if (Q.motif) {
      Acc128 r = {0, 0, 0, 0};
      if (h != kNoRow) {
        const uint32_t c = Q.colour[dst], j0 = arg.off(blockIdx.y, c), j1 = j0 + arg.mu(blockIdx.y, c);
        for (uint32_t j = j0; j < j1; ++j) {
          uint64_t w = Q.P[(uint64_t)h * k + (k - 1 - j)];
          if (o != kNoRow) w ^= Q.P[(uint64_t)o * k + (k - 1 - j)];
          gf_table(tab, w);
          gf_comb_acc(base, Q.z[(uint64_t)dst * Q.kq + j], r);
        }
      }
      s = gf_reduce(r);
    } else {
      wave_lds_fence();
      sh.h[wv][lane] = h;
      sh.o[wv][lane] = o;
      sh.d[wv][lane] = dst;
      sh.sum[wv][lane] = 0;
      wave_lds_fence();
      auto load = [&](uint32_t r, uint64_t& w, uint64_t& z) {
        const uint32_t i = r * kLanes + lane, e = min(i * inv >> 16, kLanes - 1), c = i - e * k;
        const uint32_t eh = sh.h[wv][e], eo = sh.o[wv][e];
        w = 0;
        z = 0;
        if (eh != kNoRow) {
          w = *(gu64*)(Q.P + (uint64_t)eh * k + c);
          z = *(gu64*)(Q.z + (uint64_t)sh.d[wv][e] * Q.kq + (k - 1 - c));
          if (eo != kNoRow) w ^= *(gu64*)(Q.P + (uint64_t)eo * k + c);
        }
      };
      uint64_t w, z, wn, zn;
      load(0, w, z);
      for (uint32_t r = 0; r < rounds; ++r) {
        load(r + 1 < rounds ? r + 1 : r, wn, zn);  // in flight during these products
        const uint64_t v = gf_mul(tab, z, w);
        atomicXor((unsigned long long*)&sh.sum[wv][(r * kLanes + lane) * inv >> 16], (unsigned long long)v);
        w = wn;
        z = zn;
      }
      wave_lds_fence();
      s = sh.sum[wv][lane];
    }
    const uint64_t v = gf_mul(tab, yv, s);
    if (Q.fine && in) Q.T[Q.l_e[p]] = v;
    sum ^= v;
  }
  uint32_t s0 = lo32(sum), s1 = hi32(sum);
#pragma unroll
  for (int d = 1; d < kLanes; d <<= 1) {
    s0 ^= (uint32_t)__shfl_xor((int)s0, d, kLanes);
    s1 ^= (uint32_t)__shfl_xor((int)s1, d, kLanes);
  }
  if (lane == 0) sh.part[wv] = mk64(s0, s1);
  __syncthreads();
  // Each block leaves its sum, for the host to add up: one word that all blocks
  // add to by atomics queues them up (374 blocks 21 us, 1536 blocks 45 us on the
  // 10^6-edge path query; 15 us as it is).
  if (threadIdx.x == 0)
    __hip_atomic_store(Q.result + blockIdx.x, sh.part[0] ^ sh.part[1] ^ sh.part[2] ^ sh.part[3], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// k = 2: a walk is one edge, so there are no sets and no rows, and the last
// level is y_e (z_{src,1} z_{dst,2} + z_{src,2} z_{dst,1}) (gamma in place of z and
// times det Omega for motif queries), all hashed where they are used. One launch;
// bound by its three or four products per edge. (10^5 edges, fine-grained: the
// evaluation form's eleven launches took 170 us, of which its last level 48 and
// its one-block reduction 28; 7 us here.)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_coef_pairs(OneCoef a) {
  __shared__ struct {
    uint64_t tab[4][16][kLanes];
    uint64_t part[4];
  } sh;  // the only static LDS: starts at address 0
  const CoefQuery& Q = a.q;
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  uint64_t* tab = &sh.tab[wv][0][lane];
  tab[0] = 0;
  auto omega = [&](uint32_t d, uint32_t j) { return hash1(Q.seed, 'W', (uint64_t)d | ((uint64_t)(j + 1) << 32)); };
  const uint64_t det = Q.motif ? gf_mul(tab, omega(0, 0), omega(1, 1)) ^ gf_mul(tab, omega(0, 1), omega(1, 0)) : 0;
  uint64_t sum = 0;
  for (uint64_t e = blockIdx.x * 256 + threadIdx.x; e < Q.m; e += gridDim.x * 256) {  // (m may be near 2^32)
    const uint32_t s = Q.e_src[e], u = Q.e_dst[e], t = Q.e_t[e];
    bool ok = !(Q.f.rmask && (Q.f.rmask[s] | Q.f.rmask[u])) && !(Q.f.t_max && t > Q.f.t_max) &&
              !(Q.f.smask && !Q.f.smask[s]) && !(Q.f.tmask && !Q.f.tmask[u]);
    uint64_t z[4] = {};  // src 1, 2, dst 1, 2
    if (ok && Q.motif) {
      const uint32_t c[2] = {Q.colour[s], Q.colour[u]};
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t o = a.off(0, c[i / 2]), d = i & 1u;
        if (d >= o && d < o + a.mu(0, c[i / 2])) z[i] = hash1(Q.seed, 'G', (uint64_t)(i < 2 ? s : u) | ((uint64_t)d << 32));
      }
      ok = (z[0] && z[3]) || (z[1] && z[2]);
    } else if (ok) {
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) z[i] = hash1(Q.seed, 'Z', (uint64_t)(i < 2 ? s : u) | ((uint64_t)((i & 1u) + 1) << 32));
    }
    uint64_t v = 0;
    if (ok) {
      v = gf_mul(tab, z[0], z[3]) ^ gf_mul(tab, z[1], z[2]);
      v = gf_mul(tab, hash2(Q.seed, 'Y', (uint64_t)s | ((uint64_t)u << 32), (uint64_t)t | (1ull << 32)), v);
      if (Q.motif) v = gf_mul(tab, det, v);
    }
    if (Q.fine) Q.T[e] = v;
    sum ^= v;
  }
  uint32_t s0 = lo32(sum), s1 = hi32(sum);
#pragma unroll
  for (int d = 1; d < kLanes; d <<= 1) {
    s0 ^= (uint32_t)__shfl_xor((int)s0, d, kLanes);
    s1 ^= (uint32_t)__shfl_xor((int)s1, d, kLanes);
  }
  if (lane == 0) sh.part[wv] = mk64(s0, s1);
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(Q.result + blockIdx.x, sh.part[0] ^ sh.part[1] ^ sh.part[2] ^ sh.part[3], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// Rows by iteration. The value of a single iteration L is no coefficient of the
// polynomial above, but the product sets, lists and scans serve it as well:
// with Q.iters set, value i of a row belongs to iteration Q.it0 + i, and a
// vertex factor is one product by z^L_v = XOR_{j in L} z_{v,j} per value, formed
// from the k entries of z_v where it is used.
// (10^5-edge motif query, k = 9, all 512 iterations: 1400 -> 520 us against the
// evaluation form, whose lists keep four to eight times the entries. Bound by
// latency there: 22 launches, each a chain of a few dependent loads.)
// ---------------------------------------------------------------------------
// z^L_v of the lane's iteration (v wave-uniform): the entries of z_v by scalar
// loads, all in flight together (past the row its last four again, which no bit
// of L < 2^k selects).
__device__ __forceinline__ uint64_t iter_form(const CoefQuery& Q, uint32_t v, uint32_t L) {
  const auto* z = as_const(Q.z + (uint64_t)v * Q.kq);
  uint64_t x[kCoefMaxK];
#pragma unroll
  for (uint32_t j = 0; j < kCoefMaxK; ++j) x[j] = z[min(j & ~3u, Q.kq - 4) + (j & 3u)];
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (uint32_t j = 0; j < kCoefMaxK; ++j) {
    const uint32_t m = 0u - ((L >> j) & 1u);
    lo = and_xor(lo32(x[j]), m, lo);
    hi = and_xor(hi32(x[j]), m, hi);
  }
  return mk64(lo, hi);
}

// The rows level 2 reads, at the head of P (whose own rows take over once level
// 2's scan has read them): z^L of every vertex, or, where there are many vertices
// for the list (see run_coef), of each entry's source at the entry's place. (3*10^5
// edges on 3*10^6 vertices, all but one iteration: k = 8, 4044 us by vertex, 217 by
// entry, 534 in the evaluation form; k = 12, 79.7 ms in a table of 98 GB, 391 us.
// 2*10^5 edges on 2000 vertices, k = 8: 2277 us by vertex, 2362 by entry.)
__global__ __launch_bounds__(256) void k_iter_z(OneCoef a) {
  const CoefQuery& Q = a.q;
  const uint32_t lane = threadIdx.x & 63u, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n = Q.by_entry ? *as_const(Q.count) : Q.n, co = blockIdx.y * kLanes + lane;
  for (uint64_t p = blockIdx.x * 4 + wv; p < n; p += gridDim.x * 4) {
    const uint64_t x = iter_form(Q, Q.by_entry ? as_const(Q.l_e)[p] : (uint32_t)p, Q.it0 + co);
    if (co < Q.iters) Q.P[p * Q.iters + co] = x;
  }
}

// Rows P_l of the entries some window reads: a wave takes 64 values of four
// list positions in turn; the multiples of its lanes' z^L are kept while the
// destination stays.
__global__ __launch_bounds__(256) void k_iter_mul(OneCoef a, uint32_t l) {
  __shared__ uint64_t lds[4][16][kLanes];  // the only static LDS: starts at address 0
  const CoefQuery& Q = a.q;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t C = Q.iters, co = blockIdx.y * kLanes + lane, ca = min(co, C - 1);
  const uint64_t y = l - 2;
  const Runs R = level_runs(Q, l, a.waves(0, l));
  const uint32_t* dsts = Q.l_dst + y * Q.lstride;
  const uint8_t* store = Q.store + y * flag_stride(Q.words);
  uint64_t* tab = &lds[wv][0][lane];
  tab[0] = 0;
  const uint32_t base = lds_addr(tab);
  uint32_t cur = kNoRow;
  const uint32_t units = (R.n + 3) / 4, waves = gridDim.x * 4;
  const uint64_t* carry = carries(Q, l);
  for (uint32_t u = blockIdx.x * 4 + wv; u < units; u += waves) {
    uint32_t flags = as_const((const uint32_t*)store)[u];
    if (!flags) continue;
    const uint32_t run = R.run(u / 2), oe = as_const(Q.open_end)[run];
    while (flags) {
      const uint32_t p = u * 4 + (uint32_t)__builtin_ctz(flags) / 8;
      flags &= flags - 1;
      uint64_t v = *(gu64*)(Q.Q + (uint64_t)p * C + ca);
      if (p < oe) v ^= *(gu64*)(carry + (uint64_t)run * C + ca);
      const uint32_t dst = as_const(dsts)[p];
      if (dst != cur) {
        cur = dst;
        gf_table(tab, iter_form(Q, dst, Q.it0 + ca));
      }
      Acc128 r = {0, 0, 0, 0};
      gf_comb_acc(base, v, r);
      if (co < C) Q.P[(uint64_t)p * C + co] = gf_reduce(r);
    }
  }
}

// Last level: per wave, 64 iterations and a run of entries, the sum of
// z_{dst} * (XOR of y W over the entries of a destination), left in tail[wave].
__global__ __launch_bounds__(256) void k_iter_top(OneCoef a) {
  __shared__ struct {
    uint64_t tab[4][16][kLanes];
    uint64_t ytab[4][kTile * 16];
  } sh;  // the only static LDS: starts at address 0
  const CoefQuery& Q = a.q;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t C = Q.iters, co = blockIdx.y * kLanes + lane, ca = min(co, C - 1);
  const uint64_t y = Q.k - 2;
  const uint32_t* l_hi = Q.l_hi + y * Q.lstride;
  const uint32_t* l_lo = Q.l_lo + y * Q.lstride;
  const uint32_t* l_dst = Q.l_dst + y * Q.lstride;
  const uint64_t* l_y = Q.l_y + y * Q.lstride;
  const Runs R = level_runs(Q, Q.k, a.waves(0, Q.k));
  const uint32_t run = blockIdx.x * 4 + wv;
  uint64_t* tab = &sh.tab[wv][0][lane];
  tab[0] = 0;
  const uint32_t base = lds_addr(tab), yb = lds_addr(sh.ytab[wv]);
  const uint32_t t0 = run < R.runs ? R.tile(run) : 0, t1 = run < R.runs ? R.tile(run + 1) : 0;
  uint32_t cur = kNoRow;
  uint64_t sum = 0;
  Acc128 acc = {0, 0, 0, 0};
  auto flush = [&] {
    if (cur != kNoRow) sum ^= gf_mul(tab, gf_reduce(acc), iter_form(Q, cur, Q.it0 + ca));
    acc = Acc128{0, 0, 0, 0};
  };
  for (uint32_t t = t0; t < t1; ++t) {
    const uint32_t p0 = t * kTile;
    const IdxN<kTile> h = load_idx<kTile>(l_hi + p0), o = load_idx<kTile>(l_lo + p0), d = load_idx<kTile>(l_dst + p0);
    const uint64_t yv = *(gu64*)(l_y + p0 + (lane >> 3));
    uint64_t w[kTile], w2[kTile];
#pragma unroll
    for (uint32_t i = 0; i < kTile; ++i) {
      w[i] = w2[i] = 0;
      if (h.v[i] != kNoRow) w[i] = *(gu64*)(Q.P + (uint64_t)h.v[i] * C + ca);
      if (o.v[i] != kNoRow) w2[i] = *(gu64*)(Q.P + (uint64_t)o.v[i] * C + ca);
    }
    wave_lds_fence();
    tile_tables(sh.ytab[wv], lane, yv);
    wave_lds_fence();
#pragma unroll
    for (uint32_t i = 0; i < kTile; ++i) {
      if (h.v[i] == kNoRow) continue;
      if (d.v[i] != cur) {
        flush();
        cur = d.v[i];
      }
      comb8(yb + i * 128u, w[i] ^ w2[i], acc);
    }
  }
  flush();
  if (run < R.runs && co < C) Q.tail[(uint64_t)run * C + co] = sum;
}

// f(it0 + i) for i < count: the runs' sums, 64 iterations per block.
__global__ __launch_bounds__(1024) void k_iter_fold(OneCoef a, uint32_t count) {
  __shared__ uint64_t part[16][kLanes];
  const CoefQuery& Q = a.q;
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6, co = blockIdx.x * kLanes + lane;
  const Runs R = level_runs(Q, Q.k, a.waves(0, Q.k));
  uint64_t s = 0;
  if (co < Q.iters) {
#pragma unroll 8
    for (uint32_t r = wv; r < R.runs; r += 16) s ^= Q.tail[(uint64_t)r * Q.iters + co];
  }
  part[wv][lane] = s;
  __syncthreads();
  if (wv == 0 && co < count) {
    for (uint32_t i = 1; i < 16; ++i) s ^= part[i][lane];
    __hip_atomic_store(Q.result + co, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
bool coef_applies(const QueryPlan& qp) {
  return qp.k >= 2 && qp.k <= kCoefMaxK && qp.it_begin == 0 && qp.it_end == (1ull << qp.k);
}
bool iter_rows_apply(const QueryPlan& qp) { return qp.k >= 3 && qp.k <= kCoefMaxK; }

static inline uint64_t up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

// Waves the scan of a level is cut into, over its coefficient blocks: four
// per SIMD.
constexpr uint32_t kScanWaves = 4096;
// Blocks of the last level: each leaves one sum.
constexpr uint32_t kTopBlocks = 1024;
// Blocks of the row products that go over a list in turn.
constexpr uint32_t kMulBlocks = 2048;
// Edges, over the grid slices of a launch, from which a thread of the backward pass
// takes four. (k = 8, Chung-Lu and
// uniform graphs, one edge per thread against four, us per query: 6*10^5 edges 282
// and 297, 219 and 231; 10^6 365 and 373, 237 and 241; 2*10^6 628 and 609, 354 and 336;
// 4*10^6 1076 and 1046, 545 and 508. 24 queries on 10^6
// edges: 5725 and 5506; one on 10^6 edges and 199 on 300: 3156 and 2411.)
constexpr uint64_t kWideSets = 1400000;
// Entries per run from which the carries get a launch of their own.
constexpr uint64_t kLongRun = 32;
// Runs that one destination may span from which the carries come from prefix
// sums: two short launches more against a sum over the square of the runs.
constexpr uint64_t kFarRuns = 1024;

// Device buffers of one query carved from one region, each 256-byte aligned.
struct Carver {
  uint8_t* base;
  uint64_t off = 0;
  template <class T>
  void take(T*& p, uint64_t count) {
    p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += up(count * sizeof(T), 256);
  }
};

// Values per row of the window rows that level l reads, and of the rows it forms.
static uint32_t width_in(const CoefQuery& q, uint32_t l) { return q.iters ? q.iters : binom(q.k, l - 1); }
static uint32_t width_out(const CoefQuery& q, uint32_t l) { return q.iters ? q.iters : binom(q.k, l); }
// Runs of level l's scan over `entries` entries (see level_runs).
static uint32_t scan_runs(const CoefQuery& q, const CoefShades& sh, uint64_t entries, uint32_t l) {
  return std::max(1u, run_count(sh.waves[l], width_in(q, l), (uint32_t)((entries + kTile - 1) / kTile)));
}

// The query's own fields; buffers are set by carve_setup.
static void fill_query(CoefQuery& q, CoefShades& sh, const GraphDev& G, const QueryPlan& qp, const uint32_t* dv,
                       const EdgeFilter& filt, bool fine, uint32_t waves) {
  q.e_src = G.e_src.as<uint32_t>();
  q.e_dst = G.e_dst.as<uint32_t>();
  q.e_t = G.e_t.as<uint32_t>();
  q.in_off = G.in_off.as<uint32_t>();
  q.hi = G.hi.as<uint32_t>();
  q.colour = G.colour.as<uint8_t>();
  q.dv = dv;
  q.f = filt;
  q.seed = qp.seed;
  q.n = G.n;
  q.m = (uint32_t)G.m;
  q.k = qp.k;
  q.kq = qp.kq;
  q.delta = qp.delta;
  q.motif = qp.motif ? 1 : 0;
  std::copy(qp.mu, qp.mu + RS_MAX_COLOURS, sh.mu);
  std::copy(qp.shade_off, qp.shade_off + RS_MAX_COLOURS, sh.off);
  q.blocks = (uint32_t)up((G.m + kSetBlock - 1) / kSetBlock, 4);
  q.words = q.blocks * 16;
  q.nested = filt.smask ? 0 : 1;
  // with a source restriction a walk's tail need not be a walk from a source,
  // so the forward sets are not nested and every level needs its own
  q.fwd = filt.smask ? qp.k : std::min(qp.k, kForwardLevels);
  q.plain = !filt.any() && !qp.motif ? 1 : 0;
  q.fine = fine ? 1 : 0;
  std::fill(sh.waves, sh.waves + kCoefMaxK + 1, waves);
  q.lstride = up(G.m + kTile, 64);  // all m edges and the padding a tile reads
}

// Windows, bitmaps, ranks, lists and tails (base null: only sizes).
static uint64_t carve_setup(CoefQuery& q, const CoefShades& sh, uint8_t* base) {
  Carver c{base};
  const uint64_t L = q.k - 1, fw = (uint64_t)q.words + q.words / 64;
  uint64_t tails = 0, width = q.iters;
  for (uint32_t l = 2; l < q.k; ++l) width = std::max<uint64_t>(width, width_in(q, l));
  for (uint32_t l = 2; l < q.k; ++l)
    tails = std::max<uint64_t>(tails, (uint64_t)scan_runs(q, sh, q.m, l) * width_in(q, l));
  // (rows by iteration may be made narrower later, and the last level leaves its sums here)
  if (q.iters) tails = std::min<uint64_t>(64ull * sh.waves[2], up(q.iters, 64) * ((q.m + kTile - 1) / kTile));
  c.take(q.win, q.m);
  c.take(q.valid, q.words);
  c.take(q.fbits, (q.fwd - 1) * fw);
  c.take(q.mark, (q.k - 2) * mark_stride(q.blocks));
  c.take(q.sbits, L * q.words);
  c.take(q.wrank, L * q.words);
  c.take(q.bsum, L * q.blocks);
  c.take(q.boff, L * q.blocks);
  c.take(q.store, L * flag_stride(q.words));
  c.take(q.restart, L * flag_stride(q.words));
  c.take(q.l_hi, L * q.lstride);
  c.take(q.l_lo, L * q.lstride);
  c.take(q.l_dst, L * q.lstride);
  c.take(q.l_y, L * q.lstride);
  c.take(q.l_e, q.lstride);
  c.take(q.tail, tails);
  c.take(q.carry, tails);
  const uint64_t runs = std::min<uint64_t>(4 * kScanWaves, (q.m + kTile - 1) / kTile);  // (a run has a tile at least)
  c.take(q.started, runs);
  c.take(q.open_end, runs);
  c.take(q.seg, runs);
  c.take(q.group, tails / 64 + width);
  return c.off;
}

// Bytes of the P and Q rows with these set sizes.
static void row_bytes(const CoefQuery& qy, const uint32_t* cnt, uint64_t* p, uint64_t* q) {
  *p = *q = 256;
  for (uint32_t l = 2; l < qy.k; ++l) {
    *p = std::max<uint64_t>(*p, up(8ull * cnt[l - 2] * width_out(qy, l), 256));
    *q = std::max<uint64_t>(*q, up(8ull * cnt[l - 2] * width_in(qy, l), 256));
  }
}
static uint32_t carried_levels(const CoefQuery& q, const CoefShades& sh, const uint32_t* cnt) {
  uint32_t b = 0;
  for (uint32_t l = 2; l < q.k; ++l)
    if (cnt[l - 2] > kLongRun * scan_runs(q, sh, cnt[l - 2], l)) b |= 1u << (l - 2);
  return b;
}
// Levels where one destination may span more than kFarRuns runs. A list with
// known size is taken to hold a vertex's arrivals at up to eight times the rate at
// which it holds all edges. Sizes that are only bounds (sized false) leave a run's
// length open, and it is taken as one tile, on graphs with a sixteenth of all
// arrivals at one vertex: with less, the tails one by one cost no more than the two
// launches. (Us per query one by one and with prefix sums: 40000 of 50000 edges into
// one vertex, k = 3, 308 and 98; 700000 of 10^6, 1846 and 214; 160000 of 8*10^5, most
// others unused, k = 3, 376 and 153, k = 6, 250 and 213; 12000 of 6*10^4, k = 6, where a
// list holds few of them, 110 and 140. Sized, 4*10^6-edge motif query, 84000 arrivals
// at one vertex, few of them in the lists: 1484 and 1527.)
static uint32_t far_levels(const CoefQuery& q, const CoefShades& sh, const uint32_t* cnt, bool sized, uint64_t m,
                           uint64_t most_arrivals) {
  uint32_t b = 0;
  for (uint32_t l = 2; l < q.k; ++l) {
    const uint64_t n = cnt[l - 2], runs = scan_runs(q, sh, n, l);
    const uint64_t span = sized ? std::min({n, most_arrivals, 8 * most_arrivals * n / m + 1}) * runs / std::max<uint64_t>(n, 1)
                                : (16 * most_arrivals >= m ? most_arrivals / kTile : 0);
    if (std::min(runs, span) > kFarRuns) b |= 1u << (l - 2);
  }
  return b;
}

// Grid sizes of the launches over one or more queries: the largest any needs.
struct CoefGrid {
  uint32_t queries = 0, begin = 1, blocks = 1, k_max = 0, fwd_max = 0, fwd_min = 16, carried = 0, far = 0;
  bool small = true;
  uint32_t runs[kCoefMaxK] = {}, waves[kCoefMaxK] = {}, cblocks[kCoefMaxK] = {}, mul[kCoefMaxK] = {}, carry_mul[kCoefMaxK] = {},
           lds[kCoefMaxK] = {}, carry_lds[kCoefMaxK] = {}, top = 1, per_wave = 64;
  uint64_t last = 0;  // last-level entries, over the queries and the largest
  uint64_t last_max = 0;
  void sets(const CoefQuery& q) {
    ++queries;
    begin = std::max(begin, q.blocks + (uint32_t)(((uint64_t)q.n * q.kq + 1023) / 1024) + q.motif);
    blocks = std::max(blocks, q.blocks);
    k_max = std::max(k_max, q.k);
    fwd_max = std::max(fwd_max, q.fwd);
    fwd_min = std::min(fwd_min, q.plain && q.fwd > 3 ? 4u : 3u);
    small = small && q.words <= kSmallWords;
  }
  void levels(const CoefQuery& q, const CoefShades& sh, const uint32_t* cnt) {
    const uint32_t k = q.k;
    carried |= q.carried;
    far |= q.far;
    for (uint32_t l = 2; l < k; ++l) {
      const uint64_t n = cnt[l - 2];
      const uint32_t r = scan_runs(q, sh, n, l), wl = q.iters ? 0 : mul_lds(k, binom(k, l - 1), binom(k, l));
      runs[l - 1] = std::max(runs[l - 1], r);
      // (A query with fewer entries than the bound may run unpacked.)
      const uint32_t c = width_in(q, l), per = runs_packed(sh.waves[l], c, r) ? 64 / run_lanes(c) : 1;
      waves[l - 1] = std::max({waves[l - 1], (r + per - 1) / per, std::min<uint32_t>(r, sh.waves[l])});
      cblocks[l - 1] = std::max(cblocks[l - 1], (c + 63) / 64);
      if ((q.carried >> (l - 2)) & 1u) {
        carry_mul[l - 1] = std::max(carry_mul[l - 1], (uint32_t)std::min<uint64_t>((n + 15) / 16, kMulBlocks));
        carry_lds[l - 1] = std::max(carry_lds[l - 1], wl);
      } else {
        mul[l - 1] = std::max(mul[l - 1], std::min<uint32_t>(r, sh.waves[l]));
        lds[l - 1] = std::max(lds[l - 1], wl);
      }
    }
    last += cnt[k - 2];
    last_max = std::max<uint64_t>(last_max, cnt[k - 2]);
    for (per_wave = 64; per_wave > 8 && last < 6144ull * per_wave; per_wave /= 2) {
    }
    top = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((last_max + 4 * per_wave - 1) / (4 * per_wave), kTopBlocks));
  }
};

template <class A>
static hipError_t launch_coef_sets(const A& a, const CoefGrid& g, hipStream_t st) {
  const uint32_t nq = g.queries;
  hipLaunchKernelGGL(k_coef_begin<A>, dim3(g.begin, nq), dim3(1024), 0, st, a);
  if (g.small) {
    hipLaunchKernelGGL(k_coef_sets_small<A>, dim3(1, nq), dim3(1024), 0, st, a);
    return hipGetLastError();
  }
  for (uint32_t l = g.fwd_min; l <= g.fwd_max; ++l)
    hipLaunchKernelGGL(k_coef_fwd<A>, dim3(g.blocks, nq), dim3(1024), 0, st, a, l);
  for (uint32_t d = 1; d + 2 <= g.k_max; ++d) {
    if ((uint64_t)g.blocks * nq * kSetBlock >= kWideSets)
      hipLaunchKernelGGL((k_coef_bwd<A, 4>), dim3(g.blocks / 4, nq), dim3(1024), 0, st, a, d);
    else
      hipLaunchKernelGGL((k_coef_bwd<A, 1>), dim3(g.blocks, nq), dim3(1024), 0, st, a, d);
  }
  hipLaunchKernelGGL(k_coef_offsets<A>, dim3(g.k_max - 1, nq), dim3(1024), 0, st, a);
  return hipGetLastError();
}

template <class A>
static hipError_t launch_coef_lists(const A& a, const CoefGrid& g, hipStream_t st) {
  hipLaunchKernelGGL(k_coef_lists<A>, dim3(g.blocks, g.k_max - 1, g.queries), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <class A, bool FAR>
static void launch_coef_mul(const A& a, const CoefGrid& g, uint32_t l, hipStream_t st) {
  const uint32_t i = l - 1, nq = g.queries;
  if (g.carry_mul[i]) {
    hipLaunchKernelGGL(k_coef_carry<A>, dim3((g.runs[i] + 3) / 4, g.cblocks[i], nq), dim3(256), 0, st, a, l);
    hipLaunchKernelGGL((k_coef_mul<A, true, FAR>), dim3(g.carry_mul[i], 1, nq), dim3(256), 4 * g.carry_lds[i], st, a, l,
                       g.carry_lds[i]);
  }
  if (g.mul[i])  // the carry lies behind the waves' rows: at most one row
    hipLaunchKernelGGL((k_coef_mul<A, false, FAR>), dim3(g.mul[i], 1, nq), dim3(256), 5 * g.lds[i], st, a, l, g.lds[i]);
}

template <class A>
static hipError_t launch_coef_level(const A& a, const CoefGrid& g, uint32_t l, hipStream_t st) {
  const uint32_t i = l - 1, nq = g.queries;
  hipLaunchKernelGGL(k_coef_scan<A>, dim3((g.waves[i] + 3) / 4, g.cblocks[i], nq), dim3(256), 0, st, a, l);
  if ((g.far >> (l - 2)) & 1u) {
    hipLaunchKernelGGL(k_coef_fold<A>, dim3((g.runs[i] + 63) / 64, g.cblocks[i], nq), dim3(1024), 0, st, a, l);
    hipLaunchKernelGGL(k_coef_prefix<A>, dim3((g.runs[i] + 63) / 64, g.cblocks[i], nq), dim3(1024), 0, st, a, l);
    launch_coef_mul<A, true>(a, g, l, st);
  } else {
    launch_coef_mul<A, false>(a, g, l, st);
  }
  return hipGetLastError();
}

static hipError_t launch_iter_level(const OneCoef& a, const CoefGrid& g, uint32_t l, hipStream_t st) {
  const uint32_t i = l - 1, cb = g.cblocks[i];
  hipLaunchKernelGGL(k_coef_scan<OneCoef>, dim3((g.waves[i] + 3) / 4, cb, 1), dim3(256), 0, st, a, l);
  if ((g.far >> (l - 2)) & 1u) {
    hipLaunchKernelGGL(k_coef_fold<OneCoef>, dim3((g.runs[i] + 63) / 64, cb, 1), dim3(1024), 0, st, a, l);
    hipLaunchKernelGGL(k_coef_prefix<OneCoef>, dim3((g.runs[i] + 63) / 64, cb, 1), dim3(1024), 0, st, a, l);
  }
  hipLaunchKernelGGL(k_coef_carry<OneCoef>, dim3((g.runs[i] + 3) / 4, cb, 1), dim3(256), 0, st, a, l);
  hipLaunchKernelGGL(k_iter_mul, dim3(std::max(1u, g.carry_mul[i]), cb), dim3(256), 0, st, a, l);
  return hipGetLastError();
}

template <class A>
static hipError_t launch_coef_top(const A& a, const CoefGrid& g, hipStream_t st) {
  hipLaunchKernelGGL(k_coef_top<A>, dim3(g.top, g.queries), dim3(256), 0, st, a, g.per_wave);
  return hipGetLastError();
}

// Rows are sized for all m edges up to this many bytes; above it the set sizes
// are read back first: a synchronisation and an idle GPU of 40 to 50 us, against
// memory for edges no set holds (10^6 edges, k = 8: 1.1 GB, half of what the
// evaluation form's prefix state takes; 407 us with the read-back, 370 without;
// with 70% of the edges in the sets 3080 and 3050, although runs are then
// taken to be short).
constexpr uint64_t kUnsizedRows = 1200ull << 20;
// Rows by iteration are made narrower, for more passes, down to this many bytes.
constexpr uint64_t kIterRows = 4ull << 30;

// By iteration, an entry costs a shared-table product and two rows of traffic,
// and a stored row a product by z^L; the evaluation form spends one lane-wise
// product per entry and no second row, after a longer setup. Where most edges
// are in the sets and the setup is small against the levels, that is the
// faster one (10^6 edges, k = 8, 73% of the edges per level: 9.1 ms against
// 9.5 to 10.0; with 4%: 1.55 against 1.0; 10^5 edges with 72%: 1.32 against 1.15;
// 10^6 uniform edges, k = 10, 14%: 13.3 against 12.0).
static bool dense_sets(const CoefQuery& q, const uint32_t* cnt, uint64_t span) {
  uint64_t total = 0;
  for (uint32_t y = 0; y + 1 < q.k; ++y) total += cnt[y];
  return q.m * span >= 100000000ull && 2 * total > (uint64_t)q.m * (q.k - 1);
}

// Whether run_coef may take this much for the setup and lists (see there).
static bool setup_fits(uint64_t setup, uint64_t eval_lists) { return setup <= std::max<uint64_t>(eval_lists, 8 << 20); }

uint64_t coef_list_bytes(const rs_graph* g, const QueryPlan& qp, uint64_t eval_lists) {
  uint64_t most = 0;
  if (!iter_rows_apply(qp)) return 0;
  for (const uint64_t iters : {uint64_t(0), qp.it_end - qp.it_begin}) {
    CoefQuery q{};
    CoefShades sh{};
    fill_query(q, sh, g->g, qp, nullptr, EdgeFilter(), false, kScanWaves);
    q.iters = (uint32_t)iters;
    const uint64_t b = carve_setup(q, sh, nullptr);
    if (setup_fits(b, eval_lists)) most = std::max(most, b);
  }
  return most;
}
uint64_t coef_batch_query_bytes(const rs_graph* g, const QueryPlan& qp) {
  if (qp.k < 3 || !coef_applies(qp)) return 0;
  CoefQuery q{};
  CoefShades sh{};
  fill_query(q, sh, g->g, qp, nullptr, EdgeFilter(), false, kScanWaves);
  return up(8ull * q.n * q.kq, 256) + up(carve_setup(q, sh, nullptr), 256) + sizeof(CoefQuery) + sizeof(CoefShades) + 256;
}

rs_status run_coef(rs_graph* g, PlainWorkspace& ws, const PlainSizes& sz, const QueryPlan& qp, const QueryExtras* ex,
                   const uint32_t* dv, const EdgeFilter& filt, uint64_t* T, hipStream_t st, bool timed,
                   std::vector<uint64_t>* sums_host, uint32_t* n_sums, bool by_iteration) {
  const uint64_t m = g->g.m, n = g->g.n;
  const uint32_t k = qp.k;
  *n_sums = 0;
  OneCoef a{};
  CoefQuery& q = a.q;
  fill_query(q, a.sh, g->g, qp, dv, filt, ex && ex->fine, kScanWaves);
  q.T = T;
  const uint32_t span = (uint32_t)(qp.it_end - qp.it_begin);
  if (by_iteration) {
    q.iters = span;
    q.carried = (1u << (k - 2)) - 1;
  }
  const uint32_t max_sums = std::max<uint32_t>(kTopBlocks, 1u << kCoefMaxK);
  uint64_t *out = nullptr, *sums = nullptr;
  if (k == 2) {
    if (ws.scratch) {
      if (8 * kTopBlocks > ws.scratch_bytes) return RS_OK;
      sums = reinterpret_cast<uint64_t*>(ws.scratch);
    } else {
      if (!ws.host_result) RS_HIP(hipHostMalloc((void**)&ws.host_result, 8 * max_sums, hipHostMallocDefault));
      sums = ws.host_result;
    }
    q.result = sums;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>((m + 255) / 256, kTopBlocks);
    {
      ProfScope ps(KC_TOP, st, 0.0, timed);
      hipLaunchKernelGGL(k_coef_pairs, dim3(blocks), dim3(256), 0, st, a);
      RS_HIP(hipGetLastError());
    }
    if (ws.scratch) {
      sums_host->resize(blocks);
      RS_HIP(hipMemcpyAsync(sums_host->data(), sums, 8ull * blocks, hipMemcpyDeviceToHost, st));
    }
    *n_sums = blocks;
    return RS_OK;
  }
  // Buffers. The setup and lists take the place of the evaluation form's lists,
  // the rows that of its prefix state: a workspace sized for the evaluation
  // form holds the coefficient form too (small graphs: a few MB over).
  const uint64_t setup_bytes = carve_setup(q, a.sh, nullptr);
  if (!ws.scratch && !setup_fits(setup_bytes, sz.lists)) return RS_OK;
  uint32_t cnt[kCoefMaxK - 1];
  for (uint32_t y = 0; y + 1 < k; ++y) cnt[y] = (uint32_t)m;
  uint64_t p_bytes, q_bytes;
  row_bytes(q, cnt, &p_bytes, &q_bytes);
  uint8_t* scratch_rows = nullptr;
  uint64_t scratch_left = 0;
  if (ws.scratch) {
    Carver c{ws.scratch};
    uint8_t* setup;
    c.take(q.z, sz.z / 8);
    c.take(setup, setup_bytes);
    c.take(out, 16);
    c.take(sums, max_sums);
    if (c.off > ws.scratch_bytes) return RS_OK;
    scratch_rows = ws.scratch + c.off;
    scratch_left = ws.scratch_bytes - c.off;
    carve_setup(q, a.sh, setup);
  } else {
    if (ws.z.reserve(sz.z, st, false) || ws.lists.reserve(setup_bytes, st, false) || ws.out.reserve(128, st, false))
      return RS_ENOMEM;
    if (!ws.host_result) RS_HIP(hipHostMalloc((void**)&ws.host_result, 8 * max_sums, hipHostMallocDefault));
    sums = ws.host_result;
    out = ws.out.as<uint64_t>();
    q.z = ws.z.as<uint64_t>();
    carve_setup(q, a.sh, ws.lists.as<uint8_t>());
  }
  q.det = out;
  q.count = reinterpret_cast<uint32_t*>(out + 4);
  q.result = sums;
  q.z1 = q.z;
  q.z1_stride = q.kq;

  CoefGrid grid;
  grid.sets(q);
  if (by_iteration && q.motif) {  // the forms themselves, not their shades' coefficients
    grid.begin = q.blocks;  // no vertex rows, no determinant
    RS_HIP(launch_ztable(q.z, (uint32_t)n, qp, q.colour, st));
  }
  {
    ProfScope ps(KC_WINDOW, st, 20.0 * m, timed);
    RS_HIP(launch_coef_sets(a, grid, st));
  }
  uint32_t counted[kCoefMaxK] = {};
  auto fits = [&] { return ws.scratch ? p_bytes + q_bytes <= scratch_left : p_bytes <= sz.p && q_bytes <= sz.p; };
  bool sized = !fits() || p_bytes + q_bytes > kUnsizedRows;
  if (!sized && timed && profiling_on()) {  // the byte accounting wants the sizes
    RS_HIP(hipMemcpyAsync(counted, q.count, 4 * (k - 1), hipMemcpyDeviceToHost, st));
    RS_HIP(hipStreamSynchronize(st));
  }
  if (sized) {
    RS_HIP(hipMemcpyAsync(cnt, q.count, 4 * (k - 1), hipMemcpyDeviceToHost, st));
    RS_HIP(hipStreamSynchronize(st));
    row_bytes(q, cnt, &p_bytes, &q_bytes);
    while (q.iters > 64 && (!fits() || p_bytes + q_bytes > kIterRows)) {
      q.iters = (q.iters / 2 + 63) / 64 * 64;
      row_bytes(q, cnt, &p_bytes, &q_bytes);
    }
    if (!fits() || (by_iteration && dense_sets(q, cnt, span))) return RS_OK;
    if (!by_iteration) q.carried = carried_levels(q, a.sh, cnt);
    std::copy(cnt, cnt + k - 1, counted);
  }
  q.far = far_levels(q, a.sh, cnt, sized, m, g->info.max_in_degree);
  // by vertex only where the table fits P, and, the list's size unknown, where it is
  // small against the edges
  q.by_entry = by_iteration && n > (sized ? cnt[0] : m / 8) ? 1 : 0;
  // bytes a level's scan and products cannot do without: per entry its list
  // entry and the two window rows it reads
  auto level_bytes = [&](uint32_t l) { return (double)counted[l - 2] * (22.0 + 16.0 * width_in(q, l)); };
  if (ws.scratch) {
    q.P = reinterpret_cast<uint64_t*>(scratch_rows);
    q.Q = reinterpret_cast<uint64_t*>(scratch_rows + p_bytes);
  } else {
    // an eighth to spare, so that the next query's slightly larger sets fit too
    if (ws.p0.reserve(p_bytes > ws.p0.bytes ? std::min(sz.p, p_bytes + p_bytes / 8) : 8, st, false) ||
        ws.p1.reserve(q_bytes > ws.p1.bytes ? std::min(sz.p, q_bytes + q_bytes / 8) : 8, st, false))
      return RS_ENOMEM;
    q.P = ws.p0.as<uint64_t>();
    q.Q = ws.p1.as<uint64_t>();
  }
  grid.levels(q, a.sh, cnt);
  {
    ProfScope ps(KC_QTABLE, st, 40.0 * m, timed);
    RS_HIP(launch_coef_lists(a, grid, st));
  }
  uint32_t sums_out = grid.top;
  if (by_iteration) {
    q.z1 = q.P;
    q.z1_stride = q.iters;
    const uint32_t top_runs = scan_runs(q, a.sh, cnt[k - 2], k), cb = (q.iters + 63) / 64;
    for (uint32_t i = 0; i < span; i += q.iters) {
      q.it0 = (uint32_t)qp.it_begin + i;
      q.result = sums + i;
      hipLaunchKernelGGL(k_iter_z, dim3(std::max(1u, std::min((uint32_t)((q.by_entry ? cnt[0] : n) + 3) / 4, kMulBlocks)), cb), dim3(256), 0, st, a);
      RS_HIP(hipGetLastError());
      for (uint32_t l = 2; l < k; ++l) {
        ProfScope ps(l == 2 ? KC_FIRST : KC_SCAN, st, level_bytes(l), timed);
        RS_HIP(launch_iter_level(a, grid, l, st));
      }
      ProfScope ps(KC_TOP, st, 0.0, timed);
      hipLaunchKernelGGL(k_iter_top, dim3((top_runs + 3) / 4, cb), dim3(256), 0, st, a);
      hipLaunchKernelGGL(k_iter_fold, dim3(cb), dim3(1024), 0, st, a, std::min(q.iters, span - i));
      RS_HIP(hipGetLastError());
    }
    sums_out = span;
  } else {
    for (uint32_t l = 2; l < k; ++l) {
      ProfScope ps(l == 2 ? KC_FIRST : KC_SCAN, st, level_bytes(l), timed);
      RS_HIP(launch_coef_level(a, grid, l, st));
    }
    ProfScope ps(KC_TOP, st, level_bytes(k), timed);
    RS_HIP(launch_coef_top(a, grid, st));
  }
  // the sums: in pinned memory once the stream is done, or read back
  if (ws.scratch) {
    sums_host->resize(sums_out);
    RS_HIP(hipMemcpyAsync(sums_host->data(), sums, 8ull * sums_out, hipMemcpyDeviceToHost, st));
  }
  *n_sums = sums_out;
  return RS_OK;
}

// ---------------------------------------------------------------------------
// Many queries at once.
// ---------------------------------------------------------------------------
struct CoefBatch {
  DevBuf desc;
  uint8_t* host = nullptr;  // pinned: descriptors to upload, set sizes and results read back
  uint64_t host_bytes = 0;
};
CoefBatch* coef_batch_create() { return new CoefBatch(); }
void coef_batch_release(CoefBatch* b) {
  b->desc.release();
  if (b->host) (void)hipHostFree(b->host);
  b->host = nullptr;
  b->host_bytes = 0;
}
void coef_batch_destroy(CoefBatch* b) {
  coef_batch_release(b);
  delete b;
}
uint64_t coef_batch_bytes(const CoefBatch* b) { return b->desc.bytes; }

// Queries of one launch share its LDS size, which follows the widest row; a row
// product of k = 12 holds 61 KB per block (77 KB where it sums the carries itself),
// one of k = 9 13 KB (16 KB), so the widths are kept apart in these classes.
static uint32_t width_class(uint32_t k) { return k <= 9 ? 0 : (k <= 11 ? 1 : 2); }

rs_status run_coef_batch(CoefBatch& B, DevBuf& setup, DevBuf& rows, const rs_graph* const* graphs, const std::vector<QueryPlan>& plans,
                         const std::vector<uint32_t>& idx_in, rs_result* results, hipStream_t st, uint64_t budget,
                         std::vector<uint32_t>* left) {
  std::vector<uint32_t> idx = idx_in;
  std::stable_sort(idx.begin(), idx.end(), [&](uint32_t x, uint32_t y) {
    const uint32_t cx = width_class(plans[x].k), cy = width_class(plans[y].k);
    return cx != cy ? cx < cy : plans[x].k > plans[y].k;
  });
  const uint32_t nq = (uint32_t)idx.size();
  if (!nq) return RS_OK;
  // pinned staging: descriptors, shades, set sizes, results
  const uint64_t b_desc = up(sizeof(CoefQuery) * nq, 256), b_sh = up(sizeof(CoefShades) * nq, 256), b_cnt = up(64ull * nq, 256),
                 b_out = up(8ull * nq, 256);
  const uint32_t top_cap = std::max(32u, kTopBlocks * 4 / nq);  // last-level blocks per query
  const uint64_t b_res = 8ull * top_cap * nq;
  const uint64_t host_need = b_desc + b_sh + b_cnt + b_res;
  if (B.host_bytes < host_need) {
    if (B.host) (void)hipHostFree(B.host);
    B.host = nullptr;
    B.host_bytes = 0;
    RS_HIP(hipHostMalloc((void**)&B.host, host_need, hipHostMallocDefault));
    B.host_bytes = host_need;
  }
  CoefQuery* qs = reinterpret_cast<CoefQuery*>(B.host);
  CoefShades* sh = reinterpret_cast<CoefShades*>(B.host + b_desc);
  uint32_t* cnt = reinterpret_cast<uint32_t*>(B.host + b_desc + b_sh);
  uint64_t* res = reinterpret_cast<uint64_t*>(B.host + b_desc + b_sh + b_cnt);
  if (B.desc.reserve(b_desc + b_sh + b_cnt + b_out, st, false)) return RS_ENOMEM;
  uint8_t* dd = B.desc.as<uint8_t>();
  // most waves of one query in a level's launch (see below); the blocks that a
  // smaller query leaves empty cost little up to this many
  const uint32_t waves = std::min(kScanWaves, std::max(256u, 8 * kScanWaves / nq));
  uint64_t setup_bytes = 0;
  std::vector<uint64_t> z_off(nq), s_off(nq);
  for (uint32_t i = 0; i < nq; ++i) {
    const QueryPlan& qp = plans[idx[i]];
    qs[i] = CoefQuery{};
    fill_query(qs[i], sh[i], graphs[idx[i]]->g, qp, nullptr, EdgeFilter(), false, waves);
    z_off[i] = setup_bytes;
    setup_bytes += up(8ull * qs[i].n * qs[i].kq, 256);
    s_off[i] = setup_bytes;
    setup_bytes += up(carve_setup(qs[i], sh[i], nullptr), 256);
  }
  if (setup.reserve(setup_bytes, st, false)) return RS_ENOMEM;
  uint32_t* d_cnt = reinterpret_cast<uint32_t*>(dd + b_desc + b_sh);
  uint64_t* d_out = reinterpret_cast<uint64_t*>(dd + b_desc + b_sh + b_cnt);
  CoefGrid all;
  for (uint32_t i = 0; i < nq; ++i) {
    CoefQuery& q = qs[i];
    q.z = reinterpret_cast<uint64_t*>(setup.as<uint8_t>() + z_off[i]);
    q.z1 = q.z;
    q.z1_stride = q.kq;
    carve_setup(q, sh[i], setup.as<uint8_t>() + s_off[i]);
    q.count = d_cnt + 16 * i;
    q.det = d_out + i;
    q.result = res + (uint64_t)top_cap * i;
    all.sets(q);
  }
  const ManyCoef many{reinterpret_cast<const CoefQuery*>(dd), reinterpret_cast<const CoefShades*>(dd + b_desc)};
  RS_HIP(hipMemcpyAsync(dd, B.host, b_desc + b_sh, hipMemcpyHostToDevice, st));
  RS_HIP(launch_coef_sets(many, all, st));
  RS_HIP(hipMemcpyAsync(cnt, d_cnt, 64ull * nq, hipMemcpyDeviceToHost, st));
  RS_HIP(hipStreamSynchronize(st));
  // A level's launch shares two GPUs' worth of waves over its queries by their
  // products: queries differ by orders of magnitude, and few reach the high
  // levels. (24 queries on 10^6 edges, levels 2 to 8: the scans took 280, 211,
  // 285, 298, 256, 242 and 163 us with equal shares, 229, 193, 173, 157, 119, 112
  // and 59 so.)
  for (uint32_t l = 2; l <= kCoefMaxK; ++l) {
    auto work = [&](uint32_t i) { return l < qs[i].k ? (double)cnt[16 * i + l - 2] * binom(qs[i].k, l - 1) : 0.0; };
    double total = 1;
    for (uint32_t i = 0; i < nq; ++i) total += work(i);
    for (uint32_t i = 0; i < nq; ++i)
      sh[i].waves[l] = (uint32_t)std::min<double>(waves, std::max(64.0, 2.0 * kScanWaves * work(i) / total));
  }
  // rounds of consecutive queries whose rows fit the budget
  std::vector<uint64_t> p_off(nq), q_off(nq);
  std::vector<std::pair<uint32_t, uint32_t>> rounds;
  std::vector<bool> run(nq, true);
  std::vector<uint32_t> sums(nq, 0);
  uint64_t at = 0, most = 256;
  uint32_t first = 0;
  for (uint32_t i = 0; i < nq; ++i) {
    uint64_t p, q;
    row_bytes(qs[i], cnt + 16 * i, &p, &q);
    qs[i].carried = carried_levels(qs[i], sh[i], cnt + 16 * i);
    qs[i].far = far_levels(qs[i], sh[i], cnt + 16 * i, true, qs[i].m, graphs[idx[i]]->info.max_in_degree);
    if (p + q > budget) {  // too large for this form: left to the caller
      run[i] = false;
      left->push_back(idx[i]);
      p = q = 0;
    }
    if (at + p + q > budget || (i > first && width_class(qs[i].k) != width_class(qs[first].k))) {
      rounds.push_back({first, i});
      first = i;
      at = 0;
    }
    p_off[i] = at;
    q_off[i] = at + p;
    at += p + q;
    most = std::max(most, at);
  }
  rounds.push_back({first, nq});
  if (rows.reserve(most > rows.bytes ? std::min(std::max(budget, most), most + most / 8) : 8, st, false))
    return RS_ENOMEM;
  for (uint32_t i = 0; i < nq; ++i) {
    qs[i].P = reinterpret_cast<uint64_t*>(rows.as<uint8_t>() + p_off[i]);
    qs[i].Q = reinterpret_cast<uint64_t*>(rows.as<uint8_t>() + q_off[i]);
    if (!run[i]) qs[i].k = 0;  // (no kernel takes a query of no levels)
  }
  RS_HIP(hipMemcpyAsync(dd, B.host, b_desc + b_sh, hipMemcpyHostToDevice, st));
  for (const auto& rd : rounds) {
    CoefGrid g;
    const ManyCoef part{many.qs + rd.first, many.sh + rd.first};
    for (uint32_t i = rd.first; i < rd.second; ++i) {
      if (!run[i]) {
        ++g.queries;
        continue;
      }
      g.sets(qs[i]);
      g.levels(qs[i], sh[i], cnt + 16 * i);
    }
    if (g.k_max == 0) continue;
    g.top = std::min(g.top, top_cap);
    for (uint32_t i = rd.first; i < rd.second; ++i) sums[i] = g.top;
    RS_HIP(launch_coef_lists(part, g, st));
    for (uint32_t l = 2; l < g.k_max; ++l) RS_HIP(launch_coef_level(part, g, l, st));
    RS_HIP(launch_coef_top(part, g, st));
  }
  RS_HIP(hipStreamSynchronize(st));
  for (uint32_t i = 0; i < nq; ++i) {
    if (!run[i]) continue;
    rs_result& r = results[idx[i]];
    r.fingerprint = 0;
    for (uint32_t b = 0; b < sums[i]; ++b) r.fingerprint ^= ((volatile uint64_t*)res)[(uint64_t)top_cap * i + b];
    r.yes = r.fingerprint != 0;
    r.status = RS_OK;
  }
  return RS_OK;
}


// ---------------------------------------------------------------------------
// The literal reading (rs_literal.hip) in the coefficient form.
//
// Its y variables belong to a window term, not to an edge: slot s = (u, i) holds
//   chi_l(s) = z_u * XOR over in-edges e = (v -> u, i), window slots q of v
//                    of y(e, time of q, l-1) * chi_{l-1}(q),
// so a level is no prefix sum, but the walk polynomial is the same and a slot
// holds C(k,l) coefficients. The sets are over slots: forward, those with an
// edge whose window holds a slot of the set below; backward, those in a window
// of a set slot above. A window's slots are consecutive in the set below, so an
// edge's terms are a range of its rows. One wave forms a slot's row: terms in
// tiles of eight (a lane hashes one term's y and writes two of its multiples),
// then the vertex product. (10^6-edge path query, k = 8: the levels took 3.3 ms
// and the last one 1.2 in the evaluation form, with every slot some window
// reads and 256 values each; here 24 to 39 us each and 83, the sets and lists
// 200. Bound by latency: a wave's four dependent loads against one to two terms
// per slot.)
// ---------------------------------------------------------------------------
struct LitCoef {
  const uint32_t *slot_e, *slot_t, *v_soff;  // edges of a slot [ns + 1], its time, first slot of a vertex
  const uint32_t* slot;                      // [m] slot of an edge
  uint32_t *wlo, *whi;                       // [m] window of each edge, in slots
  uint64_t* fb;                              // [fwd - 1][words] forward sets of levels 2..fwd
  uint8_t* mark;                             // [k - 2][words * 64] levels 2..k-1: slots some window reads
  uint4* ls;                                 // lists: first edge, end, vertex, slot
  uint32_t* rt;                              // time of a list entry
  uint4* te;                                 // [k - 1][m] by edge: first row and rows of its terms, edge key (level 2: Y2)
  uint64_t* zs;                              // [ns] value of each slot
  uint32_t m, ns, nbe, nbz;
  uint64_t hp;
};

__device__ __forceinline__ uint32_t slot_search(const uint32_t* t, uint32_t a, uint32_t b, uint32_t x) {  // first >= x
  while (a < b) {
    const uint32_t mid = a + ((b - a) >> 1);
    if (t[mid] < x) a = mid + 1; else b = mid;
  }
  return a;
}

// Block roles: edges (their windows), slots (the level-2 set), vertex rows, and
// for motif queries one block for det Omega. Clears the marks and the values.
__global__ __launch_bounds__(1024) void k_litc_begin(OneCoef a, LitCoef T) {
  __shared__ DetShared sh;
  const CoefQuery& Q = a.q;
  const uint32_t tid = threadIdx.x;
  uint32_t b = blockIdx.x;
  {
    const uint64_t i0 = (uint64_t)b * 1024 + tid, step = (uint64_t)gridDim.x * 1024, nm = (uint64_t)(Q.k - 2) * Q.words * 8;
    for (uint64_t i = i0; i < nm; i += step) reinterpret_cast<uint64_t*>(T.mark)[i] = 0;
    for (uint64_t i = i0; i < T.ns; i += step) T.zs[i] = 0;
    for (uint64_t i = Q.words + i0; i < (uint64_t)(Q.fwd - 1) * Q.words; i += step) T.fb[i] = 0;
  }
  if (b < T.nbe) {
    const uint32_t e = b * 1024 + tid;
    if (e < T.m) {
      const uint32_t v = Q.e_src[e], i = Q.e_t[e], dv = Q.dv ? Q.dv[v] : Q.delta;
      const uint32_t lo = T.v_soff[v], hi = T.v_soff[v + 1];
      const uint32_t x = slot_search(T.slot_t, lo, hi, i > dv ? i - dv : 1u);
      T.wlo[e] = x;
      T.whi[e] = i == 0xFFFFFFFFu ? hi : slot_search(T.slot_t, x, hi, i + 1);
    }
    return;
  }
  b -= T.nbe;
  if (b < Q.blocks) {
    const uint32_t s = b * kSetBlock + tid;
    bool in = s < T.ns;
    if (in && Q.motif) {
      const uint32_t e0 = T.slot_e[s], e1 = T.slot_e[s + 1];
      in = false;
      if (a.mu(0, Q.colour[Q.e_dst[e0]]))
        for (uint32_t e = e0; e < e1 && !in; ++e) in = a.mu(0, Q.colour[Q.e_src[e]]) != 0;
    }
    const uint64_t f = __ballot(in);
    if ((tid & 63u) == 0) T.fb[b * 16 + (tid >> 6)] = f;
    return;
  }
  b -= Q.blocks;
  if (b < T.nbz) {
    const uint64_t idx = (uint64_t)b * 1024 + tid;
    if (idx < (uint64_t)Q.n * Q.kq) Q.z[idx] = vertex_form(a, Q, 0, idx);
    return;
  }
  if (Q.motif && b == T.nbz) shade_det(Q, sh);
}

// The set passes and the lists take an edge per thread, 1024 edges per block: a
// hub holds any number of edges per slot. (90 per slot, 3*10^5 edges, k = 3, with
// each slot's edges gone over by the slot's thread: forward pass 42 us, backward
// passes 82, lists 460, and 12 ms with delta = 400, where an edge's level-2
// constant sums 401 hashes; 4, 4, 13 and 167 us so.)

// Forward set of level l (3..fwd): the slots of the set below with an edge whose
// window holds one of its slots. The set's bits are zero before (k_litc_begin).
__global__ __launch_bounds__(1024) void k_litc_fwd(OneCoef a, LitCoef T, uint32_t l) {
  __shared__ uint64_t hit[17];  // the slots of 1024 edges
  const CoefQuery& Q = a.q;
  const uint64_t* below = T.fb + (uint64_t)(l - 3) * Q.words;
  uint64_t* here = T.fb + (uint64_t)(l - 2) * Q.words;
  const uint32_t tid = threadIdx.x, e = blockIdx.x * 1024 + tid, w0 = T.slot[blockIdx.x * 1024] >> 6;
  if (tid < 17) hit[tid] = 0;
  __syncthreads();
  if (e < T.m) {
    const uint32_t s = T.slot[e], x = T.wlo[e], y = T.whi[e];
    const uint64_t bit = 1ull << (s & 63u);
    if (x < y && (below[s >> 6] & bit)) {
      bool in = false;
      const uint32_t wa = x >> 6, wb = (y - 1) >> 6;
      for (uint32_t i = wa; i <= wb && !in; ++i)
        in = (below[i] & (i == wa ? bits_from(x) : ~0ull) & (i == wb ? bits_below_incl(y - 1) : ~0ull)) != 0;
      if (in) atomicOr((unsigned long long*)&hit[(s >> 6) - w0], (unsigned long long)bit);
    }
  }
  __syncthreads();
  if (tid < 17 && hit[tid]) atomicOr((unsigned long long*)&here[w0 + tid], (unsigned long long)hit[tid]);
}

// Is slot s in the set of level l: in the forward set and, below the last
// level, in a window of the level above.
__device__ __forceinline__ bool lit_in_set(const CoefQuery& Q, const LitCoef& T, uint32_t l, uint32_t s) {
  return ((T.fb[(uint64_t)(min(l, Q.fwd) - 2) * Q.words + (s >> 6)] >> (s & 63u)) & 1u) &&
         (l == Q.k || T.mark[(uint64_t)(l - 2) * Q.words * 64 + s]);
}

// Set of level l (k .. 2) with its ranks, by the first Q.blocks blocks; the others
// mark the windows of its edges for the level below.
__global__ __launch_bounds__(1024) void k_litc_bwd(OneCoef a, LitCoef T, uint32_t l) {
  __shared__ uint64_t sl[16];
  const CoefQuery& Q = a.q;
  if (blockIdx.x >= Q.blocks) {
    const uint32_t e = (blockIdx.x - Q.blocks) * 1024 + threadIdx.x;
    if (l == 2 || e >= T.m || !lit_in_set(Q, T, l, T.slot[e])) return;
    uint8_t* mk = T.mark + (uint64_t)(l - 3) * Q.words * 64;
    const uint32_t y = T.whi[e];
    for (uint32_t q = T.wlo[e]; q < y; ++q) mk[q] = 1;
    return;
  }
  const uint32_t s = blockIdx.x * kSetBlock + threadIdx.x;
  set_word(Q, l - 2, s >> 6, __ballot(lit_in_set(Q, T, l, s)), sl);
  set_ranks(Q, l - 2, blockIdx.x, sl);
}

// Lists of levels 2..k (as k_coef_lists): the first Q.blocks blocks of a level
// write its slots, the others its edges, 1024 each. Either gathers what is in the
// set in LDS first, so that all lanes are busy.
__global__ __launch_bounds__(256) void k_litc_lists(OneCoef a, LitCoef T) {
  __shared__ uint16_t at[kSetBlock];
  __shared__ uint32_t count;
  const CoefQuery& Q = a.q;
  const uint32_t y = blockIdx.y, l = y + 2, lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  const uint64_t* bits = Q.sbits + (uint64_t)y * Q.words;
  if (blockIdx.x < Q.blocks) {
    const uint32_t n = Q.bsum[(uint64_t)y * Q.blocks + blockIdx.x];
    if (n == 0) return;
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
      const uint32_t lw = r * 4 + wv, w = blockIdx.x * 16 + lw;
      const uint64_t b = bits[w];
      if ((b >> lane) & 1ull)
        at[Q.wrank[(uint64_t)y * Q.words + w] + __popcll(b & ((1ull << lane) - 1))] = (uint16_t)(lw * 64 + lane);
    }
    __syncthreads();
    const uint64_t p0 = y * Q.lstride + Q.boff[(uint64_t)y * Q.blocks + blockIdx.x];
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
      const uint32_t s = blockIdx.x * kSetBlock + at[i], e0 = T.slot_e[s];
      T.ls[p0 + i] = make_uint4(e0, T.slot_e[s + 1], Q.e_dst[e0], s);
      T.rt[p0 + i] = T.slot_t[s];
    }
    return;
  }
  const uint32_t eb = (blockIdx.x - Q.blocks) * 1024;
  if (threadIdx.x == 0) count = 0;
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < 4; ++r) {
    const uint32_t i = r * 256 + threadIdx.x, s = eb + i < T.m ? T.slot[eb + i] : 0u;
    const uint64_t in = __ballot(eb + i < T.m && ((bits[s >> 6] >> (s & 63u)) & 1u));
    uint32_t p = 0;
    if (lane == 0 && in) p = atomicAdd(&count, (uint32_t)__popcll(in));
    p = __shfl(p, 0, 64);
    if ((in >> lane) & 1u) at[p + __popcll(in & ((1ull << lane) - 1))] = (uint16_t)i;
  }
  __syncthreads();
  uint4* te = T.te + (uint64_t)y * T.m;
  const uint32_t n = count;
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    const uint32_t e = eb + at[i], v = Q.e_src[e];
    const uint64_t h = lit_edge_key(T.hp, v, Q.e_dst[e]);
    if (l == 2) {
      const uint32_t t = Q.e_t[e], dv = Q.dv ? Q.dv[v] : Q.delta;
      uint64_t y2 = 0;  // the window sum of y over every time t - j >= 1, j <= delta(v)
      for (uint64_t p = t > dv ? t - dv : 1u; p <= t; ++p) y2 ^= lit_y(h, (uint32_t)p, 1);
      te[e] = make_uint4(v, 1, lo32(y2), hi32(y2));
    } else {
      const uint32_t ra = set_rank(Q, y - 1, T.wlo[e]), rb = set_rank(Q, y - 1, T.whi[e]);
      te[e] = make_uint4(ra, rb - ra, lo32(h), hi32(h));
    }
  }
}

__device__ __forceinline__ uint4 load_const4(const uint4* p) {  // by scalar loads
  const auto* q = as_const((const uint32_t*)p);
  return make_uint4(q[0], q[1], q[2], q[3]);
}

// XOR of the terms of a slot's edges, coefficient ca of each (l: the slot's level).
__device__ __forceinline__ uint64_t lit_terms(const CoefQuery& Q, const LitCoef& T, uint32_t l, uint4 s, uint32_t C,
                                              uint32_t ca, uint32_t lane, uint64_t* region) {
  const uint4* te = T.te + (uint64_t)(l - 2) * T.m;
  const uint32_t* rt = T.rt + (uint64_t)(l - 3) * Q.lstride;  // (l > 2)
  const uint32_t tb = lds_addr(region);
  Acc128 acc = {0, 0, 0, 0};
  for (uint32_t e = s.x; e < s.y; ++e) {
    const uint4 t = load_const4(te + e);
    const uint64_t h = mk64(t.z, t.w);
    if (l == 2) {
      const uint64_t w = *(gu64*)(Q.z + (uint64_t)t.x * Q.kq + ca);
      wave_lds_fence();
      if (lane < 16) region[lane] = multiple(h, lane);
      wave_lds_fence();
      comb8(tb, w, acc);
      continue;
    }
    for (uint32_t r = t.x, end = t.x + t.y; r < end; r += kTile) {
      const uint32_t nt = min(kTile, end - r);
      const uint32_t time = rt[r + min(lane >> 3, nt - 1)];
      uint64_t w[kTile];
#pragma unroll
      for (uint32_t i = 0; i < kTile; ++i) {
        w[i] = 0;
        if (i < nt) w[i] = *(gu64*)(Q.P + (uint64_t)(r + i) * C + ca);
      }
      const uint64_t yv = lit_y(h, time, l - 1);
      wave_lds_fence();
      tile_tables(region, lane, yv);
      wave_lds_fence();
#pragma unroll
      for (uint32_t i = 0; i < kTile; ++i)
        if (i < nt) comb8(tb + i * 128u, w[i], acc);
    }
  }
  return gf_reduce(acc);
}

// Rows of level l (2..k-1), one wave per slot of its set (in turn past kLitBlocks
// blocks).
__global__ __launch_bounds__(256) void k_litc_level(OneCoef a, LitCoef T, uint32_t l, uint32_t wave_lds, uint64_t* rows) {
  extern __shared__ uint64_t dyn_lds[];  // [4][wave_lds]: tables of a tile, then the row product's
  const CoefQuery& Q = a.q;
  const uint32_t lane = threadIdx.x & 63u, k = Q.k;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n = *as_const(Q.count + (l - 2));
  uint64_t* region = dyn_lds + wv * (wave_lds / 8);
  RowMul M;
  M.c_in = kBinomD.v[k][l - 1];
  M.c_out = kBinomD.v[k][l];
  M.per = kBinomD.v[k - 1][l - 1];
  M.tab = region + kTile * 16;
  M.q = M.tab + k * 16;
  M.out = M.q + M.c_in;
  M.pairs = kPairTable.v + kPairTable.base[k][l];
  M.lane = lane;
  M.cur = kNoRow;
  M.j0 = 0;
  M.nj = k;
  for (uint64_t p = blockIdx.x * 4 + wv; p < n; p += gridDim.x * 4) {
    const uint4 s = load_const4(T.ls + (uint64_t)(l - 2) * Q.lstride + p);
    for (uint32_t cb = 0; cb < M.c_in; cb += kLanes) {
      const uint32_t co = cb + lane;
      const uint64_t v = lit_terms(Q, T, l, s, M.c_in, min(co, M.c_in - 1), lane, region);
      if (co < M.c_in) M.q[co] = v;
    }
    M.form(a, Q, s.z, rows + p * M.c_out);
    wave_lds_fence();  // the row has been read before the next one is begun
  }
}

// Last level: the value of each slot of its set.
__global__ __launch_bounds__(256) void k_litc_top(OneCoef a, LitCoef T) {
  __shared__ struct {
    uint64_t tab[4][16][kLanes];
    uint64_t ytab[4][kTile * 16];
    uint64_t part[4];
  } sh;  // the only static LDS: starts at address 0
  const CoefQuery& Q = a.q;
  const uint32_t lane = threadIdx.x & 63u, k = Q.k;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint64_t* tab = &sh.tab[wv][0][lane];
  tab[0] = 0;
  const uint32_t n = *as_const(Q.count + (k - 2)), ca = min(lane, k - 1);
  uint64_t sum = 0;
  for (uint64_t p = blockIdx.x * 4 + wv; p < n; p += gridDim.x * 4) {
    const uint4 s = load_const4(T.ls + (uint64_t)(k - 2) * Q.lstride + p);
    const uint64_t z = lane < k ? *(gu64*)(Q.z + (uint64_t)s.z * Q.kq + (k - 1 - lane)) : 0;
    uint64_t v = gf_mul(tab, lit_terms(Q, T, k, s, k, ca, lane, sh.ytab[wv]), z);
    uint32_t v0 = lo32(v), v1 = hi32(v);
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      v0 ^= (uint32_t)__shfl_xor((int)v0, d, kLanes);
      v1 ^= (uint32_t)__shfl_xor((int)v1, d, kLanes);
    }
    v = mk64(v0, v1);  // (lanes 0..15 hold the k <= 12 products)
    if (Q.motif) v = gf_mul(tab, v, *Q.det);
    if (lane == 0) T.zs[s.w] = v;
    sum ^= v;
  }
  if (lane == 0) sh.part[wv] = sum;
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(Q.result + blockIdx.x, sh.part[0] ^ sh.part[1] ^ sh.part[2] ^ sh.part[3], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// Blocks of a level's rows at most: a launch takes fewer than 2^32 work items along
// a dimension, and a level may hold as many slots.
constexpr uint64_t kLitBlocks = 1 << 20;

bool lit_coef_applies(const LiteralState& L, uint64_t m, const QueryPlan& qp) {
  if (qp.k < 3 || !coef_applies(qp) || !L.ns || L.max_slot_edges > kLitSlotEdges) return false;
  // Edges that the longest slot's wave goes over, a pass per 64 coefficients, over
  // the levels, against the edges that the evaluation form's time allows, which is per
  // level a latency and the edges and chunks of all slots. Evaluation and coefficient
  // form beyond the line: 100 edges a slot, k = 3, 336 us and 627; 12000 edges, up to 84
  // parallel ones, k = 8, 406 and 728. Within it: 300000 edges with a hub, k = 6, 27.0 ms
  // and 16.6; 172000 edges, k = 7, 2.88 ms and 1.15.
  uint64_t passes = 0;
  for (uint32_t l = 2; l < qp.k; ++l) passes += (binom(qp.k, l - 1) + 63) / 64;
  return L.max_slot_edges * passes <= (qp.k - 1) * (8 + m * (qp.chunk_last - qp.chunk_first) / 2560);
}

rs_status run_literal_coef(const GraphDev& G, LiteralState& L, const QueryPlan& qp, const uint32_t* dv, uint64_t hp,
                           hipStream_t st, uint32_t* n_sums) {
  *n_sums = 0;
  const uint64_t m = G.m, ns = L.ns;
  const uint32_t n = G.n, k = qp.k;
  OneCoef a{};
  CoefQuery& q = a.q;
  fill_query(q, a.sh, G, qp, dv, EdgeFilter{}, false, kScanWaves);
  q.m = (uint32_t)ns;  // the sets are over slots
  q.blocks = (uint32_t)up((ns + kSetBlock - 1) / kSetBlock, 4);
  q.words = q.blocks * 16;
  q.lstride = up(ns, 64);
  LitCoef T{};
  T.slot_e = L.slot_e.as<uint32_t>();
  T.slot_t = L.slot_t.as<uint32_t>();
  T.v_soff = L.v_soff.as<uint32_t>();
  T.slot = L.slot.as<uint32_t>();
  T.m = (uint32_t)m;
  T.ns = (uint32_t)ns;
  T.hp = hp;
  T.nbe = (uint32_t)((m + 1023) / 1024);
  T.nbz = (uint32_t)(((uint64_t)n * qp.kq + 1023) / 1024);
  auto carve = [&](uint8_t* base) {
    Carver c{base};
    const uint64_t lv = k - 1;
    c.take(q.z, (uint64_t)n * qp.kq);
    c.take(q.det, 1);
    c.take(q.count, 16);
    c.take(q.sbits, lv * q.words);
    c.take(q.wrank, lv * q.words);
    c.take(q.bsum, lv * q.blocks);
    c.take(q.boff, lv * q.blocks);
    c.take(T.wlo, m);
    c.take(T.whi, m);
    c.take(T.fb, (uint64_t)(q.fwd - 1) * q.words);
    c.take(T.mark, (uint64_t)(k - 2) * q.words * 64);
    c.take(T.ls, lv * q.lstride);
    c.take(T.rt, lv * q.lstride);
    c.take(T.te, lv * m);
    return c.off;
  };
  if (L.coef.reserve(carve(nullptr), st, false)) return RS_OK;
  carve(L.coef.as<uint8_t>());
  T.zs = L.zs.as<uint64_t>();
  if (!L.host_result) RS_HIP(hipHostMalloc((void**)&L.host_result, 8 * (kTopBlocks + kCoefMaxK), hipHostMallocDefault));
  if (!L.counted) RS_HIP(hipEventCreateWithFlags(&L.counted, hipEventDisableTiming));
  q.result = L.host_result;
  {
    ProfScope ps(KC_LITERAL, st, 0.0);
    hipLaunchKernelGGL(k_litc_begin, dim3(T.nbe + q.blocks + T.nbz + q.motif), dim3(1024), 0, st, a, T);
    for (uint32_t l = 3; l <= q.fwd; ++l) hipLaunchKernelGGL(k_litc_fwd, dim3(T.nbe), dim3(1024), 0, st, a, T, l);
    for (uint32_t l = k; l >= 2; --l)
      hipLaunchKernelGGL(k_litc_bwd, dim3(q.blocks + (l > 2 ? T.nbe : 0)), dim3(1024), 0, st, a, T, l);
    hipLaunchKernelGGL(k_coef_offsets<OneCoef>, dim3(k - 1, 1), dim3(1024), 0, st, a);
    RS_HIP(hipGetLastError());
  }
  // The set sizes come back while the lists are formed, which do not need them: with
  // the stream idle during the copy and the wait (45 us), small queries took longer
  // than in the evaluation form (1515 edges, k = 7: 200 us, 173 so, 161 there).
  uint32_t* cnt = reinterpret_cast<uint32_t*>(L.host_result + kTopBlocks);
  RS_HIP(hipMemcpyAsync(cnt, q.count, 4 * (k - 1), hipMemcpyDeviceToHost, st));
  RS_HIP(hipEventRecord(L.counted, st));
  ProfScope ps(KC_LITERAL, st, 0.0);
  hipLaunchKernelGGL(k_litc_lists, dim3(q.blocks + T.nbe, k - 1), dim3(256), 0, st, a, T);
  RS_HIP(hipGetLastError());
  RS_HIP(hipEventSynchronize(L.counted));
  uint64_t rows = 256;  // two buffers in turn
  for (uint32_t l = 2; l < k; ++l) rows = std::max<uint64_t>(rows, 8ull * cnt[l - 2] * binom(k, l));
  if (2 * rows > kLitRows) return RS_OK;
  if (L.chi0.reserve(rows, st, false) || L.chi1.reserve(rows, st, false)) return RS_OK;
  uint64_t *below = L.chi0.as<uint64_t>(), *here = L.chi1.as<uint64_t>();
  for (uint32_t l = 2; l < k; ++l) {
    q.P = below;
    const uint32_t lds = mul_lds(k, binom(k, l - 1), binom(k, l)) + kTile * 128;
    if (cnt[l - 2])
      hipLaunchKernelGGL(k_litc_level, dim3((uint32_t)std::min<uint64_t>((cnt[l - 2] + 3ull) / 4, kLitBlocks)), dim3(256),
                         4 * lds, st, a, T, l, lds, here);
    RS_HIP(hipGetLastError());
    std::swap(below, here);
  }
  q.P = below;
  *n_sums = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((cnt[k - 2] + 3ull) / 4, kTopBlocks));
  hipLaunchKernelGGL(k_litc_top, dim3(*n_sums), dim3(256), 0, st, a, T);
  RS_HIP(hipGetLastError());
  return RS_OK;
}

}  // namespace rs

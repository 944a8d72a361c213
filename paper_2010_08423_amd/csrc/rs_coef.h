// Coefficient form of the sieve: shared declarations of the kernels and their
// host side (rs_coef.hip).
#pragma once

#include "rs_internal.h"

namespace rs {

// Largest k the coefficient form takes: its rows grow as C(k, k/2) (924
// entries at k = 12), and the pair tables are compiled in up to here.
constexpr uint32_t kCoefMaxK = 12;
constexpr uint32_t kNoRow = 0xFFFFFFFFu;

// Edges per block of the set kernels, one per thread (16 bitmap words). Their
// work per edge is a chain of a few dependent loads, so a small graph wants as
// many blocks as it can give (10^4-edge path query: 128 us with four edges per
// thread one after another, 115 with one).
constexpr uint32_t kSetBlock = 1024;

// Forward passes stop at this level (see k_coef_fwd): the set of level l > it
// is cut with level kForwardLevels' condition only. On the 10^6-edge path
// query (k = 8), cutting every level exactly leaves 79723 last-level edges,
// stopping at 6 leaves 94668, at 5 114053; each further pass is a launch.
constexpr uint32_t kForwardLevels = 6;

// Bytes of one level's flags by list position: all edges, and what a tile reads
// past them.
__host__ __device__ inline uint64_t flag_stride(uint64_t words) { return words * 64 + 64; }

// Bytes of one level's window marks: one per edge, one per block of edges. The
// backward pass reads them 16 at a time.
__host__ __device__ constexpr uint64_t mark_stride(uint64_t blocks) { return blocks * kSetBlock + ((blocks + 15) & ~15ull); }
static_assert(mark_stride(4) % 16 == 0 && mark_stride(20) % 16 == 0, "each level's marks start on 16 bytes");

// One query in the coefficient form: its graph, constraints and buffers.
struct CoefQuery {
  const uint32_t *e_src, *e_dst, *e_t, *in_off, *hi;
  const uint8_t* colour;
  const uint32_t* dv;  // per-vertex resting times, or null
  EdgeFilter f;
  uint64_t seed;
  uint32_t n, m, k, kq, delta, motif;
  uint32_t words, blocks;        // bitmap words (16 per block), blocks of kSetBlock edges (a multiple of 4)
  uint32_t fwd;                  // last forward level, 2..min(k, kForwardLevels)
  uint32_t nested;               // 1: every forward set lies inside the one before (no source restriction)
  uint32_t plain;                // 1: every edge is valid and may start a walk (level 3's set is known at once)
  uint32_t fine;                 // 1: per-edge sums T are kept
  uint2* win;                    // [m] window [x, y) of edge ids over the in-edges of the edge's source
  uint64_t* z;                   // [n][kq] linear forms of the vertices
  uint64_t* valid;               // [words] edges some walk may use
  uint64_t* fbits;               // [fwd - 1][words + words/64] forward sets of levels 2..fwd, each with a bit per non-zero word
  uint8_t* mark;                 // [k - 2][mark_stride] levels 2..k-1: window ends by edge, then by block
  uint64_t* sbits;               // [k - 1][words] product sets of levels 2..k
  uint32_t* wrank;               // [k - 1][words] set bits before a word inside its block
  uint32_t* bsum;                // [k - 1][blocks] set bits per block
  uint32_t* boff;                // [k - 1][blocks] their exclusive prefix
  uint32_t* count;               // [k - 1] set sizes
  uint8_t* store;                // [k - 1][flag_stride] by list position: rows some window reads
  uint8_t* restart;              // [k - 1][flag_stride] by list position: first entry of its destination
  uint64_t* det;                 // [1] determinant of the shade matrix (motif queries)
  uint64_t* result;              // one sum per block of the last level, whose XOR is the fingerprint (host-visible)
  // lists of levels 2..k: level l at entry (l - 2) * lstride
  uint32_t *l_hi, *l_lo, *l_dst, *l_e;
  uint64_t* l_y;
  uint64_t lstride;
  uint32_t carried;      // bit y: the level with index y has long runs (carries in a launch of their own)
  uint32_t far;          // bit y: a destination of that level may span very many runs (carries from prefix sums)
  uint32_t iters, it0;   // rows by iteration: values per row (0: coefficient rows), iteration of the first
  uint32_t by_entry;     // by iteration: level 2's rows lie by list entry, not by source
  const uint64_t* z1;    // rows that level 2 reads: z, or by iteration z^L
  uint32_t z1_stride;
  uint64_t *P, *Q;  // rows of the level below, prefix rows of this level
  uint64_t* tail;        // [runs][C(k, l-1)] XOR of each run's open part
  uint64_t* carry;       // [runs][C(k, l-1)] XOR of its segment in the runs before it (long runs), or of all tails
                         // before it (far runs)
  uint32_t* open_end;    // [runs] end of the entries before its first segment start (long runs)
  uint64_t* group;       // [runs / 64][C(k, l-1)] sums of 64 tails (far runs)
  uint32_t* seg;         // [runs] the run in which the segment that it continues starts (far runs)
  uint8_t* started;      // [runs] whether a segment starts in the run
  uint64_t* T;           // [m] per-edge sums (fine-grained queries)
};
// Arrays that kernels index at run time, apart from the query (a copy of it
// indexed so would live in memory, not in registers).
struct CoefShades {
  uint8_t mu[RS_MAX_COLOURS], off[RS_MAX_COLOURS];  // multiplicity and first shade of each colour (motif queries)
  uint32_t waves[kCoefMaxK + 1];  // [level] waves its scan is cut into, over its coefficient blocks
};

// True if the plan and its extras can run in the coefficient form.
bool coef_applies(const QueryPlan& qp);
// True if its single iterations can run on the same lists (rows by iteration).
bool iter_rows_apply(const QueryPlan& qp);
// Enqueues one query in the coefficient form on ws. *n_sums = 0 (and RS_OK)
// when its rows do not fit what sz allows the evaluation form; only scratch was
// written then. Constraint arrays are on the device already; T is the per-edge sum
// array of a fine-grained query, cleared or written whole here. Once the caller has synchronised
// st, the fingerprint is the XOR of *n_sums words in ws.host_result, or, on a
// workspace without it (no allocation), in *sums. by_iteration: the words are the
// values of the plan's iterations in turn.
rs_status run_coef(rs_graph* g, PlainWorkspace& ws, const PlainSizes& sz, const QueryPlan& qp, const QueryExtras* ex,
                   const uint32_t* dv, const EdgeFilter& filt, uint64_t* T, hipStream_t st, bool timed,
                   std::vector<uint64_t>* sums, uint32_t* n_sums, bool by_iteration);

// The literal reading of one query in the coefficient form: zeta per slot in
// L.zs; the fingerprint is the XOR of *n_sums words of L.host_result once st is
// synchronised. *n_sums = 0 (and RS_OK): its rows exceed kLitRows or its buffers
// the device's memory, only scratch was written. (It may need more than the
// evaluation form: 16 bytes per edge and level against 1 KB per slot.)
//
// A slot's row is formed by one wave, 64 coefficients and an edge at a time, so
// graphs with more than kLitSlotEdges edges into one vertex at one time are left
// to the evaluation form, which cuts slots into tiles, and so are shorter slots
// whose chain is long against that form's work (lit_coef_applies).
constexpr uint32_t kLitSlotEdges = 128;
constexpr uint64_t kLitRows = 16ull << 30;  // what the evaluation form's two buffers may hold together
bool lit_coef_applies(const LiteralState& L, uint64_t m, const QueryPlan& qp);
rs_status run_literal_coef(const GraphDev& G, LiteralState& L, const QueryPlan& qp, const uint32_t* dv, uint64_t hp,
                           hipStream_t st, uint32_t* n_sums);

// Device bytes of the setup and lists that run_coef reserves in ws.lists for this
// plan or a part of its range (0: the plan runs in the evaluation form only).
uint64_t coef_list_bytes(const rs_graph* g, const QueryPlan& qp, uint64_t eval_lists);

// Many queries at once: each level is one launch over all of them (per class of
// row widths). idx: the positions in graphs / plans / results to run. Queries
// whose rows do not fit `budget` bytes are appended to *left and not run. setup
// and rows are the caller's, who uses them for other things between calls.
// A launch has a grid slice per query, along y or z, where it takes 65536: calls
// run at most kCoefQueries at once.
constexpr size_t kCoefQueries = 32768;
struct CoefBatch;  // its descriptors, kept between calls
// Device bytes of one query in a batch, without its rows.
uint64_t coef_batch_query_bytes(const rs_graph* g, const QueryPlan& qp);
CoefBatch* coef_batch_create();
void coef_batch_destroy(CoefBatch* b);
void coef_batch_release(CoefBatch* b);
uint64_t coef_batch_bytes(const CoefBatch* b);
rs_status run_coef_batch(CoefBatch& B, DevBuf& setup, DevBuf& rows, const rs_graph* const* graphs, const std::vector<QueryPlan>& plans,
                         const std::vector<uint32_t>& idx, rs_result* results, hipStream_t st, uint64_t budget,
                         std::vector<uint32_t>* left);

}  // namespace rs

// Weakly-connected components of the thresholded edge graph: the step after
// the edge classifier in the track-finding pipeline (paper section 2.1: the
// GNN edge scores are passed to WCC; section 2.3: the custom backend returns
// one integer label per space point).
//
// A union-find over the nodes in a fixed number of launches.  Links only ever
// point to a smaller id of the same component (parent[v] <= v), so a walk
// along them ends, a root is the smallest id of its tree, and once every kept
// edge has its ends in one tree the roots are the smallest ids of the
// components: a unique answer, whatever order the GPU worked in.
//
//   init      parent[v] = v
//   hook      parent[larger end] = smaller end, for every kept edge: in a
//             detector graph this already gives each hit of a track its
//             predecessor
//   round     for every kept edge, both ends are pointed at their roots, and
//             the larger root at the smaller one
//   unite     the same, but the root is linked by an atomic minimum, repeated
//             until both ends share a root
//   compress  parent[v] = root of v
//
// hook and round link by stores: where several edges link one root, some
// link is lost, which unite makes good.  No minimum there: an atomic minimum
// goes to the memory side, and once large trees meet, a hundred thousand of
// them hit one root.  The rounds leave unite almost nothing to do (a root
// survives a round only if no neighbouring tree has a smaller one), which
// keeps its minima from contending.
//
// Walks read the links through the caches (an agent-scope load goes past the
// XCD's L2, several times its latency).  A link read that way may be old, but
// it was a valid link of the same component; a node that once had a smaller
// link is never a root again; and only unite's atomic minimum, on the value
// at the memory side, decides whether a root is still one.  On a node that is
// none any more it returns the link so far, smaller than the node; whichever
// of the two links the node keeps, that one and the smaller root still have to
// share a root, and the walk goes on from there.  So every loop strictly
// descends in the node ids and ends, and the host has nothing to check.
//
// Whole call, us, against hook rounds by agent-scope walks and atomic minima
// with a convergence flag read by the host every four rounds: 300k hits with
// track-like scores (270k of 1.0M edges kept) 244 -> 97; 150k hits, all 500k
// edges kept (one giant component) 519 -> 90; chain of 300k ids 295 -> 90;
// hub of 300k edges, with the largest id 1366 -> 85, with the middle one 967 ->
// 100 (means: from call to call 55 to 1200); random graph, 1.2M edges,
// 369 -> 163.
#include "gnn_internal.h"

namespace gnn {
namespace {

constexpr int WT = 256;  // threads per workgroup
constexpr int WE = 4;    // edges per thread: their walks are in flight together

__device__ __forceinline__ int32_t clampi(int32_t v, int32_t n) {
  return v < 0 ? 0 : (v >= n ? n - 1 : v);
}

// Links as this XCD's caches have them (workgroup scope: not kept in a
// register between reads), and stores to them (whole ones: other threads read
// and lower the same words).
__device__ __forceinline__ int32_t link_of(const int32_t *parent, int32_t v) {
  return __hip_atomic_load(parent + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void set_link(int32_t *parent, int32_t v, int32_t to) {
  __hip_atomic_store(parent + v, to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Walks of at most NEAR links (a detector graph's trees are as deep as it has
// layers): v's ancestor that far up, or its root, with `root` telling which.
constexpr int NEAR = 16;

__device__ __forceinline__ int32_t walk_near(const int32_t *parent, int32_t v, bool &root) {
  root = false;
  for (int s = 0; s < NEAR; ++s) {
    const int32_t p = link_of(parent, v);
    if (p == v) {
      root = true;
      return v;
    }
    v = p;
  }
  return v;
}

// Full walks: past NEAR links at the memory side, halving the path behind
// (a minimum, which other XCDs see), so that the walks of a chain's nodes
// shorten one another's.
__device__ __forceinline__ int32_t find_root(int32_t *parent, int32_t v) {
  bool root;
  v = walk_near(parent, v, root);
  while (!root) {
    const int32_t p = __hip_atomic_load(parent + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (p == v) return v;
    const int32_t q = __hip_atomic_load(parent + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (q == p) return p;
    atomicMin(&parent[v], q);
    v = q;
  }
  return v;
}

struct WccEdges {
  const int32_t *ei;
  const float *scores;
  float threshold;
  int64_t n_edges;
  int32_t n_nodes;
};

// Larger and smaller end of edge j (equal: nothing to do).
__device__ __forceinline__ void load_edge(const WccEdges &E, int64_t j, int32_t &hi, int32_t &lo) {
  const bool in = j < E.n_edges;
  const bool keep = in && (!E.scores || E.scores[j] > E.threshold);
  const int32_t s = in ? clampi(E.ei[j], E.n_nodes) : 0;
  const int32_t d = in ? clampi(E.ei[E.n_edges + j], E.n_nodes) : 0;
  hi = s > d ? s : d;
  lo = s > d ? d : s;
  if (!keep) hi = lo = 0;
}

// This thread's edges.
__device__ __forceinline__ void load_edges(const WccEdges &E, int32_t (&hi)[WE],
                                           int32_t (&lo)[WE]) {
#pragma unroll
  for (int k = 0; k < WE; ++k)
    load_edge(E, ((int64_t)blockIdx.x * WE + k) * WT + threadIdx.x, hi[k], lo[k]);
}

// Both ends' roots in place of the ends, larger first; an end that was not
// linked to its root directly is now.  FULL = false: walks of NEAR links
// (shortening the rest of a long path by as much); an edge with an end whose
// root was not reached gets equal ends.
template <bool FULL>
__device__ __forceinline__ void find_roots(int32_t *parent, int32_t (&hi)[WE], int32_t (&lo)[WE]) {
  int32_t ph[WE], pl[WE];
#pragma unroll
  for (int k = 0; k < WE; ++k) {
    ph[k] = link_of(parent, hi[k]);
    pl[k] = link_of(parent, lo[k]);
  }
#pragma unroll
  for (int k = 0; k < WE; ++k) {
    if (hi[k] == lo[k]) continue;
    bool all = true;
    auto walk = [&](int32_t v, int32_t p) {  // p: v's link
      if (p == v) return v;
      bool root = true;
      const int32_t r = FULL ? find_root(parent, p) : walk_near(parent, p, root);
      all = all && root;
      if (r != p) set_link(parent, v, r);
      return r;
    };
    const int32_t rh = walk(hi[k], ph[k]), rl = walk(lo[k], pl[k]);
    hi[k] = rh > rl ? rh : rl;
    lo[k] = !all ? hi[k] : rh > rl ? rl : rh;
  }
}

// The pairs of a hub, or between two large trees, all have one larger end.
// Each for itself they leave it whichever link comes last (a hub then keeps a
// random leaf, and a round settles only the larger ones), and what the rounds
// leave queues in unite at one word, 100 ns each: one call in ten of the
// 300k-edge hubs took 3.4 to 8 ms, and now and then 1 ms was added where all
// edges are kept.  So a workgroup takes one larger end of its open pairs, one
// that neighbouring edges share where there is such, and the least of its
// partners: these are pointed at the least, and thread 0 gets the pair (r, m)
// of the two.  r = m: nothing done, fewer than `few` threads have that end.
// False: no open pair in the workgroup.  In unite and in the first round, where
// that end is common: of 1500 calls of a hub half take 90 us, one in a hundred
// 250 to 500, the longest 1.2 ms.  In all rounds, or before the round's own
// links, the hubs never take more than 0.1 ms, but a graph of large trees meets
// a round later (500k edges, all kept, 91 -> 99 us).
__device__ __forceinline__ bool fold_common(int32_t (&hi)[WE], int32_t (&lo)[WE], int few,
                                            int32_t &r, int32_t &m) {
  __shared__ int32_t root[2], least;  // root: of a neighbouring edge too, of any
  int32_t any = -1, both = -1;
#pragma unroll
  for (int k = 0; k < WE; ++k) {
    const int32_t mine = hi[k] != lo[k] ? hi[k] : -1, next = __shfl_xor(mine, 1);
    if (mine >= 0) any = mine;
    if (mine >= 0 && mine == next) both = mine;
  }
  if (threadIdx.x == 0) {
    root[0] = -1;
    least = INT32_MAX;
  }
  if (!__syncthreads_or(any >= 0)) return false;
  if (both >= 0)
    __hip_atomic_store(&root[0], both, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if (any >= 0) __hip_atomic_store(&root[1], any, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __syncthreads();
  r = m = root[0] >= 0 ? root[0] : root[1];
  int32_t mine = INT32_MAX;
#pragma unroll
  for (int k = 0; k < WE; ++k)
    if (hi[k] != lo[k] && hi[k] == r) mine = lo[k] < mine ? lo[k] : mine;
  if (__syncthreads_count(mine < INT32_MAX) < few) return true;
  if (mine < INT32_MAX) atomicMin(&least, mine);
  __syncthreads();
  m = least;
#pragma unroll
  for (int k = 0; k < WE; ++k)
    if (hi[k] != lo[k] && hi[k] == r) {
      hi[k] = lo[k];
      lo[k] = m;
    }
  return true;
}

// Links root (or fresh node) a to c < a on the lanes with `active`.  Links
// already smaller stay, and where all active lanes of the wave link the same
// node, the smallest c is taken (a hub's edges would otherwise leave it a
// random link, and the smaller ends one round each).
__device__ __forceinline__ void link_to(int32_t *parent, bool active, int32_t a, int32_t c) {
  const uint64_t m = __ballot(active);
  if (m == 0) return;
  const int first = __builtin_ctzll(m);
  const int32_t a0 = __builtin_amdgcn_readlane(a, first);
  if (__popcll(m) > 1 && __ballot(active && a == a0) == m) {
    int32_t x = active ? c : INT32_MAX;
    for (int off = 32; off > 0; off >>= 1) {
      const int32_t y = __shfl_xor(x, off);
      x = y < x ? y : x;
    }
    c = x;
    active = ((int)threadIdx.x & 63) == first;
  }
  if (active && c < link_of(parent, a)) set_link(parent, a, c);
}

__global__ __launch_bounds__(WT) void wcc_init(int32_t *__restrict__ parent, int32_t n) {
  const int64_t v = (int64_t)blockIdx.x * WT + threadIdx.x;
  if (v < n) parent[v] = (int32_t)v;
}

__global__ __launch_bounds__(WT) void wcc_hook(WccEdges E, int32_t *parent) {
  int32_t hi[WE], lo[WE];
  load_edges(E, hi, lo);
#pragma unroll
  for (int k = 0; k < WE; ++k) link_to(parent, hi[k] != lo[k], hi[k], lo[k]);
}

// With `check`, a workgroup first looks at WT edges spread over the list (the
// same ones for all) and leaves the rest to unite once all but a few of them
// are settled: no flag has to be kept, cleared or counted.
__global__ __launch_bounds__(WT) void wcc_round(WccEdges E, int32_t *parent, bool check,
                                               bool fold) {
  int32_t hi[WE], lo[WE];
  if (check) {
    load_edge(E, (int64_t)threadIdx.x * E.n_edges / WT, hi[0], lo[0]);
    const bool open = hi[0] != lo[0] && link_of(parent, hi[0]) != link_of(parent, lo[0]);
    if (__syncthreads_count(open) <= WT / 32) return;
  }
  load_edges(E, hi, lo);
  find_roots<false>(parent, hi, lo);
#pragma unroll
  for (int k = 0; k < WE; ++k) link_to(parent, hi[k] != lo[k], hi[k], lo[k]);
  // (behind the links: a barrier before them holds back what other workgroups
  // can already follow)
  int32_t r, m;
  if (!fold || !fold_common(hi, lo, WT / 4, r, m) || r == m) return;
#pragma unroll
  for (int k = 0; k < WE; ++k) link_to(parent, hi[k] != lo[k], hi[k], lo[k]);
  if (threadIdx.x == 0 && m < link_of(parent, r)) set_link(parent, r, m);
}

// Until roots a and b are one.
__device__ __forceinline__ void unite(int32_t *parent, int32_t a, int32_t b) {
  while (a != b) {
    if (a < b) {
      const int32_t t = a;
      a = b;
      b = t;
    }
    const int32_t old = atomicMin(&parent[a], b);
    if (old == a) break;
    a = find_root(parent, old);
  }
}

__global__ __launch_bounds__(WT) void wcc_unite(WccEdges E, int32_t *parent) {
  int32_t hi[WE], lo[WE], r, m;
  load_edges(E, hi, lo);
  find_roots<true>(parent, hi, lo);
  if (!fold_common(hi, lo, 1, r, m)) return;
  if (threadIdx.x == 0) unite(parent, r, m);
#pragma unroll
  for (int k = 0; k < WE; ++k) unite(parent, hi[k], lo[k]);
}

// (A node whose own link another thread shortens meanwhile reads either
// link; both lead to the same root.)
__global__ __launch_bounds__(WT) void wcc_compress(int32_t *parent, int32_t n) {
  const int64_t v = (int64_t)blockIdx.x * WT + threadIdx.x;
  if (v < n) {
    const int32_t p = link_of(parent, (int32_t)v), r = find_root(parent, p);
    if (r != p) set_link(parent, (int32_t)v, r);
  }
}

// Rounds launched: a round with nothing left to do costs 4 us, one too few
// leaves unite contending (1.0M edges, tracks / 500k edges, all kept: 3 rounds
// 92 / 86 us, 4 97 / 90, 5 101 / 95; 2 rounds 87 / 105 to 240).  Four keep the
// grid of random ids (547 x 547) and hubs of 300k edges at 3 too.
constexpr int ROUNDS = 4;

}  // namespace

hipError_t launch_wcc(const int32_t *edge_index, const float *scores, float threshold,
                      int64_t n_edges, int32_t n_nodes, int32_t *labels, hipStream_t stream) {
  if (n_nodes <= 0) return hipSuccess;
  const WccEdges E{edge_index, scores, threshold, n_edges, n_nodes};
  const unsigned nv = (unsigned)(((int64_t)n_nodes + WT - 1) / WT);
  const unsigned ne = (unsigned)((n_edges + WT * WE - 1) / (WT * WE));
  hipError_t e = launch(wcc_init, nv, WT, 0, stream, labels, n_nodes);
  if (e != hipSuccess || n_edges <= 0) return e;
  if ((e = launch(wcc_hook, ne, WT, 0, stream, E, labels))) return e;
  for (int r = 0; r < ROUNDS; ++r)
    if ((e = launch(wcc_round, ne, WT, 0, stream, E, labels, r > 0, r == 0))) return e;
  if ((e = launch(wcc_unite, ne, WT, 0, stream, E, labels))) return e;
  return launch(wcc_compress, nv, WT, 0, stream, labels, n_nodes);
}

}  // namespace gnn

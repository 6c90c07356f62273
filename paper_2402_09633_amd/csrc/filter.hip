// Edge filtering before the GNN (paper section 2.1: after the embedding
// step a Filtering MLP scores the candidate edges and applyFiltering keeps
// the edges above a fixed threshold).
//
// filter      one wave per 32 candidate edges: the raw features of both
//             endpoints, two hidden layers (small_mlp.h), H -> 1 head,
//             sigmoid; the unit's kept edges (score > threshold) go out as
//             one 32-bit mask.
// compaction  in input order.  A workgroup of the scoring launch takes one run
//             of consecutive units and counts its kept edges, so the scatter
//             launch (same runs) adds up the counts before its own and needs
//             no launches to count or scan; within a run it ranks by popcounts
//             of the masks.  The kept edges are written as a contiguous
//             [2][n_kept] edge_index, ready for gnn_infer.
//
// 2.0M candidates, H = 64: whole call 278 -> 125 us, scoring 247 -> 86 us (one
// unit per workgroup slot, weights from L2, layer 0 on the VALU before),
// compaction 16 us in three launches -> 8.5 in one.  Counters of the scoring
// launch: VALU busy 50%, matrix cores 37% of the time, the two hardly
// overlapping; LDS and gather waits cover the rest.  12 or 16 waves per
// workgroup take the same time (the parameters spill or U falls to 1).
#include "small_mlp.h"

namespace gnn {
namespace {

constexpr int CTHREADS = 1024;

__host__ __device__ inline int64_t units_of(int64_t n_edges) { return (n_edges + 31) / 32; }

// Run of units of workgroup b of `wgs`: [b * per, b * per + per) clipped.
__host__ __device__ inline int64_t run_len(int64_t units, int32_t wgs) {
  return (units + wgs - 1) / wgs;
}

// U units at a time per wave (small_mlp.h).
template <int MB, bool SPLIT, bool FOLD, int FK>
__global__ __launch_bounds__(64 * SM_WAVES) void filter_mlp(FilterArgs a) {
  constexpr int U = MB == 2 && FOLD ? 2 : 1;
  using M = SmallMlp<MB, SPLIT, FOLD, U>;
  constexpr int H = 32 * MB;
  __shared__ typename M::Lds lds;
  __shared__ alignas(16) float head[H];
  __shared__ int32_t kept[SM_WAVES];
  const int lane = threadIdx.x & 63, hh = lane >> 5, n = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t units = units_of(a.n_edges), per = run_len(units, gridDim.x);
  const int64_t u0 = (int64_t)blockIdx.x * per, u1 = u0 + per < units ? u0 + per : units;
  const int F = FK ? FK : a.F;
  constexpr int STEP = U * SM_WAVES;

  auto load_idx = [&](int64_t u, int32_t (&s)[U], int32_t (&d)[U]) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int64_t row = (u + i) * 32 + n, r = row < a.n_edges ? row : a.n_edges - 1;
      s[i] = a.edge_index[r];
      d[i] = a.edge_index[a.n_edges + r];
    }
  };
  // Feature 2 step + hh of the rows [x_src; x_dst].
  auto load_x = [&](const int32_t (&s)[U], const int32_t (&d)[U], int step, float (&xk)[U]) {
    const int k = 2 * step + hh;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int64_t v = clamp_idx(k < F ? s[i] : d[i], a.n_nodes);
      xk[i] = a.x[v * F + (k < F ? k : k - F)];
    }
  };
  // The indices are requested two rounds ahead and, for the template's F, the
  // features one round ahead.
  int64_t u = u0 + U * wv;
  int32_t s[U], d[U], s1[U], d1[U];
  float xv[FK ? FK : 1][U];
  if (u < u1) load_idx(u, s, d);
  if (u + STEP < u1) load_idx(u + STEP, s1, d1);
  if constexpr (FK > 0)
    if (u < u1)
#pragma unroll
      for (int k = 0; k < FK; ++k) load_x(s, d, k, xv[k]);
  M::load(lds, a.mlp);
  for (int i = threadIdx.x; i < H; i += 64 * SM_WAVES) head[i] = a.w2[i];
  __syncthreads();
  const float b2 = a.b2[0];

  int32_t cnt = 0;
  for (; u < u1; u += STEP) {
    // keeps the LDS reads of the weights inside the loop
    asm volatile("" ::: "memory");
    f16v acc[U][MB], acc2[U][MB];
    M::bias(acc, lds.prm, hh);
    if constexpr (FK > 0) {
#pragma unroll
      for (int k = 0; k < FK; ++k) M::step0(acc, lds, k, xv[k], lane);
    } else {
      for (int k = 0; k < F; ++k) {
        load_x(s, d, k, xv[0]);
        M::step0(acc, lds, k, xv[0], lane);
      }
    }
    if (u + STEP < u1) {
#pragma unroll
      for (int i = 0; i < U; ++i) {
        s[i] = s1[i];
        d[i] = d1[i];
      }
      if (u + 2 * STEP < u1) load_idx(u + 2 * STEP, s1, d1);
      if constexpr (FK > 0)
#pragma unroll
        for (int k = 0; k < FK; ++k) load_x(s, d, k, xv[k]);
    }
    M::rest(acc, acc2, lds, a.mlp, lane, hh);
    float part[U];
#pragma unroll
    for (int i = 0; i < U; ++i) part[i] = 0.f;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4 ww = *(const f4 *)(head + mb * 32 + 8 * q + 4 * hh);
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
          for (int t = 0; t < 4; ++t) part[i] += acc2[i][mb][4 * q + t] * ww[t];
      }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      part[i] += __shfl_xor(part[i], 32);
      const float score = sigmoidf_stable(part[i] + b2);
      const int64_t row = (u + i) * 32 + n;
      const bool mine = hh == 0 && u + i < u1 && row < a.n_edges;
      if (mine) a.scores[row] = score;
      const uint32_t m = (uint32_t)__ballot(mine && score > a.threshold);
      if (lane == 0 && u + i < u1) a.masks[u + i] = m;
      cnt += __popc(m);
    }
  }
  if (lane == 0) kept[wv] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t t = 0;
    for (int w = 0; w < SM_WAVES; ++w) t += kept[w];
    a.counts[blockIdx.x] = t;
  }
}

// Stable scatter of the kept edges, workgroup b the run of units that
// workgroup b of the scoring launch took: position = kept edges of the runs
// before + kept edges before this one in the run.  CTHREADS units at a time:
// a block scan of their popcounts, then each half-wave writes one unit.
__global__ __launch_bounds__(CTHREADS) void compact_scatter(
    const int32_t *__restrict__ edge_index, int64_t n, const uint32_t *__restrict__ masks,
    const int32_t *__restrict__ counts, int32_t *__restrict__ total, int32_t *__restrict__ out) {
  __shared__ int32_t wsum[2][CTHREADS / 64];
  __shared__ int32_t base[CTHREADS];
  __shared__ uint32_t msk[CTHREADS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int32_t wgs = gridDim.x, blk = blockIdx.x;
  auto wave_sum = [](int32_t v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
  };
  int32_t before = 0, all = 0;
  for (int32_t i = tid; i < wgs; i += CTHREADS) {
    const int32_t c = counts[i];
    all += c;
    before += i < blk ? c : 0;
  }
  before = wave_sum(before);
  all = wave_sum(all);
  if (lane == 0) {
    wsum[0][w] = before;
    wsum[1][w] = all;
  }
  __syncthreads();
  int32_t run = 0, tot = 0;
  for (int i = 0; i < CTHREADS / 64; ++i) {
    run += wsum[0][i];
    tot += wsum[1][i];
  }
  if (blk == 0 && tid == 0) *total = tot;
  const int64_t units = units_of(n), per = run_len(units, wgs);
  const int64_t u0 = (int64_t)blk * per, u1 = u0 + per < units ? u0 + per : units;
  for (int64_t ub = u0; ub < u1; ub += CTHREADS) {
    const uint32_t m = ub + tid < u1 ? masks[ub + tid] : 0u;
    const int32_t c = __popc(m);
    int32_t incl = c;
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t v = __shfl_up(incl, off);
      if (lane >= off) incl += v;
    }
    __syncthreads();  // (the previous round's and the first sums' readers)
    if (lane == 63) wsum[0][w] = incl;
    msk[tid] = m;
    __syncthreads();
    int32_t pre = run;
    for (int i = 0; i < CTHREADS / 64; ++i) {
      pre += i < w ? wsum[0][i] : 0;
      run += wsum[0][i];
    }
    base[tid] = pre + incl - c;
    __syncthreads();
    const int64_t here = u1 - ub < CTHREADS ? u1 - ub : CTHREADS;
    const uint32_t b = lane & 31, lt = (1u << b) - 1u;
    for (int64_t j = tid >> 5; j < here; j += CTHREADS / 32) {
      const uint32_t mj = msk[j];
      if (mj >> b & 1u) {
        const int64_t i = (ub + j) * 32 + b;
        const int32_t pos = base[j] + __popc(mj & lt);
        out[pos] = edge_index[i];
        out[(int64_t)tot + pos] = edge_index[n + i];
      }
    }
  }
}

template <int MB>
hipError_t scores_h(const FilterArgs &a, int32_t wgs, hipStream_t stream) {
  if (!a.mlp.w1r) return launch(filter_mlp<MB, false, false, 0>, wgs, 64 * SM_WAVES, 0, stream, a);
  if (!a.mlp.fold) return launch(filter_mlp<MB, true, false, 0>, wgs, 64 * SM_WAVES, 0, stream, a);
  // hits have three features; any other width takes the loop over its steps
  if (a.F == 3) return launch(filter_mlp<MB, true, true, 3>, wgs, 64 * SM_WAVES, 0, stream, a);
  return launch(filter_mlp<MB, true, true, 0>, wgs, 64 * SM_WAVES, 0, stream, a);
}

}  // namespace

int32_t filter_wgs(int64_t n_edges, int n_cu) {
  const int64_t units = units_of(n_edges), most = (int64_t)n_cu * SM_WGS_PER_CU;
  return (int32_t)(units < most ? units : most);
}

hipError_t launch_filter_scores(int hidden, const FilterArgs &a, int32_t wgs, hipStream_t stream) {
  if (a.n_edges <= 0) return hipSuccess;
  if (wgs < 1 || a.mlp.steps != a.F || a.F < 1 || a.F > MAX_F) return hipErrorInvalidValue;
  switch (hidden) {
    case 64: return scores_h<2>(a, wgs, stream);
    case 128: return scores_h<4>(a, wgs, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_compact(const int32_t *edge_index, int64_t n, const uint32_t *masks,
                          const int32_t *counts, int32_t wgs, int32_t *total, int32_t *out,
                          hipStream_t stream) {
  if (n <= 0 || wgs < 1) return hipErrorInvalidValue;
  return launch(compact_scatter, wgs, CTHREADS, 0, stream, edge_index, n, masks, counts, total,
                out);
}

}  // namespace gnn

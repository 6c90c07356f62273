// Graph construction, the first stage of the pipeline (paper section 2.1: an
// embedding network maps every space point into a latent space, and a
// fixed-radius nearest-neighbour search there proposes the candidate edges
// that the filter and the GNN then score).
//
// embed       one wave per 32 points: two hidden layers (small_mlp.h), then
//             the D outputs (D <= 16), on the fp16 matrix cores from three-part
//             splits (VALU dot products where the gains are not folded).
//             300k points, 3 -> 128 -> 128 -> 8: 100 -> 40 us (47 with the
//             outputs on the VALU: its weights alone were half of the LDS
//             reads, which bounded it).
// frnn        every pair i < j with d2(i, j) < r2, where d2 is evaluated in
//             fp32 as d = fmaf(t, t, d) over the coordinates in ascending
//             order (t = z_i[k] - z_j[k]).  Points are binned on a grid over
//             the first min(3, D) coordinates with cells no narrower than the
//             radius, so a pair within the radius sits in the same or
//             adjacent cells; cells are hashed into a power-of-two table that
//             is turned into buckets by the CSR builder (a stable sort of the
//             points by bucket).  A point scans the buckets of the 3^g
//             neighbouring cells, each bucket once, so hash collisions never
//             produce a pair twice.  One pass counts the pairs and keeps each
//             point's first partners; after an exclusive scan of the counts
//             they are written grouped by i (within one i in cell-scan
//             order), which is deterministic.  300k clustered 8-d points,
//             544k pairs, whole call: 494 -> 240 us (two full scans of 190 us
//             became one of 100, bound by its scattered loads; one sort of
//             the keys instead of two; the write queued behind the count).
#include "small_mlp.h"

namespace gnn {
namespace {

constexpr int FTHREADS = 256;
constexpr int MAX_D = 16;

// Slots of a point in the pair search.  The fewest take no memory of their
// own: a sort pass leaves 16 bytes a point.
constexpr int32_t FRNN_SLOTS_LEAST = 4, FRNN_SLOTS_MOST = 32;
static_assert(FRNN_SLOTS_LEAST * sizeof(int32_t) == 2 * sizeof(uint2), "slots in place of pairs");

// Parts of the output layer's split products: with x = x1 + x2 + x3 and
// w = w1 + w2 + w3 in fp16 (33 bits each), the six products of order up to
// 2^-22 leave an error below fp32's own rounding.  (Rows of W2 that their
// scales do not keep clear of fp16's subnormal floor are not folded:
// row_scale() in gnn_api.hip.)
constexpr int OUT_PARTS = 3;

template <int MB, bool SPLIT, bool FOLD, int FK>
__global__ __launch_bounds__(64 * SM_WAVES) void embed_mlp(EmbedArgs a) {
  using M = SmallMlp<MB, SPLIT, FOLD, 1>;
  constexpr int H = 32 * MB;
  constexpr int KS = (FK + 1) / 2;  // layer-0 steps (the odd feature's partner is zero)
  constexpr int NOUT = 2 * MB * OUT_PARTS * 64;
  __shared__ typename M::Lds lds;
  __shared__ h8 out_r[FOLD ? NOUT : 1];
  __shared__ alignas(16) float out_w[FOLD ? 1 : MAX_D * H];
  __shared__ alignas(16) float out_b[32];
  __shared__ alignas(16) float out_s[32];
  const int lane = threadIdx.x & 63, hh = lane >> 5, n = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int F = FK ? FK : a.F;
  const int64_t units = (a.n + 31) / 32, nw = (int64_t)gridDim.x * SM_WAVES;
  auto load_x = [&](int64_t u, int step, float (&xk)[1]) {
    const int64_t row = u * 32 + n, r = row < a.n ? row : a.n - 1;
    const int k = 2 * step + hh;
    xk[0] = k < F ? a.x[r * F + k] : 0.f;
  };
  // one unit per workgroup before any workgroup takes a second
  int64_t u = (int64_t)wv * gridDim.x + blockIdx.x;
  float xv[FK ? KS : 1][1];
  if constexpr (FK > 0)
    if (u < units)
#pragma unroll
      for (int k = 0; k < KS; ++k) load_x(u, k, xv[k]);
  M::load(lds, a.mlp);
  if constexpr (FOLD) {
    for (int i = threadIdx.x; i < NOUT; i += 64 * SM_WAVES) out_r[i] = ((const h8 *)a.w2r)[i];
    if (threadIdx.x < 32) out_s[threadIdx.x] = a.s2inv[threadIdx.x];
  } else {
    for (int i = threadIdx.x; i < a.D * H; i += 64 * SM_WAVES) out_w[i] = a.w2[i];
  }
  if (threadIdx.x < 32) out_b[threadIdx.x] = (int)threadIdx.x < a.D ? a.b2[threadIdx.x] : 0.f;
  __syncthreads();
  for (; u < units; u += nw) {
    // keeps the LDS reads of the weights inside the loop
    asm volatile("" ::: "memory");
    f16v acc[1][MB], acc2[1][MB];
    M::bias(acc, lds.prm, hh);
    if constexpr (FK > 0) {
#pragma unroll
      for (int k = 0; k < KS; ++k) M::step0(acc, lds, k, xv[k], lane);
      if (u + nw < units)
#pragma unroll
        for (int k = 0; k < KS; ++k) load_x(u + nw, k, xv[k]);
    } else {
      for (int k = 0; k < a.mlp.steps; ++k) {
        load_x(u, k, xv[0]);
        M::step0(acc, lds, k, xv[0], lane);
      }
    }
    M::rest(acc, acc2, lds, a.mlp, lane, hh);
    const int64_t row = u * 32 + n;
    if constexpr (FOLD) {
      // z = W2 a on the matrix cores, one 32-wide output block of which D
      // rows are used; lane (n, hh) then holds outputs 8 q + 4 hh + t.
      // The five small products have a sum of their own: in one sum they
      // would round the large one six times as often.
      f16v z, zl;
#pragma unroll
      for (int v = 0; v < 16; ++v) z[v] = zl[v] = 0.f;
#pragma unroll
      for (int g = 0; g < 2 * MB; ++g) {
        const h8 *r = out_r + g * OUT_PARTS * 64 + lane;
        const f8 x = acc_x<MB>(acc2[0], g);
        const h8 x1 = __builtin_convertvector(x, h8);
        const f8 y = residual16(x, x1);
        const h8 x2 = __builtin_convertvector(y, h8);
        const h8 x3 = __builtin_convertvector(residual16(y, x2), h8);
        const h8 w1 = r[0], w2 = r[64], w3 = r[128];
        zl = mma_h(w3, x1, zl);
        zl = mma_h(w2, x2, zl);
        zl = mma_h(w1, x3, zl);
        zl = mma_h(w2, x1, zl);
        zl = mma_h(w1, x2, zl);
        z = mma_h(w1, x1, z);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) z[v] += zl[v];
      if (row < a.n) {
#pragma unroll
        for (int q = 0; q < MAX_D / 8; ++q) {
          const int d0 = 8 * q + 4 * hh;
          float *o = a.z + row * a.D + d0;
          const f4 v = f4{z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]} * *(const f4 *)(out_s + d0) +
                       *(const f4 *)(out_b + d0);
          if (d0 + 4 <= a.D && a.z16) {
            *(f4 *)o = v;
          } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
              if (d0 + t < a.D) o[t] = v[t];
          }
        }
      }
    } else {
      for (int d = 0; d < a.D; ++d) {
        const float *wd = out_w + d * H + 4 * hh;
        float part = 0.f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f4 ww = *(const f4 *)(wd + mb * 32 + 8 * q);
#pragma unroll
            for (int t = 0; t < 4; ++t) part += acc2[0][mb][4 * q + t] * ww[t];
          }
        part += __shfl_xor(part, 32);
        if (row < a.n && hh == 0) a.z[row * a.D + d] = part + out_b[d];
      }
    }
  }
}

// Grid cell of a point along the first g coordinates (coordinates clamped so
// that the cell index fits comfortably in an int).
__device__ __forceinline__ void cell_of(const float *zp, int g, float inv_cell, int (&c)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float v = k < g ? floorf(zp[k] * inv_cell) : 0.f;
    v = fminf(fmaxf(v, -1.0e9f), 1.0e9f);
    c[k] = (int)v;
  }
}

__device__ __forceinline__ uint32_t cell_hash(const int (&c)[3], uint32_t mask) {
  return ((uint32_t)c[0] * 73856093u ^ (uint32_t)c[1] * 19349663u ^ (uint32_t)c[2] * 83492791u) &
         mask;
}

__global__ __launch_bounds__(FTHREADS) void frnn_keys(FrnnArgs a, int32_t *__restrict__ keys) {
  const int64_t i = (int64_t)blockIdx.x * FTHREADS + threadIdx.x;
  if (i >= a.n) return;
  int c[3];
  cell_of(a.z + i * a.D, a.D < 3 ? a.D : 3, a.inv_cell, c);
  keys[i] = (int32_t)cell_hash(c, a.mask);
}

// A point's word in `count`: the pairs, and whether they are left to the
// second scan.
constexpr int32_t FRNN_COUNT = INT32_MAX, FRNN_AGAIN = INT32_MIN;

// The points' coordinates in bucket order, the first four apart.
__global__ __launch_bounds__(FTHREADS) void frnn_gather(FrnnArgs a, bool vec) {
  const int64_t p = (int64_t)blockIdx.x * FTHREADS + threadIdx.x;
  if (p >= a.n) return;
  const float *src = a.z + (int64_t)a.perm[p] * a.D;
  f4 v = {0.f, 0.f, 0.f, 0.f};
  float z_4 = 0.f;
  if (vec) {  // rows of whole 16-byte pieces, D % 4 == 0
    v = *(const f4 *)src;
    for (int k = 4; k < a.D; k += 4) {
      const f4 w = *(const f4 *)(src + k);
      if (k == 4) z_4 = w[0];
      *(f4 *)(a.zr + p * (a.D - 4) + k - 4) = w;
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k < a.D) v[k] = src[k];
    for (int k = 4; k < a.D; ++k) a.zr[p * (a.D - 4) + k - 4] = src[k];
    if (a.D > 4) z_4 = src[4];
  }
  *(f4 *)(a.z4 + 4 * p) = v;
  if (a.D > 4) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    *(f2 *)(a.z2 + 2 * p) = f2{v[3], z_4};
  }
}

// Calls emit(j) for the partners j > i of the point at bucket position p (id
// i), in the order of the cells and of the ids within a bucket.
//
// The neighbouring cells' buckets are scanned once each (a bucket that two
// cells share through the hash is skipped the second time), so every other
// point is tested at most once; a point of a colliding far cell simply fails
// the distance test.
//
// Bound by the number of scattered loads: a wave's lanes scan unrelated
// buckets, and the texture unit takes about one lane a cycle.  So a candidate
// is first tested on as little as rejects nearly all of them.  The distance
// only grows as its coordinates are added (each fmaf rounds a sum of
// non-negative terms upwards from the partial sum), so a candidate fails as
// soon as a partial sum, or the square of any one coordinate's difference,
// reaches r2.  With five or more coordinates (PAIRS) that is tested on two of
// those that the grid does not separate, 8 bytes a candidate and two
// candidates a load; with fewer, on the first four, 16 bytes.  Only the
// survivors' other coordinates and ids are read, and those later, from a list
// in LDS, LIST at a time: done where they are found, one lane's survivor makes
// the whole wave wait for its loads.  The lanes empty their lists together
// when one is full; each for itself, the wave waited for the loads of one lane
// after the other where the two coordinates separate nothing (both constant,
// 300k points: 735 us, together 440; without a first test 490).  Lists of 24:
// of 16 are full too often (1.0M points 390 against 370 us for the launch), of
// 32 cost a workgroup per CU (300k points 98 -> 139 us).  Candidates are taken
// U at a time and the next three cells' bounds are requested ahead.
//
// direct: no first test, every candidate's id and coordinates read at once.
// AGAIN: compiled for direct only.
constexpr int LIST = 24;
template <int D, bool AGAIN, typename Emit>
__device__ __forceinline__ void scan_point(const FrnnArgs &a, int64_t p, int32_t i, bool direct,
                                           Emit emit) {
  constexpr int U = 4;
  constexpr bool PAIRS = D >= 5;
  typedef int32_t i2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef float f4u __attribute__((ext_vector_type(4), aligned(8)));
  constexpr int NY = D > 1 ? 3 : 1, NZ = D > 2 ? 3 : 1;
  const f4 *z4 = (const f4 *)a.z4;
  const f4 zi = z4[p];
  // coordinates from the fifth on of the point at bucket position q
  auto load_rest = [&](int64_t q, float (&v)[D > 4 ? D - 4 : 1]) {
    if constexpr (D > 4 && D % 4 == 0) {
#pragma unroll
      for (int k = 0; k < D - 4; k += 4) {
        const f4 w = *(const f4 *)(a.zr + q * (D - 4) + k);
#pragma unroll
        for (int t = 0; t < 4; ++t) v[k + t] = w[t];
      }
    } else {
#pragma unroll
      for (int k = 0; k < D - 4; ++k) v[k] = a.zr[q * (D - 4) + k];
    }
  };
  float zri[D > 4 ? D - 4 : 1];
  load_rest(p, zri);
  auto dist2 = [&](const f4 &v, const float (&w)[D > 4 ? D - 4 : 1]) {
    float acc = 0.f;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const float t = k < 4 ? zi[k < 4 ? k : 0] - v[k < 4 ? k : 0]
                            : zri[k < 4 ? 0 : k - 4] - w[k < 4 ? 0 : k - 4];
      acc = __builtin_fmaf(t, t, acc);
    }
    return acc;
  };
  int ci[3];
  {
    const float zc[3] = {zi[0], zi[1], zi[2]};
    cell_of(zc, D < 3 ? D : 3, a.inv_cell, ci);
  }
  auto key_of = [&](int c) {  // c = 3 * (3 * z + y) + x
    const int nc[3] = {ci[0] + c % 3 - 1, ci[1] + (NY > 1 ? c / 3 % 3 - 1 : 0),
                       ci[2] + (NZ > 1 ? c / 9 - 1 : 0)};
    return cell_hash(nc, a.mask);
  };
  // Whether any two of the cells share a bucket.  The hash is an exclusive or
  // of one term per axis, so two cells collide when the differences of their
  // terms cancel; each axis has three nonzero differences.
  bool collide = false;
  {
    uint32_t d[3][4];
    const uint32_t mul[3] = {73856093u, 19349663u, 83492791u};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const uint32_t t0 = (uint32_t)(ci[k] - 1) * mul[k], t1 = (uint32_t)ci[k] * mul[k],
                     t2 = (uint32_t)(ci[k] + 1) * mul[k];
      d[k][0] = 0;
      d[k][1] = t0 ^ t1;
      d[k][2] = t0 ^ t2;
      d[k][3] = t1 ^ t2;
    }
#pragma unroll
    for (int z = 0; z < (NZ > 1 ? 4 : 1); ++z)
#pragma unroll
      for (int y = 0; y < (NY > 1 ? 4 : 1); ++y)
#pragma unroll
        for (int x = 0; x < 4; ++x)
          if (x + y + z > 0) collide |= ((d[0][x] ^ d[1][y] ^ d[2][z]) & a.mask) == 0;
  }
  // Bucket bounds of row r's three cells (r = 3 z + y), empty when skipped.
  auto bounds = [&](int r, int32_t (&qb)[3], int32_t (&qe)[3]) {
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      const int c = 3 * r + x;
      const uint32_t key = key_of(c);
      const i2 q = *(const i2 *)(a.rp + key);  // one load for both bounds
      qb[x] = q[0];
      qe[x] = q[1];
      if (collide)
        for (int e = 0; e < c; ++e) qe[x] = key_of(e) == key ? qb[x] : qe[x];
    }
  };
  if (direct) {
    for (int c = 0; c < 3 * NY * NZ; ++c) {
      const uint32_t key = key_of(c);
      const i2 b = *(const i2 *)(a.rp + key);
      bool seen = false;
      if (collide)
        for (int e = 0; e < c; ++e) seen |= key_of(e) == key;
      if (seen) continue;
      for (int32_t q0 = b[0]; q0 < b[1]; q0 += U) {
        int32_t j[U];
        f4 zq[U];
        float zrq[U][D > 4 ? D - 4 : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {  // (past the bucket's end: its last point again)
          const int32_t q = q0 + u < b[1] ? q0 + u : b[1] - 1;
          j[u] = a.perm[q];
          if constexpr (D >= 4) {
            zq[u] = z4[q];
          } else {  // (what the lanes get back bounds a scan of shared buckets)
#pragma unroll
            for (int k = 0; k < D; ++k) zq[u][k] = a.z4[4 * (int64_t)q + k];
          }
          load_rest(q, zrq[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (q0 + u < b[1] && j[u] > i && dist2(zq[u], zrq[u]) < a.r2) emit(j[u]);
      }
    }
    return;
  }
  if constexpr (AGAIN) return;
  __shared__ int32_t list[LIST][FTHREADS];
  int n_list = 0;
  // (one entry at a time: two or four cost the registers of a wave per SIMD,
  // 300k points 238 -> 270 us for the call)
  auto flush = [&]() {
    for (int k = 0; k < n_list; ++k) {
      const int32_t q = list[k][threadIdx.x];
      const int32_t j = a.perm[q];
      bool near = true;
      if constexpr (PAIRS) {  // (else the list holds only pairs)
        float w[D > 4 ? D - 4 : 1];
        load_rest(q, w);
        near = dist2(z4[q], w) < a.r2;
      }
      if (near && j > i) emit(j);
    }
    n_list = 0;
  };
  auto push = [&](int32_t q) {
    if (q != p) list[n_list++][threadIdx.x] = q;
  };
  struct Batch {
    f4 v[PAIRS ? U / 2 : U];
  };
  auto load = [&](Batch &w, int32_t q0, int32_t qe) {
    if constexpr (PAIRS) {
      // (past the bucket's end: other points' coordinates, not used)
      const f4u *pr = (const f4u *)(a.z2 + 2 * (int64_t)q0);
      w.v[0] = pr[0];
      if (q0 + 2 < qe) w.v[1] = pr[1];
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q0 + u < qe) w.v[u] = z4[q0 + u];
    }
  };
  auto test = [&](const Batch &w, int32_t q0, int32_t qe) {
    if (__any(n_list > LIST - U)) flush();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      bool near;
      if constexpr (PAIRS) {
        const float t3 = zi[3] - w.v[u / 2][2 * (u % 2)],
                    t4 = zri[0] - w.v[u / 2][2 * (u % 2) + 1];
        near = !(t3 * t3 >= a.r2) && !(t4 * t4 >= a.r2);
      } else {
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < D; ++k) {
          const float t = zi[k] - w.v[u][k];
          acc = __builtin_fmaf(t, t, acc);
        }
        near = acc < a.r2;
      }
      if (q0 + u < qe && near) push(q0 + u);
    }
  };
  int32_t nb[3], ne[3];
  bounds(0, nb, ne);
  for (int r = 0; r < NY * NZ; ++r) {
    int32_t qb[3], qe[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      qb[x] = nb[x];
      qe[x] = ne[x];
    }
    if (r + 1 < NY * NZ) bounds(r + 1, nb, ne);
    // The first U candidates of the three cells are requested together.
    Batch first[3];
#pragma unroll
    for (int x = 0; x < 3; ++x)
      if (qb[x] < qe[x]) load(first[x], qb[x], qe[x]);
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      test(first[x], qb[x], qe[x]);
      for (int32_t q0 = qb[x] + U; q0 < qe[x]; q0 += U) {
        Batch more;
        load(more, q0, qe[x]);
        test(more, q0, qe[x]);
      }
    }
  }
  flush();
}

// Whether the point at bucket position p has one `step` places on in its
// bucket that the first test lets through.
template <int D>
__device__ __forceinline__ bool dense_at(const FrnnArgs &a, int64_t p, int step) {
  const f4 z = ((const f4 *)a.z4)[p];
  const float zc[3] = {z[0], z[1], z[2]};
  int ci[3];
  cell_of(zc, D < 3 ? D : 3, a.inv_cell, ci);
  const uint32_t key = cell_hash(ci, a.mask);
  bool near = (threadIdx.x & 63) + step < 64 && __shfl_down(key, step) == key;
  if constexpr (D >= 5) {
    const float z_4 = a.z2[2 * p + 1];
    const float t3 = z[3] - __shfl_down(z[3], step), t4 = z_4 - __shfl_down(z_4, step);
    near = near && t3 * t3 < a.r2 && t4 * t4 < a.r2;
  } else {
    float d2 = 0.f;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const float t = z[k] - __shfl_down(z[k], step);
      d2 = __builtin_fmaf(t, t, d2);
    }
    near = near && d2 < a.r2;
  }
  return near;
}

// Pairs of every point: the count, and up to a.n_slots partners.  Thread
// p handles the point at bucket position p (neighbouring threads handle
// neighbouring points, whose candidates they share in the caches).  Notes in
// a.again whether points of the workgroup have to be scanned again.
//
// In groups of points that are all near one another the first test rejects
// too little to pay.  A workgroup where DENSE_LANES points have a partner by
// the first test DENSE_STEP places on in their bucket (groups of about 40 and
// more in few cells) does without it; where MANY_LANES have one MANY_STEP
// places on, most points have more partners than slots, and it only counts.
// Whole call, us, test and slots for all -> without the test -> only counting,
// 100k points, 8 dimensions: groups of 20 255 -> 270 -> 335, of 60 (width
// 0.005) 540 -> 510 -> 490, of 100 600 -> 515 -> 497, of 250 1000 -> 820 -> 770;
// 300k points in groups of 10 stay with the test (235; 445 without).
// Five waves per SIMD up to 11 dimensions, a few registers spilled for them
// in 10 and 11: 300k points 299 -> 264 and 304 -> 276.  In 12 the spills cost
// what they gain (300k 280 -> 264, 220k, which four waves hold, 87 -> 100 for
// the launch).
constexpr int DENSE_STEP = 4, DENSE_LANES = 7 * FTHREADS / 16;
constexpr int MANY_STEP = 16, MANY_LANES = FTHREADS / 4;
template <int D>
__global__ __launch_bounds__(FTHREADS, D >= 5 && D <= 11 ? 5 : 4) void frnn_collect(FrnnArgs a) {
  const int64_t p = (int64_t)blockIdx.x * FTHREADS + threadIdx.x;
  const bool in = p < a.n;
  const bool dense = __syncthreads_count(in && dense_at<D>(a, p, DENSE_STEP)) >= DENSE_LANES;
  const bool many = dense && __syncthreads_count(in && dense_at<D>(a, p, MANY_STEP)) >= MANY_LANES;
  int32_t cnt = 0;
  if (in) {
    const int32_t i = a.perm[p];
    int32_t *slot = a.slots + (int64_t)i * a.n_slots;
    scan_point<D, false>(a, p, i, dense, [&](int32_t j) {
      if (!many && cnt < a.n_slots) slot[cnt] = j;
      ++cnt;
    });
    a.count[i] = many || cnt > a.n_slots ? cnt | FRNN_AGAIN : cnt;
  }
  const int again = __syncthreads_or(many || cnt > a.n_slots);
  if (threadIdx.x == 0) a.again[blockIdx.x] = again;
}

// Writes the pairs where there is room for all of them.  The first half of
// the workgroups scans a second time, in bucket order like the first, the
// points whose partners were not all collected (in the order of the ids a
// wave's lanes share nothing: 100k points in groups of 100, 1060 us against
// 220), without the first test: they have many partners.  The second half
// writes the collected partners of the others in the order of the ids, so
// that neighbouring threads write neighbouring pairs (in bucket order every
// store had a line of its own: 40 us against 9).
template <int D>
__global__ __launch_bounds__(FTHREADS) void frnn_write(FrnnArgs a, unsigned half) {
  const int64_t total = *a.total;
  if (total > a.max_pairs) return;
  const bool again = blockIdx.x < half;
  if (again && !a.again[blockIdx.x]) return;
  const int64_t k = (int64_t)(again ? blockIdx.x : blockIdx.x - half) * FTHREADS + threadIdx.x;
  if (k >= a.n) return;
  const int64_t i = again ? a.perm[k] : k;
  const int32_t cnt = a.count[i];
  if (again != (cnt < 0)) return;
  int64_t o = a.offs[i];
  auto put = [&](int32_t j) {
    a.out[o] = (int32_t)i;
    a.out[total + o] = j;
    ++o;
  };
  if (again) {
    scan_point<D, true>(a, k, (int32_t)i, true, put);
  } else {
    typedef int32_t i4 __attribute__((ext_vector_type(4)));
    const int32_t *slot = a.slots + i * a.n_slots;
    for (int32_t c = 0; c < cnt; c += 4) {
      const i4 v = *(const i4 *)(slot + c);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (c + t < cnt) put(v[t]);
    }
  }
}

template <bool WRITE>
hipError_t launch_points(const FrnnArgs &a, hipStream_t stream) {
  const unsigned blocks = (unsigned)((a.n + FTHREADS - 1) / FTHREADS);
  switch (a.D) {
#define GNN_FRNN_D(d) \
  case d:                                                                                  \
    if constexpr (WRITE)                                                                   \
      return launch(frnn_write<d>, 2 * blocks, FTHREADS, 0, stream, a, blocks);            \
    else                                                                                   \
      return launch(frnn_collect<d>, blocks, FTHREADS, 0, stream, a);
    GNN_FRNN_D(1) GNN_FRNN_D(2) GNN_FRNN_D(3) GNN_FRNN_D(4) GNN_FRNN_D(5) GNN_FRNN_D(6)
    GNN_FRNN_D(7) GNN_FRNN_D(8) GNN_FRNN_D(9) GNN_FRNN_D(10) GNN_FRNN_D(11) GNN_FRNN_D(12)
    GNN_FRNN_D(13) GNN_FRNN_D(14) GNN_FRNN_D(15) GNN_FRNN_D(16)
#undef GNN_FRNN_D
    default: return hipErrorInvalidValue;
  }
}

// Exclusive scan of the per-point counts into offs (int64), total -> *total:
// per-tile sums (tiles of 2048 counts), then each tile's own scan on top of
// the sums before it.  Those are added up by the tile itself for up to
// SCAN_DIRECT tiles (at most 16 reads a thread; a launch less), above that
// they are scanned by a launch in between.  Thread t of a tile owns its 8
// consecutive counts.
constexpr int ST = 256, SI = 8, STILE = ST * SI, SCAN_DIRECT = 16 * ST;

// Exclusive scan of v over the block; *sum gets the block total.
__device__ __forceinline__ int64_t block_excl_scan(int64_t v, int64_t *sum) {
  __shared__ int64_t part[ST];
  const int t = threadIdx.x;
  part[t] = v;
  __syncthreads();
  for (int off = 1; off < ST; off <<= 1) {
    const int64_t u = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += u;
    __syncthreads();
  }
  const int64_t incl = part[t];
  *sum = part[ST - 1];
  __syncthreads();
  return incl - v;
}

__global__ __launch_bounds__(ST) void scan_tiles(const int32_t *__restrict__ count, int64_t n,
                                                 int64_t *__restrict__ bsum) {
  const int64_t base = (int64_t)blockIdx.x * STILE + (int64_t)threadIdx.x * SI;
  int64_t s = 0;
#pragma unroll
  for (int k = 0; k < SI; ++k)
    if (base + k < n) s += count[base + k] & FRNN_COUNT;
  int64_t tot;
  (void)block_excl_scan(s, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// In place over the nb tile sums, ST at a time with a running carry.
__global__ __launch_bounds__(ST) void scan_sums(int64_t *__restrict__ bsum, int64_t nb,
                                                int64_t *__restrict__ total) {
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += ST) {
    const int64_t i = b0 + threadIdx.x;
    const int64_t v = i < nb ? bsum[i] : 0;
    int64_t tot;
    const int64_t ex = block_excl_scan(v, &tot);
    if (i < nb) bsum[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) *total = carry;
}

// direct: bsum holds the tiles' sums, else their exclusive scan.
__global__ __launch_bounds__(ST) void scan_down(const int32_t *__restrict__ count, int64_t n,
                                                const int64_t *__restrict__ bsum, bool direct,
                                                int64_t *__restrict__ offs,
                                                int64_t *__restrict__ total) {
  int64_t before = 0;
  if (direct) {
    int64_t all = 0;
    for (int64_t b = threadIdx.x; b < (int64_t)gridDim.x; b += ST) {
      const int64_t v = bsum[b];
      before += b < (int64_t)blockIdx.x ? v : 0;
      all += v;
    }
    int64_t sum;
    (void)block_excl_scan(before, &sum);
    before = sum;
    if (blockIdx.x == 0) {  // (uniform over the block)
      (void)block_excl_scan(all, &sum);
      if (threadIdx.x == 0) *total = sum;
    }
  } else {
    before = bsum[blockIdx.x];
  }
  const int64_t base = (int64_t)blockIdx.x * STILE + (int64_t)threadIdx.x * SI;
  int32_t c[SI];
  int64_t s = 0;
#pragma unroll
  for (int k = 0; k < SI; ++k) {
    c[k] = base + k < n ? count[base + k] & FRNN_COUNT : 0;
    s += c[k];
  }
  int64_t tot;
  int64_t run = before + block_excl_scan(s, &tot);
#pragma unroll
  for (int k = 0; k < SI; ++k)
    if (base + k < n) {
      offs[base + k] = run;
      run += c[k];
    }
}

}  // namespace

namespace {

template <int MB>
hipError_t embed_h(const EmbedArgs &a, unsigned wgs, hipStream_t stream) {
  if (!a.mlp.w1r) return launch(embed_mlp<MB, false, false, 0>, wgs, 64 * SM_WAVES, 0, stream, a);
  if (!a.mlp.fold) return launch(embed_mlp<MB, true, false, 0>, wgs, 64 * SM_WAVES, 0, stream, a);
  // hits have three features; any other width takes the loop over its steps
  if (a.F == 3) return launch(embed_mlp<MB, true, true, 3>, wgs, 64 * SM_WAVES, 0, stream, a);
  return launch(embed_mlp<MB, true, true, 0>, wgs, 64 * SM_WAVES, 0, stream, a);
}

}  // namespace

hipError_t launch_embed(int hidden, const EmbedArgs &args, int n_cu, hipStream_t stream) {
  EmbedArgs a = args;
  if (a.n <= 0) return hipSuccess;
  if (a.D < 1 || a.D > MAX_D || a.F < 1 || a.F > MAX_F || a.mlp.steps != (a.F + 1) / 2)
    return hipErrorInvalidValue;
  // 16-byte stores where every row's pieces of four outputs are aligned
  a.z16 = a.D % 4 == 0 && (uintptr_t)a.z % 16 == 0;
  const int64_t units = (a.n + 31) / 32, most = (int64_t)n_cu * SM_WGS_PER_CU;
  const unsigned wgs = (unsigned)(units < most ? units : most);
  switch (hidden) {
    case 64: return embed_h<2>(a, wgs, stream);
    case 128: return embed_h<4>(a, wgs, stream);
  }
  return hipErrorInvalidValue;
}

size_t frnn_scan_blocks(int64_t n) { return (size_t)((n + STILE - 1) / STILE); }

hipError_t launch_frnn_keys(const FrnnArgs &a, int32_t *keys, hipStream_t stream) {
  if (a.n <= 0) return hipSuccess;
  return launch(frnn_keys, (unsigned)((a.n + FTHREADS - 1) / FTHREADS), FTHREADS, 0, stream, a,
                keys);
}

hipError_t launch_frnn_pairs(const FrnnArgs &a, hipStream_t stream) {
  if (a.n <= 0) return hipSuccess;
  hipError_t e =
      launch(frnn_gather, (unsigned)((a.n + FTHREADS - 1) / FTHREADS), FTHREADS, 0, stream, a,
             a.D % 4 == 0 && (uintptr_t)a.z % 16 == 0);
  if (e == hipSuccess) e = launch_points<false>(a, stream);
  if (e != hipSuccess) return e;
  const unsigned nb = (unsigned)frnn_scan_blocks(a.n);
  const bool direct = nb <= a.scan_direct;
  if ((e = launch(scan_tiles, nb, ST, 0, stream, a.count, a.n, a.bsum))) return e;
  if (!direct)
    if ((e = launch(scan_sums, 1, ST, 0, stream, a.bsum, (int64_t)nb, a.total))) return e;
  if ((e = launch(scan_down, nb, ST, 0, stream, a.count, a.n, a.bsum, direct, a.offs, a.total)))
    return e;
  return a.out ? launch_points<true>(a, stream) : hipSuccess;
}

}  // namespace gnn

// ---------------------------------------------------------------- host ---

#include <cmath>

#include "../../include/gnn.h"

namespace {

size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

}  // namespace

namespace {

using namespace gnn;

// Workspace of one search.
struct FrnnPlan {
  uint32_t buckets = 64;
  size_t bytes = 0;
  size_t keys, rp, perm, pairs, status, count, offs, total, bsum, z4, zr, z2, slots, again;

  FrnnPlan(int64_t n, int32_t dim, int32_t n_slots) {
    while ((int64_t)buckets < 2 * n && buckets < (1u << 30)) buckets <<= 1;
    auto take = [&](size_t b) {
      const size_t o = bytes;
      bytes += align256(b > 0 ? b : 1);
      return o;
    };
    keys = take((size_t)n * 4);
    rp = take(((size_t)buckets + 1) * 4);
    perm = take((size_t)n * 4);
    pairs = take((size_t)n * 16);
    status = take(csr_scratch_bytes(n, buckets, 1));
    count = take((size_t)n * 4);
    offs = take((size_t)n * 8);
    total = take(8);
    bsum = take(frnn_scan_blocks(n) * 8);
    z4 = take((size_t)n * 16);
    zr = dim > 4 ? take((size_t)n * (dim - 4) * 4) : 0;
    z2 = dim > 4 ? take(((size_t)n + 4) * 8) : 0;  // (read up to 3 points past the end)
    // few enough, the slots go where the sorted pairs were
    slots = n_slots <= FRNN_SLOTS_LEAST ? pairs : take((size_t)n * n_slots * 4);
    again = take((size_t)((n + FTHREADS - 1) / FTHREADS) * 4);
  }
};

int frnn(const float *z, int64_t n_nodes, int32_t dim, float r2, int32_t *edge_index,
         int64_t max_pairs, int64_t *n_pairs, int32_t n_slots, int64_t scan_direct,
         hipStream_t stream) {
  if (!n_pairs) return set_error(GNN_E_INVALID_ARG, "n_pairs is NULL");
  *n_pairs = 0;
  if (n_nodes < 0 || n_nodes > INT32_MAX)
    return set_error(GNN_E_INVALID_ARG, "n_nodes outside 0..INT32_MAX");
  if (n_nodes >= CSR_MAX_ITEMS)
    return set_error(GNN_E_UNSUPPORTED, "the cell sort takes at most 2^30 - 1 points");
  if (dim < 1 || dim > 16) return set_error(GNN_E_INVALID_ARG, "dim outside 1..16");
  if (max_pairs < 0) return set_error(GNN_E_INVALID_ARG, "max_pairs is negative");
  if (n_nodes > 0 && !z) return set_error(GNN_E_INVALID_ARG, "z is NULL");
  if (std::isnan(r2)) return set_error(GNN_E_INVALID_ARG, "r2 is NaN");
  if (n_nodes < 2 || !(r2 > 0.f)) return GNN_OK;

  FrnnArgs a;
  a.z = z;
  a.n = n_nodes;
  a.D = dim;
  a.r2 = r2;
  // Cells a little wider than the radius: a pair that passes the fp32 test
  // differs by less than that along every coordinate.
  const double cell = 1.001 * std::sqrt((double)r2);
  a.inv_cell = std::isfinite(cell) && cell > 0.0 ? (float)(1.0 / cell) : 0.f;

  const int64_t n = n_nodes;
  FrnnPlan w(n, dim, n_slots);
  void *base = nullptr;
  hipError_t e = hipMallocAsync(&base, w.bytes, stream);
  if (e != hipSuccess && n_slots > FRNN_SLOTS_LEAST) {
    // no room for that many slots: the fewest, and more points scanned twice
    (void)hipGetLastError();
    n_slots = FRNN_SLOTS_LEAST;
    w = FrnnPlan(n, dim, n_slots);
    e = hipMallocAsync(&base, w.bytes, stream);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return set_error(GNN_E_OOM, "frnn workspace allocation failed");
  }
  unsigned char *b = (unsigned char *)base;
  int32_t *keys = (int32_t *)(b + w.keys);
  CsrScratch cs;
  cs.pairs_a = (uint2 *)(b + w.pairs);
  cs.pairs_b = cs.pairs_a + n;
  cs.status = (uint32_t *)(b + w.status);
  a.mask = w.buckets - 1;
  a.rp = (const int32_t *)(b + w.rp);
  a.perm = (const int32_t *)(b + w.perm);
  a.z4 = (float *)(b + w.z4);
  a.zr = (float *)(b + w.zr);
  a.z2 = (float *)(b + w.z2);
  a.n_slots = n_slots;
  a.slots = (int32_t *)(b + w.slots);
  a.again = (int32_t *)(b + w.again);
  a.count = (int32_t *)(b + w.count);
  a.offs = (int64_t *)(b + w.offs);
  a.total = (int64_t *)(b + w.total);
  a.bsum = (int64_t *)(b + w.bsum);
  a.scan_direct = scan_direct;
  a.out = edge_index;
  a.max_pairs = max_pairs < INT32_MAX ? max_pairs : INT32_MAX;

  // The write is queued behind the count and checks it on the device, so the
  // stream does not run dry while the host reads the count.
  int rc = GNN_OK;
  int64_t total = 0;
  e = launch_frnn_keys(a, keys, stream);
  if (e == hipSuccess)
    e = build_buckets(keys, (int32_t)n, (int32_t)w.buckets, (int32_t *)(b + w.rp),
                      (int32_t *)(b + w.perm), cs, stream);
  if (e == hipSuccess) e = launch_frnn_pairs(a, stream);
  if (e == hipSuccess) e = hipMemcpyAsync(&total, a.total, 8, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    rc = set_error(GNN_E_HIP, hipGetErrorString(e));
  } else {
    *n_pairs = total;
    if (total > INT32_MAX)
      rc = set_error(GNN_E_UNSUPPORTED, "more than INT32_MAX pairs");
    else if (edge_index && total > max_pairs)
      rc = set_error(GNN_E_INVALID_ARG, "edge_index holds fewer pairs than found (see n_pairs)");
  }
  if (hipFreeAsync(base, stream) != hipSuccess && rc == GNN_OK)
    rc = set_error(GNN_E_HIP, "frnn workspace release failed");
  return rc;
}

}  // namespace

extern "C" int gnn_frnn(const float *z, int64_t n_nodes, int32_t dim, float r2,
                        int32_t *edge_index, int64_t max_pairs, int64_t *n_pairs,
                        hipStream_t stream) {
  // Room for 32 partners a point (a cluster's first point has most of the
  // cluster; one point that is scanned twice costs the write launch 25 us);
  // for very many points, whose workspace counts, the fewest.
  const int32_t n_slots = n_nodes <= (1 << 24) ? FRNN_SLOTS_MOST : FRNN_SLOTS_LEAST;
  return frnn(z, n_nodes, dim, r2, edge_index, max_pairs, n_pairs, n_slots, SCAN_DIRECT, stream);
}

extern "C" int gnn_debug_frnn(const float *z, int64_t n_nodes, int32_t dim, float r2,
                              int32_t *edge_index, int64_t max_pairs, int64_t *n_pairs,
                              int32_t n_slots, int64_t scan_direct, hipStream_t stream) {
  if (n_slots < FRNN_SLOTS_LEAST || n_slots > FRNN_SLOTS_MOST || n_slots % 4 != 0)
    return set_error(GNN_E_INVALID_ARG, "n_slots is none of 4, 8 .. 32");
  if (scan_direct < 0 || scan_direct > SCAN_DIRECT)
    return set_error(GNN_E_INVALID_ARG, "scan_direct outside 0..4096");
  return frnn(z, n_nodes, dim, r2, edge_index, max_pairs, n_pairs, n_slots, scan_direct, stream);
}

extern "C" size_t gnn_debug_frnn_bytes(int64_t n_nodes, int32_t dim, int32_t n_slots) {
  if (n_nodes < 1 || n_nodes >= CSR_MAX_ITEMS || dim < 1 || dim > 16) return 0;
  if (n_slots < FRNN_SLOTS_LEAST || n_slots > FRNN_SLOTS_MOST || n_slots % 4 != 0) return 0;
  return FrnnPlan(n_nodes, dim, n_slots).bytes;
}

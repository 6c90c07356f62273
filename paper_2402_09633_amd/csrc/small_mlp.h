// The two hidden layers shared by the edge filter and the embedding: a raw
// input row of a few features -> H (LayerNorm/ReLU) -> H (LayerNorm/ReLU),
// one wave per U 32-row units.
//
// The kernels are persistent: a workgroup copies the weights into LDS once
// and its waves walk 32-row units.  The rows themselves are a few words each,
// so a unit is bound by its instructions: VALU, matrix and LDS cycles are of
// the same size, and all three are kept down:
//  - layer 0 runs on the fp32 matrix cores (v_mfma_f32_32x32x2_f32, two input
//    features per step): lane half hh supplies feature 2 k + hh of row n,
//    so a lane loads half of its row.  On the VALU it took 16 MB FMAs and
//    4 MB loads of weights per feature;
//  - both layers' weights are centred (gnn_api.hip), so the LayerNorms form
//    no mean, and their biases are the accumulators' starting values;
//  - layer 1 runs on the fp16 matrix cores from split operands (SPLIT) with
//    its records in LDS, or on the fp32 ones when the first LayerNorm's
//    output bound leaves the fp16 range;
//  - FOLD: the LayerNorms' gains are folded into the next layer's weights
//    (relu(g y + b) = |g| relu(+-y + b / |g|), the sign into this layer's
//    rows): one multiply and one LDS read per value fewer.  The folded
//    outputs carry FOLD_SCALE, which keeps the low parts of their fp16
//    splits out of the subnormal range;
//  - U = 2 (H = 64, where the registers allow it): every record and parameter
//    read from LDS serves two units.  LDS returns 128 bytes a cycle to the
//    whole CU, 16 bytes per lane take 8 cycles even when all lanes ask for
//    the same address, and at U = 1 that was the bound.
#pragma once

#include "device_common.h"

namespace gnn {
namespace {

constexpr int SM_WAVES = 8;

// Workgroups of a persistent launch per CU.
constexpr int SM_WGS_PER_CU = 1;

// split2 with the residual formed by one mixed-precision fma per value
// (x1 * -1 + x, the fp16 source converted exactly): the same bits, 8
// instructions fewer per 8 values.
__device__ __forceinline__ f8 residual16(const f8 &x, const h8 &x1) {
  typedef unsigned u4v __attribute__((ext_vector_type(4)));
  const u4v p = __builtin_bit_cast(u4v, x1);
  f8 r;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const unsigned pj = p[j];
    const float lo = x[2 * j], hi = x[2 * j + 1];
    float rl, rh;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(rl) : "v"(pj), "v"(lo));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
        : "=v"(rh)
        : "v"(pj), "v"(hi));
    r[2 * j] = rl;
    r[2 * j + 1] = rh;
  }
  return r;
}

template <int MB, bool SPLIT, bool FOLD, int U>
struct SmallMlp {
  static constexpr int H = 32 * MB;
  static constexpr int KS = MAX_F;  // layer-0 steps of two features, at most
  static constexpr int NREC = SPLIT ? 2 * MB * MB * 2 * 64 : 1;
  struct Lds {
    h8 rec[NREC];           // layer 1: f16x2 records of s1 W1
    float w0[KS * MB * 64];  // layer 0: [step][mb][lane], W0[32 mb + lane % 32][2 step + lane / 32]
    alignas(16) float prm[6 * H];  // b0 g0 beta0 | s1 b1, g1, beta1 (FOLD: g unused)
  };

  static __device__ __forceinline__ void load(Lds &s, const SmallMlpArgs &a) {
    if constexpr (SPLIT)
      for (int i = threadIdx.x; i < NREC; i += 64 * SM_WAVES) s.rec[i] = ((const h8 *)a.w1r)[i];
    for (int i = threadIdx.x; i < a.steps * MB * 64; i += 64 * SM_WAVES) s.w0[i] = a.w0a[i];
    for (int i = threadIdx.x; i < H; i += 64 * SM_WAVES) {
      s.prm[i] = a.b0[i];
      s.prm[H + i] = a.g0[i];
      s.prm[2 * H + i] = a.beta0[i];
      s.prm[3 * H + i] = a.b1[i] * a.s1;
      s.prm[4 * H + i] = a.g1[i];
      s.prm[5 * H + i] = a.beta1[i];
    }
  }

  static __device__ __forceinline__ void bias(f16v (&acc)[U][MB], const float *b, int hh) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4 v = *(const f4 *)(b + mb * 32 + 8 * q + 4 * hh);
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[i][mb][4 * q + t] = v[t];
      }
  }

  // One layer-0 step: xk[i] is feature 2 step + hh of this lane's row in unit i.
  static __device__ __forceinline__ void step0(f16v (&acc)[U][MB], const Lds &s, int step,
                                               const float (&xk)[U], int lane) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const float w = s.w0[(step * MB + mb) * 64 + lane];
#pragma unroll
      for (int i = 0; i < U; ++i)
        acc[i][mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, xk[i], acc[i][mb], 0, 0, 0);
    }
  }

  // LayerNorm/ReLU of centred sums, prm = (.., g, beta).
  static __device__ __forceinline__ void ln(f16v (&acc)[U][MB], const float *prm, float eps,
                                            int hh) {
    constexpr float inv_h = 1.0f / H;
    float rstd[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      float var = 0.f;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) var += acc[i][mb][v] * acc[i][mb][v];
      var += __shfl_xor(var, 32);
      rstd[i] = ln_rstd(var * inv_h + eps) * (FOLD ? FOLD_SCALE : 1.f);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = mb * 32 + 8 * q + 4 * hh;
        const f4 bt = *(const f4 *)(prm + 2 * H + f);
        f4 gg = {1.f, 1.f, 1.f, 1.f};
        if constexpr (!FOLD) gg = *(const f4 *)(prm + H + f);
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float y = acc[i][mb][4 * q + t];
            acc[i][mb][4 * q + t] =
                fmaxf(FOLD ? __builtin_fmaf(y, rstd[i], bt[t]) : y * rstd[i] * gg[t] + bt[t], 0.f);
          }
      }
  }

  // From layer 0's sums (bias included) to the second LayerNorm/ReLU's
  // outputs in acc2.
  static __device__ __forceinline__ void rest(f16v (&acc)[U][MB], f16v (&acc2)[U][MB],
                                              const Lds &s, const SmallMlpArgs &a, int lane,
                                              int hh) {
    ln(acc, s.prm, a.eps, hh);
    if constexpr (SPLIT) {
      bias(acc2, s.prm + 3 * H, hh);
      const h8 *rec = s.rec + lane;
#pragma unroll
      for (int g = 0; g < 2 * MB; ++g) {
        h8 w1[MB], w2[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          w1[mb] = rec[(g * 2 * MB + 2 * mb) * 64];
          w2[mb] = rec[(g * 2 * MB + 2 * mb + 1) * 64];
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const f8 x = acc_x<MB>(acc[i], g);
          const h8 x1 = __builtin_convertvector(x, h8);
          const h8 x2 = __builtin_convertvector(residual16(x, x1), h8);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) acc2[i][mb] = mma_h(w1[mb], x1, acc2[i][mb]);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) acc2[i][mb] = mma_h(w2[mb], x1, acc2[i][mb]);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) acc2[i][mb] = mma_h(w1[mb], x2, acc2[i][mb]);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < U; ++i) {
        gemm_acc_f32<MB, MB>(acc2[i], acc[i], (const f4 *)a.w1 + lane, 0);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f4 v = *(const f4 *)(s.prm + 3 * H + mb * 32 + 8 * q + 4 * hh);
#pragma unroll
            for (int t = 0; t < 4; ++t) acc2[i][mb][4 * q + t] += v[t];
          }
      }
    }
    ln(acc2, s.prm + 3 * H, a.eps * a.s1 * a.s1, hh);
  }
};

}  // namespace
}  // namespace gnn

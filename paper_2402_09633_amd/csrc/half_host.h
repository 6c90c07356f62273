// fp32 to and from IEEE half bits on the host (round to nearest even), by the
// block: gnn_create makes some hundred thousand of them, and the compiler's
// call for (_Float16) was most of its time (fp32 model 13.3 ms).  With the
// CPU's own conversion (F16C) where it has one, asked at run time (1.2 ms),
// else in integers (4.5 ms).
#pragma once

#include <cstdint>
#include <cstring>

#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#define GNN_HOST_F16C 1
#include <immintrin.h>
#endif

namespace gnn {

inline uint16_t f32_to_f16(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  const uint32_t sign = (u >> 16) & 0x8000u;
  u &= 0x7fffffffu;
  if (u >= 0x47800000u)  // 2^16 and above, infinity, NaN
    return (uint16_t)(sign | (u > 0x7f800000u ? 0x7e00u : 0x7c00u));
  if (u < 0x38800000u) {  // below 2^-14: added to 0.5, whose last bit is half's 2^-24
    float m;
    memcpy(&m, &u, 4);
    m += 0.5f;
    memcpy(&u, &m, 4);
    return (uint16_t)(sign | (u - 0x3f000000u));
  }
  u += 0xfffu + ((u >> 13) & 1u);
  return (uint16_t)(sign | ((u - 0x38000000u) >> 13));
}

inline float f16_to_f32(uint16_t h) {
  const uint32_t sign = (uint32_t)(h & 0x8000u) << 16, e = (h >> 10) & 31u, m = h & 0x3ffu;
  float f = (float)m * 0x1p-24f;  // (subnormal, zero)
  uint32_t u;
  memcpy(&u, &f, 4);
  if (e == 31u) u = 0x7f800000u | m << 13;
  else if (e) u = (e + 112u) << 23 | m << 13;
  u |= sign;
  memcpy(&f, &u, 4);
  return f;
}

inline void to_f16(const float *x, uint16_t *y, int n) {
  for (int i = 0; i < n; ++i) y[i] = f32_to_f16(x[i]);
}
inline void to_f32(const uint16_t *x, float *y, int n) {
  for (int i = 0; i < n; ++i) y[i] = f16_to_f32(x[i]);
}

#ifdef GNN_HOST_F16C
// split_f16, eight values at a time
template <int PARTS, int N>
__attribute__((target("avx,f16c"))) void split_f16_hw(const double (&w)[N], uint16_t *out) {
  for (int i = 0; i < N; i += 8) {
    __m256d a = _mm256_loadu_pd(w + i), b = _mm256_loadu_pd(w + i + 4);
    for (int p = 0; p < PARTS; ++p) {
      const __m256 x = _mm256_set_m128(_mm256_cvtpd_ps(b), _mm256_cvtpd_ps(a));
      const __m128i h = _mm256_cvtps_ph(x, _MM_FROUND_TO_NEAREST_INT);
      _mm_storeu_si128((__m128i *)(out + p * N + i), h);
      const __m256 y = _mm256_cvtph_ps(h);
      a = _mm256_sub_pd(a, _mm256_cvtps_pd(_mm256_castps256_ps128(y)));
      b = _mm256_sub_pd(b, _mm256_cvtps_pd(_mm256_extractf128_ps(y, 1)));
    }
  }
}
inline bool host_f16c() {
  static const bool yes = __builtin_cpu_supports("avx") && __builtin_cpu_supports("f16c");
  return yes;
}
#endif

// PARTS halves whose sum is w, largest first, in consecutive blocks of N
// (a multiple of 8): part p + 1 is what part p left.
template <int PARTS, int N>
inline void split_f16(const double (&w)[N], uint16_t *out) {
#ifdef GNN_HOST_F16C
  if (host_f16c()) {
    split_f16_hw<PARTS>(w, out);
    return;
  }
#endif
  double left[N];
  float x[N], y[N];
  memcpy(left, w, sizeof left);
  for (int p = 0; p < PARTS; ++p, out += N) {
    for (int i = 0; i < N; ++i) x[i] = (float)left[i];
    to_f16(x, out, N);
    to_f32(out, y, N);
    for (int i = 0; i < N; ++i) left[i] -= (double)y[i];
  }
}

}  // namespace gnn

// fp32 to and from IEEE half bits on the host (round to nearest even).  In
// integers: gnn_create makes some hundred thousand of them, and without the
// host CPU's own conversion (F16C, which not every host has) the compiler's
// call for (_Float16) is most of its time: fp32 model 13.3 ms, 1.1 so.
#pragma once

#include <cstdint>
#include <cstring>

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

}  // namespace gnn

// Device conversions to the low-precision layouts (see to_lowp_2d in internal.h).
#pragma once

#include "internal.h"

namespace ascc {

// Round-to-nearest-even FP32 -> bf16 bits (finite inputs; NaN stays NaN).
__device__ __forceinline__ unsigned short bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  const uint32_t r = u + 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(r >> 16);
}
__device__ __forceinline__ float bf16_to_f(unsigned short h) { return __uint_as_float(((uint32_t)h) << 16); }

// A shadow written by the kernel that forms its source: rows of ld values (a multiple of 32) in precision prec.
struct Shadow {
  void* p = nullptr;
  long ld = 0;
  int prec = 0;
};

// Values x .. x + 3 (x a multiple of 4) of a shadow's row, as 8- or 16-byte stores.
__device__ __forceinline__ void put_lowp4(const Shadow& s, long row, long x, const double (&d)[4]) {
  if (s.prec == kPrecBF16x3) {
    unsigned short h[4], l[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      h[j] = bf16_rne((float)d[j]);
      l[j] = bf16_rne((float)(d[j] - (double)bf16_to_f(h[j])));
    }
    unsigned short* o = static_cast<unsigned short*>(s.p) + 2 * row * s.ld + (x >> 5) * 64 + (x & 31);
    *reinterpret_cast<ushort4*>(o) = make_ushort4(h[0], h[1], h[2], h[3]);
    *reinterpret_cast<ushort4*>(o + 32) = make_ushort4(l[0], l[1], l[2], l[3]);
  } else {
    *reinterpret_cast<float4*>(static_cast<float*>(s.p) + row * s.ld + x) =
        make_float4((float)d[0], (float)d[1], (float)d[2], (float)d[3]);
  }
}

}  // namespace ascc

// Block-diagonal (random) Hadamard transform of bf16 data along K, exact
// then rounded once to bf16 (the rotation the paper applies before MixFP4
// quantization: the RHT of the training recipe, Sec. 3.2 / Fig. 7, and the
// "+RHT" rows of Sec. 4.2):
//   y[c b + j] = sum_i s_i x[c b + i] H_b[i, j] / sqrt(b),
// H_b the Sylvester matrix ((-1)^popcount(i & j)), s a vector of b signs.
//
// Layout: a lane holds one 16-element quantization block, so a Hadamard
// block of b = 16 L elements spans L lanes of one DPP row (L = 1..16):
// consecutive lanes, except that for L = 8 a block takes the lanes whose
// index has one value of bit 2 (rotated_index).  The fast Walsh-Hadamard
// butterflies run in fp64: four stages inside the lane, then log2 L stages
// across lanes through DPP lane exchanges (xor 1, 2: quad permutes; xor 8:
// row rotate by 8; xor 4, which only L = 16 needs: half-row mirror then quad
// reverse, two moves instead of one).
//
// Exactness: a bf16 value is a multiple of 2^(e-7) below 2^(e+1), so a block
// sum of b of them is exact in fp64 when the nonzero inputs of the block span
// at most 2^(45 - log2 b) in magnitude (2^37 for b = 256).  Then the sum S is
// exact, S / sqrt(b) is exact for b a power of 4 and within 2^-52 (relative)
// otherwise, and the result is rounded to bf16 once: to fp32 with round to
// odd (which keeps the correct final rounding, fp32 having 16 more bits),
// then to bf16 with ties to even.  For b = 2 * 4^m, a value whose fp32 image
// sits on a bf16 rounding midpoint is settled exactly: y > M iff
// S^2 > b M^2, with S^2 held exactly as p + e (fma) and p - b M^2 exact
// (Sterbenz).  An exactly zero result is +0.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"
#include "lanes.h"

namespace mixfp4 {

// One butterfly stage across lanes: the lane with bit kX clear keeps
// own + partner, the other partner - own (fma with +-1: one rounding, exact
// whenever the sum is).
template <int kX>
__device__ __forceinline__ void cross_stage(double (&v)[16], int lane) {
  const double sg = (lane & kX) ? -1.0 : 1.0;
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = __builtin_fma(v[j], sg, xor_f64<kX>(v[j]));
}

// Round y = S * scale to bf16 (see the header comment); returns the bits.
__device__ __forceinline__ uint32_t round_to_bf16(double S, const HadamardParams& hp) {
  const double y = __builtin_fma(S, hp.scale, 0.0);   // S * scale, and -0 -> +0
  const float f = (float)y;
  uint32_t fb = __float_as_uint(f);
  if (hp.odd && (fb & 0xFFFFu) - 0x7FFFu <= 2u) {
    // fp32 image within an ulp of the bf16 midpoint M: decide y > M exactly
    const uint32_t upper = fb & 0xFFFF0000u;
    const double M = (double)__uint_as_float((upper & 0x7FFFFFFFu) | 0x8000u);
    const double p = S * S;
    const double e = __builtin_fma(S, S, -p);
    const double diff = (p - M * M * hp.b) + e;
    return (upper >> 16) + (diff > 0.0 ? 1u : 0u);
  }
  const double back = (double)f;
  if (__builtin_fabs(back) > __builtin_fabs(y)) fb -= 1u;   // truncate toward zero
  if (back != y) fb |= 1u;                                  // round to odd
  return (fb + 0x7FFFu + ((fb >> 16) & 1u)) >> 16;
}

// The block of 16 elements that the lane of linear index g holds: for L = 8
// bits 2 and 3 of g are swapped, so that the three exchanges of a Hadamard
// block are xor 1, 2 and 8.
__device__ __forceinline__ int64_t rotated_index(int64_t g, const HadamardParams& hp) {
  if (hp.lanes_log2 != 3) return g;
  return (g & ~int64_t(12)) | ((g & 4) << 1) | ((g & 8) >> 1);
}

// Per-thread xor masks flipping the bf16 sign bits of the 16 elements of a
// lane at position `pos` within its Hadamard block (pos = lane % L).
struct SignMasks {
  uint32_t m[8];
};

__device__ __forceinline__ SignMasks load_sign_masks(const HadamardParams& hp, int pos) {
  SignMasks s;
#pragma unroll
  for (int i = 0; i < 8; ++i) s.m[i] = 0u;
  if (hp.signs) {
    const int8_t* p = hp.signs + 16 * pos;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t a = (uint32_t)(uint8_t)p[2 * i] >> 7, b = (uint32_t)(uint8_t)p[2 * i + 1] >> 7;
      s.m[i] = (a << 15) | (b << 31);
    }
  }
  return s;
}

// The 16 exact block sums S of this lane.  Every lane of a Hadamard block
// must be active.
__device__ __forceinline__ void hadamard_sums(uint4 v0, uint4 v1, const SignMasks& sm,
                                              const HadamardParams& hp, double (&v)[16]) {
  const uint32_t w[8] = {v0.x ^ sm.m[0], v0.y ^ sm.m[1], v0.z ^ sm.m[2], v0.w ^ sm.m[3],
                         v1.x ^ sm.m[4], v1.y ^ sm.m[5], v1.z ^ sm.m[6], v1.w ^ sm.m[7]};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    v[2 * i] = (double)__uint_as_float(w[i] << 16);
    v[2 * i + 1] = (double)__uint_as_float(w[i] & 0xFFFF0000u);
  }
#pragma unroll
  for (int h = 1; h < 16; h <<= 1) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (j & h) continue;
      const double a = v[j], c = v[j + h];
      v[j] = a + c;
      v[j + h] = a - c;
    }
  }
  const int lane = (int)(threadIdx.x & 63u);
  if (hp.lanes_log2 >= 1) cross_stage<1>(v, lane);
  if (hp.lanes_log2 >= 2) cross_stage<2>(v, lane);
  // ascending element bits, whatever L: beyond the exact span the result
  // depends on the order of the stages
  if (hp.lanes_log2 >= 4) cross_stage<4>(v, lane);
  if (hp.lanes_log2 >= 3) cross_stage<8>(v, lane);
}

// Rotate the lane's 16 bf16 values (v0: elements 0-7, v1: 8-15) in place.
// Every lane of a Hadamard block must be active.
//
// Rounding: the fp32 image of S * scale, rounded to bf16 with ties to even,
// is the correct result unless it lies within one fp32 ulp of a bf16
// midpoint (otherwise no midpoint lies between it and the exact value), and
// also there when S * scale and all its images are exact (b a power of 4 and
// S within 24 bits, where ties are common).  The few other lanes (3 in 65536
// elements) round all their elements with round_to_bf16; that path for every
// element cost more instructions than the butterflies (14 against 6.5 an
// element).  2^24 elements, b = 128: rotate and quantize 31.9 -> 29.1 us,
// maximum of the rotated tensor 24.0 -> 17.0 us.
__device__ __forceinline__ void hadamard_rotate(uint4& v0, uint4& v1, const SignMasks& sm,
                                                const HadamardParams& hp) {
  double v[16];
  hadamard_sums(v0, v1, sm, hp, v);
  uint32_t o[8];
  uint32_t nearest = 0xFFFFFFFFu;       // (low half of the image - 0x7FFF) << 16, least
  uint32_t below = hp.odd ? 1u << 28 : 0u;   // fp64 bits below fp32's last
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    uint32_t r[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const double y = __builtin_fma(v[2 * i + e], hp.scale, 0.0);
      const uint32_t fb = __float_as_uint((float)y);
      below |= (uint32_t)__builtin_bit_cast(uint64_t, y);
      nearest = min(nearest, (fb << 16) + 0x80010000u);
      r[e] = fb + 0x7FFFu + ((fb >> 16) & 1u);
    }
    o[i] = __builtin_amdgcn_perm(r[1], r[0], 0x07060302u);
  }
  if (nearest <= 0x20000u && (below & 0x1FFFFFFFu) != 0u) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      o[i] = round_to_bf16(v[2 * i], hp) | (round_to_bf16(v[2 * i + 1], hp) << 16);
  }
  v0 = make_uint4(o[0], o[1], o[2], o[3]);
  v1 = make_uint4(o[4], o[5], o[6], o[7]);
}

// max |rotated X| of the lane's 16 values as bf16 magnitude bits: rounding
// is monotonic, so only the largest |S| is rounded.  A block that holds an
// infinity or a NaN is rotated and compared element by element.
__device__ __forceinline__ uint32_t hadamard_absmax(uint4 v0, uint4 v1, const SignMasks& sm,
                                                    const HadamardParams& hp) {
  double v[16];
  hadamard_sums(v0, v1, sm, hp, v);
  double mx = 0.0;
#pragma unroll
  for (int j = 0; j < 16; ++j) mx = __builtin_fmax(mx, __builtin_fabs(v[j]));
  // a sum of finite values stays far below 2^1023: an infinity or a NaN
  // anywhere in the block shows in every S, also in the first
  if (__builtin_fabs(v[0]) < 0x1p1000) return round_to_bf16(mx, hp) & 0x7FFFu;
  uint32_t m = 0u;
#pragma unroll
  for (int j = 0; j < 16; ++j) m = max(m, round_to_bf16(v[j], hp) & 0x7FFFu);
  return m;
}

}  // namespace mixfp4

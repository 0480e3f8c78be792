// MixFP4 -> fp32 decode (App. B.2-B.3): value = s32 * (E4M3(scale) * v) * sign,
// v from the E2M1 grid when scale bit 7 (T) is 0 and from the INT4 grid
// {0..7} (E1M2 x2) when it is 1.  E4M3 * v is exact in fp32, so every output
// is rounded once.
//
// HBM-bound: 0.5625 B read and 4 B written per element.  A lane decodes four
// consecutive elements at a time (two code bytes, one 16-byte store), so that
// every store instruction of a wave writes 1 KB of contiguous memory; the
// code and scale bytes behind it are a few cache lines that the wave's next
// instructions reuse.  With a whole block per lane each of its four stores
// touched 64 lines for 16 bytes: 2^24 elements 24.7 us (3.1 TB/s), now
// 13.3 us (5.8 TB/s).
#include "formats.h"
#include "internal.h"

namespace mixfp4 {
namespace {

constexpr int kThreads = 256;

constexpr int kQuads = 4;             // groups of four elements per thread and iteration

__global__ __launch_bounds__(kThreads) void dequantize_kernel(
    const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales,
    const float* __restrict__ tensor_scale, int64_t nquads, float* __restrict__ out) {
  const float s32 = tensor_scale ? *tensor_scale : 1.0f;
  const uint16_t* cw = reinterpret_cast<const uint16_t*>(codes);
  constexpr int64_t kTile = kThreads * kQuads;
  for (int64_t t = (int64_t)blockIdx.x * kTile; t < nquads; t += (int64_t)gridDim.x * kTile) {
    uint32_t c[kQuads], sb[kQuads];
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
      int64_t g = t + q * kThreads + threadIdx.x;
      g = g < nquads ? g : nquads - 1;
      c[q] = cw[g];
      sb[q] = scales[g >> 2];
    }
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
      const int64_t g = t + q * kThreads + threadIdx.x;
      const bool t1 = (sb[q] & 0x80u) != 0;
      const float s8 = e4m3_value(sb[q] & 0x7Fu);
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t nib = (c[q] >> (4 * j)) & 0xFu;
        const uint32_t mag = nib & 7u;
        const float a = s32 * (s8 * (t1 ? (float)mag : e2m1_value(mag)));
        v[j] = (nib & 8u) ? -a : a;
      }
      if (g < nquads)
        reinterpret_cast<float4*>(out)[g] = make_float4(v[0], v[1], v[2], v[3]);
    }
  }
}

}  // namespace

hipError_t launch_dequantize(const uint8_t* codes, const uint8_t* scales,
                             const float* tensor_scale, int64_t rows, int64_t k, float* out,
                             hipStream_t stream) {
  const int64_t nblocks = rows * (k / kBlock);
  if (nblocks == 0) return hipSuccess;
  const int64_t nquads = nblocks * (kBlock / 4);
  int64_t g = (nquads + kThreads * kQuads - 1) / (kThreads * kQuads);
  if (g > 65536) g = 65536;
  dequantize_kernel<<<(int)g, kThreads, 0, stream>>>(codes, scales, tensor_scale, nquads, out);
  return hipGetLastError();
}

}  // namespace mixfp4

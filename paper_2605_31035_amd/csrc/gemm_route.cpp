// Which GEMM mixfp4_gemm_auto takes: host code only, apart from the kernels'
// sources, whose measured traffic is tied to their text.
#include "blocked_layout.h"
#include "internal.h"

namespace mixfp4 {

namespace {
// Expected time of the two-pass GEMM in us: both decodes (2.56 B per element
// at 5.6 TB/s and a launch each) and the rounds that launch_gemm_decoded
// makes: a round of 256 x 256 tiles costs 6 us and 93 us per 4096 of K with
// every CU busy (76 with two thirds of them or less), one of 128 x 256 tiles
// 8 and 52 us (42).
float two_pass_us(int64_t m, int64_t n, int64_t k) {
  const int64_t cus = compute_units();
  const int64_t tm = padded_rows(m) / kTileRows, tn = padded_rows(n) / kTileRows;
  const int64_t tiles = tm * tn;
  const float kf = (float)k / 4096.0f;
  auto per_k = [&](int64_t wgs, float low, float high) {
    const float f = (float)wgs / (float)cus;
    return (f <= 0.667f ? low : low + (high - low) * (f - 0.667f) * 3.0f) * kf;
  };
  float us = 6.0f + (float)(m + n) * (float)k * 2.5625f / 5.6e6f;
  if (2 * tiles <= cus) return us + 8.0f + per_k(2 * tiles, 42.0f, 52.0f);
  const int64_t full = tiles / cus;
  us += (float)full * (6.0f + 93.0f * kf);
  const int64_t rest = tiles - full * cus;
  if (rest == 0) return us;
  const int64_t half = 2 * tm * (tn - full * cus / tm);
  return us + (full > 0 && half <= cus ? 8.0f + per_k(half, 42.0f, 52.0f)
                                       : 6.0f + per_k(rest, 76.0f, 93.0f));
}
}  // namespace

// The decode shapes and K % 32 != 0 take no workspace.  Where W can be read
// packed (K % 64 == 0), the cheaper of the direct and the two-pass GEMM by
// their expected times: the direct one up to about a thousand rows, or while
// its 128 x 256 tiles fill at most one round (509 x 11008 x 4096: 58 against
// 72 us; 1024 x 8192 x 8192: 128 against 148), two passes beyond (4096 x
// 14336 x 4096: 400 against 411, 16384 x 8192 x 8192: 1643 against 1800).
// The direct one has to be 8% cheaper: its decode beside the MFMAs draws
// power that lowers the clock, most in a longer run of GEMMs (2048 x 4096 x
// 11008 alone: 173 against 178 us, but inside a layer's backward pass the
// whole pass took 553 us with it and 544 without).  K % 64 = 32: the fused
// kernel's masked loads lose to two passes from 17 rows on (17 x 11008 x
// 4000 79 against 69 us, 512 x 11008 x 4000 220 against 79, 17 x 2048 x 1056
// 23 against 22); below K = 512, where the launches count, and for K < 256,
// two passes from m n / (m + n) = 1280 on.  So too for a W whose scale bytes
// are not word aligned, which the direct kernel does not read.
GemmPlan gemm_plan(int64_t m, int64_t n, int64_t k, bool w_word_aligned) {
  if (!gemm_two_pass_applies(m, n, k)) return {GemmRoute::kNoWorkspace, 0, 0};
  const int64_t both = gemm_two_pass_workspace(m, n, k);
  if (!w_word_aligned || !gemm_direct_applies(m, n, k))
    return (k % 64 != 0 && k >= 512) || m * n >= 1280 * (m + n)
               ? GemmPlan{GemmRoute::kTwoPass, 0, both}
               : GemmPlan{GemmRoute::kNoWorkspace, 0, 0};
  float us = 0.0f;
  const int tile = gemm_direct_tile(m, n, k, &us);
  us += 3.0f + (float)m * (float)k * 2.5625f / 5.6e6f;
  if (us <= 0.92f * two_pass_us(m, n, k)) return {GemmRoute::kDirect, tile, decoded_bytes(m, k)};
  return {GemmRoute::kTwoPass, 0, both};
}

}  // namespace mixfp4

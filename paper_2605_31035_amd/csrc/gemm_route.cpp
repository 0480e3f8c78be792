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
// whole pass took 553 us with it and 544 without).
//
// Up to K = 4096 the fused kernel is the third choice: one launch, and
// neither operand written first (1536 x 1024 x 320: 11 us against 20 on the
// direct kernel, 768 x 4096 x 1024 19 against 22, 512 x 16384 x 512 20
// against 23, 3000 x 1024 x 1024 19 against 25).  The direct kernel's costs
// are those at K = 4096; below, each call takes about 5 us more than they
// say, each further round 2 to 4, and C's stores show.  Products of
// m n / (m + n) >= 1280 that would go to two passes stay there.
//
// K % 64 = 32: the fused kernel's masked loads lose to two passes as K grows
// (512 x 11008 x 4000 220 against 79 us, 17 x 2048 x 1568 33 against 24), but
// a single round of its tiles wins while W's decode is the larger cost (17 x
// 8192 x 1056 24 against 32, 17 x 28672 x 4000 114 against 139); up to
// K = 832 it does or loses by 5% at most (32 x 512 x 800: 20 against 19).
// Below K = 512, for K < 256, and for a W whose scale bytes are not word
// aligned, which the direct kernel does not read, two passes from
// m n / (m + n) = 1280 on.
GemmPlan gemm_plan(int64_t m, int64_t n, int64_t k, bool w_word_aligned) {
  const GemmPlan none{GemmRoute::kNoWorkspace, 0, 0};
  if (!gemm_two_pass_applies(m, n, k)) return none;
  const GemmPlan two{GemmRoute::kTwoPass, 0, gemm_two_pass_workspace(m, n, k)};
  const bool large = m * n >= 1280 * (m + n);
  if (!w_word_aligned || !gemm_direct_applies(m, n, k)) {
    if (large) return two;
    if (k % 64 == 0 || k < 512) return none;
    const bool one_round = ((m + 127) / 128) * ((n + 127) / 128) <= compute_units();
    return one_round && k <= 4096 &&
                   (k <= 832 || gemm_fused_us(m, n, k) <= two_pass_us(m, n, k))
               ? none
               : two;
  }
  float us = 0.0f;
  int rounds = 1;
  const int tile = gemm_direct_tile(m, n, k, &us, &rounds);
  us += 3.0f + (float)m * (float)k * 2.5625f / 5.6e6f;
  const float two_us = two_pass_us(m, n, k);
  const bool direct = us <= 0.92f * two_us;
  if (k <= 4096 && (direct || !large)) {
    const float kf = (float)k / 4096.0f, c_us = (float)m * (float)n * 4.0f / 5e6f;
    us += 5.0f - 2.4f * kf + 0.45f * c_us + 400.0f / (float)k +
          (2.0f + 400.0f / (float)k) * (float)(rounds - 1);
    if (gemm_fused_us(m, n, k) <= (direct ? us : two_us)) return none;
  }
  return direct ? GemmPlan{GemmRoute::kDirect, tile, decoded_bytes(m, k)} : two;
}

}  // namespace mixfp4

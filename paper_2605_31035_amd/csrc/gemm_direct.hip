// MixFP4 GEMM for the sizes between the decode shape (m <= 16) and the large
// prefill: C = s32_A s32_W A W^T with A decoded once to exact fp16 values in
// the blocked layout (decode_operand.hip) and W read packed and decoded on
// its way into the matrix instructions (Sec. 3.3, App. B.5).
//
// Why.  The two-pass GEMM writes and reads W as fp16: 2.56 B per element of W
// before the first MFMA (20 us for 11008 x 4096), which a product of a few
// hundred rows does not earn back.  The fused kernel (gemm.hip) decodes both
// operands in every tile and needs 128 x 128 tiles, which leave most CUs idle
// at these sizes (64 x 14336 x 4096: 112 tiles).  Here A, the small operand,
// is decoded once (3 us), W leaves HBM once at 4.5 bits, and no wave shares
// W, so W never passes through LDS as fp16: a wave decodes its own columns'
// fragments in registers, between the MFMAs of the previous slice.
//
// Tiling.  A workgroup of KW x NW waves owns 32 TM rows and 32 TN NW columns
// of C; wave (kg, nw) computes all the rows of its own 32 TN columns over
// share kg of K, as TM x TN v_mfma_f32_32x32x16_f16 tiles (W first, as in
// gemm_f16.hip), and the KW partial sums are added through LDS in the order
// of K.  Narrow or short products take small tiles and split K over the
// waves, so that every CU has a workgroup and two waves per SIMD hide each
// other's latency; wide ones share A between column waves.
//
// Loads.  All operands but the scales go straight from memory to LDS
// (16-byte buffer loads): A in blocks of 32 K through a ring of ST stages
// (one per share of K, its loads dealt over the NW waves), W in a ring of WR
// windows of 128 K, 64 bytes per row and load, private to each wave.  Loaded by every
// lane into registers instead, a W row's 16-byte pieces and 4-byte scale
// words cost the texture unit a line each and held up the MFMAs: 128 x 11008
// x 4096 on TM = 4, NW = 4 took 66 us with them and 60 us without.  Scales
// come 16 bytes (256 K) at a time per row.
//
// Measured (with A's decode; before = the faster of the fused and two-pass
// kernels): 32 x 14336 x 4096 44.8 -> 16.2 us, 64 x 14336 x 4096 45.7 ->
// 19.2, 64 x 4096 x 11008 110.9 -> 20.1, 128 x 11008 x 4096 45.8 -> 25.3,
// 256 x 4096 x 4096 45.2 -> 19, 509 x 11008 x 4096 74.8 -> 56.5, 1024 x 4096
// x 4096 50.4 -> 45.  The decode
// costs nothing beside the MFMAs from TM = 4 on; the MFMAs alone (no loads,
// no decode) take 44 of the 60 us of a lone 128 x 256 tile at K = 4096.
#include <type_traits>

#include "blocked_layout.h"
#include "decode.h"
#include "internal.h"
#include "tile_order.h"

typedef int mixfp4_i32x4d __attribute__((ext_vector_type(4)));
// The 16-byte buffer load that writes straight into LDS (destination M0 +
// offset + 16 * lane).
__device__ void mixfp4_d_buffer_load_lds(mixfp4_i32x4d rsrc,
                                         __attribute__((address_space(3))) uint32_t* lds,
                                         int size, int voffset, int soffset, int offset,
                                         int aux) __asm("llvm.amdgcn.raw.buffer.load.lds");

namespace mixfp4 {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef mixfp4_i32x4d i32x4;

__device__ __forceinline__ i32x4 raw_range(const void* base, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  i32x4 r;
  r[0] = (int)(uint32_t)b;
  r[1] = (int)(uint32_t)(b >> 32);
  r[2] = (int)bytes;
  r[3] = 0x00020000;
  return r;
}

constexpr int kStepK64 = 64;       // K step of the main loop: four 16-K slices

// Four dwords at a 4-byte aligned address.
typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// Order of one slice's instructions: after each of the 2 TM MFMAs, a share
// of the next slice's LDS reads, of its decode and of the block loads.
template <int TM, int TN, int LD>
__device__ __forceinline__ void slice_order() {
  constexpr int kM = TM * TN;
#pragma unroll
  for (int i = 0; i < kM; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (i < TM) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, (24 * TN + kM - 1) / kM, 0);
    if (i >= kM / 2 && i - kM / 2 < LD) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
  }
}

template <int TM, int TN, int KW, int NW, int ST, int WR, int MINB>
__global__ __launch_bounds__(64 * KW * NW, MINB) void gemm_direct_kernel(
    const uint8_t* __restrict__ ablk, const uint8_t* __restrict__ w_codes,
    const uint8_t* __restrict__ w_scales, const float* __restrict__ a_ts,
    const float* __restrict__ w_ts, int64_t m, int64_t n, int64_t k, float* __restrict__ c,
    int64_t ldc) {
  constexpr int kWaveCols = 32 * TN;
  constexpr int kRows = 32 * TM, kCols = kWaveCols * NW;
  constexpr int kBlkA = kRows * 64;                  // bytes of one stage: kRows x 32 K
  constexpr int L = 2 * TM / NW;                     // 1 KB loads of A per wave and stage
  constexpr int kWinBytes = kWaveCols * 64;          // W codes of a wave over 128 K: one window
  constexpr int kUnits = TM * TN * 4;                // accumulator quads of a wave
  static_assert(L * NW == 2 * TM, "the waves share a stage's loads evenly");
  constexpr int kRingA = ST * kBlkA;
  constexpr int kRingW = WR * kWinBytes;
  constexpr int kRedBytes = KW == 1 ? 0 : KW == 2 ? NW * kUnits * 1024 : KW * NW * kUnits * 1024;
  constexpr int kRings = KW * kRingA + KW * NW * kRingW;
  constexpr int kLds = kRings > kRedBytes ? kRings : kRedBytes;
  // a W window must have landed when its first step is read: with WR = 3
  // it is issued 8 blocks before, with WR = 2 4, and read after the wait of
  // the sixth (second) block after it
  static_assert(ST >= 3 && (WR == 3 ? ST <= 8 : WR == 2 && ST <= 4), "window distance");
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kLds];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NW, nw = wave % NW;          // share of K, column range
  const int half = lane >> 5, lrow = lane & 31;
  const int64_t blocks = k / kStepK;                 // 32-K blocks of A
  const int64_t ntm = (m + kRows - 1) / kRows, ntn = (n + kCols - 1) / kCols;
  const int64_t tile = grouped_tile(xcd_item(blockIdx.x, gridDim.x), ntm, ntn);
  const int64_t m0 = (tile / ntn) * kRows;
  const int64_t n0 = (tile % ntn) * kCols + nw * kWaveCols;
  // this wave's K steps [u0, u0 + steps) of 64
  const int total = (int)(k / kStepK64);
  const int u0 = (int)((int64_t)total * kg / KW);
  const int steps = (int)((int64_t)total * (kg + 1) / KW) - u0;

  const i32x4 rsrc = raw_range(ablk + (m0 / kTileRows) * blocks * kBlkBytes + (m0 % kTileRows) * 64,
                               (uint32_t)(blocks * kBlkBytes - (m0 % kTileRows) * 64));
  uint8_t* ring_a = lds + kg * kRingA;
  uint8_t* ring_w = lds + KW * kRingA + wave * kRingW;
  const int last = 2 * steps - 1;                    // last block of the range
  auto lds_at = [&](uint8_t* base, int ofs) {
    return (__attribute__((address_space(3))) uint32_t*)(uintptr_t)(
        reinterpret_cast<uintptr_t>(base) + ofs);
  };
  auto issue = [&](int slot, int s, int p) {
    const int src = (s < last ? s : last) + 2 * u0;
    const int ofs = (nw * L + p) * 1024;
    mixfp4_d_buffer_load_lds(rsrc, lds_at(ring_a, slot + ofs), 16, lane * 16,
                             src * kBlkBytes + ofs, 0, 0);
  };
  // Window v of W: 128 K of this wave's 64 rows, 64 code bytes per row, row r
  // at 64 r with its 16-byte piece p in slot p ^ ((r >> 2) & 3).  Rows past
  // n load zeros (range check); a window past the row's end holds the next
  // row's codes there, never used.
  const int64_t pitch = k / 2;
  const int64_t wrows = n - n0 < 0 ? 0 : (n - n0 < kWaveCols ? n - n0 : kWaveCols);
  const uint8_t* wbase = w_codes + n0 * pitch + u0 * 32;
  const int wbytes = (int)(wrows * pitch) - u0 * 32;
  const int last_win = (steps - 1) / 2;
  int wofs[2 * TN];
#pragma unroll
  for (int q = 0; q < 2 * TN; ++q) {
    const int r = 16 * q + (lane >> 2);
    wofs[q] = r * (int)pitch + 16 * ((lane & 3) ^ ((r >> 2) & 3));
  }
  auto issue_w = [&](int slot, int v) {
    v = v < last_win ? v : last_win;
    const i32x4 rw = raw_range(wbase + 64 * v, (uint32_t)(wbytes > 64 * v ? wbytes - 64 * v : 0));
#pragma unroll
    for (int q = 0; q < 2 * TN; ++q)
      mixfp4_d_buffer_load_lds(rw, lds_at(ring_w, slot + q * 1024), 16, wofs[q], 0, 0, 0);
  };
  // the 16 code bytes of both of this lane's rows for step `odd` of a window
  typedef uint4 Raw[TN];
  auto read_w = [&](Raw& x, int slot, int odd) {
#pragma unroll
    for (int g = 0; g < TN; ++g) {
      const int r = 32 * g + lrow;
      x[g] = *reinterpret_cast<const uint4*>(ring_w + slot + r * 64 +
                                             slot_of(r, 2 * odd + half) * 16);
    }
  };
  // Scale bytes of this lane's rows: 16 bytes serve four steps.  The last
  // load of a row is moved back to end with the row; `shift` drops the
  // dwords of earlier steps.
  const uint8_t* ws[TN];
#pragma unroll
  for (int g = 0; g < TN; ++g) {
    int64_t r = n0 + 32 * g + lrow;
    r = r < n ? r : n - 1;
    ws[g] = w_scales + r * (k / kBlock);
  }
  auto load_s = [&](u32x4a4 (&x)[TN], int u) {
    int at = u0 + u;
    at = at < total - 4 ? at : total - 4;
#pragma unroll
    for (int g = 0; g < TN; ++g) x[g] = *reinterpret_cast<const u32x4a4*>(ws[g] + 4 * at);
  };
  auto take_s = [&](uint32_t (&d)[TN][4], const u32x4a4 (&x)[TN], int u) {
    const int shift = u0 + u - (total - 4);
#pragma unroll
    for (int g = 0; g < TN; ++g) {
      uint32_t a = x[g][0], b = x[g][1], e = x[g][2];
      const uint32_t f = x[g][3];
      if (shift > 0) {
        a = shift == 1 ? b : shift == 2 ? e : f;
        b = shift == 1 ? e : f;
        e = f;
      }
      d[g][0] = a;
      d[g][1] = b;
      d[g][2] = e;
      d[g][3] = f;
    }
  };
  // The codes of one step dealt to the MFMA's lane halves: dword sl is the
  // 8-element group 2 sl + h of slice sl.
  typedef uint32_t Codes[TN][4];
  auto deal = [&](Codes& f, const Raw& x) {
#pragma unroll
    for (int g = 0; g < TN; ++g) {
      auto r = __builtin_amdgcn_permlane32_swap(x[g].x, x[g].y, false, false);
      auto q = __builtin_amdgcn_permlane32_swap(x[g].z, x[g].w, false, false);
      f[g][0] = r[0];
      f[g][2] = r[1];
      f[g][1] = q[0];
      f[g][3] = q[1];
    }
  };
  typedef f16x8 AFrag[TM];
  typedef f16x8 BFrag[TN];
  auto read_a = [&](AFrag& fa, int slot, int sl) {
    const uint8_t* b = ring_a + slot;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int r = 32 * i + lrow;
      fa[i] = *reinterpret_cast<const f16x8*>(b + r * 64 + slot_of(r, 2 * sl + half) * 16);
    }
  };
  auto decode_w = [&](BFrag& fb, const Codes& f, const uint32_t (&sc)[TN][4], int j, int sl) {
#pragma unroll
    for (int g = 0; g < TN; ++g) {
      BlockDec d[4];
      block_dec4(sc[g][j], d);
      fb[g] = __builtin_bit_cast(f16x8, decode8(f[g][sl], d[sl]));
    }
  };
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;
  auto mfma = [&](const AFrag& fa, const BFrag& fb) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[j], fa[i], acc[i][j], 0, 0, 0);
  };

  if (steps > 0) {
    u32x4a4 sn[TN];
    uint32_t sc[TN][4];
    load_s(sn, 0);
#pragma unroll
    for (int v = 0; v < WR - 1; ++v) issue_w(v * kWinBytes, v);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < ST - 1; ++s)
#pragma unroll
      for (int p = 0; p < L; ++p) issue(s * kBlkA, s, p);
    wait_vm<(ST - 2) * L>();
    if (NW > 1) __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    AFrag pa, qa;
    BFrag pb, qb;
    Raw raw;
    Codes cur;
    take_s(sc, sn, 0);
    read_w(raw, 0, 0);
    deal(cur, raw);
    read_a(pa, 0, 0);
    decode_w(pb, cur, sc, 0, 0);
    int rd = 0, wr = (ST - 1) * kBlkA;               // slots of block s and of block s + ST - 1
    int wcur = 0, wfill = (WR - 1) * kWinBytes;       // slots of this W window and of the one WR - 1 ahead
    // One 64-K step u (step j of four whose scales are in sc): two blocks of
    // 32 K, each two slices.  Slice by slice, the next slice's A fragments
    // are read and its W fragments decoded while this slice's MFMAs run.
    auto step = [&](auto J_, int u) {
      constexpr int j = decltype(J_)::value;
      if constexpr (j == 0) load_s(sn, u + 4);
      if constexpr (j % 2 == 0) issue_w(wfill, u / 2 + WR - 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int s = 2 * u + b;
        if (b == 0) {
          if constexpr (j % 2 == 1) {
            wfill = wcur;
            wcur = wcur + kWinBytes == kRingW ? 0 : wcur + kWinBytes;
          }
          read_w(raw, wcur, j % 2 == 0 ? 1 : 0);
        }
        read_a(qa, rd, 1);
        decode_w(qb, cur, sc, j, 2 * b + 1);
        mfma(pa, pb);
#pragma unroll
        for (int p = 0; p < L; ++p) issue(wr, s + ST - 1, p);
        slice_order<TM, TN, L>();
        __builtin_amdgcn_sched_barrier(0);
        // block s + 1 has landed: at least the (ST - 2) L loads of the blocks
        // after it were issued later
        wait_vm<(ST - 2) * L>();
        if (NW > 1) __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        wr = rd;
        rd = rd + kBlkA == kRingA ? 0 : rd + kBlkA;
        read_a(pa, rd, 0);
        if (b == 0) {
          decode_w(pb, cur, sc, j, 2);
        } else {
          deal(cur, raw);
          if constexpr (j == 3) take_s(sc, sn, u + 1);
          decode_w(pb, cur, sc, (j + 1) % 4, 0);
        }
        mfma(qa, qb);
        slice_order<TM, TN, 0>();
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    using std::integral_constant;
    for (int u = 0;;) {
      step(integral_constant<int, 0>{}, u);
      if (++u >= steps) break;
      step(integral_constant<int, 1>{}, u);
      if (++u >= steps) break;
      step(integral_constant<int, 2>{}, u);
      if (++u >= steps) break;
      step(integral_constant<int, 3>{}, u);
      if (++u >= steps) break;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }

  const float scale = (a_ts ? *a_ts : 1.0f) * (w_ts ? *w_ts : 1.0f);
  const bool vec = (ldc % 4) == 0 && (reinterpret_cast<uintptr_t>(c) & 15u) == 0;
  // 32 x 32 accumulator layout of C^T: lane holds row 32 i + lane % 32;
  // register q holds column 32 j + 8 (q / 4) + 4 (lane / 32) + q % 4
  auto store4 = [&](int i, int j, int qq, float4 v) {
    const int64_t row = m0 + 32 * i + lrow, col = n0 + 32 * j + 8 * qq + 4 * half;
    if (row >= m) return;
    float* p = c + row * ldc + col;
    v = make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale);
    if (vec) {
      if (col < n) *reinterpret_cast<float4*>(p) = v;
    } else {
      if (col < n) p[0] = v.x;
      if (col + 1 < n) p[1] = v.y;
      if (col + 2 < n) p[2] = v.z;
      if (col + 3 < n) p[3] = v.w;
    }
  };
  auto quad = [&](int i, int j, int qq) {
    const f32x16& v = acc[i][j];
    return make_float4(v[4 * qq], v[4 * qq + 1], v[4 * qq + 2], v[4 * qq + 3]);
  };
  if constexpr (KW == 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) store4(i, j, qq, quad(i, j, qq));
  } else if constexpr (KW == 2) {
    // each half of K hands the other half's two register quads of every tile
    // over through LDS and finishes its own
    float4* red = reinterpret_cast<float4*>(lds) + nw * kUnits * 64;
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (kg != h) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int qq = 2 * h; qq < 2 * h + 2; ++qq)
              red[((i * TN + j) * 4 + qq) * 64 + lane] = quad(i, j, qq);
      }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (kg == h) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int qq = 2 * h; qq < 2 * h + 2; ++qq) {
              const float4 o = red[((i * TN + j) * 4 + qq) * 64 + lane];
              const float4 t = quad(i, j, qq);
              store4(i, j, qq, make_float4(t.x + o.x, t.y + o.y, t.z + o.z, t.w + o.w));
            }
      }
  } else {
    // partial sums through LDS, added in the order of K: share kg of the
    // waves finishes every KW-th register quad
    float4* red = reinterpret_cast<float4*>(lds);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq)
          red[((kg * NW + nw) * kUnits + (i * TN + j) * 4 + qq) * 64 + lane] = quad(i, j, qq);
    __syncthreads();
#pragma unroll
    for (int e0 = 0; e0 < kUnits; e0 += KW) {
      const int e = e0 + kg;
      if (e >= kUnits) continue;
      float4 t = red[(nw * kUnits + e) * 64 + lane];
#pragma unroll
      for (int w = 1; w < KW; ++w) {
        const float4 o = red[((w * NW + nw) * kUnits + e) * 64 + lane];
        t = make_float4(t.x + o.x, t.y + o.y, t.z + o.z, t.w + o.w);
      }
      store4(e / (4 * TN), (e / 4) % TN, e % 4, t);
    }
  }
}

template <int TM, int TN, int KW, int NW, int ST, int WR, int MINB>
hipError_t launch(const uint8_t* ablk, const float* a_ts, const uint8_t* w_codes,
                  const uint8_t* w_scales, const float* w_ts, int64_t m, int64_t n, int64_t k,
                  float* c, hipStream_t stream) {
  const int64_t tiles = ((m + 32 * TM - 1) / (32 * TM)) * ((n + 32 * TN * NW - 1) / (32 * TN * NW));
  gemm_direct_kernel<TM, TN, KW, NW, ST, WR, MINB><<<(unsigned)tiles, 64 * KW * NW, 0, stream>>>(
      ablk, w_codes, w_scales, a_ts, w_ts, m, n, k, c, n);
  return hipGetLastError();
}

// The tile configurations, with what one round of workgroups (`per_cu` on
// every CU) costs, one launch included: `fixed` us and `per_k` us for every
// 4096 of K, or `low` in a round that leaves a third of the CUs idle (per_cu
// = 1) or gives each only one workgroup of two.  Measured at K = 4096 with
// 128, 256, 344 and 512 workgroups (two rows of tiles from 256 on), us:
//   32 x 32    7.6   7.8  14.0  14.3     64 x 128  27.4  29.6  51.6   57.0
//   32 x 64   11.2  11.9  22.6  25.2    128 x 64   20.9  24.5  42.7   48.5
//   64 x 32    9.3  10.8  19.1  20.8    128 x 128  39.1  41.5  58.7   69.7
//   64 x 64   13.1  16.2  28.7  33.1    128 x 256  54.4  67.4 113.1  132.0
//   128 x 256, two on a CU: 64.0 75.0 104.6 126.8 (97 with 258, and 109 a
//   round over eight rounds of a 16384 x 8192 x 8192 product)
// The first three and the fourth split K over eight waves: 64 x 14336 x 4096
// on 64 x 64 tiles takes 16.3 us with eight waves and two W windows, 18.6
// with four waves and three.
struct DirectTile {
  int rows, cols, per_cu;
  int k_multiple;          // shares of K must be equal where waves step together
  float fixed, per_k, low;
};
constexpr DirectTile kTiles[] = {
    {32, 32, 2, 64, 0.5f, 13.8f, 7.2f},        {32, 64, 1, 64, 1.3f, 11.5f, 10.0f},
    {64, 32, 1, 64, 2.0f, 8.5f, 7.3f},         {64, 64, 1, 64, 1.5f, 15.0f, 11.8f},
    {64, 128, 1, 64 * 4, 1.5f, 28.0f, 26.0f},  {128, 64, 1, 64, 1.5f, 22.5f, 19.5f},
    {128, 128, 2, 64 * 2, 3.0f, 66.5f, 37.0f}, {128, 256, 1, 64 * 2, 5.0f, 61.0f, 48.5f},
    {128, 256, 2, 64, 6.0f, 108.0f, 61.0f},
};
constexpr int kTileCount = (int)(sizeof(kTiles) / sizeof(kTiles[0]));

float tile_cost(const DirectTile& t, int64_t m, int64_t n, int64_t k, int64_t cus) {
  const int64_t wgs = ((m + t.rows - 1) / t.rows) * ((n + t.cols - 1) / t.cols);
  const float kf = (float)k / 4096.0f;
  const int64_t full = wgs / (cus * t.per_cu), rest = wgs % (cus * t.per_cu);
  float us = (float)full * (t.fixed + t.per_k * kf);
  const float kk = kf * t.per_k;
  if (rest > cus)                 // two workgroups on some CUs
    us += t.fixed + kk * (0.83f + 0.17f * (float)(rest - cus) / (float)cus);
  else if (rest > 0)
    us += t.fixed + (t.per_cu == 2 || 3 * rest <= 2 * cus + 16 ? t.low * kf : kk);
  return us;
}

}  // namespace

bool gemm_direct_applies(int64_t m, int64_t n, int64_t k) {
  return gemm_two_pass_applies(m, n, k) && k % kStepK64 == 0 && k >= 256;
}

int gemm_direct_tile(int64_t m, int64_t n, int64_t k, float* us, int* rounds) {
  const int64_t cus = compute_units();
  int best = -1;
  float cost = 0.0f;
  for (int i = 0; i < kTileCount; ++i) {
    if (k % kTiles[i].k_multiple != 0) continue;
    const float t = tile_cost(kTiles[i], m, n, k, cus);
    if (best < 0 || t < cost) {
      best = i;
      cost = t;
    }
  }
  *us = cost;
  const DirectTile& t = kTiles[best];
  const int64_t wgs = ((m + t.rows - 1) / t.rows) * ((n + t.cols - 1) / t.cols);
  *rounds = (int)((wgs + cus * t.per_cu - 1) / (cus * t.per_cu));
  return best;
}

hipError_t launch_gemm_direct(int tile, const uint8_t* ablk, const float* a_ts,
                              const uint8_t* w_codes, const uint8_t* w_scales, const float* w_ts,
                              int64_t m, int64_t n, int64_t k, float* c, hipStream_t stream) {
  if (tile < 0 || tile >= kTileCount || k < 256 || k % kTiles[tile].k_multiple != 0)
    return hipErrorInvalidValue;
  switch (tile) {
    case 0: return launch<1, 1, 8, 1, 4, 2, 2>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
    case 1: return launch<1, 2, 8, 1, 4, 2, 1>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
    case 2: return launch<2, 1, 8, 1, 4, 2, 1>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
    case 3: return launch<2, 2, 8, 1, 3, 2, 1>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
    case 4: return launch<2, 2, 4, 2, 3, 3, 1>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
    case 5: return launch<4, 2, 4, 1, 3, 3, 1>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
    case 6: return launch<4, 2, 2, 2, 3, 2, 2>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
    case 7: return launch<4, 2, 2, 4, 4, 2, 1>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
    default: return launch<4, 2, 1, 4, 4, 3, 2>(ablk, a_ts, w_codes, w_scales, w_ts, m, n, k, c, stream);
  }
}

}  // namespace mixfp4

// Column transforms of the t passes: one column of F complex values by G <= 64
// lanes of a wave (lane s holds positions G r + s, r < E, natural order), and
// its spectrum in the block's LDS staging tile.
//
// F = 256, 512, 1024 (G = 64, E = 4, 8, 16): register passes of radix E (the last
// one of 1024: radix 4), natural order in, with lane twiddles from tables laid
// out in lane order; between passes registers and lane bits change places, by
// v_permlane swaps and row DPP or through the column's own LDS, which only its
// wave touches (no barrier).  Other lengths (2 values per lane at 128 and below,
// 32 at 2048; passes were not tried there): radix-2 stages, in registers for
// spans of G and more and across lanes below (fft_device.h).  At 512 points the
// passes take 0.6 of the vector instructions and 16 instead of 64 LDS exchanges.
#pragma once
#include "fft_device.h"
#include "fft_quad.h"

namespace cnlos {

template <int LOGF>
struct FftCol {
  static constexpr int F = 1 << LOGF;
  static constexpr int G = (F / 2) < 64 ? (F / 2) : 64;
  static constexpr int E = F / G;
  static constexpr bool PASS = LOGF >= 8 && LOGF <= 10;
  // entries of the twiddle tables: [k - 1][lane], W_F^{lane k} (a) and the later
  // passes' (b; E = 4 appends W_16^j, j < 16)
  static constexpr int TA = PASS ? (E - 1) * 64 : 0;
  static constexpr int TB = PASS ? (E - 1) * 64 + (E == 4 ? 16 : 0) : 0;
};

// Row of the staging tile that holds frequency k: where the passes leave it
// (lane + 64 r), so that a wave reads and writes 64 consecutive rows.
template <int LOGF>
__device__ __forceinline__ int z_row(int k) {
  using C = FftCol<LOGF>;
  if constexpr (!C::PASS) return k;
  const int l = k & 63, hi = k & ~63;
  if constexpr (C::E == 8) return hi + ((l & 7) << 3) + (l >> 3);
  if constexpr (C::E == 4) return hi + ((l & 3) << 4) + (l & 12) + (l >> 4);
  return hi + ((l & 15) << 2) + (l >> 4);
}
// LDS index of (row, column b) of the staging tile: rows of J + 1 (odd: 32
// consecutive rows of a column fall into different banks); the radix-2 form's
// bit-reversed rows with one more slot every 8 rows
template <int LOGF, int J>
__device__ __forceinline__ int z_at(int row, int b) {
  return row * (J + 1) + (FftCol<LOGF>::PASS ? 0 : (row >> 3)) + b;
}

// lane twiddles of the passes, loaded ahead of their use
template <int LOGF>
struct FftTw {
  using C = FftCol<LOGF>;
  static constexpr int N = C::PASS ? C::E - 1 : 1;
  float2 a[N], b[N], c[3];
  __device__ __forceinline__ void load_a(const float2* __restrict__ ta, int s) {
    if constexpr (C::PASS) {
#pragma unroll
      for (int k = 0; k < N; ++k) a[k] = ta[64 * k + s];
    }
  }
  __device__ __forceinline__ void load_b(const float2* __restrict__ tb, int s) {
    if constexpr (C::PASS) {
#pragma unroll
      for (int k = 0; k < N; ++k) b[k] = tb[64 * k + s];
      if constexpr (C::E == 4) {
#pragma unroll
        for (int k = 0; k < 3; ++k) c[k] = tb[192 + (k + 1) * (s & 3)];
      }
    }
  }
};

// registers (bit 0: P, Q) and lane bit 3 change places: the upper 8 lanes of a
// row take Q of the lower ones into P, these P of the upper ones into Q
__device__ __forceinline__ void lane_swap8(float& p, float& q) {
  const int a = __float_as_int(p), b = __float_as_int(q);
  p = __int_as_float(__builtin_amdgcn_update_dpp(a, b, 0x128, 0xf, 0xc, false));   // row_ror:8
  q = __int_as_float(__builtin_amdgcn_update_dpp(b, a, 0x128, 0xf, 0x3, false));
}
// 8 x 8: registers <-> lane bits 3 .. 5
__device__ __forceinline__ void exchange_hi8(float2 (&x)[8]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    lane_swap32(x[r].x, x[r + 4].x);
    lane_swap32(x[r].y, x[r + 4].y);
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    if (r & 2) continue;
    lane_swap16(x[r].x, x[r + 2].x);
    lane_swap16(x[r].y, x[r + 2].y);
  }
#pragma unroll
  for (int r = 0; r < 8; r += 2) {
    lane_swap8(x[r].x, x[r + 1].x);
    lane_swap8(x[r].y, x[r + 1].y);
  }
}
// Registers <-> the lane bits [SH, SH + log2 W) through the column's LDS, for
// each group of W registers.  One wave's LDS accesses are in order.
template <int E, int W, int SH>
__device__ __forceinline__ void exchange_lds(float2 (&x)[E], float2* slot, int s) {
  constexpr int mask = (W - 1) << SH;
  // E = 4: rows of 4 with a pad every 4 lanes (the column's LDS holds 292)
  auto at = [](int lane, int j) { return E == 4 ? 4 * lane + (lane >> 2) + j : (E + 1) * lane + j; };
  const int own = (s & mask) >> SH, rest = s & ~mask;
#pragma unroll
  for (int j = 0; j < E; ++j) slot[at(s, j)] = x[j];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int j = 0; j < E; ++j) x[j] = slot[at(rest | ((j % W) << SH), (j / W) * W + own)];
  __builtin_amdgcn_wave_barrier();
}

template <int N>
__device__ __forceinline__ void tw_mul(float2 (&x)[N + 1], const float2 (&w)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) x[k + 1] = cmul(x[k + 1], w[k]);
}
template <int N>
__device__ __forceinline__ void tw_mulc(float2 (&x)[N + 1], const float2 (&w)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) x[k + 1] = cmulc(x[k + 1], w[k]);
}

// radix-E pass whose upper half input is zero / of whose output only the lower
// half is wanted
template <int E>
__device__ __forceinline__ void dft_half_in(float2 (&x)[E]) {
  constexpr int H = E / 2;
  float2 a[H], b[H];
#pragma unroll
  for (int n = 0; n < H; ++n) {
    a[n] = x[n];
    b[n] = cmul_w64<false>(x[n], (64 / E) * n);
  }
  dft_reg<H, false>(a);
  dft_reg<H, false>(b);
#pragma unroll
  for (int k = 0; k < H; ++k) {
    x[2 * k] = a[k];
    x[2 * k + 1] = b[k];
  }
}
template <int E>
__device__ __forceinline__ void idft_half_out(float2 (&x)[E]) {
  constexpr int H = E / 2;
  float2 a[H], b[H];
#pragma unroll
  for (int k = 0; k < H; ++k) {
    a[k] = x[2 * k];
    b[k] = x[2 * k + 1];
  }
  dft_reg<H, true>(a);
  dft_reg<H, true>(b);
#pragma unroll
  for (int n = 0; n < H; ++n) x[n] = cadd(a[n], cmul_w64<true>(b[n], (64 / E) * n));
}

// Forward passes: x natural (HALF: the upper half of the registers is zero) ->
// x[r] = spectrum row s + 64 r of z_row.
template <int LOGF, bool HALF>
__device__ __forceinline__ void passes_fwd(float2 (&x)[FftCol<LOGF>::E], float2* slot,
                                           const FftTw<LOGF>& tw, int s) {
  constexpr int E = FftCol<LOGF>::E;
  if constexpr (HALF) dft_half_in<E>(x);
  else dft_reg<E, false>(x);
  tw_mul(x, tw.a);
  if constexpr (E == 8) {
    exchange_hi8(x);
    dft_reg<8, false>(x);
    tw_mul(x, tw.b);
    exchange_lds<8, 8, 0>(x, slot, s);
    dft_reg<8, false>(x);
  } else if constexpr (E == 4) {
    quad_transpose(x[0], x[1], x[2], x[3]);
    dft_reg<4, false>(x);
    tw_mul(x, tw.b);
    exchange_lds<4, 4, 2>(x, slot, s);
    dft_reg<4, false>(x);
    tw_mul(x, tw.c);
    exchange_lds<4, 4, 0>(x, slot, s);
    dft_reg<4, false>(x);
  } else {
    exchange_lds<16, 16, 2>(x, slot, s);
    dft_reg<16, false>(x);
    tw_mul(x, tw.b);
    exchange_lds<16, 4, 0>(x, slot, s);
    float2 y[16];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      dft4<false>(x[4 * e], x[4 * e + 1], x[4 * e + 2], x[4 * e + 3]);
#pragma unroll
      for (int d = 0; d < 4; ++d) y[e + 4 * d] = x[4 * e + d];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = y[r];
  }
}

// Inverse passes (the mirror): rows s + 64 r -> natural (CROP: only the lower
// half of the registers is formed).
template <int LOGF, bool CROP>
__device__ __forceinline__ void passes_inv(float2 (&x)[FftCol<LOGF>::E], float2* slot,
                                           const FftTw<LOGF>& tw, int s) {
  constexpr int E = FftCol<LOGF>::E;
  if constexpr (E == 8) {
    dft_reg<8, true>(x);
    exchange_lds<8, 8, 0>(x, slot, s);
    tw_mulc(x, tw.b);
    dft_reg<8, true>(x);
    exchange_hi8(x);
  } else if constexpr (E == 4) {
    dft_reg<4, true>(x);
    exchange_lds<4, 4, 0>(x, slot, s);
    tw_mulc(x, tw.c);
    dft_reg<4, true>(x);
    exchange_lds<4, 4, 2>(x, slot, s);
    tw_mulc(x, tw.b);
    dft_reg<4, true>(x);
    quad_transpose(x[0], x[1], x[2], x[3]);
  } else {
    float2 y[16];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int d = 0; d < 4; ++d) y[4 * e + d] = x[e + 4 * d];
      dft4<true>(y[4 * e], y[4 * e + 1], y[4 * e + 2], y[4 * e + 3]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = y[r];
    exchange_lds<16, 4, 0>(x, slot, s);
    tw_mulc(x, tw.b);
    dft_reg<16, true>(x);
    exchange_lds<16, 16, 2>(x, slot, s);
  }
  tw_mulc(x, tw.a);
  if constexpr (CROP) idft_half_out<E>(x);
  else dft_reg<E, true>(x);
}

}  // namespace cnlos

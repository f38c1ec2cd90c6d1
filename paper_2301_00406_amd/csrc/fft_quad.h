// Four-lane register FFT of the plane kernels.
//
// A transform of length N = 4 E is held by the four lanes j, j + 16, j + 32,
// j + 48 of a wave (g = lane / 16), E values each, so a wave carries 16
// transforms.  All butterflies run in registers: a length-E transform per lane
// with compile-time twiddles, one 4 x 4 transpose between the four lanes and
// their registers (v_permlane32_swap and v_permlane16_swap, one instruction per
// register and no LDS), and radix-4 butterflies.  Against eight lanes with
// cross-lane stages of spans 4, 2 and 1 (a lane exchange and a full complex
// product per value and stage) that is a third fewer vector instructions.
//
// A zero-padded transform of length 2N is its two halves by the parity h of
// the frequency 2 k + h: a length-N transform of x (h = 0) and of x[n] W_2N^n
// (h = 1); the twist is a compile-time factor per register and a change of the
// lane twiddles' index.  The inverses of both halves add up.
//
// Two arrangements, mirrored between a forward transform and its inverse:
//   rows     x[n1 + E n2] at lane g = n1 / (E/4) (E/4 neighbours per lane: wide
//            global accesses) <-> X[4 k1 + g] at lane g, register k1;
//   columns  x[4 n1 + g] at lane g, register n1 <-> X[k1 + E k2] with k1 =
//            quad(h, i, g), register (i, k2).
// In the columns' spectrum, -k sits in the lane of k (quad()), so the two
// frequencies can share a kernel value and be combined without an exchange.
#pragma once
#include "fft_device.h"

namespace cnlos {

// cos(2 pi k / 64), k = 0 .. 16
__device__ constexpr float kCos64[17] = {
    1.0f,                0.99518472667219693f, 0.98078528040323044f, 0.95694033573220886f,
    0.92387953251128674f, 0.88192126434835503f, 0.83146961230254524f, 0.77301045336273696f,
    0.70710678118654752f, 0.63439328416364549f, 0.55557023301960222f, 0.47139673682599764f,
    0.38268343236508977f, 0.29028467725446236f, 0.19509032201612827f, 0.09801714032956060f,
    0.0f};

// a exp(-+ 2 pi i k / 64) for a compile-time k (forward: minus; INV: plus)
template <bool INV>
__device__ __forceinline__ float2 cmul_w64(float2 a, int k) {
  k &= 63;
  if (INV) k = (64 - k) & 63;
  // quarter turns first: k = 16 q + r
  const int q = k >> 4, r = k & 15;
  if (q == 1) a = make_float2(a.y, -a.x);
  if (q == 2) a = make_float2(-a.x, -a.y);
  if (q == 3) a = make_float2(-a.y, a.x);
  if (r == 0) return a;
  if (r == 8) return make_float2(kCos64[8] * (a.x + a.y), kCos64[8] * (a.y - a.x));
  const float c = kCos64[r], s = kCos64[16 - r];
  return make_float2(a.x * c + a.y * s, a.y * c - a.x * s);
}

// radix-4 butterfly, natural order
template <bool INV>
__device__ __forceinline__ void dft4(float2& a0, float2& a1, float2& a2, float2& a3) {
  const float2 s02 = cadd(a0, a2), d02 = csub(a0, a2), s13 = cadd(a1, a3), d13 = csub(a1, a3);
  a0 = cadd(s02, s13);
  a2 = csub(s02, s13);
  if (INV) {
    a1 = make_float2(d02.x - d13.y, d02.y + d13.x);
    a3 = make_float2(d02.x + d13.y, d02.y - d13.x);
  } else {
    a1 = make_float2(d02.x + d13.y, d02.y - d13.x);
    a3 = make_float2(d02.x - d13.y, d02.y + d13.x);
  }
}

// E = 32: one group at a time (its successor's twiddles are already on their
// way); without the fence the twiddles of all groups are held at once and the
// kernel spills
template <int E>
__device__ __forceinline__ void quad_group_end() {
  if constexpr (E == 32) __builtin_amdgcn_sched_barrier(0);
}

// in-register transform of length E, natural order in and out
template <int E, bool INV>
__device__ __forceinline__ void dft_reg(float2 (&v)[E]) {
  if constexpr (E == 2) {
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (E == 4) {
    dft4<INV>(v[0], v[1], v[2], v[3]);
  } else {
    // n = B a + b: length A over a, twiddle W_E^{b k1}, length B over b
    constexpr int B = E == 8 ? 2 : 4, A = E / B;
    float2 t[B][A];
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
      for (int a = 0; a < A; ++a) t[b][a] = v[B * a + b];
      dft_reg<A, INV>(t[b]);
#pragma unroll
      for (int k = 0; k < A; ++k) t[b][k] = cmul_w64<INV>(t[b][k], (64 / E) * b * k);
      quad_group_end<E>();
    }
#pragma unroll
    for (int k = 0; k < A; ++k) {
      if constexpr (B == 2) {
        v[k] = cadd(t[0][k], t[1][k]);
        v[k + A] = csub(t[0][k], t[1][k]);
      } else {
        dft4<INV>(t[0][k], t[1][k], t[2][k], t[3][k]);
#pragma unroll
        for (int b = 0; b < 4; ++b) v[k + A * b] = t[b][k];
      }
    }
  }
}

// swap the upper 32 lanes of a with the lower 32 of b; the odd rows of 16
// lanes of a with the even rows of b
__device__ __forceinline__ void lane_swap32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void lane_swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
// 4 x 4 transpose: register r at lane g takes register g of lane r
__device__ __forceinline__ void quad_transpose(float2& r0, float2& r1, float2& r2, float2& r3) {
  lane_swap32(r0.x, r2.x);
  lane_swap32(r0.y, r2.y);
  lane_swap32(r1.x, r3.x);
  lane_swap32(r1.y, r3.y);
  lane_swap16(r0.x, r1.x);
  lane_swap16(r0.y, r1.y);
  lane_swap16(r2.x, r3.x);
  lane_swap16(r2.y, r3.y);
}

// The column spectrum's k1 at lane g of register group i, half h.  E >= 8:
// groups 2t and 2t + 1 hold k1 and its negative (E - k1 for h = 0, where 0 and
// E/2 are their own negatives and share lane 0; E - 1 - k1 for h = 1).
template <int E>
__host__ __device__ constexpr int quad(int h, int i, int g) {
  if (E == 4) return g;
  const int a = 4 * (i >> 1) + g;
  if (!(i & 1)) return a;
  if (h) return E - 1 - a;
  return a == 0 ? E / 2 : E - a;
}

// the lane number, opaque to the compiler: the twiddle addresses that follow
// from it are formed anew by each transform (a few additions) instead of being
// kept in registers through the kernel
__device__ __forceinline__ int fresh(int g) {
  asm volatile("" : "+v"(g));
  return g;
}
// row twiddles W_2N^{n1 (2c + H)}, n1 = (E/4) g + i, at wb[c][i (2c + H)]
template <int E, int H>
__device__ __forceinline__ void quad_row_tw(const float2* (&wb)[4], const float2* tw2, int g) {
  const int f = fresh(g);
#pragma unroll
  for (int c = 0; c < 4; ++c) wb[c] = tw2 + (E / 4) * (2 * c + H) * f;
}

// Forward row transform, half H: x[4 i + n2] = element n1 + E n2, n1 =
// (E/4) g + i, into v[k1] = X[4 k1 + g].  tw2[t] = W_2N^t, t < 2N (LDS).
template <int E, int H>
__device__ __forceinline__ void quad_row_fwd(const float2 (&x)[E], float2 (&v)[E],
                                             const float2* tw2, int g) {
  const float2* wb[4];
  quad_row_tw<E, H>(wb, tw2, g);
#pragma unroll
  for (int i = 0; i < E / 4; ++i) {
    float2 a[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) a[c] = H ? cmul_w64<false>(x[4 * i + c], 8 * c) : x[4 * i + c];
    dft4<false>(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int c = H ? 0 : 1; c < 4; ++c) a[c] = cmul(a[c], wb[c][i * (2 * c + H)]);
    quad_transpose(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int c = 0; c < 4; ++c) v[(E / 4) * c + i] = a[c];
    if (i & 1) quad_group_end<E>();
  }
  dft_reg<E, false>(v);
}

// Inverse row transform of half H, into x (ADD: added to it).
template <int E, int H, bool ADD>
__device__ __forceinline__ void quad_row_inv(float2 (&v)[E], float2 (&x)[E], const float2* tw2,
                                             int g) {
  dft_reg<E, true>(v);
  const float2* wb[4];
  quad_row_tw<E, H>(wb, tw2, g);
#pragma unroll
  for (int i = 0; i < E / 4; ++i) {
    float2 a[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) a[c] = v[(E / 4) * c + i];
    quad_transpose(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int c = H ? 0 : 1; c < 4; ++c) a[c] = cmulc(a[c], wb[c][i * (2 * c + H)]);
    dft4<true>(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float2 y = H ? cmul_w64<true>(a[c], 8 * c) : a[c];
      x[4 * i + c] = ADD ? cadd(x[4 * i + c], y) : y;
    }
    if (i & 1) quad_group_end<E>();
  }
}

// Lane twiddles of a column transform: W_2N^{q kk}, kk = 2 quad(H, i, g) + H,
// q = 1 .. 3.  Even groups i = 2t: kk = 8 t + (2 g + H); odd ones: kk = 2 E - H
// - 8 t - 2 g (lane 0 of group 1 of the even half: E).
template <int E, int H>
struct QuadColTw {
  const float2 *lo[3], *hi[3], *h0[3];
  static constexpr int TM = E >= 8 ? E / 8 - 1 : 0;     // the last t
  __device__ __forceinline__ QuadColTw(const float2* tw2, int g) {
    const int f = fresh(g);
#pragma unroll
    for (int q = 1; q < 4; ++q) {
      lo[q - 1] = tw2 + q * (2 * f + H);
      if constexpr (E >= 8) {
        hi[q - 1] = tw2 + q * (2 * E - H - 8 * TM - 2 * f);
        h0[q - 1] = tw2 + q * (f ? 2 * E - 2 * f : E);
      }
    }
  }
  __device__ __forceinline__ void get(float2 (&w)[3], int i) const {
    const int t = i >> 1;
#pragma unroll
    for (int q = 1; q < 4; ++q) {
      if (E == 4 || !(i & 1)) w[q - 1] = lo[q - 1][8 * t * q];
      else if (H == 0 && t == 0) w[q - 1] = h0[q - 1][0];
      else w[q - 1] = hi[q - 1][8 * (TM - t) * q];
    }
  }
};

// Forward column transform, half H, in place: c[n1] = x[4 n1 + g] into
// c[4 i + k2] = X[quad(H, i, g) + E k2].
template <int E, int H>
__device__ __forceinline__ void quad_col_fwd(float2 (&c)[E], const float2* tw2, int g) {
  if constexpr (H) {
#pragma unroll
    for (int n = 1; n < E; ++n) c[n] = cmul_w64<false>(c[n], (32 / E) * n);
  }
  dft_reg<E, false>(c);
  float2 s[E];
  float2 w[3];
  const QuadColTw<E, H> tw(tw2, g);
  tw.get(w, 0);
#pragma unroll
  for (int i = 0; i < E / 4; ++i) {
    float2 a[4], wn[3];
    if (i + 1 < E / 4) tw.get(wn, i + 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = c[quad<E>(H, i, q)];
    quad_transpose(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int q = 1; q < 4; ++q) a[q] = cmul(a[q], w[q - 1]);
    dft4<false>(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int q = 0; q < 4; ++q) s[4 * i + q] = a[q];
    if (i + 1 < E / 4) {
#pragma unroll
      for (int q = 0; q < 3; ++q) w[q] = wn[q];
    }
    quad_group_end<E>();
  }
#pragma unroll
  for (int r = 0; r < E; ++r) c[r] = s[r];
}

// Inverse column transform, half H, in place (the mirror of quad_col_fwd).
template <int E, int H>
__device__ __forceinline__ void quad_col_inv(float2 (&c)[E], const float2* tw2, int g) {
  float2 s[E];
  float2 w[3];
  const QuadColTw<E, H> tw(tw2, g);
  tw.get(w, 0);
#pragma unroll
  for (int i = 0; i < E / 4; ++i) {
    float2 a[4], wn[3];
    if (i + 1 < E / 4) tw.get(wn, i + 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = c[4 * i + q];
    dft4<true>(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int q = 1; q < 4; ++q) a[q] = cmulc(a[q], w[q - 1]);
    quad_transpose(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int q = 0; q < 4; ++q) s[quad<E>(H, i, q)] = a[q];
    if (i + 1 < E / 4) {
#pragma unroll
      for (int q = 0; q < 3; ++q) w[q] = wn[q];
    }
    quad_group_end<E>();
  }
  dft_reg<E, true>(s);
#pragma unroll
  for (int n = 0; n < E; ++n) c[n] = H ? cmul_w64<true>(s[n], (32 / E) * n) : s[n];
}

}  // namespace cnlos

// Spectral kernels: the zero-padded 3-D FFT convolution of the light-cone
// transform (the H of eq. (3)) and the FFT-diagonal solve of eq. (11).
//
// Both are split the same way over the [n][n][m] volume (t fastest):
//   t pass   : per scan column, resample (R_z, convolution only), real-to-
//              complex FFT along t, written as spectrum planes [kt][n*n];
//   plane    : per kt plane, 2-D FFT over (x, y), pointwise spectral operation
//              (multiply by H^ / its conjugate, or divide by c + mu*sigma),
//              inverse 2-D FFT, in place;
//   t pass   : per scan column, complex-to-real inverse FFT along t, crop,
//              R_t^{-1} (S^T and the falloff weight), fused epilogue.
// The t axis of the convolution is padded to 2m and the real input makes only
// kt = 0..m necessary (the two real bins kt = 0, m share one plane);
// the (x, y) padding to 2n x 2n lives only inside the plane kernel: rows and
// columns are transformed with their zero halves folded into twists, and the
// n x n crop is taken before anything leaves the CU (n = 128 takes the ky
// parities one after the other to fit LDS).
#include <math.h>

#include "cnlos_internal.h"
#include "fft_device.h"
#include "fft_quad.h"
#include "fft_column.h"
#include "stencil_device.h"

namespace cnlos {

// the volume behind v for this launch's scene (zo: the scene's byte offset)
__device__ __forceinline__ const float* vol_in(const Vol& v, const CtlHead& h, size_t zo) {
  return vol_resolve(v, h, zo);
}
__device__ __forceinline__ float* vol_out(const Vol& v, const CtlHead& h, size_t zo) {
  return vol_resolve(v, h, zo);
}
// ---------------------------------------------------------------------------
// t passes.  A block handles J scan columns (t_columns); each column's FFT
// lives in the registers of a group of G <= 64 lanes, so within one wave
// (lane s keeps positions G*r + s).  Spectrum planes are exchanged with global
// memory through an LDS staging tile [kt][J], so every plane access is a
// J * 8-byte segment (64 bytes from m = 256 on).  Fewer lanes per column (more
// elements per lane, fewer cross-lane stages) measured slower: the passes are
// bound by the latency of their phases, and fewer waves hide less of it.
// ---------------------------------------------------------------------------
// Columns per block of a t pass of length 2^logf: 8 for lengths 256 to 1024,
// where a block's 512 threads, its LDS (37 KB at 512, 75 KB at 1024) and registers
// leave room for two blocks per CU, so one block's loads overlap the other's
// transform (16-column blocks of 1024 threads, one per CU, write 128-byte
// segments: forward pass of 128x128x1024 84 -> 73 us, but inverse 60 -> 77, and
// 13 -> 18 and 11 -> 17 at 32x32x1024); 16 for shorter transforms (the solve phase
// of a fused pass needs whole waves), 4 at 2048 (LDS).
constexpr int t_columns(int logf) { return logf <= 7 ? 16 : (logf <= 10 ? 8 : 4); }

// waves per SIMD that a t pass is compiled for: two blocks of 512 threads per CU
// at length 1024 (their LDS allows it; the epilogues' registers need the cap, which
// spills 12 of k_tinv_conv_rhs<FWD_DUAL>'s and 8 of k_tinv_conv<FWD_OBJ>'s)
constexpr int t_waves(int logf) { return logf == 10 ? 4 : 1; }

template <int LOGF>
struct TGeo {                                 // transform of length F = 2^LOGF
  static constexpr int F = 1 << LOGF;
  static constexpr int G = (F / 2) < 64 ? (F / 2) : 64;   // lanes per column
  static constexpr int E = F / G;                         // elements per lane (>= 2)
  static constexpr int J = t_columns(LOGF);               // columns per block
  static constexpr int NT = J * G;
};

// A block-strided copy with compile-time extents, split into its loads (into
// registers, indices clamped into range) and its stores: a loop whose trip count
// depends on the thread index is not unrolled, and each of its iterations waits
// for its own load before its store.  Copies whose loads are all issued before the
// first store (copy_together) cost one memory round trip together, where
// copies done one after the other wait for each in turn.
template <int NT, int COUNT, typename T, typename Ld, typename St>
struct SplitCopy {
  static constexpr int NS = (COUNT + NT - 1) / NT;
  Ld ld;
  St st;
  T v[NS];
  __device__ __forceinline__ void load(int tid) {
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int it = tid + j * NT;
      v[j] = ld(it < COUNT ? it : COUNT - 1);
    }
  }
  // unconditional: a lane past the end stores the last element's value to
  // the last element, as its owner does (a store under a per-lane condition
  // lets the compiler sink its load into the branch, behind a wait for every
  // load before it)
  __device__ __forceinline__ void store(int tid) {
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int it = tid + j * NT;
      st(it < COUNT ? it : COUNT - 1, v[j]);
    }
  }
};
template <int NT, int COUNT, typename Ld, typename St>
__device__ __forceinline__ auto split_copy(Ld ld, St st) {
  using T = decltype(ld(0));
  return SplitCopy<NT, COUNT, T, Ld, St>{ld, st, {}};
}
template <typename... C>
__device__ __forceinline__ void copy_together(int tid, C&&... c) {
  (c.load(tid), ...);
  (c.store(tid), ...);
}
template <int NT, int COUNT, typename T>
__device__ __forceinline__ auto table_copy(T* dst, const T* __restrict__ src) {
  return split_copy<NT, COUNT>([=](int i) { return src[i]; }, [=](int i, T v) { dst[i] = v; });
}

template <int J>
constexpr int stg_size(int rows) { return rows * (J + 1) + rows / 8 + J; }   // see z_at
// The real transforms' (un)tangling.  A real column of 2F samples is one
// complex transform Z of length F of its pairs; its spectrum X[0 .. F] and Z
// are related per pair of frequencies (k, F - k), so the thread that moves
// such a pair between the planes and the LDS staging tile does both at once (one
// complex product for two frequencies, and the tile holds Z in natural order).
// Planes: kt = 0 .. F - 1, plane 0 holding X_0 + i X_F (both real).  The pair
// of k = 0 is k = F/2, whose twiddle is -i: Z = conj(X) there.
// W^k = exp(-pi i k / F) = tw[STEP k].
//
// planes -> Z: loads and stores split as in SplitCopy
template <int J, int NT, int LOGF, int STEP>
struct TangleCopy {
  static constexpr int F = 1 << LOGF, COUNT = F / 2 * J, NS = (COUNT + NT - 1) / NT;
  float2* lds;
  const float2* __restrict__ spec;
  const float2* __restrict__ tw;
  int nn, col0;
  float2 a[NS], b[NS], w[NS];
  __device__ __forceinline__ static int at(int tid, int j) {
    const int it = tid + j * NT;
    return it < COUNT ? it : COUNT - 1;
  }
  __device__ __forceinline__ void load(int tid) {
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int it = at(tid, j), k = it / J, c = col0 + it % J, kp = k ? F - k : F / 2;
      a[j] = spec[(size_t)k * nn + c];
      b[j] = spec[(size_t)kp * nn + c];
      w[j] = tw[STEP * k];
    }
  }
  __device__ __forceinline__ void store(int tid) {
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int it = at(tid, j), k = it / J, c = it % J, kp = k ? F - k : F / 2;
      const float2 e = make_float2(0.5f * (a[j].x + b[j].x), 0.5f * (a[j].y - b[j].y));
      const float2 o = make_float2(0.5f * (a[j].x - b[j].x), 0.5f * (a[j].y + b[j].y));
      const float2 q = cmulc(o, w[j]);
      const bool z = k == 0;
      const float2 zk = make_float2(z ? 0.5f * (a[j].x + a[j].y) : e.x - q.y,
                                    z ? 0.5f * (a[j].x - a[j].y) : e.y + q.x);
      const float2 zp = make_float2(z ? b[j].x : e.x + q.y, z ? -b[j].y : q.x - e.y);
      lds[z_at<LOGF, J>(z_row<LOGF>(k), c)] = zk;
      lds[z_at<LOGF, J>(z_row<LOGF>(kp), c)] = zp;
    }
  }
};
template <int J, int NT, int LOGF, int STEP>
__device__ __forceinline__ auto tangle_copy(float2* lds, const float2* __restrict__ spec,
                                            const float2* __restrict__ tw, int nn, int col0) {
  return TangleCopy<J, NT, LOGF, STEP>{lds, spec, tw, nn, col0, {}, {}, {}};
}
// Z (staged) -> planes
template <int J, int NT, int LOGF, int STEP>
__device__ __forceinline__ void untangle_to_planes(const float2* lds, const float2* __restrict__ tw,
                                                   float2* __restrict__ spec, int nn, int col0,
                                                   int tid) {
  constexpr int F = 1 << LOGF, COUNT = F / 2 * J, NS = (COUNT + NT - 1) / NT;
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const int it = tid + j * NT;
    if (NS * NT > COUNT && it >= COUNT) break;
    const int k = it / J, c = it % J, kp = k ? F - k : F / 2;
    const float2 zk = lds[z_at<LOGF, J>(z_row<LOGF>(k), c)];
    const float2 zp = lds[z_at<LOGF, J>(z_row<LOGF>(kp), c)];
    const float2 e = make_float2(0.5f * (zk.x + zp.x), 0.5f * (zk.y - zp.y));
    const float2 o = make_float2(0.5f * (zk.x - zp.x), 0.5f * (zk.y + zp.y));
    const float2 q = cmul(o, tw[STEP * k]);
    const bool z = k == 0;
    spec[(size_t)k * nn + col0 + c] =
        make_float2(z ? zk.x + zk.y : e.x + q.y, z ? zk.x - zk.y : e.y - q.x);
    spec[(size_t)kp * nn + col0 + c] =
        make_float2(z ? zp.x : e.x - q.y, z ? -zp.y : -e.y - q.x);
  }
}

// A column's spectrum between its lanes' registers and the staging tile.
// Radix-2 form: position G r + s holds the bit-reversed frequency.
template <int LOGF, int J>
__device__ __forceinline__ void stage_put(float2* lds, const float2 (&x)[FftCol<LOGF>::E], int b,
                                          int s) {
  using C = FftCol<LOGF>;
#pragma unroll
  for (int r = 0; r < C::E; ++r)
    lds[z_at<LOGF, J>(C::PASS ? 64 * r + s : brev(C::G * r + s, LOGF), b)] = x[r];
}
template <int LOGF, int J>
__device__ __forceinline__ void stage_get(const float2* lds, float2 (&x)[FftCol<LOGF>::E], int b,
                                          int s) {
  using C = FftCol<LOGF>;
#pragma unroll
  for (int r = 0; r < C::E; ++r)
    x[r] = lds[z_at<LOGF, J>(C::PASS ? 64 * r + s : brev(C::G * r + s, LOGF), b)];
}
// The transforms (tws, twc: the radix-2 form's tables in LDS; slot: the column's
// LDS).  HALF: zero upper half (the padded input); CROP: lower half only.
template <int LOGF, bool HALF, int TSTEP>
__device__ __forceinline__ void col_transform_fwd(float2 (&x)[FftCol<LOGF>::E], float2* slot,
                                                  const FftTw<LOGF>& tw, const float2* tws,
                                                  const float2* twc, int s) {
  using C = FftCol<LOGF>;
  if constexpr (C::PASS) {
    passes_fwd<LOGF, HALF>(x, slot, tw, s);
  } else {
    if constexpr (HALF) {
#pragma unroll
      for (int r = 0; r < C::E / 2; ++r)
        x[r + C::E / 2] = cmul(x[r], tws[TSTEP * 2 * (C::G * r + s)]);
    }
    dif_inlane<C::G, C::E, HALF ? C::E / 4 : C::E / 2>(x, s, twc);
    dif_xlane<C::G, C::E>(x, s, twc);
  }
}
template <int LOGF, bool CROP, int TSTEP>
__device__ __forceinline__ void col_transform_inv(float2 (&x)[FftCol<LOGF>::E], float2* slot,
                                                  const FftTw<LOGF>& tw, const float2* tws,
                                                  const float2* twc, int s) {
  using C = FftCol<LOGF>;
  if constexpr (C::PASS) {
    passes_inv<LOGF, CROP>(x, slot, tw, s);
  } else {
    dit_xlane<C::G, C::E>(x, s, twc);
    dit_inlane<C::G, C::E, CROP ? C::E / 4 : C::E / 2>(x, s, twc);
    if constexpr (CROP) {
#pragma unroll
      for (int r = 0; r < C::E / 2; ++r)
        x[r] = cadd(x[r], cmulc(x[r + C::E / 2], tws[TSTEP * 2 * (C::G * r + s)]));
    }
  }
}
// Twiddle tables of a launch: the radix-2 form's (tw: exp(-pi i j / m); twc per
// span) and the passes' (fa, fb: the convolution's, then the solve's).
struct TwTabs {
  const float2* tw;
  const float2* twc;
  const float2* fa;
  const float2* fb;
};
__device__ __forceinline__ void zsh_tw(TwTabs& t, size_t zo) {
  t.tw = zsh(t.tw, zo);
  t.twc = zsh(t.twc, zo);
  t.fa = zsh(t.fa, zo);
  t.fb = zsh(t.fb, zo);
}

// The resampling rows and columns as descriptors of one 16-byte read (built on
// the host): weights of three neighbouring samples from a base on (0 where the
// row has fewer; the base is clamped so that all three exist), or for an R_z
// row of more than 3 taps, whose interior weights are exactly 1, the end
// weights (x, z) with both ends' indices, the interior coming from the prefix
// sums pf.  Such rows lie below m/8 (resample_long_rows; LONG: the row may be one).
template <bool LONG, typename PT>
__device__ __forceinline__ float rz_row(const float4 d, const float* xf, const PT* pf) {
  const RzIndex x = rz_index(__float_as_int(d.w));
  const float s = fmaf(d.y, xf[x.k0 + 1], d.x * xf[x.k0]);
  if constexpr (!LONG) {
    return fmaf(d.z, xf[x.k0 + 2], s);
  } else {
    const float in = (float)(pf[x.p2] - pf[x.p0]);
    return fmaf(d.z, xf[x.k2], s + (x.lg ? in : 0.f));   // k2: k0 + 2, or the row's end
  }
}
__device__ __forceinline__ float st_taps(const float4 d, const float* g) {
  const int x = __float_as_int(d.w);
  return fmaf(d.z, g[x + 2], fmaf(d.y, g[x + 1], d.x * g[x]));
}

// Inclusive prefix sum over the 64 lanes (DPP: within rows of 16 lanes, then
// across them).  In FP64: an R_z row takes the difference of two prefix sums,
// and with FP32 sums in this order the dual model's volumes were half as far
// again from the FP64 result (32x32x256, 16 iterations: 8.6e-7 against 5.8e-7).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xf, false);
  return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_scan(double v) {
  v = dpp_add<0x111, 0xf>(v);       // row_shr:1, 2, 4, 8
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);       // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xc>(v);    // row_bcast:31 into rows 2 and 3
}
// type of the prefix sums: FP64 where a column has a whole wave
template <int LOGM>
using Prefix = typename std::conditional<TGeo<LOGM>::G == 64, double, float>::type;

// t pass, forward, convolution: x -> R_z x -> zero-pad to 2m -> R2C -> planes.
// The real length-2m transform is a complex length-m transform of the packed
// pairs (x[2p], x[2p+1]); its upper half is zero, so the first DIF stage is a
// twist.  The two real bins kt = 0 and kt = m share plane 0 as X_0 + i X_m, so
// the transform fills exactly m planes.
// Forward t pass of the convolution from a column whose real input is in
// LDS (xf, with xv[r] = xf[G r + s] in registers): R_z, packed real-to-complex
// transform of length 2m, staged and untangled into the planes.  Only the
// staging tile is shared by the block's waves: two barriers.
template <int LOGM>
__device__ __forceinline__ void tfwd_conv_from_lds(float2* lds, const TwTabs& tt, const float2* tws,
                                                   const float2* twc,
                                                   const float4* __restrict__ rows,
                                                   float (&xv)[TGeo<LOGM>::E], int tid, int col0,
                                                   float2* __restrict__ spec, int nn) {
  using T = TGeo<LOGM>;
  constexpr int M = 1 << LOGM, G = T::G, E = T::E, J = T::J, NT = T::NT;
  constexpr int ZS = M + M / 8 + 4;
  const int b = tid / G, s = tid % G;
  float2* slot = lds + b * ZS;
  float* xf = reinterpret_cast<float*>(slot);
  Prefix<LOGM>* pf = reinterpret_cast<Prefix<LOGM>*>(xf + M);
  static_assert(resample_scan_rows(M, G) * G * sizeof(*pf) <= M * sizeof(float), "prefix sums fit");
  float4 d[E];                                     // descriptors of the rows 2p, 2p + 1
#pragma unroll
  for (int r = 0; r < E; ++r) d[r] = rows[2 * (G * (r >> 1) + s) + (r & 1)];
  FftTw<LOGM> tw;
  tw.load_a(tt.fa, s);
  // R_z rows of more than 3 taps (small q, where a z bin spans many t bins)
  // have interior weights exactly 1, so they are computed as w x[k0] +
  // (P[k1] - P[k0 + 1]) + w' x[k1] from exclusive prefix sums P of the first
  // RS G inputs (those rows end below m/4 + 8, checked when the tables are
  // built); rows of at most 3 taps are summed directly.  No row loops, so no
  // lane waits for the longest row of its wave.
  constexpr int RS = resample_scan_rows(M, G);
  Prefix<LOGM> carry = 0;
#pragma unroll
  for (int r = 0; r < RS; ++r) {
    Prefix<LOGM> inc = xv[r];
    if constexpr (G == 64) {
      inc = wave_scan(inc);
      pf[G * r + s] = carry + (inc - (double)xv[r]);
      const unsigned long long u = (unsigned long long)__double_as_longlong(inc);
      const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)u, 63);
      const unsigned hi = __builtin_amdgcn_readlane((int)(u >> 32), 63);
      carry += __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    } else {
#pragma unroll
      for (int d1 = 1; d1 < G; d1 <<= 1) {
        const float y = __shfl_up(inc, d1, G);
        if (s >= d1) inc += y;
      }
      pf[G * r + s] = carry + (inc - xv[r]);
      carry += __shfl(inc, G - 1, G);
    }
  }
  __builtin_amdgcn_wave_barrier();                 // a column belongs to one wave
  // R_z rows 2p, 2p+1 packed as one complex value, lower half of the transform
  float2 x[E];
#pragma unroll
  for (int r = 0; r < E / 2; ++r) {
    if (2 * G * r < resample_long_rows(M))
      x[r] = make_float2(rz_row<true>(d[2 * r], xf, pf), rz_row<true>(d[2 * r + 1], xf, pf));
    else
      x[r] = make_float2(rz_row<false>(d[2 * r], xf, pf), rz_row<false>(d[2 * r + 1], xf, pf));
  }
  __builtin_amdgcn_wave_barrier();
  tw.load_b(tt.fb, s);
  col_transform_fwd<LOGM, true, 1>(x, slot, tw, tws, twc, s);
  __syncthreads();                                 // every column's LDS is free
  stage_put<LOGM, J>(lds, x, b, s);
  __syncthreads();
  untangle_to_planes<J, NT, LOGM, 1>(lds, tt.tw, spec, nn, col0, tid);
}

template <int LOGM>
__global__ void __launch_bounds__(TGeo<LOGM>::NT, t_waves(LOGM))
k_tfwd_conv(ConvSrc src, ResampleTables S, TwTabs tt, float2* __restrict__ spec, int nn,
            const DevCtl* ctl, size_t zs, int gate) {
  using T = TGeo<LOGM>;
  constexpr int M = 1 << LOGM, G = T::G, E = T::E, J = T::J, NT = T::NT;
  constexpr int ZS = M + M / 8 + 4;               // per-column LDS stride (float2)
  constexpr int LDS2 = (J * ZS > stg_size<J>(M)) ? J * ZS : stg_size<J>(M);
  constexpr bool OLD = !FftCol<LOGM>::PASS;
  __shared__ float2 lds[LDS2];
  __shared__ float2 tws[OLD ? M : 1];
  __shared__ float2 twc[OLD ? M : 1];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  const CtlHead hd = ctl_head(ctl);
  const float* sa = vol_in(src.a, hd, zo);
  const float* sb = vol_in(src.b, hd, zo);
  const float* sc_ = vol_in(src.c, hd, zo);
  if (gated_off(hd, gate)) return;
  S.rows = zsh(S.rows, zo);
  zsh_tw(tt, zo);
  spec = zsh(spec, zo);
  src.w = zsh(src.w, zo);
  src.mask = zsh(src.mask, zo);
  src.scale_div = zsh(src.scale_div, zo);
  const int tid = threadIdx.x, b = tid / G, s = tid % G;
  const int col0 = xcd_block(blockIdx.x, gridDim.x) * J, col = col0 + b;
  // the tables' loads issue with the operands' (one round trip for both);
  // they reach LDS after the operands are loaded
  auto t_tws = table_copy<NT, OLD ? M : 1>(tws, tt.tw);
  auto t_twc = table_copy<NT, OLD ? M : 1>(twc, tt.twc);
  if constexpr (OLD) {
    t_tws.load(tid);
    t_twc.load(tid);
  }

  float ca = 1.f, cb = 0.f;
  if (src.lincache) {
    const double beta = ctl->beta;
    ca = (float)(1.0 + beta);
    cb = (float)(-beta);
  }
  const float sc = src.scale_div ? (float)(1.0 / *src.scale_div) : 1.f;
  const float mk = src.mask ? (float)src.mask[col] : 1.f;
  float* xf = reinterpret_cast<float*>(lds + b * ZS);     // this column's real input
  // every operand is loaded unconditionally (an absent one from a stand-in,
  // a, and replaced by the identity), so all of a lane's loads issue at once:
  // a load under a condition compiles to a branch with a wait after it
  const bool hb = sb != nullptr, hc = sc_ != nullptr, hw = src.w != nullptr;
  const float* pb = hb ? sb : sa;
  const float* pc = hc ? sc_ : sa;
  const float* pw = hw ? src.w : sa;
  float va[E], vb[E], vc[E], vw[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int k = G * r + s;
    const size_t g = (size_t)col * M + k;
    va[r] = sa[g];
    vb[r] = pb[g];
    vc[r] = pc[g];
    vw[r] = pw[k];
  }
  if constexpr (OLD) {
    t_tws.store(tid);
    t_twc.store(tid);
  }
  float xv[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int k = G * r + s;
    float x = ca * va[r];
    x += cb * (hb ? vb[r] : 0.f);
    x -= hc ? vc[r] : 0.f;
    x *= hw ? vw[r] : 1.f;
    xv[r] = x * sc * mk;
    xf[k] = xv[r];
  }
  if constexpr (OLD) __syncthreads();              // the tables
  tfwd_conv_from_lds<LOGM>(lds, tt, tws, twc, S.rows, xv, tid, col0, spec, nn);
}

// A column's inverse transform up to its m real samples g2 (packed pairs) in
// LDS: spectrum from the staging tile, transform, crop.  g2 of column b is at
// lds + b (m/2 + 2).
template <int LOGM>
__device__ __forceinline__ float2* tinv_conv_samples(float2* lds, const FftTw<LOGM>& tw,
                                                     const float2* tws, const float2* twc,
                                                     float scale, int b, int s) {
  using T = TGeo<LOGM>;
  constexpr int M = 1 << LOGM, G = T::G, E = T::E, J = T::J, ZS = M + M / 8 + 4;
  float2 x[E];
  stage_get<LOGM, J>(lds, x, b, s);
  __syncthreads();                                 // staging consumed: the columns' LDS
  col_transform_inv<LOGM, true, 1>(x, lds + b * ZS, tw, tws, twc, s);
  if constexpr (FftCol<LOGM>::PASS) __syncthreads();   // every column's exchanges are done
  float2* g2 = lds + b * (M / 2 + 2);
#pragma unroll
  for (int r = 0; r < E / 2; ++r) g2[G * r + s] = cscale(x[r], scale);
  __builtin_amdgcn_wave_barrier();                 // a column belongs to one wave
  return g2;
}

// t pass, inverse, convolution: planes -> C2R (length 2m) -> crop -> S^T -> epilogue
// (plane 0 holds X_0 + i X_m, as written by the forward pass)
template <int LOGM, int EPI>
__global__ void __launch_bounds__(TGeo<LOGM>::NT, t_waves(LOGM))
k_tinv_conv(const float2* __restrict__ spec, int nn, ResampleTables S, TwTabs tt, ConvEpi ep,
            float scale, const DevCtl* ctl, size_t zs, int gate) {
  using T = TGeo<LOGM>;
  constexpr int M = 1 << LOGM, G = T::G, E = T::E, J = T::J, NT = T::NT;
  constexpr int ZS = M + M / 8 + 4;
  constexpr int LDS2 = (J * ZS > stg_size<J>(M)) ? J * ZS : stg_size<J>(M);
  constexpr bool OLD = !FftCol<LOGM>::PASS;
  __shared__ float2 lds[LDS2];
  __shared__ float2 tws[OLD ? M : 1];
  __shared__ float2 twc[OLD ? M : 1];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  const CtlHead hd = ctl_head(ctl);
  float* eout = vol_out(ep.out, hd, zo);
  const float* eau = (EPI == EPI_FWD_OBJ || EPI == EPI_FWD_DUAL) ? vol_in(ep.au, hd, zo) : nullptr;
  const float* eaup =
      (EPI == EPI_FWD_OBJ || EPI == EPI_FWD_DUAL) ? vol_in(ep.au_prev, hd, zo) : nullptr;
  if (gated_off(hd, gate)) return;
  S.cols = zsh(S.cols, zo);
  zsh_tw(tt, zo);
  spec = zsh(spec, zo);
  ep.w = zsh(ep.w, zo);
  ep.mask = zsh(ep.mask, zo);
  ep.tau0 = zsh(ep.tau0, zo);
  ep.partials = zsh(ep.partials, zo);
  const int tid = threadIdx.x, b = tid / G, s = tid % G;
  const int col0 = xcd_block(blockIdx.x, gridDim.x) * J, col = col0 + b;
  FftTw<LOGM> tw;
  // tables and the block's planes: one round trip
  if constexpr (OLD)
    copy_together(tid, table_copy<NT, M>(tws, tt.tw), table_copy<NT, M>(twc, tt.twc),
                  tangle_copy<J, NT, LOGM, 1>(lds, spec, tt.tw, nn, col0));
  else
    copy_together(tid, tangle_copy<J, NT, LOGM, 1>(lds, spec, tt.tw, nn, col0));
  tw.load_b(tt.fb, s);
  tw.load_a(tt.fa, s);
  __syncthreads();
  const float* g = reinterpret_cast<const float*>(
      tinv_conv_samples<LOGM>(lds, tw, tws, twc, scale, b, s));
  double acc0 = 0.0, acc1 = 0.0;
  float ca = 1.f, cb = 0.f;
  if (EPI == EPI_FWD_OBJ || EPI == EPI_FWD_DUAL) {
    const double beta = ctl->beta;
    ca = (float)(1.0 + beta);
    cb = (float)(-beta);
  }
  const float mk = ep.mask ? (float)ep.mask[col] : 1.f;
  // global operands loaded unconditionally, absent ones from a stand-in (the
  // output column) and replaced by the identity, so the loads issue at once
  const bool hw = ep.w != nullptr;
  const float* pw = hw ? ep.w : eout + (size_t)col * M;
  float vw[E], vau[E], vaup[E], vt0[E];
  float4 sc[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int k = G * r + s;
    const size_t gi = (size_t)col * M + k;
    sc[r] = S.cols[k];
    vw[r] = pw[k];
    if constexpr (EPI == EPI_FWD_OBJ || EPI == EPI_FWD_DUAL) {
      vau[r] = eau[gi];
      vaup[r] = eaup[gi];
    }
    if constexpr (EPI == EPI_FWD_OBJ) vt0[r] = ep.tau0[gi];
  }
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int k = G * r + s;
    float tk = st_taps(sc[r], g);
    tk *= hw ? vw[r] : 1.f;
    const size_t gi = (size_t)col * M + k;
    if (EPI == EPI_PLAIN || EPI == EPI_NORM) {
      tk *= mk;
      eout[gi] = tk;
      if (EPI == EPI_NORM) acc0 += (double)tk * (double)tk;
    } else {
      eout[gi] = tk;
      const float d = tk - (ca * vau[r] + cb * vaup[r]);
      if (EPI == EPI_FWD_OBJ) {
        const float rr = tk - vt0[r];
        const bool kept = mk != 0.f;
        acc0 += kept ? (double)d * (double)d : 0.0;
        acc1 += kept ? (double)rr * (double)rr : 0.0;
      } else {
        acc0 += (double)d * (double)d;
      }
    }
  }
  if (EPI == EPI_NORM) {
    double v[1] = {acc0};
    const int slots[1] = {SL_NORM};
    block_sum_store<1>(v, ep.partials, slots, kMaxBlocks);
  } else if (EPI == EPI_FWD_OBJ) {
    double v[2] = {acc0, acc1};
    const int slots[2] = {SL_CHECK, SL_DATA};
    block_sum_store<2>(v, ep.partials, slots, kMaxBlocks);
  } else if (EPI == EPI_FWD_DUAL) {
    double v[1] = {acc0};
    const int slots[1] = {SL_CHECK};
    block_sum_store<1>(v, ep.partials, slots, kMaxBlocks);
  }
}

// ---------------------------------------------------------------------------
// Plane kernel of the convolution on eight-lane transforms, for n = 8 (where
// four lanes would hold two values each; larger planes: k_plane_conv_quad).
// Rows: 8 lanes per row transform the zero-padded row (length 2n) with the upper
// half of the first stage folded into a twist; the 2n spectrum positions go to
// LDS.  Columns: 8 lanes per spectrum column transform the zero-padded column,
// multiply by H^ (or its conjugate) at the position's frequency, transform back
// and keep the first n rows.  Rows again: inverse, keep the first n.
//
// Block 0 holds the two real planes kt = 0 and kt = m packed as
// Z = P_0 + i P_m.  H^ is real on both (h is even in x and y, and the t phase
// is +-1), and the spectra of the real planes are Hermitian, so the product
// separates with the partner frequency -k (see plane_conv_cols_packed); the
// result is conv(P_0) + i conv(P_m).
// ---------------------------------------------------------------------------
// YS: LDS row stride of the transposes, L + PAD (here and in QuadCfg's kernels).
// The pad changes only where values sit in LDS (bank conflicts of the column
// accesses), never a result; the plan picks it per shape (1, 2 or 4; 2 when
// untuned).
template <int LOGN>
struct PlaneRegCfg {
  static constexpr int N = 1 << LOGN, L = 2 * N, NT = 8 * N;
  static constexpr int RE = L / 8;
};

// forward column transform of a zero-padded column whose first n entries are
// in c[0 .. RE/2): twist (folded first stage), then the remaining DIF stages
template <int LOGN>
__device__ __forceinline__ void col_fwd(float2 (&c)[PlaneRegCfg<LOGN>::RE], int s,
                                        const float2* tws, const float2* twc) {
  constexpr int RE = PlaneRegCfg<LOGN>::RE;
#pragma unroll
  for (int r = 0; r < RE / 2; ++r) c[r + RE / 2] = cmul(c[r], tws[8 * r + s]);
  dif_inlane<8, RE, RE / 4>(c, s, twc);
  dif_xlane<8, RE>(c, s, twc);
}

// inverse column transform, keeping the first n outputs in c[0 .. RE/2)
template <int LOGN>
__device__ __forceinline__ void col_inv(float2 (&c)[PlaneRegCfg<LOGN>::RE], int s,
                                        const float2* tws, const float2* twc) {
  constexpr int RE = PlaneRegCfg<LOGN>::RE;
  dit_xlane<8, RE>(c, s, twc);
  dit_inlane<8, RE, RE / 4>(c, s, twc);
#pragma unroll
  for (int r = 0; r < RE / 2; ++r) c[r] = cadd(c[r], cmulc(c[r + RE / 2], tws[8 * r + s]));
}

// column pass of block 0 (the packed real planes kt = 0 and kt = m).  The
// forward column spectra Z^ of all 2n columns go to LDS (2n rows), then each
// position combines its own value with the partner at (-kx, -ky):
//   Y(k) = Z^(k) (H_0 + H_m)/2 + conj(Z^(-k)) (H_0 - H_m)/2,
// the spectrum of conv(P_0) + i conv(P_m) (H_0, H_m real and even).  Plane 0
// of H^ holds the two factors as one pair (k_hq_pack_real).
// h0: plane 0 of H^ at this lane's positions of its first column, loaded by
// the caller before the column transforms.
template <int LOGN, int PAD>
__device__ __forceinline__ void plane_conv_cols_packed(float2* Y, const float2* Hab,
                                                       const float2 (&h0)[PlaneRegCfg<LOGN>::RE],
                                                       const float2* tws, const float2* twc,
                                                       int tid) {
  using PC = PlaneRegCfg<LOGN>;
  constexpr int N = PC::N, L = PC::L, LOGL = LOGN + 1, RE = PC::RE, YS = L + PAD;
  const int s = tid & 7;
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
    const int col = (tid >> 3) + half * N;
    float2 c[RE];
#pragma unroll
    for (int r = 0; r < RE / 2; ++r) c[r] = Y[(8 * r + s) * YS + col];
    col_fwd<LOGN>(c, s, tws, twc);
#pragma unroll
    for (int r = 0; r < RE; ++r) Y[(8 * r + s) * YS + col] = c[r];
  }
  __syncthreads();
  float2 w[2][RE];
  // the partner of position 8r + s: frequency brev(8r + s) = 16 brev3(s) +
  // brev4(r) (the register part is a constant), negated; the column's once
  const int kxs = brev(s, 3) << (LOGL - 3);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int col = (tid >> 3) + half * N;
    const int colp = brev((L - brev(col, LOGL)) & (L - 1), LOGL);
#pragma unroll
    for (int r = 0; r < RE; ++r) {
      const int p = 8 * r + s;
      const int fx = kxs + brev(r, LOGL - 3);
      const int pp = brev((L - fx) & (L - 1), LOGL);
      const float2 own = Y[p * YS + col], par = Y[pp * YS + colp];
      const float2 ab = half == 0 ? h0[r] : Hab[(r * L + col) * 8 + s];   // lane-ordered H^ plane 0
      w[half][r] = make_float2(ab.x * own.x + ab.y * par.x, ab.x * own.y - ab.y * par.y);
    }
  }
  __syncthreads();                                 // every partner read before write-back
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int col = (tid >> 3) + half * N;
    col_inv<LOGN>(w[half], s, tws, twc);
#pragma unroll
    for (int r = 0; r < RE / 2; ++r) Y[(8 * r + s) * YS + col] = w[half][r];
  }
}

template <int LOGN, bool ADJ, int PAD>
__global__ void __launch_bounds__(PlaneRegCfg<LOGN>::NT)
k_plane_conv_reg(float2* __restrict__ spec, const float2* __restrict__ hq,
                 const float2* __restrict__ tw, const float2* __restrict__ twcg, const DevCtl* ctl,
                 size_t zs, size_t hzs, int gate) {
  using PC = PlaneRegCfg<LOGN>;
  constexpr int N = PC::N, L = PC::L, LOGL = LOGN + 1, NT = PC::NT;
  constexpr int RE = PC::RE, YS = L + PAD;
  // n rows of row spectra; block 0 uses all 2n rows for its column spectra
  __shared__ float2 Y[2 * N * YS];
  __shared__ float2 tws[N];
  __shared__ float2 twc[L];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  if (gated_off(ctl, gate)) return;
  spec = zsh(spec, zo);
  hq = zsh(hq, (size_t)blockIdx.z * hzs);   // 0: one H^ for every scene
  tw = zsh(tw, zo);
  twcg = zsh(twcg, zo);
  const int tid = threadIdx.x, row = tid >> 3, s = tid & 7;
  float2* P = spec + (size_t)blockIdx.x * N * N;
  const float2* Hp = hq + (size_t)blockIdx.x * L * L;     // lane-ordered H^ of this plane
  // the block's rows and both twiddle tables in one round trip (NT >= L >=
  // N: every thread copies the entry of its index modulo the table size, so
  // entries are written more than once, always with their own value)
  float2 x[RE], h0[RE];
#pragma unroll
  for (int r = 0; r < RE / 2; ++r) x[r] = P[row * N + 8 * r + s];
  const float2 tv_s = tw[tid % N];
  const float2 tv_c = twcg[tid % L];
  tws[tid % N] = tv_s;
  twc[tid % L] = tv_c;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RE / 2; ++r) x[r + RE / 2] = cmul(x[r], tws[8 * r + s]);
  dif_inlane<8, RE, RE / 4>(x, s, twc);
  dif_xlane<8, RE>(x, s, twc);
#pragma unroll
  for (int r = 0; r < RE; ++r) Y[row * YS + 8 * r + s] = x[r];
  __syncthreads();
  // H^ at this lane's positions of a spectrum column (a wave's load of
  // register r reads 64 consecutive entries) is loaded before the column's
  // transforms, whose work hides its latency
#pragma unroll
  for (int r = 0; r < RE; ++r) h0[r] = Hp[(r * L + row) * 8 + s];
  if (blockIdx.x == 0) {
    plane_conv_cols_packed<LOGN, PAD>(Y, hq, h0, tws, twc, tid);
  } else {
    // 2n spectrum columns, 8 lanes each, two columns per lane group
    auto column = [&](int col, const float2 (&h)[RE]) {
      float2 c[RE];
#pragma unroll
      for (int r = 0; r < RE / 2; ++r) c[r] = Y[(8 * r + s) * YS + col];
      col_fwd<LOGN>(c, s, tws, twc);
#pragma unroll
      for (int r = 0; r < RE; ++r) c[r] = ADJ ? cmulc(c[r], h[r]) : cmul(c[r], h[r]);
      col_inv<LOGN>(c, s, tws, twc);
#pragma unroll
      for (int r = 0; r < RE / 2; ++r) Y[(8 * r + s) * YS + col] = c[r];
    };
    column(row, h0);
    float2 h1[RE];
#pragma unroll
    for (int r = 0; r < RE; ++r) h1[r] = Hp[(r * L + row + N) * 8 + s];
    column(row + N, h1);
  }
  __syncthreads();
  {
    const int row = tid >> 3, s = tid & 7;
    float2 x[RE];
#pragma unroll
    for (int r = 0; r < RE; ++r) x[r] = Y[row * YS + 8 * r + s];
    dit_xlane<8, RE>(x, s, twc);
    dit_inlane<8, RE, RE / 4>(x, s, twc);
#pragma unroll
    for (int r = 0; r < RE / 2; ++r) x[r] = cadd(x[r], cmulc(x[r + RE / 2], tws[8 * r + s]));
#pragma unroll
    for (int r = 0; r < RE / 2; ++r) P[row * N + 8 * r + s] = x[r];
  }
}

// ---------------------------------------------------------------------------
// Plane kernels of the convolution for n >= 16, on the four-lane transforms of
// fft_quad.h: 16 rows or columns per wave, both zero-padded transforms as two
// halves by the parity of ky and kx.
//
// H^ in memory.  H^ is even in kx and ky.  A lane group takes the columns ky
// and -ky (n <= 64), or the two columns' groups read the same entries (n =
// 128), and -kx sits in the lane of kx, so the table holds the quarter 0 <= kx,
// ky <= n once: [slot][ky pair][lane group], in the order in which a wave's
// loads read 64 consecutive entries, then the column ky = n (n = 16, where -kx
// is in another lane: all kx, [slot] per register).
template <int LOGN>
struct QuadCfg {
  static constexpr int N = 1 << LOGN, L = 2 * N, E = N / 4, NT = 4 * N;
  // kernel values per lane and half, and per plane
  static constexpr int S0 = E == 4 ? 4 : E / 2 + 1, S1 = E == 4 ? 4 : E / 2, SLOTS = S0 + S1;
  static constexpr int PITCH = SLOTS * (4 * N + 4);
  static constexpr int EXTRA = SLOTS * 4 * N;           // the column ky = n: [slot][g]
};
// entries of one kt plane of H^
constexpr int hq_pitch(int logn) {
  return logn == 4   ? QuadCfg<4>::PITCH
         : logn == 5 ? QuadCfg<5>::PITCH
         : logn == 6 ? QuadCfg<6>::PITCH
         : logn == 7 ? QuadCfg<7>::PITCH
                     : 4 << (2 * logn);
}
static_assert(QuadCfg<4>::PITCH <= 4 << 8 && QuadCfg<7>::PITCH <= 4 << 14,
              "a plane of H^ within the 4 n^2 entries that the workspace holds");

// element o of q: a 32-bit offset from a base that is the same for the wave
// (one address register per access instead of two)
__device__ __forceinline__ float2 at32(const float2* __restrict__ q, uint32_t o) {
  return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(q) + (o << 3));
}
__device__ __forceinline__ void put32(float2* __restrict__ q, uint32_t o, float2 v) {
  *reinterpret_cast<float2*>(reinterpret_cast<char*>(q) + (o << 3)) = v;
}
// elements n2 = C of a lane's row part, x[4 i + C], from and to memory (16-byte
// accesses from E = 8 on: the E/4 elements are neighbours, 16-byte aligned)
template <int E>
__device__ __forceinline__ void row_get(float2 (&x)[E], const float2* __restrict__ q, uint32_t p0,
                                        int c) {
  if constexpr (E == 4) {
    x[c] = at32(q, p0 + E * c);
  } else {
#pragma unroll
    for (int i = 0; i < E / 4; i += 2) {
      const float4 v = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(q) +
                                                        ((p0 + E * c + i) << 3));
      x[4 * i + c] = make_float2(v.x, v.y);
      x[4 * i + 4 + c] = make_float2(v.z, v.w);
    }
  }
}
template <int E>
__device__ __forceinline__ void row_put(const float2 (&x)[E], float2* __restrict__ q, uint32_t p0,
                                        int c) {
  if constexpr (E == 4) {
    put32(q, p0 + E * c, x[c]);
  } else {
#pragma unroll
    for (int i = 0; i < E / 4; i += 2) {
      typedef float f4 __attribute__((ext_vector_type(4)));
      const f4 v = {x[4 * i + c].x, x[4 * i + c].y, x[4 * i + 4 + c].x, x[4 * i + 4 + c].y};
      f4* to = reinterpret_cast<f4*>(reinterpret_cast<char*>(q) + ((p0 + E * c + i) << 3));
      // n <= 64: past L2, where the lines would only wait for the t pass that
      // reads them on other XCDs (64x64x512: 24.0 -> 22.6 us; n = 128 reads its
      // first half back: 121 -> 123)
      if constexpr (E < 32) __builtin_nontemporal_store(v, to);
      else *to = v;
    }
  }
}
// this lane's kernel values of half H, from place `first` of the plane on
template <int LOGN, int H>
__device__ __forceinline__ void quad_hq_load(float2 (&hs)[QuadCfg<LOGN>::S0],
                                             const float2* __restrict__ hp, uint32_t first,
                                             uint32_t stride) {
  using QC = QuadCfg<LOGN>;
  constexpr int B = H ? QC::S0 : 0, CNT = H ? QC::S1 : QC::S0;
#pragma unroll
  for (int s = 0; s < CNT; ++s) hs[s] = at32(hp, first + (B + s) * stride);
}
// the value of register (i, k2)
template <int E, int H, int S>
__device__ __forceinline__ float2 quad_hq(const float2 (&hs)[S], int i, int k2, int g) {
  if constexpr (E == 4) {
    return hs[k2];
  } else {
    const int t = 4 * (i >> 1);
    if (H == 1 || t > 0) return hs[t + ((i & 1) ? 3 - k2 : k2)];
    // lane 0: k1 = 0 (i = 0, its k2 = 1 and 3 are negatives) and k1 = E/2
    const bool z = g == 0;
    auto sel = [&](int a, int b) {
      return make_float2(z ? hs[a].x : hs[b].x, z ? hs[a].y : hs[b].y);
    };
    if (i == 0) return k2 == 3 ? sel(1, 3) : hs[k2];
    return k2 == 0 ? hs[3] : k2 == 1 ? sel(S - 1, 2) : k2 == 2 ? sel(S - 1, 1) : sel(3, 0);
  }
}
template <int LOGN, bool ADJ, int H>
__device__ __forceinline__ void quad_product(float2 (&c)[QuadCfg<LOGN>::E],
                                             const float2 (&hs)[QuadCfg<LOGN>::S0], int g) {
  constexpr int E = QuadCfg<LOGN>::E;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const float2 h = quad_hq<E, H>(hs, r >> 2, r & 3, g);
    c[r] = ADJ ? cmulc(c[r], h) : cmul(c[r], h);
  }
}
// Block 0 holds the two real planes kt = 0 and kt = m packed as P_0 + i P_m;
// H^ is real on both, and the product separates with the partner frequency
// (-kx, -ky):  Y(k) = Z(k) (H_0 + H_m)/2 + conj(Z(-k)) (H_0 - H_m)/2, the
// spectrum of conv(P_0) + i conv(P_m).  Plane 0 of H^ holds the two factors as
// one pair (k_hq_pack_real).
__device__ __forceinline__ float2 quad_pair_product(float2 own, float2 par, float2 ab) {
  return make_float2(ab.x * own.x + ab.y * par.x, ab.x * own.y - ab.y * par.y);
}
// place in a column's spectrum (stored at [4 r + g], r = 4 i + k2) of the
// negative of register n of half H
template <int E, int H>
__device__ __forceinline__ int quad_negative(int n, int g) {
  const int i = n >> 2, k2 = n & 3;
  if constexpr (E == 4) {
    if (H) return 4 * (3 - k2) + 3 - g;
    return 4 * (g ? 3 - k2 : (4 - k2) & 3) + ((4 - g) & 3);
  } else {
    const int np = 4 * (i ^ 1) + 3 - k2;
    if (H == 1 || i > 1) return 4 * np + g;
    return 4 * (g ? np : 4 * i + (i ? 3 - k2 : (4 - k2) & 3)) + g;
  }
}

// A lane group's columns of a plane (one, or a column and its negative), in
// place in LDS (element 4 n + g at Yc[4 n YS]): both kx halves forward, product,
// inverse, summed.  The kernel values of a half are read before its transform,
// which hides their latency; the two columns share them unless `apart` (the
// columns 0 and n; the same for a wave).
// PACKED (block 0; every thread of the block takes part): the partner column's
// spectrum half, at Yp, has as many values as that column has places in Y.
template <int LOGN, bool ADJ, int YS, bool PACKED, int NC, typename Fn>
__device__ __forceinline__ void quad_columns(float2* const (&Yc)[NC], const float2* const (&Yp)[NC],
                                             const float2* Hp, const uint32_t (&h0)[NC],
                                             const uint32_t (&hst)[NC], bool apart,
                                             const float2* tw2, int g, Fn before_last) {
  using QC = QuadCfg<LOGN>;
  constexpr int E = QC::E;
  float2 c[PACKED ? NC : 1][E], r[NC][E], in[PACKED ? NC : 1][PACKED ? E : 1];
  if constexpr (PACKED) {
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int n = 0; n < E; ++n) in[k][n] = Yc[k][4 * n * YS];
  }
  auto kx_half = [&](auto hc) {
    constexpr int H = decltype(hc)::value;
    float2 hs[QC::S0];
    if constexpr (!PACKED) {
      quad_hq_load<LOGN, H>(hs, Hp, h0[0], hst[0]);
#pragma unroll
      for (int k = 0; k < NC; ++k) {
#pragma unroll
        for (int n = 0; n < E; ++n) c[0][n] = Yc[k][4 * n * YS];
        if (k > 0 && apart) quad_hq_load<LOGN, H>(hs, Hp, h0[k], hst[k]);
        quad_group_end<E>();
        quad_col_fwd<E, H>(c[0], tw2, g);
        quad_group_end<E>();
        quad_product<LOGN, ADJ, H>(c[0], hs, g);
        if constexpr (H == 1) before_last();
        quad_group_end<E>();
        quad_col_inv<E, H>(c[0], tw2, g);
#pragma unroll
        for (int n = 0; n < E; ++n) r[k][n] = H ? cadd(r[k][n], c[0][n]) : c[0][n];
        quad_group_end<E>();
      }
    } else {
#pragma unroll
      for (int k = 0; k < NC; ++k) {
#pragma unroll
        for (int n = 0; n < E; ++n) c[k][n] = in[k][n];
        quad_col_fwd<E, H>(c[k], tw2, g);
#pragma unroll
        for (int n = 0; n < E; ++n) Yc[k][4 * n * YS] = c[k][n];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        quad_hq_load<LOGN, H>(hs, Hp, h0[k], hst[k]);
#pragma unroll
        for (int n = 0; n < E; ++n)
          c[k][n] = quad_pair_product(c[k][n], Yp[k][quad_negative<E, H>(n, g) * YS],
                                      quad_hq<E, H>(hs, n >> 2, n & 3, g));
      }
      __syncthreads();
      if constexpr (H == 1) before_last();
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        quad_col_inv<E, H>(c[k], tw2, g);
#pragma unroll
        for (int n = 0; n < E; ++n) r[k][n] = H ? cadd(r[k][n], c[k][n]) : c[k][n];
      }
    }
  };
  kx_half(std::integral_constant<int, 0>{});
  kx_half(std::integral_constant<int, 1>{});
#pragma unroll
  for (int k = 0; k < NC; ++k)
#pragma unroll
    for (int n = 0; n < E; ++n) Yc[k][4 * n * YS] = r[k][n];
}

// n <= 64: a block per kt plane, Y [n][2 n] with the even ky first.  Bound by
// vector issue (64x64x512: 77 to 82 % of the SIMDs' busy cycles, 44 to 47 % of each
// wave's; 0.58 of the instructions of the eight-lane form, whose cross-lane stages
// took half).
// SPLIT = 1 (n = 64): 4 n threads; a lane group takes both ky halves of its row
// and the columns ky and -ky.  SPLIT = 2 (n <= 32): 8 n threads; the second half
// of the waves takes the odd ky and the columns -ky, and the two halves of a
// row's sum meet in LDS: twice the waves with half the chain each, for planes
// too small to fill a CU (32x32x256: 7.0 against 8.6 us per pass; at n = 64,
// where two blocks per CU already do, 25.1 against 23.6).
template <int LOGN>
constexpr int quad_split() { return LOGN < 6 ? 2 : 1; }
template <int LOGN, bool ADJ, int PAD>
__global__ void __launch_bounds__(quad_split<LOGN>() * QuadCfg<LOGN>::NT, 2 * quad_split<LOGN>())
k_plane_conv_quad(float2* __restrict__ spec, const float2* __restrict__ hq,
                  const float2* __restrict__ tw, const DevCtl* ctl, size_t zs, size_t hzs,
                  int gate) {
  using QC = QuadCfg<LOGN>;
  constexpr int N = QC::N, L = QC::L, E = QC::E, YS = L + PAD;
  constexpr bool SPLIT = quad_split<LOGN>() == 2;
  __shared__ float2 Y[N * YS];
  __shared__ float2 tw2[L];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  if (gated_off(ctl, gate)) return;
  spec = zsh(spec, zo);
  hq = zsh(hq, (size_t)blockIdx.z * hzs);   // 0: one H^ for every scene
  tw = zsh(tw, zo);
  const int tid = threadIdx.x, j = tid & 15, g = (tid >> 4) & 3;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool second = SPLIT && wv >= N / 16;         // the same for a wave
  const int row = (16 * wv + j) & (N - 1);
  float2* P = spec + (size_t)blockIdx.x * N * N;
  const uint32_t p0 = row * N + (E / 4) * g;
  const float2* Hp = hq + (size_t)blockIdx.x * QC::PITCH;
  // the block's rows and the twiddles in one round trip; W_2N^(t + N) = -W_2N^t
  float2 x[E], v[E];
#pragma unroll
  for (int c = 0; c < 4; ++c) row_get<E>(x, P, p0, c);
  {
    const int t = tid & (L - 1);
    const float2 tv = tw[t & (N - 1)];
    tw2[t] = t < N ? tv : make_float2(-tv.x, -tv.y);
  }
  __syncthreads();
  float2* Yr = Y + row * YS + g;                     // even ky 2 (4 k + g) at Yr[4 k], odd at + N
  if (!second) {
    quad_row_fwd<E, 0>(x, v, tw2, g);
#pragma unroll
    for (int k = 0; k < E; ++k) Yr[4 * k] = v[k];
  }
  if (!SPLIT || second) {
    quad_row_fwd<E, 1>(x, v, tw2, g);
#pragma unroll
    for (int k = 0; k < E; ++k) Yr[N + 4 * k] = v[k];
  }
  __syncthreads();
  // pair `row` of columns: even ky = 2 q with 2 (n - q) (0 with n), odd ky =
  // 2 q + 1 with 2 (n - 1 - q) + 1
  {
    const int odd = row >= N / 2 ? 1 : 0, q = row & (N / 2 - 1);
    const int ca = odd * N + q, cb = odd * N + (odd ? N - 1 - q : (q ? N - q : N / 2));
    const bool self = row == 0;
    const uint32_t ha = tid & (4 * N - 1), hb = self ? QC::EXTRA + g : ha;
    const uint32_t sb = self ? 4 : 4 * N;
    float2* Yg = Y + g * YS;
    if constexpr (SPLIT) {
      float2* const Yc[1] = {Yg + (second ? cb : ca)};
      const float2* const Yp[1] = {Y + (second != self ? ca : cb)};
      const uint32_t h0[1] = {second ? hb : ha}, st[1] = {second ? sb : 4u * N};
      if (blockIdx.x == 0)
        quad_columns<LOGN, ADJ, YS, true, 1>(Yc, Yp, Hp, h0, st, true, tw2, g, [] {});
      else
        quad_columns<LOGN, ADJ, YS, false, 1>(Yc, Yp, Hp, h0, st, true, tw2, g, [] {});
    } else {
      float2* const Yc[2] = {Yg + ca, Yg + cb};
      const float2* const Yp[2] = {Y + (self ? ca : cb), Y + (self ? cb : ca)};
      const uint32_t h0[2] = {ha, hb}, st[2] = {4u * N, sb};
      if (blockIdx.x == 0)
        quad_columns<LOGN, ADJ, YS, true, 2>(Yc, Yp, Hp, h0, st, true, tw2, g, [] {});
      else
        quad_columns<LOGN, ADJ, YS, false, 2>(Yc, Yp, Hp, h0, st, wv == 0, tw2, g, [] {});
    }
  }
  __syncthreads();
  if constexpr (!SPLIT) {
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = Yr[4 * k];
    quad_row_inv<E, 0, false>(v, x, tw2, g);
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = Yr[N + 4 * k];
    quad_row_inv<E, 1, true>(v, x, tw2, g);
#pragma unroll
    for (int c = 0; c < 4; ++c) row_put<E>(x, P, p0, c);
  } else {
    // each half's inverse, then their sum: a lane group gives half of its
    // elements to the other half's group through its own places in Y
    float2* Ym = Yr + (second ? N : 0);
    const float2* Yo = Yr + (second ? 0 : N);
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = Ym[4 * k];
    if (second) quad_row_inv<E, 1, false>(v, x, tw2, g);
    else quad_row_inv<E, 0, false>(v, x, tw2, g);
    auto give = [&](auto sc) {                         // elements n2 = C, C + 1
      constexpr int C = decltype(sc)::value;
#pragma unroll
      for (int c = C; c < C + 2; ++c)
#pragma unroll
        for (int i = 0; i < E / 4; ++i) Ym[4 * (4 * i + c)] = x[4 * i + c];
    };
    auto finish = [&](auto sc) {
      constexpr int C = decltype(sc)::value;
#pragma unroll
      for (int c = C; c < C + 2; ++c) {
#pragma unroll
        for (int i = 0; i < E / 4; ++i) x[4 * i + c] = cadd(x[4 * i + c], Yo[4 * (4 * i + c)]);
        row_put<E>(x, P, p0, c);
      }
    };
    if (second) give(std::integral_constant<int, 0>{});
    else give(std::integral_constant<int, 2>{});
    __syncthreads();
    if (second) finish(std::integral_constant<int, 2>{});
    else finish(std::integral_constant<int, 0>{});
  }
}

// n = 128: the padded plane does not fit LDS, so the ky halves follow one
// another through Y [n][n], and a lane group takes one column; waves 4 to 7
// take the partner columns of waves 0 to 3 and read the same kernel values.
// 128x128x1024: 313 us on eight-lane transforms -> 243 by events, 245 in the trace of
// a reconstruction.  Vector issue takes 65 % of the SIMDs' busy cycles; the rest is
// the latency that two waves per SIMD leave open between barriers that all eight
// meet.  Planes and H^ held in L2 took 222 instead of 237 us (operator alone), so
// memory is the smaller part, although the plane that is read a second time, and H^
// passing through L2 between, make 2.05 times the bytes that the pass cannot do
// without.  14 registers are spilled (52 bytes per lane).
template <int LOGN, bool ADJ, int PAD, bool PACKED>
__device__ __forceinline__ void plane_conv_wide_body(float2* __restrict__ P, const float2* Hp,
                                                     float2* Y, float2* tw2, float2 tv, int tid) {
  using QC = QuadCfg<LOGN>;
  constexpr int N = QC::N, L = QC::L, E = QC::E, YS = N + PAD;
  const int j = tid & 15, g = (tid >> 4) & 3, row = 16 * (tid >> 6) + j;
  const uint32_t p0 = row * N + (E / 4) * g;
  float2 x[E];
  auto load_rows = [&]() {
#pragma unroll
    for (int c = 0; c < 4; ++c) row_get<E>(x, P, p0, c);
  };
  load_rows();
  {
    const int t = tid & (L - 1);
    tw2[t] = t < N ? tv : make_float2(-tv.x, -tv.y);
  }
  __syncthreads();
  float2* Yr = Y + row * YS + g;
  const int q = row & (N / 2 - 1), mem = row >= N / 2 ? 1 : 0;
  // the rows that the next step takes from memory (the odd half's input, then
  // the even half's output) are read before the last column transform, which
  // hides their latency (250 -> 243 us at 128x128x1024)
  auto ky_half = [&](auto yc) {
    constexpr int HY = decltype(yc)::value;
    {
      float2 v[E];
      quad_row_fwd<E, HY>(x, v, tw2, g);
#pragma unroll
      for (int k = 0; k < E; ++k) Yr[4 * k] = v[k];
    }
    __syncthreads();
    // column q, or its partner: n - q (0 with n/2) for even ky, n - 1 - q for odd
    const int partner = HY ? N - 1 - q : (q ? N - q : N / 2);
    float2* const Yc[1] = {Y + g * YS + (mem ? partner : q)};
    const float2* const Yp[1] = {Y + (HY == 0 && q == 0 ? (mem ? N / 2 : 0) : (mem ? q : partner))};
    const bool extra = HY == 0 && mem && q == 0;
    const uint32_t first = extra ? QC::EXTRA + g : HY * 2 * N + (tid & (2 * N - 1));
    const uint32_t h0[1] = {first}, hst[1] = {extra ? 4u : 4u * N};
    quad_columns<LOGN, ADJ, YS, PACKED, 1>(Yc, Yp, Hp, h0, hst, true, tw2, g, load_rows);
    __syncthreads();
  };
  ky_half(std::integral_constant<int, 0>{});
  // x: the odd half's input; the even half's output takes its place in memory
  float2 v[E], o[E];
#pragma unroll
  for (int k = 0; k < E; ++k) v[k] = Yr[4 * k];
  quad_row_inv<E, 0, false>(v, o, tw2, g);
#pragma unroll
  for (int c = 0; c < 4; ++c) row_put<E>(o, P, p0, c);
  __syncthreads();                                 // Y is rewritten by the odd half
  ky_half(std::integral_constant<int, 1>{});
  // x: the even half's output
#pragma unroll
  for (int k = 0; k < E; ++k) v[k] = Yr[4 * k];
  quad_row_inv<E, 1, true>(v, x, tw2, g);
#pragma unroll
  for (int c = 0; c < 4; ++c) row_put<E>(x, P, p0, c);
}

template <int LOGN, bool ADJ, int PAD>
__global__ void __launch_bounds__(QuadCfg<LOGN>::NT, 2)
k_plane_conv_wide(float2* __restrict__ spec, const float2* __restrict__ hq,
                  const float2* __restrict__ tw, const DevCtl* ctl, size_t zs, size_t hzs,
                  int gate) {
  using QC = QuadCfg<LOGN>;
  constexpr int N = QC::N, YS = N + PAD;
  __shared__ float2 Y[N * YS];
  __shared__ float2 tw2[QC::L];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  if (gated_off(ctl, gate)) return;
  spec = zsh(spec, zo);
  hq = zsh(hq, (size_t)blockIdx.z * hzs);   // 0: one H^ for every scene
  tw = zsh(tw, zo);
  const int tid = threadIdx.x;
  float2* P = spec + (size_t)blockIdx.x * N * N;
  const float2* Hp = hq + (size_t)blockIdx.x * QC::PITCH;
  const float2 tv = tw[tid & (N - 1)];
  // block 0: the packed real planes, a separate path so that its register
  // demand does not weigh on the other blocks' code
  if (blockIdx.x == 0) plane_conv_wide_body<LOGN, ADJ, PAD, true>(P, Hp, Y, tw2, tv, tid);
  else plane_conv_wide_body<LOGN, ADJ, PAD, false>(P, Hp, Y, tw2, tv, tid);
}

// Register-resident plane kernel of the diagonal solve (n <= 128): rows and
// columns of length n by LN lanes each (16 at n = 64, so that a block has 16
// waves to hide its phases' latencies; 8 otherwise), divide at the column step.
// YS is the LDS row stride of the transpose, N + PAD (a layout choice only;
// the plan picks 2, 4 or 8 per shape; untuned: 2 at n = 64, 4 at n = 128 and
// 8 otherwise, the fastest of the pads measured by hand).
template <int LOGN, int PAD = (LOGN == 6 ? 2 : LOGN == 7 ? 4 : 8)>
struct PlaneSolveCfg {
  static constexpr int N = 1 << LOGN, LN = LOGN == 6 ? 16 : 8, NT = LN * N, E = N / LN,
                       YS = N + PAD;
};

template <int LOGN, int PAD>
__global__ void __launch_bounds__(PlaneSolveCfg<LOGN>::NT)
k_plane_solve_reg(float2* __restrict__ spec, const float2* __restrict__ twcg,
                  const float* __restrict__ sig_xy, const float* __restrict__ sig_t,
                  const double* c_dev, float c_val, float mu, const DevCtl* ctl, size_t zs,
                  int gate) {
  using PC = PlaneSolveCfg<LOGN, PAD>;
  constexpr int N = PC::N, LN = PC::LN, NT = PC::NT, E = PC::E, YS = PC::YS;
  __shared__ float2 Y[N * YS];
  __shared__ float2 twc[N];
  __shared__ float sg[N];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  if (gated_off(ctl, gate)) return;
  spec = zsh(spec, zo);
  twcg = zsh(twcg, zo);
  sig_xy = zsh(sig_xy, zo);
  sig_t = zsh(sig_t, zo);
  c_dev = zsh(c_dev, zo);
  const int tid = threadIdx.x;
  const int plane = blockIdx.x;
  float2* P = spec + (size_t)plane * N * N;
  const int g = tid / LN, s = tid % LN;
  // the plane's loads issue before the tables' copy waits for its own
  float2 x[E];
#pragma unroll
  for (int r = 0; r < E; ++r) x[r] = P[g * N + LN * r + s];
  for (int i = tid; i < N; i += NT) {
    twc[i] = twcg[i];
    sg[i] = sig_xy[i];
  }
  __syncthreads();
  dif_inlane<LN, E, E / 2>(x, s, twc);
  dif_xlane<LN, E>(x, s, twc);
#pragma unroll
  for (int r = 0; r < E; ++r) Y[g * YS + LN * r + s] = x[r];
  __syncthreads();
  const float c = c_dev ? (float)(*c_dev) : c_val;
  if (plane == 0) {
    // the real planes kt = 0 and kt = m/2, packed as P_0 + i P_{m/2}: separate
    // their row spectra with the partner column -ky, divide each by its own
    // eigenvalue, recombine as Y_0 + i Y_{m/2}
    const int gp = brev((N - brev(g, LOGN)) & (N - 1), LOGN);
    float2 xh[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const float2 a = Y[(LN * r + s) * YS + g];
      const float2 d = Y[(LN * r + s) * YS + gp];
      x[r] = make_float2(0.5f * (a.x + d.x), 0.5f * (a.y - d.y));
      xh[r] = make_float2(0.5f * (a.y + d.y), 0.5f * (d.x - a.x));
    }
    __syncthreads();                               // partners read before any write-back
    dif_inlane<LN, E, E / 2>(x, s, twc);
    dif_xlane<LN, E>(x, s, twc);
    dif_inlane<LN, E, E / 2>(xh, s, twc);
    dif_xlane<LN, E>(xh, s, twc);
    const float base0 = c + mu * (sig_t[0] + sg[brev(g, LOGN)]);
    const float baseh = c + mu * (sig_t[gridDim.x] + sg[brev(g, LOGN)]);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const float sk = mu * sg[brev(LN * r + s, LOGN)];
      const float2 y0 = cscale(x[r], 1.f / (base0 + sk)), yh = cscale(xh[r], 1.f / (baseh + sk));
      x[r] = make_float2(y0.x - yh.y, y0.y + yh.x);
    }
  } else {
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = Y[(LN * r + s) * YS + g];
    dif_inlane<LN, E, E / 2>(x, s, twc);
    dif_xlane<LN, E>(x, s, twc);
    const float base = c + mu * (sig_t[plane] + sg[brev(g, LOGN)]);
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = cscale(x[r], 1.f / (base + mu * sg[brev(LN * r + s, LOGN)]));
  }
  dit_xlane<LN, E>(x, s, twc);
  dit_inlane<LN, E, E / 2>(x, s, twc);
#pragma unroll
  for (int r = 0; r < E; ++r) Y[(LN * r + s) * YS + g] = x[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < E; ++r) x[r] = Y[g * YS + LN * r + s];
  dit_xlane<LN, E>(x, s, twc);
  dit_inlane<LN, E, E / 2>(x, s, twc);
#pragma unroll
  for (int r = 0; r < E; ++r) P[g * N + LN * r + s] = x[r];
}

// ---------------------------------------------------------------------------
// FFT-diagonal solve, eq. (11):  (c I + mu nabla^* nabla) x = rhs, periodic.
// t pass forward (R2C, length m), plane (2-D FFT, divide, inverse), t pass inverse.
// ---------------------------------------------------------------------------
// t pass, forward, diagonal solve: real length m -> complex length m/2 of the
// packed pairs -> untangle -> planes kt = 0 .. m/2 - 1, the two real bins
// kt = 0 and kt = m/2 sharing plane 0 as X_0 + i X_{m/2}.
//
// With SRC != RHS_LOAD the source is the solve's right-hand side, computed
// here per bin (RhsSrc) instead of being read from a stored volume; the u
// solve's instance is the first kernel of an iteration slot
// and clears the previous slot's rejection (G_FIRST).
// p = mu v + Lambda at the two bins k, k + 1 (k even) of one scan column,
// v = shrink(grad xbar - Lambda/mu, phi/mu) as in the v-step (eq. (7)).
// c, cxp, cyp: offsets of the column and of its x + 1 and y + 1 neighbours;
// kn = (k + 2) mod m.  Offsets are per scene and below 2^31.
struct PPair {
  float2 xb;                 // xbar at the two bins
  float px[2], py[2], pt[2];
};

__device__ __forceinline__ PPair p_pair(const float* __restrict__ xb, const float* __restrict__ lam,
                                        const float* __restrict__ phi, float mu, float inv_mu,
                                        uint32_t V, uint32_t c, uint32_t cxp, uint32_t cyp,
                                        uint32_t k, uint32_t kn) {
  PPair r;
  const float2 a = ld2(xb, c + k), ax = ld2(xb, cxp + k), ay = ld2(xb, cyp + k);
  const float an = ld1(xb, c + kn);
  const float2 l0 = ld2(lam, c + k), l1 = ld2(lam, V + c + k), l2 = ld2(lam, 2 * V + c + k);
  const float2 ph = ld2(phi, c + k);
  r.xb = a;
  const float gx[2] = {ax.x - a.x, ax.y - a.y};
  const float gy[2] = {ay.x - a.x, ay.y - a.y};
  const float gt[2] = {a.y - a.x, an - a.y};
  const float lx[2] = {l0.x, l0.y}, ly[2] = {l1.x, l1.y}, lt[2] = {l2.x, l2.y};
  const float pv[2] = {ph.x, ph.y};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float bx = gx[h] - lx[h] * inv_mu;
    const float by = gy[h] - ly[h] * inv_mu;
    const float bt = gt[h] - lt[h] * inv_mu;
    const float sh = shrink_factor(bx * bx + by * by + bt * bt, pv[h] * inv_mu);
    r.px[h] = mu * (bx * sh) + lx[h];
    r.py[h] = mu * (by * sh) + ly[h];
    r.pt[h] = mu * (bt * sh) + lt[h];
  }
  return r;
}

// Right-hand side of a diagonal solve at the bin pairs (2p, 2p + 1),
// p = G r + s, of the block's J scan columns, into x[r] as (rhs_2p, rhs_2p+1):
//   u side:   rhs = L ubar - grad f + nabla^*(mu v + Lambda)             (eqs. (10), (11))
//   tau side: rhs = A u+ + mu3 f + Lambda3 + nabla^*(mu2 w + Lambda2)   (tau-subproblem)
// with nabla^* q = -(backward-difference divergence of q).  Each p = mu v +
// Lambda is formed at the lane's own voxels and at their x - 1 neighbours; the
// y - 1 neighbour's p_y comes from the neighbouring column through LDS (a
// halo column when that column is in another block) and the t - 1
// neighbour's p_t from the previous lane.
// (PL: the pointwise operand of the block's columns is in LDS, gfl [J][m]:
// grad f (RHS_U) instead of rs.gf, A u+ (RHS_TAU) instead of au;
// active: this thread's wave takes part, the others only meet the barrier)
template <int SRC, int G, int E, int J, int M, int NT, bool PL = false>
__device__ __forceinline__ void rhs_pairs(float2 (&x)[E], const RhsSrc& rs, const DevCtl* ctl,
                                          const float* __restrict__ xb,
                                          const float* __restrict__ au, int col0, int b, int s,
                                          int tid, int nn, float* pyl,
                                          const float* gfl = nullptr, bool active = true) {
  const int logn = rs.logn;
  const uint32_t N = 1u << logn, V = (uint32_t)nn * M;
  const float mu = rs.mu, inv_mu = 1.f / mu;
  auto cof = [&](uint32_t i, uint32_t j) { return (((i & (N - 1)) << logn) | (j & (N - 1))) * (uint32_t)M; };
  const uint32_t col = col0 + b, i = col >> logn, j = col & (N - 1);
  const uint32_t c = cof(i, j), cxp = cof(i + 1, j), cyp = cof(i, j + 1);
  const uint32_t cxm = cof(i - 1, j), cxmyp = cof(i - 1, j + 1);
  // p_y of the column before the block's first one (y - 1 of column col0)
  if (J < (int)N) {
    const uint32_t i0 = (uint32_t)col0 >> logn, j0 = col0 & (N - 1);
    const uint32_t ch = cof(i0, j0 - 1), chxp = cof(i0 + 1, j0 - 1), chyp = cof(i0, j0);
    for (int h = tid; h < M / 2; h += NT) {
      const PPair q = p_pair(xb, rs.lam, rs.phi, mu, inv_mu, V, ch, chxp, chyp, 2 * h,
                             (2 * h + 2) & (M - 1));
      pyl[2 * h] = q.py[0];
      pyl[2 * h + 1] = q.py[1];
    }
  }
  // x gets everything but the two neighbour terms that other lanes supply
  float t1[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    if (!active) break;
    const uint32_t k = 2 * (G * r + s), kn = (k + 2) & (M - 1);
    const PPair q = p_pair(xb, rs.lam, rs.phi, mu, inv_mu, V, c, cxp, cyp, k, kn);
    const PPair qm = p_pair(xb, rs.lam, rs.phi, mu, inv_mu, V, cxm, c, cxmyp, k, kn);
    pyl[(b + 1) * M + k] = q.py[0];
    pyl[(b + 1) * M + k + 1] = q.py[1];
    float b0, b1;
    if constexpr (SRC == RHS_U) {
      const float L = (float)ctl->L;
      float2 g;
      if constexpr (PL) g = *reinterpret_cast<const float2*>(gfl + b * M + k);
      else g = ld2(rs.gf, c + k);
      b0 = L * q.xb.x - g.x;
      b1 = L * q.xb.y - g.y;
    } else {
      float2 a;
      if constexpr (PL) a = *reinterpret_cast<const float2*>(gfl + b * M + k);
      else a = ld2(au, c + k);
      const float2 l3 = ld2(rs.lam3, c + k), t0 = ld2(rs.tau0, c + k);
      const bool kept = rs.mask[col] != 0;
      const float ik = 1.f / (rs.lambda + rs.mu3), im = 1.f / rs.mu3;
      const float f0 = f_at(q.xb.x, l3.x, t0.x, kept, rs.lambda, rs.mu3, ik, im);
      const float f1 = f_at(q.xb.y, l3.y, t0.y, kept, rs.lambda, rs.mu3, ik, im);
      b0 = a.x + rs.mu3 * f0 + l3.x;
      b1 = a.y + rs.mu3 * f1 + l3.y;
    }
    x[r].x = b0 - ((q.px[0] - qm.px[0]) + q.py[0] + q.pt[0]);
    x[r].y = b1 - ((q.px[1] - qm.px[1]) + q.py[1] + (q.pt[1] - q.pt[0]));
    t1[r] = q.pt[1];
    // finish every second pair here (no sinking of its arithmetic past the
    // loop): two pairs' loads in flight at a time, without spills
    if ((r & 1) == 1 || r == E - 1) {
      if (r & 1) asm volatile("" : "+v"(x[r - 1].x), "+v"(x[r - 1].y), "+v"(t1[r - 1]));
      asm volatile("" : "+v"(x[r].x), "+v"(x[r].y), "+v"(t1[r]));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // p_t at bin k - 1: the second bin of the previous lane's pair (lane G - 1
  // of the previous r for s = 0; bin m - 1 for k = 0)
  float up[E];
#pragma unroll
  for (int r = 0; r < E; ++r) up[r] = active ? __shfl(t1[r], (s + G - 1) & (G - 1), G) : 0.f;
  __syncthreads();
  if (!active) return;
  // slot of the y - 1 neighbour column: previous column, the same row's last
  // column when the block holds whole rows, else the halo
  const int ym = j > 0 ? b : (J >= (int)N ? b + (int)N : 0);
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int k = 2 * (G * r + s);
    x[r].x += pyl[ym * M + k] + (s > 0 ? up[r] : up[(r + E - 1) % E]);
    x[r].y += pyl[ym * M + k + 1];
  }
}

// Forward t pass of a diagonal solve from the right-hand side in registers
// (x[r] = bins 2p, 2p + 1, p = G r + s): complex transform of length m/2,
// planes kt = 0 .. m/2 - 1 (bins 0 and m/2 packed in plane 0).  J columns per
// block; waves with !act only meet the barriers.
template <int LOGM, int J, int NT>
__device__ __forceinline__ void tfwd_solve_from_regs(float2 (&x)[TGeo<LOGM - 1>::E], bool act,
                                                     float2* lds, const FftTw<LOGM - 1>& tw,
                                                     const TwTabs& tt, const float2* tws,
                                                     const float2* twc, int tid, int col0,
                                                     float2* __restrict__ spec, int nn) {
  using T = TGeo<LOGM - 1>;
  constexpr int M = 1 << LOGM, H = M / 2, LOGH = LOGM - 1;
  constexpr int G = T::G, ZS = H + H / 8 + 4;
  const int b = tid / G, s = tid % G;
  __syncthreads();
  if (act) col_transform_fwd<LOGH, false, 2>(x, lds + b * ZS, tw, tws, twc, s);
  if constexpr (FftCol<LOGH>::PASS) __syncthreads();   // every column's exchanges are done
  if (act) stage_put<LOGH, J>(lds, x, b, s);
  __syncthreads();
  untangle_to_planes<J, NT, LOGH, 2>(lds, tt.tw, spec, nn, col0, tid);
}

template <int LOGM, int SRC>
__global__ void __launch_bounds__(TGeo<LOGM - 1>::NT)
k_tfwd_solve(const float* __restrict__ src, RhsSrc rs, TwTabs tt, float2* __restrict__ spec, int nn,
             DevCtl* ctl, size_t zs, int gate) {
  using T = TGeo<LOGM - 1>;
  constexpr int M = 1 << LOGM, H = M / 2, LOGH = LOGM - 1;
  constexpr int G = T::G, E = T::E, J = T::J, NT = T::NT, ZS = H + H / 8 + 4;
  constexpr int LDS2 = (J * ZS > stg_size<J>(H)) ? J * ZS : stg_size<J>(H);
  constexpr bool OLD = !FftCol<LOGH>::PASS;
  __shared__ float2 lds[LDS2];
  __shared__ float2 twc[OLD ? H : 1];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  const CtlHead hd = ctl_head(ctl);
  const float* xb = SRC != RHS_LOAD ? vol_resolve(rs.xb, hd, zo) : nullptr;
  const float* au = SRC == RHS_TAU ? vol_resolve(rs.au, hd, zo) : nullptr;
  if (gated_off(hd, gate)) return;
  if ((gate & G_FIRST) && blockIdx.x == 0 && threadIdx.x == 0) ctl->reject = 0;
  zsh_tw(tt, zo);
  spec = zsh(spec, zo);
  const int tid = threadIdx.x, b = tid / G, s = tid % G;
  const int col0 = xcd_block(blockIdx.x, gridDim.x) * J, col = col0 + b;
  // the table's loads issue with the operands' (one round trip for both)
  auto t_twc = table_copy<NT, OLD ? H : 1>(twc, tt.twc);
  if constexpr (OLD) t_twc.load(tid);
  float2 x[E];
  if constexpr (SRC == RHS_LOAD) {
    src = zsh(src, zo);
    const float2* src2 = reinterpret_cast<const float2*>(src) + (size_t)col * H;
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = src2[G * r + s];
  } else {
    rs.gf = zsh(rs.gf, zo);
    rs.lam = zsh(rs.lam, zo);
    rs.phi = zsh(rs.phi, zo);
    rs.lam3 = zsh(rs.lam3, zo);
    rs.tau0 = zsh(rs.tau0, zo);
    rs.mask = zsh(rs.mask, zo);
    // p_y of the halo column and of the block's columns: [J + 1][m] floats
    static_assert((J + 1) * M <= 2 * LDS2, "p_y staging does not fit the transform's LDS");
    rhs_pairs<SRC, G, E, J, M, NT>(x, rs, ctl, xb, au, col0, b, s, tid, nn,
                                   reinterpret_cast<float*>(lds));
  }
  if constexpr (OLD) t_twc.store(tid);
  FftTw<LOGH> tw;
  tw.load_a(tt.fa + FftCol<LOGM>::TA, s);
  tw.load_b(tt.fb + FftCol<LOGM>::TB, s);
  tfwd_solve_from_regs<LOGM, J, NT>(x, true, lds, tw, tt, nullptr, twc, tid, col0, spec, nn);
}

// t pass, inverse, diagonal solve: planes kt = 0 .. m/2 - 1 (plane 0 packed
// as above) -> C2R (length m).
template <int LOGM>
__global__ void __launch_bounds__(TGeo<LOGM - 1>::NT)
k_tinv_solve(const float2* __restrict__ spec, int nn, TwTabs tt, SolveEpi ep, float scale,
             const DevCtl* ctl, size_t zs, int gate) {
  using T = TGeo<LOGM - 1>;
  constexpr int M = 1 << LOGM, H = M / 2, LOGH = LOGM - 1;
  constexpr int G = T::G, E = T::E, J = T::J, NT = T::NT, ZS = H + H / 8 + 4;
  constexpr int LDS2 = (J * ZS > stg_size<J>(H)) ? J * ZS : stg_size<J>(H);
  constexpr bool OLD = !FftCol<LOGH>::PASS;
  __shared__ float2 lds[LDS2];
  __shared__ float2 twc[OLD ? H : 1];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  const CtlHead hd = ctl_head(ctl);
  float* eout = vol_out(ep.out, hd, zo);
  const float* eref = vol_in(ep.ref, hd, zo);
  if (gated_off(hd, gate)) return;
  spec = zsh(spec, zo);
  zsh_tw(tt, zo);
  ep.partials = zsh(ep.partials, zo);
  const int tid = threadIdx.x, b = tid / G, s = tid % G;
  const int col0 = xcd_block(blockIdx.x, gridDim.x) * J, col = col0 + b;
  if constexpr (OLD)
    copy_together(tid, table_copy<NT, H>(twc, tt.twc),
                  tangle_copy<J, NT, LOGH, 2>(lds, spec, tt.tw, nn, col0));
  else
    copy_together(tid, tangle_copy<J, NT, LOGH, 2>(lds, spec, tt.tw, nn, col0));
  FftTw<LOGH> tw;
  tw.load_b(tt.fb + FftCol<LOGM>::TB, s);
  tw.load_a(tt.fa + FftCol<LOGM>::TA, s);
  __syncthreads();
  float2 x[E];
  stage_get<LOGH, J>(lds, x, b, s);
  if constexpr (!OLD) __syncthreads();             // staging consumed: the columns' LDS
  col_transform_inv<LOGH, false, 2>(x, lds + b * ZS, tw, nullptr, twc, s);
  float2* out2 = reinterpret_cast<float2*>(eout) + (size_t)col * H;
  if (!eref) {
#pragma unroll
    for (int r = 0; r < E; ++r) out2[G * r + s] = cscale(x[r], scale);
    return;
  }
  // with a reference (the same for the whole launch): its loads issue
  // together, ahead of the stores and the step partial
  const float2* ref2 = reinterpret_cast<const float2*>(eref) + (size_t)col * H;
  float2 rv[E];
#pragma unroll
  for (int r = 0; r < E; ++r) rv[r] = ref2[G * r + s];
  double acc = 0.0;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int p = G * r + s;
    const float2 y = cscale(x[r], scale);
    out2[p] = y;
    const float d0 = y.x - rv[r].x, d1 = y.y - rv[r].y;
    acc += (double)d0 * (double)d0 + (double)d1 * (double)d1;
  }
  double v[1] = {acc};
  const int slots[1] = {SL_STEP};
  block_sum_store<1>(v, ep.partials, slots, kMaxBlocks);
}

// Inverse t pass of A fused with the forward t pass of the A^T that follows it
// in the power iteration: the samples are weighted and masked as A's output and
// again as A^T's input, and stay in LDS.  Bound by HBM and its phases' latencies
// as the two passes are: 17.0 us at 64x64x512 against 10.3 + 10.6 for the two.
template <int LOGM>
__global__ void __launch_bounds__(TGeo<LOGM>::NT, t_waves(LOGM))
k_tinv_conv_fwd(float2* __restrict__ spec, int nn, ResampleTables S, TwTabs tt, ConvEpi ep,
                float scale, const DevCtl* ctl, size_t zs, int gate) {
  using T = TGeo<LOGM>;
  constexpr int M = 1 << LOGM, G = T::G, E = T::E, J = T::J, NT = T::NT;
  constexpr int ZS = M + M / 8 + 4;
  constexpr int LDS2 = (J * ZS > stg_size<J>(M)) ? J * ZS : stg_size<J>(M);
  constexpr bool OLD = !FftCol<LOGM>::PASS;
  __shared__ float2 lds[LDS2];
  __shared__ float2 tws[OLD ? M : 1];
  __shared__ float2 twc[OLD ? M : 1];
  const size_t zo = (size_t)blockIdx.z * zs;
  if (gated_off(zsh(ctl, zo), gate)) return;
  S.rows = zsh(S.rows, zo);
  S.cols = zsh(S.cols, zo);
  zsh_tw(tt, zo);
  spec = zsh(spec, zo);
  ep.w = zsh(ep.w, zo);
  ep.mask = zsh(ep.mask, zo);
  const int tid = threadIdx.x, b = tid / G, s = tid % G;
  const int col0 = xcd_block(blockIdx.x, gridDim.x) * J, col = col0 + b;
  FftTw<LOGM> tw;
  if constexpr (OLD)
    copy_together(tid, table_copy<NT, M>(tws, tt.tw), table_copy<NT, M>(twc, tt.twc),
                  tangle_copy<J, NT, LOGM, 1>(lds, spec, tt.tw, nn, col0));
  else
    copy_together(tid, tangle_copy<J, NT, LOGM, 1>(lds, spec, tt.tw, nn, col0));
  tw.load_b(tt.fb, s);
  tw.load_a(tt.fa, s);
  __syncthreads();
  const float* g = reinterpret_cast<const float*>(
      tinv_conv_samples<LOGM>(lds, tw, tws, twc, scale, b, s));
  const float mk = ep.mask ? (float)ep.mask[col] : 1.f;
  float xv[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const float w = ep.w[G * r + s], t = st_taps(S.cols[G * r + s], g) * w * mk;
    xv[r] = t * w * mk;
  }
  __syncthreads();                                 // every column's samples are read
  float* xf = reinterpret_cast<float*>(lds + b * ZS);
#pragma unroll
  for (int r = 0; r < E; ++r) xf[G * r + s] = xv[r];
  // the forward phase loads its tables anew: kept from the inverse they would spill
  tfwd_conv_from_lds<LOGM>(lds, tt, tws, twc, S.rows, xv, fresh(tid), col0, spec, nn);
}

// Inverse t pass of a convolution fused with the forward t pass of the
// diagonal solve that consumes its output pointwise:
//   EPI_PLAIN:    the adjoint, grad f = A^T (A ubar - tau0) (eq. (10)), into
//                 the u solve's right-hand side (eq. (11)); grad f is not
//                 written to HBM;
//   EPI_FWD_DUAL: the forward operator, A u+ (written, with the backtracking
//                 partial), into the tau solve's right-hand side (Algorithm 2).
// The output of the block's columns stays in LDS, where the right-hand side
// reads it; the right-hand side's neighbour terms come from volumes this
// launch does not change.  Block geometry of the convolution pass; the solve
// phase runs on J x G_s threads (whole waves).  The spectrum buffer is
// reused in place.
template <int LOGM, int EPI>
__global__ void __launch_bounds__(TGeo<LOGM>::NT, t_waves(LOGM))
k_tinv_conv_rhs(float2* __restrict__ spec, int nn, ResampleTables S, TwTabs tt, ConvEpi ep,
                float scale, RhsSrc rs, DevCtl* ctl, size_t zs, int gate) {
  static_assert(EPI == EPI_PLAIN || EPI == EPI_FWD_DUAL, "fused epilogues");
  constexpr int SRC = EPI == EPI_PLAIN ? RHS_U : RHS_TAU;
  using T = TGeo<LOGM>;
  using TS = TGeo<LOGM - 1>;
  constexpr int M = 1 << LOGM, G = T::G, E = T::E, J = T::J, NT = T::NT;
  constexpr int GS = TS::G, ES = TS::E;
  static_assert(J * GS <= NT && (J * GS) % 64 == 0, "solve phase on whole waves");
  constexpr int ZS = M + M / 8 + 4;
  constexpr int LDS2 = (J * ZS > stg_size<J>(M)) ? J * ZS : stg_size<J>(M);
  // LDS as floats: the C2R samples [0, J (m + 4)), the p_y rows of the
  // right-hand side [0, (J + 1) m), grad f at the top [2 LDS2 - J m, 2 LDS2)
  static_assert(2 * LDS2 >= J * (2 * M + 4) && 2 * LDS2 >= (2 * J + 1) * M, "LDS regions");
  constexpr int GFL = 2 * LDS2 - J * M;
  constexpr bool OLD = !FftCol<LOGM>::PASS, OLDS = !FftCol<LOGM - 1>::PASS;
  constexpr int NTWC = OLD ? M : OLDS ? M / 2 : 1;
  __shared__ float2 lds[LDS2];
  __shared__ float2 tws[OLD ? M : 1];
  __shared__ float2 twc[NTWC];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  const CtlHead hd = ctl_head(ctl);
  const float* xb = vol_resolve(rs.xb, hd, zo);
  float* eout = EPI == EPI_FWD_DUAL ? vol_out(ep.out, hd, zo) : nullptr;
  const float* eau = EPI == EPI_FWD_DUAL ? vol_in(ep.au, hd, zo) : nullptr;
  const float* eaup = EPI == EPI_FWD_DUAL ? vol_in(ep.au_prev, hd, zo) : nullptr;
  if (gated_off(hd, gate)) return;
  if ((gate & G_FIRST) && blockIdx.x == 0 && threadIdx.x == 0) ctl->reject = 0;
  S.cols = zsh(S.cols, zo);
  zsh_tw(tt, zo);
  spec = zsh(spec, zo);
  ep.w = zsh(ep.w, zo);
  ep.mask = zsh(ep.mask, zo);
  ep.partials = zsh(ep.partials, zo);
  rs.lam = zsh(rs.lam, zo);
  rs.phi = zsh(rs.phi, zo);
  rs.lam3 = zsh(rs.lam3, zo);
  rs.tau0 = zsh(rs.tau0, zo);
  rs.mask = zsh(rs.mask, zo);
  const int tid = threadIdx.x, b = tid / G, s = tid % G;
  const int col0 = xcd_block(blockIdx.x, gridDim.x) * J, col = col0 + b;
  // tables and the block's planes: one round trip
  if constexpr (OLD)
    copy_together(tid, table_copy<NT, M>(tws, tt.tw), table_copy<NT, NTWC>(twc, tt.twc),
                  tangle_copy<J, NT, LOGM, 1>(lds, spec, tt.tw, nn, col0));
  else if constexpr (OLDS)
    copy_together(tid, table_copy<NT, NTWC>(twc, tt.twc),
                  tangle_copy<J, NT, LOGM, 1>(lds, spec, tt.tw, nn, col0));
  else
    copy_together(tid, tangle_copy<J, NT, LOGM, 1>(lds, spec, tt.tw, nn, col0));
  float* gfl = reinterpret_cast<float*>(lds) + GFL;
  {
    FftTw<LOGM> tw;
    tw.load_b(tt.fb, s);
    tw.load_a(tt.fa, s);
    __syncthreads();
    const float* g = reinterpret_cast<const float*>(
        tinv_conv_samples<LOGM>(lds, tw, tws, twc, scale, b, s));
    const float mk = ep.mask ? (float)ep.mask[col] : 1.f;
    float ca = 1.f, cb = 0.f;
    if constexpr (EPI == EPI_FWD_DUAL) {
      const double beta = ctl->beta;
      ca = (float)(1.0 + beta);
      cb = (float)(-beta);
    }
    double acc0 = 0.0;
    // global operands loaded up front, unconditionally (see k_tinv_conv)
    const bool hw = ep.w != nullptr;
    const float* pw = hw ? ep.w : xb + (size_t)col * M;
    float vw[E], vau[E], vaup[E];
    float4 sc[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int k = G * r + s;
      sc[r] = S.cols[k];
      vw[r] = pw[k];
      if constexpr (EPI == EPI_FWD_DUAL) {
        const size_t gi = (size_t)col * M + k;
        vau[r] = eau[gi];
        vaup[r] = eaup[gi];
      }
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int k = G * r + s;
      float tk = st_taps(sc[r], g);
      tk *= hw ? vw[r] : 1.f;
      if constexpr (EPI == EPI_PLAIN) {
        gfl[b * M + k] = tk * mk;
      } else {
        const size_t gi = (size_t)col * M + k;
        eout[gi] = tk;
        gfl[b * M + k] = tk;
        const float d = tk - (ca * vau[r] + cb * vaup[r]);
        acc0 += (double)d * (double)d;
      }
    }
    if constexpr (EPI == EPI_FWD_DUAL) {
      double v[1] = {acc0};
      const int slots[1] = {SL_CHECK};
      block_sum_store<1>(v, ep.partials, slots, kMaxBlocks);
    }
  }
  __syncthreads();                                 // the output in LDS; the samples are free
  // forward t pass of the u solve with its right-hand side
  const bool sact = tid < J * GS;
  const int bs = tid / GS, ss = tid % GS;
  float2 y[ES];
  rhs_pairs<SRC, GS, ES, J, M, NT, true>(y, rs, ctl, xb, nullptr, col0, bs, ss, tid, nn,
                                         reinterpret_cast<float*>(lds), gfl, sact);
  FftTw<LOGM - 1> tws_;
  tws_.load_a(tt.fa + FftCol<LOGM>::TA, ss);
  tws_.load_b(tt.fb + FftCol<LOGM>::TB, ss);
  tfwd_solve_from_regs<LOGM, J, NT>(y, sact, lds, tws_, tt, tws, twc, tid, col0, spec, nn);
}

// Inverse t pass of the u solve fused with the forward t pass of the
// convolution that follows it (A u+, Algorithms 1 and 2): the solve's real
// output column stays in LDS as the convolution's input, so u+ is not read
// back and one launch is saved.  Both passes work on the same scan columns, so
// the spectrum buffer is reused in place (a block reads its columns' solve
// planes before it writes their convolution planes).  The block has the
// convolution pass's geometry (J columns, NT threads); the solve phase runs on
// J x G_s of them (whole waves).
template <int LOGM>
__global__ void __launch_bounds__(TGeo<LOGM>::NT, t_waves(LOGM))
k_tinv_solve_fwd(float2* __restrict__ spec, int nn, ResampleTables S, TwTabs tt, SolveEpi ep,
                 float scale, const DevCtl* ctl, size_t zs, int gate) {
  using T = TGeo<LOGM>;
  using TS = TGeo<LOGM - 1>;
  constexpr int M = 1 << LOGM, H = M / 2, LOGH = LOGM - 1;
  constexpr int G = T::G, E = T::E, J = T::J, NT = T::NT;
  constexpr int GS = TS::G, ES = TS::E;
  static_assert(J * GS <= NT && (J * GS) % 64 == 0, "solve phase on whole waves");
  constexpr int ZS = M + M / 8 + 4;
  constexpr int LDS2 = (J * ZS > stg_size<J>(M)) ? J * ZS : stg_size<J>(M);
  static_assert(stg_size<J>(H) <= LDS2, "solve staging fits");
  constexpr bool OLD = !FftCol<LOGM>::PASS, OLDS = !FftCol<LOGH>::PASS;
  constexpr int NTWC = OLD ? M : OLDS ? H : 1;
  __shared__ float2 lds[LDS2];
  __shared__ float2 tws[OLD ? M : 1];
  __shared__ float2 twc[NTWC];
  const size_t zo = (size_t)blockIdx.z * zs;
  ctl = zsh(ctl, zo);
  const CtlHead hd = ctl_head(ctl);
  float* eout = vol_out(ep.out, hd, zo);
  const float* eref = vol_in(ep.ref, hd, zo);
  if (gated_off(hd, gate)) return;
  S.rows = zsh(S.rows, zo);
  spec = zsh(spec, zo);
  zsh_tw(tt, zo);
  ep.partials = zsh(ep.partials, zo);
  const int tid = threadIdx.x;
  const int col0 = xcd_block(blockIdx.x, gridDim.x) * J;
  const bool sact = tid < J * GS;
  const int bs = tid / GS, ss = tid % GS;
  // tables and the block's planes: one round trip
  if constexpr (OLD)
    copy_together(tid, table_copy<NT, M>(tws, tt.tw), table_copy<NT, NTWC>(twc, tt.twc),
                  tangle_copy<J, NT, LOGH, 2>(lds, spec, tt.tw, nn, col0));
  else if constexpr (OLDS)
    copy_together(tid, table_copy<NT, NTWC>(twc, tt.twc),
                  tangle_copy<J, NT, LOGH, 2>(lds, spec, tt.tw, nn, col0));
  else
    copy_together(tid, tangle_copy<J, NT, LOGH, 2>(lds, spec, tt.tw, nn, col0));
  FftTw<LOGH> tw;
  tw.load_b(tt.fb + FftCol<LOGM>::TB, ss);
  tw.load_a(tt.fa + FftCol<LOGM>::TA, ss);
  __syncthreads();
  // solve phase: packed real inverse of length m (as k_tinv_solve)
  float2 y[ES];
  if (sact) stage_get<LOGH, J>(lds, y, bs, ss);
  __syncthreads();                                 // staging consumed: the columns' LDS is reused
  double acc = 0.0;
  if (sact) {
    const int col = col0 + bs;
    float2* out2 = reinterpret_cast<float2*>(eout) + (size_t)col * H;
    // the reference is read unconditionally (the output column stands in
    // when there is none), so its loads are not each behind a branch and a wait
    const bool hr = eref != nullptr;
    const float2* ref2 = reinterpret_cast<const float2*>(hr ? eref : eout) + (size_t)col * H;
    float2* xf2 = lds + bs * ZS;                   // the column's real samples, as pairs
    col_transform_inv<LOGH, false, 2>(y, xf2, tw, tws, twc, ss);
    float2 rv[ES];
#pragma unroll
    for (int r = 0; r < ES; ++r) rv[r] = ref2[GS * r + ss];
#pragma unroll
    for (int r = 0; r < ES; ++r) {
      const int p = GS * r + ss;
      const float2 v = cscale(y[r], scale);
      out2[p] = v;
      xf2[p] = v;
      const float d0 = v.x - rv[r].x, d1 = v.y - rv[r].y;
      acc += hr ? (double)d0 * (double)d0 + (double)d1 * (double)d1 : 0.0;
    }
  }
  if (eref) {
    double v[1] = {acc};
    const int slots[1] = {SL_STEP};
    block_sum_store<1>(v, ep.partials, slots, kMaxBlocks);
  }
  __syncthreads();                                 // every column's u+ in LDS
  // convolution phase: R_z, packed transform of length 2m, planes
  const int b = tid / G, s = tid % G;
  const float* xf = reinterpret_cast<const float*>(lds + b * ZS);
  float xv[E];
#pragma unroll
  for (int r = 0; r < E; ++r) xv[r] = xf[G * r + s];
  tfwd_conv_from_lds<LOGM>(lds, tt, tws, twc, S.rows, xv, tid, col0, spec, nn);
}

// exponentials staged in LDS by the H^ setup (2m <= this; 32 KB at most)
constexpr int kHqStagedExp = 2048;
// Stores of the quarter entry (kx, ky), 0 <= kx, ky <= n, of a kt plane where
// the plane kernel reads it.  n >= 16: the table of QuadCfg.  n = 8: the full
// 2n x 2n spectrum in the order the eight-lane kernel multiplies it, frequency
// (fx, fy) at [r][col][s], 8 r + s = brev(fx), col = brev(fy).
template <int LOGN>
__device__ __forceinline__ void hq_store(float2* __restrict__ Hk, int kx, int ky, float2 v) {
  constexpr int N = 1 << LOGN, L = 2 * N;
  if constexpr (LOGN < 4) {
    constexpr int LOGL = LOGN + 1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int fx = (e & 1) ? (L - kx) & (L - 1) : kx;
      const int fy = (e & 2) ? (L - ky) & (L - 1) : ky;
      if (((e & 1) && (kx == 0 || kx == N)) || ((e & 2) && (ky == 0 || ky == N))) continue;
      const int p = brev(fx, LOGL);
      Hk[((p >> 3) * L + brev(fy, LOGL)) * 8 + (p & 7)] = v;
    }
  } else {
    using QC = QuadCfg<LOGN>;
    constexpr int E = QC::E;
    auto put = [&](int slot, int g) {
      if (ky == N) {
        Hk[QC::EXTRA + slot * 4 + g] = v;
      } else {
        const int pair = (ky & 1) * (N / 2) + (ky >> 1);
        Hk[slot * 4 * N + (pair >> 4) * 64 + g * 16 + (pair & 15)] = v;
      }
    };
    const int h = kx & 1, base = h ? QC::S0 : 0;
    if constexpr (E == 4) {
      const int k = kx >> 1, kn = ((h ? N - 1 : N) - k) & (N - 1);
      put(base + k / E, k % E);
      put(base + kn / E, kn % E);
    } else {
      const int k = kx >> 1, k1 = k % E, k2 = k / E;
      const bool low = k1 < E / 2;
      const int a = low ? k1 : (h ? E - 1 - k1 : E - k1);
      if (h == 0 && k1 == E / 2) put(k2 == 0 ? 3 : E / 2, 0);
      else put(base + 4 * (a / 4) + (low ? k2 : 3 - k2), a % 4);
    }
  }
}

// ---------------------------------------------------------------------------
// H^ setup: the kernel h of eq. (3) is even in dx and dy, so its padded
// spectrum is a real cosine sum in (kx, ky) and a complex exponential in kt:
//   H^[kt][kx][ky] = (1/Z) sum_{dx,dy >= 0} c_dx c_dy cos(pi kx dx / n)
//                    cos(pi ky dy / n) exp(-pi i kt dq(dx,dy) / m),
// c_0 = 1, c_d = 2.  One block per (kt, chunk of ky); FP64 accumulation; the
// inner dy sum is staged in LDS.  Computed for kx, ky in [0, n] (the
// quarter) and stored by hq_store.
// cos(pi (n - k) d / n) = (-1)^d cos(pi k d / n): the sums over even and over
// odd d give the frequencies k and n - k together, so a block takes KP pairs of
// ky, and a thread R pairs at a time, which share the exponential and its
// lookups (then one pair of kx and four ky, which share the cosine).  Bound by
// its LDS reads: one frequency per sum and thread took 247 us at 64x64x512 and
// 5.74 ms at 128x128x1024; now 74 us and 0.88 ms.
// The kernel offsets dq (n <= 64) and, with ET, the exponential table
// exp(-pi i j / m), j < 2m (dynamic LDS, 2m entries), are staged in LDS; 2m is
// a power of two, so the phase index kt q mod 2m is a mask (kt q < 2^31 for
// m <= 2^15).  Offsets outside the cone (dq < 0) enter with weight 0, so the
// sums run branch-free and unrolled (their loads issue together).  dq is laid out
// in LDS with the lane index fastest ([dy][dx]).
// ---------------------------------------------------------------------------
template <int LOGN>
struct HqCfg {
  static constexpr int N = 1 << LOGN, P = N / 2 + 1;     // pairs (k, n - k), k = 0 .. n/2
  static constexpr int KP = P < 11 ? P : 11, R = 3, NG = (KP + R - 1) / R;
  static constexpr int CH = (P + KP - 1) / KP;           // blocks per plane
  static constexpr int KYS = 4 * ((2 * NG * R + 3) / 4); // row stride of the inner sums
};

template <int LOGN, bool ET>
__global__ void __launch_bounds__(256)
k_build_hq(float2* __restrict__ hq, int m, const int* __restrict__ dq,
           const double2* __restrict__ etab, const double* __restrict__ cosn, double invZ) {
  using HC = HqCfg<LOGN>;
  constexpr int N = HC::N, P = HC::P, KP = HC::KP, R = HC::R, NG = HC::NG, KYS = HC::KYS;
  constexpr bool DQ = N <= 64;
  __shared__ double2 G[N * KYS];                   // [dx][pair, then the partners]
  __shared__ double cs[2 * N];
  __shared__ int dq_l[DQ ? N * N : 1];
  extern __shared__ double2 et_l[];
  const int kt = blockIdx.x, kp0 = blockIdx.y * KP, tid = threadIdx.x;
  const int pmask = 2 * m - 1;
  for (int i = tid; i < 2 * N; i += blockDim.x) cs[i] = cosn[i];
  if constexpr (DQ) {
    for (int i = tid; i < N * N; i += blockDim.x) dq_l[(i % N) * N + i / N] = dq[i];
  }
  if constexpr (ET) {
    for (int i = tid; i < 2 * m; i += blockDim.x) et_l[i] = etab[i];
  }
  const double2* ets = ET ? et_l : etab;
  __syncthreads();
  // inner sum over dy for this block's pairs (those beyond n/2 are not stored)
  for (int it = tid; it < NG * N; it += blockDim.x) {
    const int grp = it / N, dx = it % N, k0 = kp0 + grp * R;
    double2 s[R][2] = {};
    int at[R] = {};
#pragma unroll 2
    for (int dy = 0; dy < N; dy += 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int q = DQ ? dq_l[(dy + h) * N + dx] : dq[dx * N + dy + h];
        const bool in = q >= 0;
        const double2 e = ets[(kt * (in ? q : 0)) & pmask];
        const double w = in ? (dy + h ? 2.0 : 1.0) : 0.0, er = w * e.x, ei = w * e.y;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double c = cs[at[r]];
          s[r][h].x = fma(c, er, s[r][h].x);
          s[r][h].y = fma(c, ei, s[r][h].y);
          at[r] = (at[r] + k0 + r) & (2 * N - 1);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int c = dx * KYS + grp * R + r;
      G[c] = make_double2(s[r][0].x + s[r][1].x, s[r][0].y + s[r][1].y);
      G[c + NG * R] = make_double2(s[r][0].x - s[r][1].x, s[r][0].y - s[r][1].y);
    }
  }
  __syncthreads();
  // outer sum over dx: columns c of G, four at a time
  for (int it = tid; it < P * (KYS / 4); it += blockDim.x) {
    const int grp = it / P, kp = it % P;
    double2 a[4][2] = {};
    int at = 0;
#pragma unroll 2
    for (int dx = 0; dx < N; dx += 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double c = (dx + h ? 2.0 : 1.0) * cs[at];
        at = (at + kp) & (2 * N - 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double2 g = G[(dx + h) * KYS + 4 * grp + r];
          a[r][h].x = fma(c, g.x, a[r][h].x);
          a[r][h].y = fma(c, g.y, a[r][h].y);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = 4 * grp + r, kq = c < NG * R ? c : c - NG * R, kl = kp0 + kq;
      if (c >= 2 * NG * R || kq >= KP || kl > N / 2) continue;
      const int ky = c < NG * R ? kl : N - kl;
      if (c >= NG * R && ky == kl) continue;               // n/2 is its own partner
      float2* Hk = hq + (size_t)kt * hq_pitch(LOGN);
      hq_store<LOGN>(Hk, kp, ky, make_float2((float)((a[r][0].x + a[r][1].x) * invZ),
                                             (float)((a[r][0].y + a[r][1].y) * invZ)));
      if (kp < N / 2)
        hq_store<LOGN>(Hk, N - kp, ky, make_float2((float)((a[r][0].x - a[r][1].x) * invZ),
                                                   (float)((a[r][0].y - a[r][1].y) * invZ)));
    }
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// blocks of the t passes (their partial sums are indexed by block)
int conv_blocks(int logn, int logm) { return (1 << (2 * logn)) / t_columns(logm); }
// tables of the passes' lane twiddles (fft_column.h) for a time axis of 2^logm
// bins: the convolution's transform, then the solve's.  tw: exp(-pi i j / m), j < m,
// which holds every root that they need (a sine and a cosine per entry instead took
// 36 us of a problem's creation at 1024 bins).
void column_twiddles(int logm, const std::vector<float2>& tw, std::vector<float2>& fa,
                     std::vector<float2>& fb) {
  const int m = 1 << logm;
  fa.clear();
  fb.clear();
  auto w = [&](int num, int den) {                 // exp(-2 pi i num / den), den divides 2 m
    const int j = (num * (2 * m / den)) & (2 * m - 1);
    return j < m ? tw[j] : make_float2(-tw[j - m].x, -tw[j - m].y);
  };
  for (int logf : {logm, logm - 1}) {
    if (logf < 8 || logf > 10) continue;
    const int F = 1 << logf, E = F / 64, low = E == 8 ? 7 : E == 4 ? 15 : 3;
    for (int k = 1; k < E; ++k)
      for (int l = 0; l < 64; ++l) {
        fa.push_back(w(l * k, F));
        fb.push_back(w((l & low) * k, 64));
      }
    if (E == 4)
      for (int j = 0; j < 16; ++j) fb.push_back(w(j, 16));
  }
}

int solve_blocks(int logn, int logm) { return (1 << (2 * logn)) / t_columns(logm - 1); }
int fused_solve_blocks(int logn, int logm) { return conv_blocks(logn, logm); }

#define CNLOS_TIMED(prof, kind, st, launch)                 \
  do {                                                     \
    const bool t_ = (prof) != nullptr && (prof)->on(kind); \
    if (t_) (void)(prof)->begin(kind, st);                 \
    launch;                                                \
    if (t_) (void)(prof)->end(kind, st);                   \
  } while (0)

// plane pass of a convolution with row pad PAD
template <int LOGN, int PAD>
static void plane_conv_pad(bool adjoint, int M, const Tables& tb, float2* spec, const DevCtl* ctl,
                           size_t zs, size_t hzs, int g, int nz, hipStream_t st) {
#define CNLOS_PCONV(K, NT_, ...)                                                                \
  hipLaunchKernelGGL((K), dim3(M, 1, nz), dim3(NT_), 0, st, spec, tb.hq, tb.tw_xy, __VA_ARGS__ ctl, \
                     zs, hzs, g)
#define CNLOS_COMMA ,
  if constexpr (LOGN < 4) {
    if (adjoint) CNLOS_PCONV(k_plane_conv_reg<LOGN CNLOS_COMMA true CNLOS_COMMA PAD>, PlaneRegCfg<LOGN>::NT, tb.twc_xy CNLOS_COMMA);
    else CNLOS_PCONV(k_plane_conv_reg<LOGN CNLOS_COMMA false CNLOS_COMMA PAD>, PlaneRegCfg<LOGN>::NT, tb.twc_xy CNLOS_COMMA);
  } else if constexpr (LOGN <= 6) {
    if (adjoint) CNLOS_PCONV(k_plane_conv_quad<LOGN CNLOS_COMMA true CNLOS_COMMA PAD>, quad_split<LOGN>() * QuadCfg<LOGN>::NT, );
    else CNLOS_PCONV(k_plane_conv_quad<LOGN CNLOS_COMMA false CNLOS_COMMA PAD>, quad_split<LOGN>() * QuadCfg<LOGN>::NT, );
  } else {
    if (adjoint) CNLOS_PCONV(k_plane_conv_wide<LOGN CNLOS_COMMA true CNLOS_COMMA PAD>, QuadCfg<LOGN>::NT, );
    else CNLOS_PCONV(k_plane_conv_wide<LOGN CNLOS_COMMA false CNLOS_COMMA PAD>, QuadCfg<LOGN>::NT, );
  }
#undef CNLOS_PCONV
#undef CNLOS_COMMA
}

template <int LOGN>
static void plane_conv(bool adjoint, int M, const Tables& tb, float2* spec, const DevCtl* ctl,
                       size_t zs, size_t hzs, int g, int nz, hipStream_t st) {
  switch (tb.plan.conv_pad) {
    case 1: plane_conv_pad<LOGN, 1>(adjoint, M, tb, spec, ctl, zs, hzs, g, nz, st); break;
    case 4: plane_conv_pad<LOGN, 4>(adjoint, M, tb, spec, ctl, zs, hzs, g, nz, st); break;
    default: plane_conv_pad<LOGN, 2>(adjoint, M, tb, spec, ctl, zs, hzs, g, nz, st); break;
  }
}

// plane pass of a diagonal solve with the plan's row pad
template <int LOGN>
static void plane_solve(int M, const Tables& tb, float2* spec, const double* c_dev, float c_val,
                        float mu, const DevCtl* ctl, size_t zs, int g, int nz, hipStream_t st) {
  const int pad = tb.plan.solve_pad > 0 ? tb.plan.solve_pad : default_solve_pad(LOGN);
#define CNLOS_PSOLVE(P)                                                                         \
  hipLaunchKernelGGL((k_plane_solve_reg<LOGN, P>), dim3(M / 2, 1, nz),                          \
                     dim3(PlaneSolveCfg<LOGN, P>::NT), 0, st, spec, tb.twc_xy, tb.sig_xy, tb.sig_t, \
                     c_dev, c_val, mu, ctl, zs, g)
  switch (pad) {
    case 2: CNLOS_PSOLVE(2); break;
    case 4: CNLOS_PSOLVE(4); break;
    default: CNLOS_PSOLVE(8); break;
  }
#undef CNLOS_PSOLVE
}

template <int LOGN, int LOGM>
static hipError_t conv_impl(const Tables& tb, const ConvSrc& src, float2* spec, bool adjoint,
                            int epi, const ConvEpi& ep, const DevCtl* ctl, const Batch& bt,
                            hipStream_t st, Prof* prof, bool tfwd_done, const RhsSrc* rhs_next) {
  constexpr int N = 1 << LOGN, M = 1 << LOGM, NN = N * N;
  const TwTabs tt{tb.tw_t, tb.twc_t, tb.fa, tb.fb};
  using TG = TGeo<LOGM>;
  const int nb = NN / TG::J;
  const int nz = bt.nz, g = bt.gate;
  const size_t zs = bt.zs, hzs = bt.hq_shared ? 0 : zs;
  if (!tfwd_done)
    CNLOS_TIMED(prof, KK_T_FWD_CONV, st,
                hipLaunchKernelGGL((k_tfwd_conv<LOGM>), dim3(nb, 1, nz), dim3(TG::NT), 0, st,
                                   src, tb.S, tt, spec, NN, ctl, zs, g));
  CNLOS_TIMED(prof, KK_PLANE_CONV, st, plane_conv<LOGN>(adjoint, M, tb, spec, ctl, zs, hzs, g, nz, st));
  const float scale = (float)(1.0 / (4.0 * (double)NN * (double)M));
  if (rhs_next) {
    if (epi == EPI_FWD_DUAL)
      CNLOS_TIMED(prof, KK_T_INV_CONV, st,
                  hipLaunchKernelGGL((k_tinv_conv_rhs<LOGM, EPI_FWD_DUAL>), dim3(nb, 1, nz),
                                     dim3(TG::NT), 0, st, spec, NN, tb.S, tt, ep,
                                     scale, *rhs_next, const_cast<DevCtl*>(ctl), zs, g));
    else if (epi == EPI_PLAIN)
      CNLOS_TIMED(prof, KK_T_INV_CONV, st,
                  hipLaunchKernelGGL((k_tinv_conv_rhs<LOGM, EPI_PLAIN>), dim3(nb, 1, nz),
                                     dim3(TG::NT), 0, st, spec, NN, tb.S, tt, ep,
                                     scale, *rhs_next, const_cast<DevCtl*>(ctl), zs, g));
    else
      return hipErrorInvalidValue;
    return hipGetLastError();
  }
#define CNLOS_TINV(E)                                                                         \
  CNLOS_TIMED(prof, KK_T_INV_CONV, st,                                                        \
              hipLaunchKernelGGL((k_tinv_conv<LOGM, E>), dim3(nb, 1, nz), dim3(TG::NT), 0, \
                                 st, spec, NN, tb.S, tt, ep, scale, ctl, zs, g))
  switch (epi) {
    case EPI_PLAIN: CNLOS_TINV(EPI_PLAIN); break;
    case EPI_FWD_OBJ: CNLOS_TINV(EPI_FWD_OBJ); break;
    case EPI_FWD_DUAL: CNLOS_TINV(EPI_FWD_DUAL); break;
    case EPI_NORMAL:
      CNLOS_TIMED(prof, KK_T_INV_CONV, st,
                  hipLaunchKernelGGL((k_tinv_conv_fwd<LOGM>), dim3(nb, 1, nz), dim3(TG::NT), 0, st,
                                     spec, NN, tb.S, tt, ep, scale, ctl, zs, g));
      break;
    default: CNLOS_TINV(EPI_NORM); break;
  }
#undef CNLOS_TINV
  return hipGetLastError();
}

template <int LOGN, int LOGM>
static hipError_t solve_impl(const Tables& tb, const float* rhs, const RhsSrc& rs, float2* spec,
                             const double* c_dev, double c_val, double mu, const SolveEpi& ep,
                             const DevCtl* ctl, const Batch& bt, hipStream_t st, Prof* prof,
                             bool fwd_next, bool tfwd_done) {
  constexpr int N = 1 << LOGN, M = 1 << LOGM, NN = N * N;
  using TG = TGeo<LOGM - 1>;
  const int nb = NN / TG::J;
  const int nz = bt.nz, g = bt.gate;
  const size_t zs = bt.zs;
  DevCtl* c = const_cast<DevCtl*>(ctl);
  const TwTabs tt{tb.tw_t, tb.twc_t, tb.fa, tb.fb};
  if (!tfwd_done) {
    switch (rs.mode) {
      case RHS_U:
        CNLOS_TIMED(prof, KK_T_FWD_SOLVE, st,
                    hipLaunchKernelGGL((k_tfwd_solve<LOGM, RHS_U>), dim3(nb, 1, nz), dim3(TG::NT), 0,
                                       st, rhs, rs, tt, spec, NN, c, zs, g));
        break;
      case RHS_TAU:
        CNLOS_TIMED(prof, KK_T_FWD_SOLVE, st,
                    hipLaunchKernelGGL((k_tfwd_solve<LOGM, RHS_TAU>), dim3(nb, 1, nz), dim3(TG::NT), 0,
                                       st, rhs, rs, tt, spec, NN, c, zs, g));
        break;
      default:
        CNLOS_TIMED(prof, KK_T_FWD_SOLVE, st,
                    hipLaunchKernelGGL((k_tfwd_solve<LOGM, RHS_LOAD>), dim3(nb, 1, nz), dim3(TG::NT),
                                       0, st, rhs, rs, tt, spec, NN, c, zs, g));
        break;
    }
  }
  CNLOS_TIMED(prof, KK_PLANE_SOLVE, st,
              plane_solve<LOGN>(M, tb, spec, c_dev, (float)c_val, (float)mu, ctl, zs, g, nz, st));
  const float scale = (float)(2.0 / ((double)NN * (double)M));
  if (fwd_next) {
    // with the forward t pass of the convolution of the result
    using TC = TGeo<LOGM>;
    CNLOS_TIMED(prof, KK_T_INV_SOLVE, st,
                hipLaunchKernelGGL((k_tinv_solve_fwd<LOGM>), dim3(NN / TC::J, 1, nz),
                                   dim3(TC::NT), 0, st, spec, NN, tb.S, tt, ep,
                                   scale, ctl, zs, g));
  } else {
    CNLOS_TIMED(prof, KK_T_INV_SOLVE, st,
                hipLaunchKernelGGL(k_tinv_solve<LOGM>, dim3(nb, 1, nz), dim3(TG::NT), 0, st, spec,
                                   NN, tt, ep, scale, ctl, zs, g));
  }
  return hipGetLastError();
}

#define CNLOS_DISPATCH_M(LOGN, FN, ...)                                  \
  switch (logm) {                                                        \
    case 4: return FN<LOGN, 4>(__VA_ARGS__);                             \
    case 5: return FN<LOGN, 5>(__VA_ARGS__);                             \
    case 6: return FN<LOGN, 6>(__VA_ARGS__);                             \
    case 7: return FN<LOGN, 7>(__VA_ARGS__);                             \
    case 8: return FN<LOGN, 8>(__VA_ARGS__);                             \
    case 9: return FN<LOGN, 9>(__VA_ARGS__);                             \
    case 10: return FN<LOGN, 10>(__VA_ARGS__);                           \
    case 11: return FN<LOGN, 11>(__VA_ARGS__);                           \
    default: return hipErrorInvalidValue;                                \
  }

#define CNLOS_DISPATCH_NM(FN, ...)                                       \
  switch (logn) {                                                        \
    case 3: CNLOS_DISPATCH_M(3, FN, __VA_ARGS__)                         \
    case 4: CNLOS_DISPATCH_M(4, FN, __VA_ARGS__)                         \
    case 5: CNLOS_DISPATCH_M(5, FN, __VA_ARGS__)                         \
    case 6: CNLOS_DISPATCH_M(6, FN, __VA_ARGS__)                         \
    case 7: CNLOS_DISPATCH_M(7, FN, __VA_ARGS__)                         \
    default: return hipErrorInvalidValue;                                \
  }

hipError_t launch_conv(int logn, int logm, const Tables& tb, const ConvSrc& src, float2* spec,
                       bool adjoint, int epi, const ConvEpi& ep, const DevCtl* ctl,
                       const Batch& bt, hipStream_t st, Prof* prof, bool tfwd_done,
                       const RhsSrc* rhs_next) {
  CNLOS_DISPATCH_NM(conv_impl, tb, src, spec, adjoint, epi, ep, ctl, bt, st, prof, tfwd_done,
                    rhs_next)
}

hipError_t launch_solve(int logn, int logm, const Tables& tb, const float* rhs, const RhsSrc& rs,
                        float2* spec, const double* c_dev, double c_val, double mu,
                        const SolveEpi& ep, const DevCtl* ctl, const Batch& bt, hipStream_t st,
                        Prof* prof, bool fwd_next, bool tfwd_done) {
  CNLOS_DISPATCH_NM(solve_impl, tb, rhs, rs, spec, c_dev, c_val, mu, ep, ctl, bt, st, prof,
                    fwd_next, tfwd_done)
}

// The real planes kt = 0 and kt = m are transformed together (packed as
// P_0 + i P_m), and the product with H^ separates into (H_0 + H_m)/2 times the
// value plus (H_0 - H_m)/2 times the partner's conjugate (both H^ planes are
// real).  Plane 0 of H^ therefore holds that pair of real factors,
// ((H_0 + H_m)/2, (H_0 - H_m)/2), one load per position; plane m is not read.
__global__ void __launch_bounds__(256) k_hq_pack_real(float2* __restrict__ hq, int m, int plane) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= plane) return;
  const float h0 = hq[q].x, hm = hq[(size_t)m * plane + q].x;
  hq[q] = make_float2(0.5f * (h0 + hm), 0.5f * (h0 - hm));
}

hipError_t launch_build_hq(int logn, int logm, float2* hq, const int* dq, const double2* etab,
                           const double* cosn, double invZ, hipStream_t st) {
  const int m = 1 << logm;
  const bool et = 2 * m <= kHqStagedExp;
#define CNLOS_HQ(LN)                                                                           \
  case LN:                                                                                     \
    if (et)                                                                                    \
      hipLaunchKernelGGL((k_build_hq<LN, true>), dim3(m + 1, HqCfg<LN>::CH), dim3(256),         \
                         2 * m * sizeof(double2), st, hq, m, dq, etab, cosn, invZ);            \
    else                                                                                       \
      hipLaunchKernelGGL((k_build_hq<LN, false>), dim3(m + 1, HqCfg<LN>::CH), dim3(256), 0, st, \
                         hq, m, dq, etab, cosn, invZ);                                         \
    break;
  switch (logn) {
    CNLOS_HQ(3)
    CNLOS_HQ(4)
    CNLOS_HQ(5)
    CNLOS_HQ(6)
    CNLOS_HQ(7)
    default: return hipErrorInvalidValue;
  }
#undef CNLOS_HQ
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int plane = hq_pitch(logn);
  hipLaunchKernelGGL(k_hq_pack_real, dim3((plane + 255) / 256), dim3(256), 0, st, hq, m, plane);
  return hipGetLastError();
}

}  // namespace cnlos

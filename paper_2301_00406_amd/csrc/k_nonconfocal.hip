// Non-confocal forward model (Section 2's general model, one illumination
// point and a scanned detector grid) applied by direct summation, and its
// transpose.
//
// With the wall normals along z the direction terms reduce, as in the
// confocal case, to the volumetric albedo weight 1 / (d_i^2 d_d^2), where d_i
// is the distance from the illuminated wall point to the voxel and d_d from
// the voxel to the detector; the path d_i + d_d selects the time bin.  The
// model is not shift-invariant (every detector sees every voxel along its own
// ellipsoids), so it has no FFT form: one application evaluates n^4 m paths.
//
// Grid conventions (the confocal ones): detector and voxel column (i, j) at
// x_i = (i + 1/2) W / n - W / 2, depth bin k at z_k = (k + 1/2) R / m with
// R = m c dt / 2, and time bin b holding path lengths in [b, b + 1) c dt.
//
// The time bin is an integer that floating point decides, so it is computed
// in FP64 and decided as the operations written here in order (no contraction
// into fused multiply-adds) decide it; the weight and the sums are FP64 as
// well, and only the stored results are FP32.  Both kernels are deterministic:
// every histogram bin and every voxel is summed in a fixed order.
//
// What bounds them: FP64 vector instructions.  Written plainly, a path costs
// two correctly rounded square roots and two correctly rounded divisions (each
// a dozen dependent FP64 instructions).  Here it costs one reciprocal square
// root r of d_d^2 (v_rsq_f64 and one third-order step: full FP64 accuracy),
// since d_d = d_d^2 r and 1 / d_d^2 = r^2, and a product with 1 / (c dt) instead
// of the bin's division.  That product can fall on the other side of a whole
// number only when it is within a few rounding errors of one: such paths
// (kNearBin; one in 5 10^7) take the plain form, so every bin is the one
// that the plain form gives.
#include "cnlos_internal.h"

namespace cnlos {

namespace {

constexpr int kNcMaxWaves = 8;       // waves per block of the forward kernel
constexpr int kNcMaxGridDev = 256;   // detectors per side (the host checks it)

struct NcPath {
  int bin;      // time bin, m when the path leaves the window
  double w;     // albedo weight (1 when not literal)
};

__device__ __forceinline__ double nc_lateral(const NcGeo& g, int i) {
#pragma clang fp contract(off)
  return ((i + 0.5) * g.wall) / g.n - g.wall / 2.0;
}
__device__ __forceinline__ double nc_depth(const NcGeo& g, int k) {
#pragma clang fp contract(off)
  return ((k + 0.5) * g.range) / g.m;
}

// path of the detector at (xd, yd) through voxel (xv, yv, z), where the
// illumination distance di of the voxel is already known
__device__ __forceinline__ NcPath nc_path(const NcGeo& g, double xd, double yd, double xv,
                                          double yv, double z, double di) {
#pragma clang fp contract(off)
  const double ex = xv - xd, ey = yv - yd;
  const double dd = sqrt((ex * ex + ey * ey) + z * z);
  const double len = di + dd;
  const double fb = floor(len / g.cdt);
  NcPath r;
  r.bin = fb < (double)g.m ? (int)fb : g.m;
  r.w = g.literal ? 1.0 / (((di * di) * dd) * dd) : 1.0;
  return r;
}

__device__ __forceinline__ double nc_illum_dist(const NcGeo& g, double xv, double yv, double z) {
#pragma clang fp contract(off)
  const double ex = xv - g.ix, ey = yv - g.iy;
  return sqrt((ex * ex + ey * ey) + z * z);
}

// 1 / sqrt(x) to FP64 accuracy for x in [1e-120, 1e120] (NcGeo::plain is set
// when a geometry could leave that range): v_rsq_f64 is good to about 2^-24,
// the third-order step leaves an error of order 2^-70 before rounding
__device__ __forceinline__ double nc_rsqrt(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double h = fma(-(x * r), r, 1.0);
  return fma(r * h, fma(0.375, h, 0.5), r);
}

// z for the body of a rarely taken branch.  The compiler counts a square root
// or a division as one operation: it would compute the body for every path,
// or lift a root out of two such bodies (64x64x512, when the branch was made: 30.9
// and 14.8 ms with one and two detectors per block, 13.8 and 12.4 without); a
// value that it cannot see through keeps them where they are.
__device__ __forceinline__ double nc_in_branch(double z) {
  asm volatile("" : "+v"(z));
  return z;
}

// distance to a whole number below which the bin is decided by nc_path: the
// error of the fast quotient is below 8 roundings of at most 1024
constexpr double kNearBin = 1e-8;

// A path from its squared detector distance d2 = (ex^2 + ey^2) + z^2 and the
// voxel's illumination distance less half a bin, dh = d_i - c dt / 2: the bin
// (not limited to the window), and 1 / d_d^2.
struct NcFast {
  int bin;
  bool near;    // decide the bin with nc_path
  double r2;
};
__device__ __forceinline__ NcFast nc_fast(double d2, double dh, double inv_cdt) {
  const double r = nc_rsqrt(d2);
  const double len = fma(d2, r, dh);
  // the whole number nearest to the quotient less 1/2, through the addition of
  // 1.5 2^52 (the quotient is below 2^30, see nc_in_range): its low word is the bin
  const double t = fma(len, inv_cdt, 6755399441055744.0);
  const double off = fma(len, inv_cdt, 6755399441055744.0 - t);   // [-1/2, 1/2]
  NcFast f;
  f.bin = __double2loint(t);
  f.near = fabs(off) > 0.5 - kNearBin;
  f.r2 = r * r;
  return f;
}

// sum into one bin of a histogram that only this wave writes; the callers
// never let two lanes of an instruction name the same bin, so the order of a
// bin's terms is the program's (no return value: the wave does not wait)
__device__ __forceinline__ void nc_bin_add(double* h, double v) {
  (void)__hip_atomic_fetch_add(h, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Place of bin b in a histogram.  Lanes are S depths apart, so their bins are up
// to S apart: a pad every 8 bins keeps such strides off shared banks.
__host__ __device__ constexpr int nc_place(int b) { return b + (b >> 3); }
constexpr int kNcRow = 72;   // LDS row of u by [j][lane] (the pad spreads the transposed stores)

// Steps of 64 depths that a column needs: with more depth every path to the
// detectors leaves the window.  d_i + d_d = P = m c dt puts d_i at
// (P + (lat_i - lat_d) / P) / 2; two depths more than that are kept.
__device__ __forceinline__ int nc_steps(const NcGeo& g, double lat_i, double lat_d, int S) {
  const double P = g.m * g.cdt, di = 0.5 * (P + (lat_i - lat_d) / P);
  const double z2 = di > 0.0 && di < P ? fmax(di * di - lat_i, 0.0) : 0.0;
  const double k = fmin(sqrt(z2) * (g.m / g.range), (double)g.m);
  return min(S, ((int)k + 2 + 63) >> 6);
}

// tau[det][b] = sum over voxels with path bin b of w u.  One block per D
// detectors; wave w takes the columns w, w + W, ... in order, and lane l
// the s consecutive depths from s l on (s = ceil(m / 64), or fewer where the
// deeper paths leave the window), so that
//   - the illumination distance and u of a voxel serve D detectors;
//   - a lane's bins never decrease from one depth to the next (the path grows
//     with the depth): a lane sums a run of equal bins in a register and adds
//     it to its wave's histogram when the bin changes;
//   - two lanes never add to one bin in the same step: if lane l's run ends at
//     step j, a lane above it whose bin is the same has not reached a new bin
//     either, since all its depths are larger.  Only the runs left at the end
//     of a column can meet; they are added in lane order.
// Depths from m on need no test: their paths are longer than the window.
// A column's u is read coalesced (SM >= S loads, the next column's while this
// one is summed) and handed to the lanes through LDS: read in place, at a
// stride of S floats, the columns of a CU's waves overrun its L1 (64x64x512,
// one detector per block, when it was made: 15.0 against 13.8 ms).
// Consecutive depths in consecutive lanes, with a segmented scan over equal
// bins per 64 paths (18 lane exchanges through the LDS pipe), and the plain path
// arithmetic took 42.6 ms at 64x64x512 and 1.59 ms at 32x32x256; now 10.5
// and 0.39 ms, issuing vector instructions in about three quarters of the cycles.
// Leaving out the depths beyond the window is worth 229 -> 120 us where paths are
// long for it (24x24x224, 1.5 m wall, 12 ps bins) and nothing where all fit.
template <int D, bool LIT, int SM>
__global__ void __launch_bounds__(64 * kNcMaxWaves)
k_nc_forward(NcGeo g, const float* __restrict__ u, float* __restrict__ tau) {
  // histograms [W][M][D], then u [W][S + 1][kNcRow]; the last row is read ahead only
  extern __shared__ double nc_lds[];
  __shared__ double xs[kNcMaxGridDev];
  const int m = g.m, n = g.n, S = (m + 63) >> 6, nt = blockDim.x, W = nt >> 6;
  const int M = nc_place(m);                   // places of one histogram
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int b = threadIdx.x; b < W * D * M; b += nt) nc_lds[b] = 0.0;
  for (int i = threadIdx.x; i < n; i += nt) xs[i] = nc_lateral(g, i);
  __syncthreads();
  float* ub = reinterpret_cast<float*>(nc_lds + W * D * M) + wv * (S + 1) * kNcRow;
  float nu[SM];
  auto load_column = [&](int col) {
    const float* uc = u + (size_t)col * m;
#pragma unroll
    for (int i = 0; i < SM; ++i) nu[i] = uc[min(64 * i + lane, m - 1)];
  };
  if (wv < n * n) load_column(wv);
  double xd[D], yd[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const int det = min((int)blockIdx.x * D + d, n * n - 1);
    xd[d] = xs[det / n];
    yd[d] = xs[det % n];
  }
  const double inv_cdt = 1.0 / g.cdt, dz = g.range / m;
  double* h = nc_lds + wv * D * M;
  int place[SM];
  int s = 0, steps = S, c = 0;
  for (int col = wv; col < n * n; col += W, ++c) {
    if ((c & 63) == 0 && !g.plain) {
      // lane l: the steps of the wave's l-th column from here on
      const int cl = min(col + lane * W, n * n - 1);
      const double xv = xs[cl / n], yv = xs[cl % n];
      const double ex = xv - g.ix, ey = yv - g.iy;
      steps = 0;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const double fx = xv - xd[d], fy = yv - yd[d];
        steps = max(steps, nc_steps(g, ex * ex + ey * ey, fx * fx + fy * fy, S));
      }
    }
    const int sc = __builtin_amdgcn_readlane(steps, c & 63);
    if (sc != s) {
      // this lane's depths 64 i + lane in the order they are read from memory,
      // and their places by [j][lane]: k = s l + j (k s' >> 16 = k / s for k < 1024)
      s = sc;
      const int inv_s = (65536 + s - 1) / s;
#pragma unroll
      for (int i = 0; i < SM; ++i) {
        const int k = min(64 * i + lane, 64 * s - 1), l = (k * inv_s) >> 16;
        place[i] = (k - l * s) * kNcRow + l;
      }
    }
    const double xv = xs[col / n], yv = xs[col % n];
    double lat_i, lat_d[D];
    {
#pragma clang fp contract(off)
      const double ex = xv - g.ix, ey = yv - g.iy;
      lat_i = ex * ex + ey * ey;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const double fx = xv - xd[d], fy = yv - yd[d];
        lat_d[d] = fx * fx + fy * fy;
      }
    }
    // only this wave's lanes touch ub, and a wave's LDS accesses are in order
#pragma unroll
    for (int i = 0; i < SM; ++i)
      if (i < s) ub[place[i]] = nu[i];
    if (col + W < n * n) load_column(col + W);
    __builtin_amdgcn_wave_barrier();
    int cur[D];
    double acc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      cur[d] = m;
      acc[d] = 0.0;
    }
    double kd = s * lane + 0.5;
    float uf = ub[lane];
    for (int j = 0; j < s; ++j) {
      // the next step's operand is read before this one's arithmetic
      const float un = ub[(j + 1) * kNcRow + lane];
      const double uv = (double)uf, z = kd * dz, zz = z * z;
      const double d2i = lat_i + zz, ri = nc_rsqrt(d2i);
      const double dh = fma(d2i, ri, -0.5 * g.cdt);
      double wu = LIT ? uv * (ri * ri) : uv;
      NcFast f[D];
      bool near = g.plain != 0;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        f[d] = nc_fast(lat_d[d] + zz, dh, inv_cdt);
        near |= f[d].near;
      }
      if (near) {
        const int k = s * lane + j;
        const double zp = nc_in_branch(nc_depth(g, k));
        const double dp = nc_illum_dist(g, xv, yv, zp);
        if (g.plain) wu = uv;
#pragma unroll
        for (int d = 0; d < D; ++d) {
          const NcPath r = nc_path(g, xd[d], yd[d], xv, yv, zp, dp);
          f[d].bin = k < m ? r.bin : m;
          if (g.plain) f[d].r2 = r.w;
        }
      }
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (j == 0) cur[d] = f[d].bin;
        // a lane whose bin has left the window has nothing more to add
        if (f[d].bin != cur[d] && cur[d] < m) {
          nc_bin_add(h + nc_place(cur[d]) * D + d, acc[d]);
          cur[d] = f[d].bin;
          acc[d] = 0.0;
        }
        acc[d] = LIT ? fma(wu, f[d].r2, acc[d]) : acc[d] + wu;
      }
      kd += 1.0;
      uf = un;
    }
    __builtin_amdgcn_wave_barrier();
    // the runs left: lanes whose run continues their predecessor's add after it
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int prev = __shfl_up(cur[d], 1, 64);
      unsigned long long same = __ballot(lane > 0 && prev == cur[d] && cur[d] < m);
      unsigned long long todo = __ballot(cur[d] < m);
      while (todo) {                             // at most 64 rounds: `same` loses a lane each
        const unsigned long long now = todo & ~same;
        if ((now >> lane) & 1) nc_bin_add(h + nc_place(cur[d]) * D + d, acc[d]);
        todo &= same;
        same &= same << 1;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const int det = blockIdx.x * D + d;
    if (det >= n * n) break;
    for (int b = threadIdx.x; b < m; b += nt) {
      double sum = 0.0;
      for (int w = 0; w < W; ++w) sum += nc_lds[(w * M + nc_place(b)) * D + d];
      tau[(size_t)det * m + b] = (float)sum;
    }
  }
}

// u[p][q][k] = sum over detectors (in index order) of w tau[det][bin].  A wave
// takes 64 depths of one column, so the squared lateral distances to the
// detector rows and columns are tables in LDS that the wave reads as
// broadcasts, and a path's squared distance is two additions.  Detectors beyond
// the reach of the wave's shallowest depth are left out, row by row.  Bound by FP64
// issue: 45x45x300 2.60 -> 1.05 ms, 24x24x224 with a 1.5 m wall 0.14 -> 0.075.
constexpr int kNcTWaves = 4;
template <bool LIT>
__global__ void __launch_bounds__(64 * kNcTWaves)
k_nc_transpose(NcGeo g, const float* __restrict__ tau, float* __restrict__ u) {
  extern __shared__ double nc_lds[];            // [kNcTWaves][2][n]: squared offsets in x, in y
  const int m = g.m, n = g.n;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int nchunk = (m + 63) >> 6, items = n * n * nchunk;
  const int item = min((int)blockIdx.x * kNcTWaves + wv, items - 1);
  const int col = item / nchunk, k0 = (item - col * nchunk) * 64;
  const double xv = nc_lateral(g, col / n), yv = nc_lateral(g, col % n);
  double* lx = nc_lds + wv * (2 * n + 1);
  double* ly = lx + n;
  // one offset more, of a detector that no path reaches within the window
  const double far = m * g.cdt;
  for (int i = lane; i < n + 1; i += 64) {
#pragma clang fp contract(off)
    const double x = nc_lateral(g, i), ex = xv - x, ey = yv - x;
    if (i < n) lx[i] = ex * ex;
    ly[i] = i < n ? ey * ey : far * far;
  }
  __syncthreads();
  const int k = min(k0 + lane, m - 1);
  const double z = nc_depth(g, k);
  const double di = nc_illum_dist(g, xv, yv, z);
  double zz;
  {
#pragma clang fp contract(off)
    zz = z * z;
  }
  const double inv_cdt = 1.0 / g.cdt, dh = di - 0.5 * g.cdt;
  // squared lateral distance beyond which the paths of the first, shallowest
  // depth leave the window, and so all the wave's do
  const double z0 = nc_depth(g, k0), reach = far - nc_illum_dist(g, xv, yv, z0);
  const double lat = (reach > 0.0 ? reach * reach - z0 * z0 : -1.0) + 1e-9 * far * far;
  const double per = n / g.wall, jv = (yv / g.wall + 0.5) * n - 0.5;
  double acc = 0.0;
  for (int i = 0; i < n; ++i) {
    const double x2 = lx[i];
    // the detectors of the row within reach, and one on either side
    const double rem = lat - x2, w = sqrt(fmax(rem, 0.0)) * per;
    const int ja = __builtin_amdgcn_readfirstlane(max(0, (int)fmax(jv - w, 0.0) - 1));
    const int jb = __builtin_amdgcn_readfirstlane(
        rem < 0.0 ? 0 : min(n, (int)fmin(jv + w, (double)n) + 2));
    // four detectors at a time: their loads are unconditional (bin clamped into
    // the column, value masked) and issue together, and one branch serves the
    // rare bins of all four
    for (int j0 = ja; j0 < jb; j0 += 4) {
      NcFast f[4];
      const float* td[4];       // in scalar registers
      bool near = false;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        td[q] = tau + (size_t)__builtin_amdgcn_readfirstlane((i * n + min(j0 + q, n - 1)) * m);
        f[q] = nc_fast((x2 + ly[min(j0 + q, n)]) + zz, dh, inv_cdt);
        near |= f[q].near;
      }
      if (near) {
        const double zp = nc_in_branch(z);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const NcPath r = nc_path(g, nc_lateral(g, i), nc_lateral(g, min(j0 + q, n - 1)), xv, yv, zp, di);
          f[q].bin = j0 + q < n ? r.bin : m;
        }
      }
      float t[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        t[q] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(td[q]) +
                                               ((uint32_t)min(f[q].bin, m - 1) << 2));
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double tq = f[q].bin < m ? t[q] : 0.f;
        acc = LIT ? fma(f[q].r2, tq, acc) : acc + tq;
      }
    }
  }
  if (LIT) {
    const double ri = 1.0 / di;
    acc *= ri * ri;
  }
  if (k0 + lane < m && (int)blockIdx.x * kNcTWaves + wv < items) u[(size_t)col * m + k] = (float)acc;
}

// The same sum with a voxel per thread and the plain path: for geometries beyond
// the fast path's range, and for large grids with few bins (launch_nc_transpose).
__global__ void __launch_bounds__(256)
k_nc_transpose_plain(NcGeo g, const float* __restrict__ tau, float* __restrict__ u) {
  __shared__ double xs[kNcMaxGridDev];
  const int m = g.m, n = g.n;
  for (int i = threadIdx.x; i < n; i += 256) xs[i] = nc_lateral(g, i);
  __syncthreads();
  const size_t V = (size_t)n * n * m;
  const size_t vox = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (vox >= V) return;
  const int col = (int)(vox / m), k = (int)(vox - (size_t)col * m);
  const double xv = xs[col / n], yv = xs[col % n], z = nc_depth(g, k);
  const double di = nc_illum_dist(g, xv, yv, z);
  double acc = 0.0;
  for (int i = 0; i < n; ++i) {
    const double xd = xs[i];
    // loads are unconditional (bin clamped into the column, term masked), so
    // the unrolled iterations' loads issue together
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
      const NcPath r = nc_path(g, xd, xs[j], xv, yv, z, di);
      const int b = r.bin < m ? r.bin : m - 1;
      const float t = tau[(size_t)(i * n + j) * m + b];
      acc += r.bin < m ? r.w * (double)t : 0.0;
    }
  }
  u[vox] = (float)acc;
}

}  // namespace

// Histograms and columns of the forward kernel: at most 60 KiB with the counts
// of waves and detectors that launch_nc_forward takes.
static size_t nc_forward_lds_bytes(int m, int d, int waves) {
  const size_t s = (m + 63) / 64;
  return (size_t)waves * d * nc_place(m) * sizeof(double) + waves * (s + 1) * kNcRow * sizeof(float);
}

// Squared distances outside [1e-120, 1e120], and paths of 2^30 bins, are left
// to the plain form.
static bool nc_in_range(const NcGeo& g) {
  const double zmin = 0.5 * g.range / g.m;
  const double far = fabs(g.wall) + fabs(g.ix) + fabs(g.iy) + g.range;
  return zmin > 1e-60 && far < 1e59 && g.cdt > 1e-60 && 4.0 * far / g.cdt < 1e9;
}

hipError_t launch_nc_forward(const NcGeo& g0, const float* u, float* tau, hipStream_t st) {
  NcGeo g = g0;
  g.plain = nc_in_range(g) ? 0 : 1;
  // Two detectors per block share a voxel's illumination path, but their
  // histograms leave room for half the waves.  Measured, one against two
  // detectors with the better count of waves each: 16x16x128 37 / 50 us, 24x24x224
  // 216 / 218, 28x28x256 376 / 299, 32x32x256 494 / 390, 45x45x300 2240 / 1701,
  // 64x64x512 12.5 / 10.5 ms, 32x32x576 1168 / 912 us, 40x40x600 3.00 / 2.86 ms,
  // 40x40x1000 5.31 / 6.36 ms.  The line is the one of an earlier form of the
  // kernel (at 24x24x224 two were 10 % slower there): from n = 24 to 31 at 256 bins
  // and from 513 to about 600 bins it now leaves up to a fifth.  Eight waves while
  // two blocks of them find room on a CU, with registers for both, else four:
  // eight against four, 24x24x512 (one detector) 369 / 406 us, 33x33x320 (two)
  // 712 / 787; 24x24x560 569 / 472, 64x64x512 (two) 13.1 / 10.5 ms.
  const bool two = g.n >= 32 && g.m <= 512;
  const int waves = nc_forward_lds_bytes(g.m, two ? 2 : 1, 8) <= 60 * 1024 ? 8 : 4;
  const int nd = g.n * g.n;
  const int S = (g.m + 63) / 64;
#define CNLOS_NCF(D, LIT, SM)                                                              \
  hipLaunchKernelGGL((k_nc_forward<D, LIT, SM>), dim3((nd + D - 1) / D), dim3(64 * waves), \
                     nc_forward_lds_bytes(g.m, D, waves), st, g, u, tau)
#define CNLOS_NCF_S(D, LIT)                                                                \
  do {                                                                                     \
    if (S <= 2) CNLOS_NCF(D, LIT, 2);                                                      \
    else if (S <= 4) CNLOS_NCF(D, LIT, 4);                                                 \
    else if (S <= 8) CNLOS_NCF(D, LIT, 8);                                                 \
    else CNLOS_NCF(D, LIT, 16);                                                            \
  } while (0)
  if (two && g.literal) CNLOS_NCF_S(2, true);
  else if (two) CNLOS_NCF_S(2, false);
  else if (g.literal) CNLOS_NCF_S(1, true);
  else CNLOS_NCF_S(1, false);
#undef CNLOS_NCF_S
#undef CNLOS_NCF
  return hipGetLastError();
}

hipError_t launch_nc_transpose(const NcGeo& g, const float* tau, float* u, hipStream_t st) {
  // A wave of k_nc_transpose takes one column whatever its depths, a thread of the
  // plain form one voxel at 2.8 times the cost of a path.  With up to 64 x 64
  // columns the waves of the first fit the chip at once, so idle lanes cost nothing
  // (64x64x16: 931 us and 932 with the plain form); beyond, with few depths, the
  // plain form is faster: 100x100x8 3.29 against 4.89 ms, 128x128x8 5.25 / 12.3,
  // 128x128x20 11.3 / 12.3, 256x256x1 14.5 / 186; 128x128x24 13.3 / 12.3.
  if (!nc_in_range(g) || (g.n > 64 && g.m < 24)) {
    const size_t V = (size_t)g.n * g.n * g.m;
    hipLaunchKernelGGL(k_nc_transpose_plain, dim3((unsigned)((V + 255) / 256)), dim3(256), 0, st, g,
                       tau, u);
    return hipGetLastError();
  }
  const int items = g.n * g.n * ((g.m + 63) / 64);
  const dim3 grid((items + kNcTWaves - 1) / kNcTWaves), block(64 * kNcTWaves);
  const size_t lds = (size_t)kNcTWaves * (2 * g.n + 1) * sizeof(double);
  if (g.literal) hipLaunchKernelGGL(k_nc_transpose<true>, grid, block, lds, st, g, tau, u);
  else hipLaunchKernelGGL(k_nc_transpose<false>, grid, block, lds, st, g, tau, u);
  return hipGetLastError();
}

}  // namespace cnlos

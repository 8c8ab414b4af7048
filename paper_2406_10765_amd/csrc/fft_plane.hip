// Fused plane pass with compile-time sizes: for one z plane of one band, inverse 2D FFT of
// the stick data, multiplication by V(r), forward 2D FFT, gather of the stick positions.
//
// Each 1D FFT of length N = A * B is done in two register stages with one LDS exchange:
//   n = B n1 + n2:  Y[n2][k1] = W_N^{s n2 k1} * sum_n1 x[B n1 + n2] W_A^{s n1 k1}     (stage 1)
//                   X[k1 + A k2] = sum_n2 Y[n2][k1] W_B^{s n2 k2}                      (stage 2)
// (s = +1 inverse, -1 forward; W_M = exp(2 pi i / M)).  T = gcd(A, B) threads share a line:
// thread t takes n2 = t + T i in stage 1 and k1 = t + T j in stage 2.
// Along x the inverse transform, the V(r) multiplication and the forward transform run back to
// back: after the inverse stage 2 a thread holds y[m1 + A m2] for its m1 and every m2, which is
// exactly the input of the forward split m = m1 + A m2, q = B q1 + q2:
//   Z[m1][q2] = W_N^{-m1 q2} sum_m2 y[m1 + A m2] W_B^{-m2 q2}                        (in registers)
//   F[B q1 + q2] = sum_m1 Z[m1][q2] W_A^{-m1 q1}                                       (after one exchange)
// The small DFTs are fully unrolled with compile-time twiddles.

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "fft_small.hpp"
#include "kernels.hpp"

namespace pw {



// ---- N x N planes in LDS with wave-local lines -----------------------------------------------------
// The TT = gcd(A, B) threads of a line sit in one wave, which orders the exchange between the two
// register stages by itself; three workgroup barriers per plane:
//   y inverse   lines = active columns xa = n1 + n1max, read straight from the sticks (zeros off a stick's
//               n2 range), exchanged in place in the plane's columns
//   x           every wave keeps one group of LPW rows: inverse, * V, forward, exchanged in place in the row
//   y forward   back into the sticks
// The plane holds the active columns only, with row pitch R; BX and AX are the pitches of the in-row
// exchange words (k1 BX + n2 and q2 AX + m1).  TT threads share a line (gcd(A, B), or 8 for 96, whose
// 24 elements per thread would leave one wave per SIMD).  R, BX and AX are those with the fewest LDS bank
// conflicts over the passes' accesses, by enumeration; 64 in FP32 (R = 64) swizzles columns and exchange
// words instead and has none.  WPE: waves per SIMD the compiler must reach, set where the natural register
// count would cost a workgroup per CU.  LOOP: a workgroup takes one z plane of several bands in turn, so that
// its rows of V stay in the first cache.  V is read where it is used: held in registers across the plane
// it cost a wave per SIMD.
// Bound by the issue of the butterflies and LDS accesses; sticks and barriers of one workgroup wait under
// the others of the compute unit.  Per band of H X (us), before with a workgroup barrier per exchange and
// zeroing, scatter and gather of the whole plane, and now:
//   FP32  54^2 0.83 -> 0.60 (144 bands), 64^2 0.88 -> 0.71, 81^2 2.20 -> 1.51, 96^2 4.14 -> 3.81 (440 bands),
//         108^2 7.76 (pencil form) -> 6.18
//   FP64  54^2 1.40 -> 1.05, 64^2 1.65 -> 1.15, 81^2 5.28 -> 2.95 (128 bands), 96^2 10.3 -> 8.0
// of which leaving out the empty blocks (grid_empty) and the products with quarter turns gives 5 to 10%.
template <typename T, int N> struct PlanePitch;
template <> struct PlanePitch<float, 24> { static constexpr int TT = 2, R = 30, BX = 7, AX = 5, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<float, 27> { static constexpr int TT = 3, R = 27, BX = 9, AX = 3, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<float, 32> { static constexpr int TT = 4, R = 37, BX = 8, AX = 4, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<float, 48> { static constexpr int TT = 4, R = 60, BX = 13, AX = 5, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<float, 54> { static constexpr int TT = 3, R = 54, BX = 9, AX = 6, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<float, 64> { static constexpr int TT = 8, R = 64, BX = 8, AX = 8, WPE = 4, LOOP = 1; };
template <> struct PlanePitch<float, 81> { static constexpr int TT = 9, R = 81, BX = 9, AX = 9, WPE = 6, LOOP = 0; };
template <> struct PlanePitch<float, 96> { static constexpr int TT = 8, R = 101, BX = 12, AX = 8, WPE = 1, LOOP = 1; };
template <> struct PlanePitch<float, 108> { static constexpr int TT = 6, R = 133, BX = 19, AX = 7, WPE = 1, LOOP = 1; };
template <> struct PlanePitch<double, 24> { static constexpr int TT = 2, R = 30, BX = 7, AX = 5, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<double, 27> { static constexpr int TT = 3, R = 27, BX = 9, AX = 3, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<double, 32> { static constexpr int TT = 4, R = 44, BX = 9, AX = 5, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<double, 48> { static constexpr int TT = 4, R = 60, BX = 13, AX = 5, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<double, 54> { static constexpr int TT = 3, R = 59, BX = 9, AX = 6, WPE = 1, LOOP = 0; };
template <> struct PlanePitch<double, 64> { static constexpr int TT = 8, R = 73, BX = 9, AX = 9, WPE = 4, LOOP = 0; };
template <> struct PlanePitch<double, 81> { static constexpr int TT = 9, R = 89, BX = 9, AX = 9, WPE = 1, LOOP = 1; };
template <> struct PlanePitch<double, 96> { static constexpr int TT = 4, R = 99, BX = 12, AX = 8, WPE = 1, LOOP = 0; };

template <typename T, int A, int B>
struct PlaneShape : PlanePitch<T, A * B> {
  using P = PlanePitch<T, A * B>;
  static constexpr int N = A * B, TT = P::TT, I1 = (B + TT - 1) / TT, J2 = (A + TT - 1) / TT;
  static constexpr int LPW = 64 / TT, NW = (N + LPW - 1) / LPW;  // lines per wave; one group of rows per wave
  static constexpr size_t LDS = (size_t)(N * P::R + N) * sizeof(cplx<T>);
  static constexpr bool SWZ = P::R == 64;
  // whether thread t's transform i of stage 1 (j of stage 2) exists: all do where TT divides B (A)
  static __device__ __forceinline__ bool has1(int t, int i) { return B % TT == 0 || t + TT * i < B; }
  static __device__ __forceinline__ bool has2(int t, int j) { return A % TT == 0 || t + TT * j < A; }
  // plane word of (row, xa); in-row words of the exchanges of row y
  static __device__ __forceinline__ int at(int row, int xa) {
    return row * P::R + (SWZ ? xa ^ (4 * ((row ^ (row >> 3)) & 7)) : xa);
  }
  static __device__ __forceinline__ int inv_word(int y, int k1, int n2) {
    return SWZ ? (8 * k1 + (n2 ^ k1)) ^ (8 * (y & 3)) : k1 * P::BX + n2;
  }
  static __device__ __forceinline__ int fwd_word(int y, int q2, int m1) {
    return SWZ ? (8 * q2 + (m1 ^ q2)) ^ (8 * (y & 3)) : q2 * P::AX + m1;
  }
};

// Grid (n3, band groups), 64 NW threads; bands blockIdx.y, blockIdx.y + gridDim.y, ...
// DENS: the charge density.  A workgroup takes bands [group per, (group + 1) per), stops behind the inverse x pass
// and adds occ_b |psi_b|^2 to FP64 registers of its rows' points, bands in order: part[group][z][y][x].  Bound by
// the sticks' one read: 144 bands on 64^3 in FP64 101 us, 207 as pencil passes through HBM.
template <typename T, int A, int B, bool DENS>
__global__ __launch_bounds__((64 * PlaneShape<T, A, B>::NW))
    __attribute__((amdgpu_waves_per_eu(DENS ? 1 : PlaneShape<T, A, B>::WPE))) void k_plane_w(
        cplx<T>* __restrict__ SB, const T* __restrict__ V, const int* __restrict__ colstart, GridDesc g,
        const cplx<T>* __restrict__ twg, T scale, int nbatch, const double* __restrict__ occ, int per,
        double* __restrict__ part) {
  using S = PlaneShape<T, A, B>;
  constexpr int N = S::N, TT = S::TT, I1 = S::I1, J2 = S::J2, LPW = S::LPW, NW = S::NW;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<T>* plane = reinterpret_cast<cplx<T>*>(smem_raw);
  cplx<T>* tw = plane + N * S::R;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int l = min(lane / TT, LPW - 1), t = lane % TT;
  const bool on = lane < LPW * TT;
  const int z = blockIdx.x, n1max = g.n1max, n1a = g.n1a;
  for (int i = tid; i < N; i += 64 * NW) tw[i] = twg[i];
  const bool row_on = on && wv * LPW + l < N;  // this thread's row
  const int y = min(wv * LPW + l, N - 1);
  const T* vz = DENS ? nullptr : V + ((long)z * N + y) * N;
  double sum[DENS ? J2 : 1][DENS ? B : 1] = {};
  __syncthreads();
  const cplx<T> zero = mk<T>(0, 0);
  // W_N^{n2 k1} of stage 1 (n2 = t + TT i), conjugated for the inverse
  auto twiddle1 = [&](cplx<T>(&r)[I1][A], bool inverse) {
#pragma unroll
    for (int i = 0; i < I1; ++i)
#pragma unroll
      for (int k1 = 1; k1 < A; ++k1) {
        cplx<T> w = tw[((t + TT * i) * k1) % N];
        if (inverse) w.y = -w.y;
        r[i][k1] = cmul<T>(r[i][k1], w);
      }
  };
  // rows e = B k1 + n2 of a column <- stage 1; rows B k1 + n2 of it -> stage 2
  auto col_exchange = [&](cplx<T>(&r1)[I1][A], cplx<T>(&r2)[J2][B], int xa, bool act) {
    wave_sync();
#pragma unroll
    for (int i = 0; i < I1; ++i)
      if (act && S::has1(t, i))
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) plane[S::at(B * k1 + t + TT * i, xa)] = r1[i][k1];
    wave_sync();
#pragma unroll
    for (int j = 0; j < J2; ++j) {
      const int k1 = S::has2(t, j) ? t + TT * j : 0;
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) r2[j][n2] = plane[S::at(B * k1 + n2, xa)];
    }
  };
  auto one_band = [&](int b) {
    cplx<T>* sb = SB + ((long)b * g.n3 + z) * g.nst;
    // ---- inverse along y, active columns ----
    for (int c0 = wv * LPW; c0 < n1a; c0 += NW * LPW) {
      const int xa = min(c0 + l, n1a - 1);
      const bool act = on && c0 + l < n1a;
      const int cs = colstart[xa], m = act ? (colstart[xa + 1] - cs - 1) >> 1 : -1;
      cplx<T> r1[I1][A], r2[J2][B];
#pragma unroll
      for (int i = 0; i < I1; ++i)
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) {
          const int e = B * n1 + t + TT * i;
          const int n2 = 2 * e < N ? e : e - N;
          r1[i][n1] = (!grid_empty(N, B, n1) && n2 <= m && -n2 <= m && S::has1(t, i)) ? sb[cs + n2 + m] : zero;
        }
#pragma unroll
      for (int i = 0; i < I1; ++i) SmallDft<T, A, +1>::run(r1[i]);
      twiddle1(r1, true);
      col_exchange(r1, r2, xa, act);
#pragma unroll
      for (int j = 0; j < J2; ++j) SmallDft<T, B, +1>::run(r2[j]);
      wave_sync();
#pragma unroll
      for (int j = 0; j < J2; ++j)
        if (act && S::has2(t, j))
#pragma unroll
          for (int k2 = 0; k2 < B; ++k2) plane[S::at(t + TT * j + A * k2, xa)] = r2[j][k2];
    }
    __syncthreads();
    // ---- along x: inverse, * V, forward ----
    {
      cplx<T>* row = plane + y * S::R;
      cplx<T> r1[I1][A], r2[J2][B];
#pragma unroll
      for (int i = 0; i < I1; ++i)
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) {
          const int x = B * n1 + t + TT * i;
          const int k = 2 * x < N ? x : x - N;
          r1[i][n1] = (!grid_empty(N, B, n1) && k <= n1max && -k <= n1max && S::has1(t, i))
                          ? plane[S::at(y, k + n1max)]
                          : zero;
        }
#pragma unroll
      for (int i = 0; i < I1; ++i) SmallDft<T, A, +1>::run(r1[i]);
      twiddle1(r1, true);
      wave_sync();
#pragma unroll
      for (int i = 0; i < I1; ++i)
        if (row_on && S::has1(t, i))
#pragma unroll
          for (int k1 = 0; k1 < A; ++k1) row[S::inv_word(y, k1, t + TT * i)] = r1[i][k1];
      wave_sync();
#pragma unroll
      for (int j = 0; j < J2; ++j) {
        const int k1 = S::has2(t, j) ? t + TT * j : 0;
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) r2[j][n2] = row[S::inv_word(y, k1, n2)];
        SmallDft<T, B, +1>::run(r2[j]);
        if constexpr (DENS) {
          const double o = occ[b];
#pragma unroll
          for (int k2 = 0; k2 < B; ++k2)
            sum[j][k2] += o * ((double)r2[j][k2].x * r2[j][k2].x + (double)r2[j][k2].y * r2[j][k2].y);
          continue;
        }
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) r2[j][k2] = cscale<T>(r2[j][k2], vz[k1 + A * k2]);
        SmallDft<T, B, -1>::run(r2[j]);  // over m2 = k2, output q2
#pragma unroll
        for (int q2 = 1; q2 < B; ++q2) r2[j][q2] = cmul<T>(r2[j][q2], tw[(k1 * q2) % N]);
      }
      if constexpr (DENS) {
        __syncthreads();  // the next band's columns go over these rows
        return;
      }
      wave_sync();
#pragma unroll
      for (int j = 0; j < J2; ++j)
        if (row_on && S::has2(t, j))
#pragma unroll
          for (int q2 = 0; q2 < B; ++q2) row[S::fwd_word(y, q2, t + TT * j)] = r2[j][q2];
      wave_sync();
#pragma unroll
      for (int i = 0; i < I1; ++i) {
        const int q2 = S::has1(t, i) ? t + TT * i : 0;
#pragma unroll
        for (int m1 = 0; m1 < A; ++m1) r1[i][m1] = row[S::fwd_word(y, q2, m1)];
        SmallDft<T, A, -1>::run(r1[i]);  // r1[i][q1] = F[B q1 + q2]
      }
      wave_sync();
#pragma unroll
      for (int i = 0; i < I1; ++i)
#pragma unroll
        for (int q1 = 0; q1 < A; ++q1) {
          const int x = B * q1 + t + TT * i;
          const int k = 2 * x < N ? x : x - N;
          if (!grid_empty(N, B, q1) && row_on && S::has1(t, i) && k <= n1max && -k <= n1max)
            plane[S::at(y, k + n1max)] = r1[i][q1];
        }
    }
    __syncthreads();
    // ---- forward along y, active columns, into the sticks (the next band's columns are this wave's own) ----
    for (int c0 = wv * LPW; c0 < n1a; c0 += NW * LPW) {
      const int xa = min(c0 + l, n1a - 1);
      const bool act = on && c0 + l < n1a;
      cplx<T> r1[I1][A], r2[J2][B];
#pragma unroll
      for (int i = 0; i < I1; ++i) {
        const int n2 = S::has1(t, i) ? t + TT * i : 0;
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) r1[i][n1] = plane[S::at(B * n1 + n2, xa)];
        SmallDft<T, A, -1>::run(r1[i]);
      }
      twiddle1(r1, false);
      col_exchange(r1, r2, xa, act);
      const int cs = colstart[xa], m = act ? (colstart[xa + 1] - cs - 1) >> 1 : -1;
#pragma unroll
      for (int j = 0; j < J2; ++j) {
        SmallDft<T, B, -1>::run(r2[j]);
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) {
          const int e = t + TT * j + A * k2;
          const int n2 = 2 * e < N ? e : e - N;
          if (!grid_empty(N, A, k2) && n2 <= m && -n2 <= m && S::has2(t, j))
            sb[cs + n2 + m] = cscale<T>(r2[j][k2], scale);
        }
      }
    }
  };
  if constexpr (DENS) {
    const int b1 = min(nbatch, ((int)blockIdx.y + 1) * per);
    for (int b = blockIdx.y * per; b < b1; ++b) one_band(b);
    double* pz = part + (((long)blockIdx.y * g.n3 + z) * N + y) * N;
#pragma unroll
    for (int j = 0; j < J2; ++j)
      if (row_on && S::has2(t, j))
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) pz[t + TT * j + A * k2] = sum[j][k2];
  } else if constexpr (S::LOOP) {
    for (int b = blockIdx.y; b < nbatch; b += gridDim.y) one_band(b);
  } else {
    one_band(blockIdx.y);
  }
}

// ---- real-space projectors on 128 x 128 FP32 planes --------------------------------------------
// The projectors are truncated to the grid points within a radius R of their atom (Section III-A:
// a projector acts only near its atom).  An entry (atom, plane) holds unwrapped ranges of columns
// x0 .. x0+nx-1 and rows y0 .. y0+ny-1 (mod 128 on the plane) that contain every point of the disc
// the ball cuts from the plane; a point lies in the ball when dx^2 + (dy^2 + dz^2) <= R^2.  The
// Gaussian factors as e^{-dx^2/(2 s^2)} e^{-(dy^2 + dz^2)/(2 s^2)}.  Both passes evaluate points
// with the same expressions, so they see the same points and the same values.
//  * The projection pass holds the plane in LDS (row y in x order, word y * 128 + (x ^ 8 (y & 1))) and
//    gives each wave whole (atom, plane) entries, 8 columns x 8 rows at a time; one reduction across the
//    wave ends each entry.
//  * The pass of V(r) adds D P on the x pass itself, where lane (l, t) of wave w holds the 16 values
//    of row y = 8w + l at x = t + 8k in registers: the wave walks the entries of its 8-row band and
//    visits only the 8-column blocks that an entry's columns meet (a wave-uniform mask).
// Both are bound by the issue of vector instructions (four waves on a SIMD) and by the LDS crossbar, so the
// row factors of the D P pass and the column factors of the projections, which the lanes share, are made by
// one lane and fetched by the others; fetching the other two as well was slower.  36 bands of 512 atoms,
// 128 x 128 x 128: projections 370 us and D P pass 543 us; 506 and 660 us with every factor made by every lane
// and sums across the wave by 36 exchanges.
// value of lane k of v (k uniform over the wave)
__device__ __forceinline__ float rs_lane(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}
__device__ __forceinline__ int rs_lane(int v, int k) { return __builtin_amdgcn_readlane(v, k); }

// One entry's data, loaded by lane k of the wave, then read by the whole wave with rs_entry.
struct RsLaneEnt {
  float dz, bx, by;
  int xr, yr;  // x0 | nx << 16 and y0 | ny << 16 (x0, y0 as 16-bit two's complement)
  int mask;
};
__device__ __forceinline__ RsLaneEnt rs_load(const RsEnt& en) {
  RsLaneEnt l;
  l.dz = en.dz;
  l.bx = en.bx;
  l.by = en.by;
  l.xr = (int)(unsigned short)en.x0 | ((int)en.nx << 16);
  l.yr = (int)(unsigned short)en.y0 | ((int)en.ny << 16);
  l.mask = en.mask;
  return l;
}
__device__ __forceinline__ RsLaneEnt rs_empty() {
  RsLaneEnt l;
  l.dz = l.bx = l.by = 0.f;
  l.xr = l.yr = 0;
  l.mask = 0;
  return l;
}

struct RsEntry {
  float dz, dz2, bx, by;
  int x0, nx, y0, ny;
  unsigned mask;  // bit k: columns 8k .. 8k+7 meet x0 .. x0+nx-1 (mod 128)
};
__device__ __forceinline__ RsEntry rs_entry(const RsLaneEnt& l, int k) {
  RsEntry e;
  e.dz = rs_lane(l.dz, k);
  e.dz2 = e.dz * e.dz;
  e.bx = rs_lane(l.bx, k);
  e.by = rs_lane(l.by, k);
  const int xr = rs_lane(l.xr, k), yr = rs_lane(l.yr, k);
  e.x0 = (int)(short)(xr & 0xffff);
  e.nx = xr >> 16;
  e.y0 = (int)(short)(yr & 0xffff);
  e.ny = yr >> 16;
  e.mask = (unsigned)rs_lane(l.mask, k);
  return e;
}

// Row part of row y (0 .. 127): dy, e^{-(dy^2 + dz^2)/(2 s^2)} and the largest dx^2 inside the ball (negative
// outside the entry's rows and beyond the ball).
struct RsRow {
  float dy, gyz, lim;
};
__device__ __forceinline__ RsRow rs_rowpart(const RsDesc& d, float dy, float dz2, bool ok) {
  RsRow w;
  w.dy = dy;
  const float s = fmaf(dy, dy, dz2);
  w.gyz = __builtin_amdgcn_exp2f(s * d.k2);
  w.lim = ok ? d.r2 - s : -1.f;
  return w;
}
__device__ __forceinline__ RsRow rs_row(const RsDesc& d, const RsEntry& e, int y) {
  const int oy = (y - e.y0) & 127;
  return rs_rowpart(d, fmaf((float)oy, d.hy, e.by), e.dz2, oy < e.ny);
}
// Column part of column x (0 .. 127): dx, dx^2 and e^{-dx^2/(2 s^2)}.  A column outside the entry's
// range needs no test of its own: its dx exceeds the disc radius of the enlarged range radius, so
// the ball test dx^2 <= lim rejects it (by a margin of 2e-4 of R^2, far above FP32 rounding).
struct RsCol {
  float dx, dx2, gx;
};
__device__ __forceinline__ RsCol rs_colpart(const RsDesc& d, const RsEntry& e, int ox) {
  RsCol c;
  c.dx = fmaf((float)ox, d.hx, e.bx);
  c.dx2 = c.dx * c.dx;
  c.gx = __builtin_amdgcn_exp2f(c.dx2 * d.k2);
  return c;
}
// value of the lane at byte address a (mod 256; 4 bytes a lane)
__device__ __forceinline__ float rs_from(float v, int a) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(a, __float_as_int(v)));
}
__device__ __forceinline__ int rs_from(int v, int a) { return __builtin_amdgcn_ds_bpermute(a, v); }

// a + its partner 32 (16) lanes away in lanes with that bit clear, b + its partner in the others
__device__ __forceinline__ float rs_half32(float a, float b) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
  return __int_as_float(p[0]) + __int_as_float(p[1]);
}
__device__ __forceinline__ float rs_half16(float a, float b) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
  return __int_as_float(p[0]) + __int_as_float(p[1]);
}
template <int CTRL>
__device__ __forceinline__ float rs_ror_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// sum over each row of 16 lanes, in all of them
__device__ __forceinline__ float rs_row_sum(float v) {
  v = rs_ror_add<0x128>(v);
  v = rs_ror_add<0x124>(v);
  v = rs_ror_add<0x122>(v);
  return rs_ror_add<0x121>(v);
}

// Adds sum_a sum_m sqrt(Omega) p_m(r - tau_a) dp_{a,m} to this lane's 16 values of row y (x = t + 8k),
// atoms in the order of the band's entry list.  With p_0 = c0 g, p_m = c1 d_m g and g = gx gyz the
// term is gx (w0 + dx w1), w0 = gyz (c0 dp_0 + c1 (dy dp_y + dz dp_z)), w1 = gyz c1 dp_x.  Of eight entries,
// lane (l, t) makes w0, w1 and the ball's limit of entry t on row l.
__device__ __forceinline__ void rs_add_regs(float2 (&r)[16], const RsDesc& rd, int z, int w, int y, int t,
                                            const float2* dp, int lane) {
  // w is the same in the whole wave: so are the entries and the branches on them
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int e0 = rd.boff[16 * z + wu], e1 = rd.boff[16 * z + wu + 1];
  for (int base = e0; base < e1; base += 64) {
    // lane k: entry base + k; dp holds (c0 D P_0, c1 D P_x, c1 D P_y, c1 D P_z)
    RsLaneEnt le = rs_empty();
    float2 q0 = make_float2(0.f, 0.f), q1 = q0, q2 = q0;
    if (base + lane < e1) {
      const RsEnt en = rd.bent[base + lane];
      le = rs_load(en);
      const float2* c = dp + 4 * en.atom;
      const float2 q3 = c[3];
      q0 = c[0];
      q1 = c[1];
      q2 = c[2];
      q0.x = fmaf(en.dz, q3.x, q0.x);
      q0.y = fmaf(en.dz, q3.y, q0.y);
    }
    const int cnt = min(64, e1 - base);
    for (int k8 = 0; k8 < cnt; k8 += 8) {
      const int a8 = 4 * (k8 + t);
      const float dz = rs_from(le.dz, a8);
      const int yr = rs_from(le.yr, a8);
      const int oy = (y - yr) & 127;  // the low 16 bits hold y0
      const RsRow rw = rs_rowpart(rd, fmaf((float)oy, rd.hy, rs_from(le.by, a8)), dz * dz, oy < (yr >> 16));
      const float w0x = rw.gyz * fmaf(rw.dy, rs_from(q2.x, a8), rs_from(q0.x, a8));
      const float w0y = rw.gyz * fmaf(rw.dy, rs_from(q2.y, a8), rs_from(q0.y, a8));
      const float w1x = rw.gyz * rs_from(q1.x, a8), w1y = rw.gyz * rs_from(q1.y, a8);
      const int n8 = min(8, cnt - k8);
      int al = 4 * (lane & 56);
      for (int j = 0; j < n8; ++j, al += 4) {
        const float u0x = rs_from(w0x, al), u0y = rs_from(w0y, al), u1x = rs_from(w1x, al), u1y = rs_from(w1y, al);
        const float lim = rs_from(rw.lim, al);
        RsEntry e;
        const int xr = rs_lane(le.xr, k8 + j);
        e.bx = rs_lane(le.bx, k8 + j);
        const unsigned mask = (unsigned)rs_lane(le.mask, k8 + j);
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
          if (mask & (1u << kk)) {
            const RsCol c = rs_colpart(rd, e, (t - xr + 8 * kk) & 127);  // the low bits of xr hold x0
            const float gx = c.dx2 <= lim ? c.gx : 0.f;
            r[kk].x += gx * fmaf(c.dx, u1x, u0x);
            r[kk].y += gx * fmaf(c.dx, u1y, u0y);
          }
        }
      }
    }
  }
}

// ---- 128 x 128 FP32 planes with wave-local lines ---------------------------------------------
// The same transform as k_plane_w (inverse along y on the active columns, inverse along x, * V,
// forward along x, forward along y on the active columns), arranged so that the 8 threads of a
// line sit in one wave: the exchange between the two stages of a line is ordered by the wave
// itself and needs no workgroup barrier, and the plane needs no zero fill, scatter or gather:
//   y passes read their input straight from the sticks (zeros off the stick's n2 range) and the
//   forward one writes its stick positions straight back;
//   the plane in LDS holds only the active columns xa = n1 + n1max, at column xa ^ sy(row) of
//   each 128-word row (sy(r) = 8 ((r >> 4 ^ r) & 1));
//   the x pass uses its row as exchange space: stage-1 word (n2, k1) of the inverse at
//   16 k1 + (n2 ^ k1 ^ 8 (y & 1)), word (m1, q2) of the forward at (8 q2 + (m1 ^ (q2 & 7))) ^ 8 (y & 1).
// Each swizzle spreads the 64 lanes of a wave (8 lines x 8 threads) over all 16 eight-byte bank
// slots in every access of the three passes.  Three workgroup barriers per plane.
__device__ __forceinline__ int p128_col(int row, int xa) { return xa ^ ((((row >> 4) ^ row) & 1) << 3); }

// NL: the real-space projectors' D P term is added to V psi between the x passes (rs_add_regs).
template <bool NL>
__global__ __launch_bounds__(1024) void k_plane128(float2* __restrict__ SB, const float* __restrict__ V,
                                                   const int* __restrict__ colstart, GridDesc g,
                                                   const float2* __restrict__ twg, float scale, RsDesc rd,
                                                   const float2* __restrict__ dp, int nproj) {
  using T = float;
  constexpr int N = 128, A = 8, B = 16, LPW = 8, NW = 16;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float2* plane = reinterpret_cast<float2*>(smem_raw);
  float2* tw = plane + N * N;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int l = lane >> 3, t = lane & 7;
  const int z = blockIdx.x, b = blockIdx.y;
  const int n1max = g.n1max, n1a = g.n1a;
  const int yrow = wv * LPW + l;
  for (int i = tid; i < N; i += 1024) tw[i] = twg[i];
  float2* sb = SB + ((long)b * g.n3 + z) * g.nst;
  __syncthreads();
  const float2 zero = mk<T>(0, 0);
  // ---- inverse along y, active columns ----
  for (int grp = wv; grp * LPW < n1a; grp += NW) {
    const int xa = grp * LPW + l;
    const bool act = xa < n1a;
    int cs = 0, m = -1;
    if (act) {
      cs = colstart[xa];
      m = (colstart[xa + 1] - cs - 1) >> 1;
    }
    float2 r1[2][A];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) {
        const int y = B * n1 + t + 8 * i;
        const int n2 = y < N / 2 ? y : y - N;
        r1[i][n1] = (!grid_empty(N, B, n1) && n2 <= m && -n2 <= m) ? sb[cs + n2 + m] : zero;
      }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int n2 = t + 8 * i;
      SmallDft<T, A, +1>::run(r1[i]);
#pragma unroll
      for (int k1 = 1; k1 < A; ++k1) {
        float2 w = tw[(n2 * k1) % N];
        w.y = -w.y;
        r1[i][k1] = cmul<T>(r1[i][k1], w);
      }
      if (act)
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) {
          const int e = B * k1 + n2;
          plane[e * N + p128_col(e, xa)] = r1[i][k1];
        }
    }
    wave_sync();
    float2 r2[B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
      const int e = B * t + n2;
      r2[n2] = plane[e * N + p128_col(e, xa)];
    }
    SmallDft<T, B, +1>::run(r2);
    wave_sync();
    if (act)
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) {
        const int e = t + A * k2;
        plane[e * N + p128_col(e, xa)] = r2[k2];
      }
  }
  __syncthreads();
  // ---- along x on every row: inverse, * V, forward ----
  {
    // V(r) of this thread's row (x = t + 8 k2), issued before the inverse stages that hide it
    T vr[B];
    {
      const T* vz = V + ((long)z * N + yrow) * N + t;
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) vr[k2] = vz[A * k2];
    }
    const int y = yrow;
    const int sy = (((y >> 4) ^ y) & 1) << 3, py = (y & 1) << 3;
    float2* row = plane + y * N;
    float2 r1[2][A];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) {
        const int x = B * n1 + t + 8 * i;
        const int k = x < N / 2 ? x : x - N;
        r1[i][n1] = (!grid_empty(N, B, n1) && k <= n1max && -k <= n1max) ? row[(k + n1max) ^ sy] : zero;
      }
    wave_sync();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int n2 = t + 8 * i;
      SmallDft<T, A, +1>::run(r1[i]);
#pragma unroll
      for (int k1 = 1; k1 < A; ++k1) {
        float2 w = tw[(n2 * k1) % N];
        w.y = -w.y;
        r1[i][k1] = cmul<T>(r1[i][k1], w);
      }
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) row[B * k1 + (n2 ^ k1 ^ py)] = r1[i][k1];
    }
    wave_sync();
    float2 r2[B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) r2[n2] = row[B * t + (n2 ^ t ^ py)];
    SmallDft<T, B, +1>::run(r2);  // r2[k2] = value at x = t + 8 k2
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) r2[k2] = cscale<T>(r2[k2], vr[k2]);
    if constexpr (NL) rs_add_regs(r2, rd, z, wv, y, t, dp + (long)b * nproj, lane);
    SmallDft<T, B, -1>::run(r2);  // over m2, output q2
#pragma unroll
    for (int q2 = 1; q2 < B; ++q2) r2[q2] = cmul<T>(r2[q2], tw[(t * q2) % N]);
    wave_sync();
#pragma unroll
    for (int q2 = 0; q2 < B; ++q2) row[(A * q2 + (t ^ (q2 & 7))) ^ py] = r2[q2];
    wave_sync();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q2 = t + 8 * i;
#pragma unroll
      for (int m1 = 0; m1 < A; ++m1) r1[i][m1] = row[(A * q2 + (m1 ^ (q2 & 7))) ^ py];
      SmallDft<T, A, -1>::run(r1[i]);  // r1[i][q1] = F[16 q1 + q2]
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q1 = 0; q1 < A; ++q1) {
        const int x = B * q1 + t + 8 * i;
        const int k = x < N / 2 ? x : x - N;
        if (!grid_empty(N, B, q1) && k <= n1max && -k <= n1max) row[(k + n1max) ^ sy] = r1[i][q1];
      }
  }
  __syncthreads();
  // ---- forward along y, active columns, into the sticks ----
  for (int grp = wv; grp * LPW < n1a; grp += NW) {
    const int xa = grp * LPW + l;
    const bool act = xa < n1a;
    int cs = 0, m = -1;
    if (act) {
      cs = colstart[xa];
      m = (colstart[xa + 1] - cs - 1) >> 1;
    }
    float2 r1[2][A];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) {
        const int e = B * n1 + t + 8 * i;
        r1[i][n1] = plane[e * N + p128_col(e, xa)];
      }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int n2 = t + 8 * i;
      SmallDft<T, A, -1>::run(r1[i]);
#pragma unroll
      for (int k1 = 1; k1 < A; ++k1) r1[i][k1] = cmul<T>(r1[i][k1], tw[(n2 * k1) % N]);
    }
    wave_sync();
    if (act)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) {
          const int e = B * k1 + t + 8 * i;
          plane[e * N + p128_col(e, xa)] = r1[i][k1];
        }
    wave_sync();
    float2 r2[B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
      const int e = B * t + n2;
      r2[n2] = plane[e * N + p128_col(e, xa)];
    }
    SmallDft<T, B, -1>::run(r2);  // r2[k2] = value at y = t + 8 k2
    if (act)
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) {
        const int y = t + A * k2;
        const int n2 = y < N / 2 ? y : y - N;
        if (!grid_empty(N, A, k2) && n2 <= m && -n2 <= m) sb[cs + n2 + m] = cscale<T>(r2[k2], scale);
      }
  }
}

namespace p128 {
constexpr int N = 128, A = 8, B = 16, LPW = 8;

__device__ __forceinline__ void yinv_load(const float2* __restrict__ sb, const int* __restrict__ colstart, int n1a,
                                          int grp, int l, int t, float2 (&r)[2][A]) {
  const int xa = grp * LPW + l;
  int cs = 0, m = -1;
  if (xa < n1a) {
    cs = colstart[xa];
    m = (colstart[xa + 1] - cs - 1) >> 1;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) {
      const int y = B * n1 + t + 8 * i;
      const int n2 = y < N / 2 ? y : y - N;
      r[i][n1] = (!grid_empty(N, B, n1) && n2 <= m && -n2 <= m) ? sb[cs + n2 + m] : make_float2(0.f, 0.f);
    }
}

__device__ __forceinline__ void yinv_compute(float2* plane, const float2* tw, int n1a, int grp, int l, int t,
                                             float2 (&r1)[2][A]) {
  const int xa = grp * LPW + l;
  const bool act = xa < n1a;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int n2 = t + 8 * i;
    SmallDft<float, A, +1>::run(r1[i]);
#pragma unroll
    for (int k1 = 1; k1 < A; ++k1) {
      float2 w = tw[(n2 * k1) % N];
      w.y = -w.y;
      r1[i][k1] = cmul<float>(r1[i][k1], w);
    }
    if (act)
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) {
        const int e = B * k1 + n2;
        plane[e * N + p128_col(e, xa)] = r1[i][k1];
      }
  }
  wave_sync();
  float2 r2[B];
#pragma unroll
  for (int n2 = 0; n2 < B; ++n2) {
    const int e = B * t + n2;
    r2[n2] = plane[e * N + p128_col(e, xa)];
  }
  SmallDft<float, B, +1>::run(r2);
  wave_sync();
  if (act)
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) {
      const int e = t + A * k2;
      plane[e * N + p128_col(e, xa)] = r2[k2];
    }
}
}  // namespace p128

// Charge density on 128 x 128 FP32 planes, fused: a workgroup takes one z plane and a group of the
// batch's bands, runs the inverse y pass (as k_plane128) and the inverse x pass of each band, and
// adds occ_b |psi_b(r)|^2 to FP64 registers of its rows' grid points, bands in order; the group's
// sum goes out once (part[group][z][y][x]) instead of one |psi|^2 grid per band.  8 waves; each
// wave owns two rows per line (y0 = 8 w + l,
// y1 = 8 (w + 8) + l), so a thread keeps 32 sums.
__device__ __forceinline__ void xinv_row_acc(float2* plane, const float2* tw, int y, int t, int n1max, double occ,
                                             double (&acc)[16]) {
  constexpr int N = 128, A = 8, B = 16;
  const int sy = (((y >> 4) ^ y) & 1) << 3, py = (y & 1) << 3;
  float2* row = plane + y * N;
  float2 r1[2][A];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) {
      const int x = B * n1 + t + 8 * i;
      const int k = x < N / 2 ? x : x - N;
      r1[i][n1] = (!grid_empty(N, B, n1) && k <= n1max && -k <= n1max) ? row[(k + n1max) ^ sy] : make_float2(0.f, 0.f);
    }
  wave_sync();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int n2 = t + 8 * i;
    SmallDft<float, A, +1>::run(r1[i]);
#pragma unroll
    for (int k1 = 1; k1 < A; ++k1) {
      float2 w = tw[(n2 * k1) % N];
      w.y = -w.y;
      r1[i][k1] = cmul<float>(r1[i][k1], w);
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) row[B * k1 + (n2 ^ k1 ^ py)] = r1[i][k1];
  }
  wave_sync();
  float2 r2[B];
#pragma unroll
  for (int n2 = 0; n2 < B; ++n2) r2[n2] = row[B * t + (n2 ^ t ^ py)];
  SmallDft<float, B, +1>::run(r2);  // r2[k2] = psi at x = t + 8 k2
#pragma unroll
  for (int k2 = 0; k2 < B; ++k2) acc[k2] += occ * ((double)r2[k2].x * r2[k2].x + (double)r2[k2].y * r2[k2].y);
}

__global__ __launch_bounds__(512) void k_density128(const float2* __restrict__ SB, const int* __restrict__ colstart,
                                                    GridDesc g, const float2* __restrict__ twg,
                                                    const double* __restrict__ occ, int nbt, int per,
                                                    double* __restrict__ part, int add) {
  constexpr int N = 128, A = 8, LPW = 8, NW = 8;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float2* plane = reinterpret_cast<float2*>(smem_raw);
  float2* tw = plane + N * N;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int l = lane >> 3, t = lane & 7;
  const int z = blockIdx.x, grp = blockIdx.y;
  const int n1max = g.n1max, n1a = g.n1a;
  const int ngrp = (n1a + LPW - 1) / LPW;
  const int y0 = wv * LPW + l, y1 = (wv + NW) * LPW + l;
  const int b_lo = grp * per, b_hi = min(nbt, b_lo + per);
  for (int i = tid; i < N; i += 64 * NW) tw[i] = twg[i];
  double acc0[16], acc1[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) acc0[k] = acc1[k] = 0.0;
  __syncthreads();
  for (int b = b_lo; b < b_hi; ++b) {
    const float2* sb = SB + ((long)b * g.n3 + z) * g.nst;
    for (int cg = wv; cg < ngrp; cg += NW) {
      float2 r[2][A];
      p128::yinv_load(sb, colstart, n1a, cg, l, t, r);
      p128::yinv_compute(plane, tw, n1a, cg, l, t, r);
    }
    __syncthreads();
    const double o = occ[b];
    xinv_row_acc(plane, tw, y0, t, n1max, o, acc0);
    __builtin_amdgcn_sched_barrier(0);
    xinv_row_acc(plane, tw, y1, t, n1max, o, acc1);
    __syncthreads();
  }
  double* pz = part + ((long)grp * g.n3 + z) * N * N;
#pragma unroll
  for (int k2 = 0; k2 < 16; ++k2) {
    double* q0 = pz + (long)y0 * N + t + A * k2;
    double* q1 = pz + (long)y1 * N + t + A * k2;
    *q0 = add ? *q0 + acc0[k2] : acc0[k2];
    *q1 = add ? *q1 + acc1[k2] : acc1[k2];
  }
}

// rho[r] = (first ? 0 : rho[r]) + sum over groups of part[group][r], groups in order
__global__ void k_density_groups(const double* __restrict__ part, int ngroups, long nr, double* __restrict__ rho,
                                 int first) {
  PW_GRID_STRIDE(r, nr) {
    double s = first ? 0.0 : rho[r];
    for (int q = 0; q < ngroups; ++q) s += part[(long)q * nr + r];
    rho[r] = s;
  }
}

// the spheres that the plane kernels carry (grid_empty)
static bool alias_free(const GridDesc& g) { return g.n1max <= plane_top(g.n1) && g.n2max <= plane_top(g.n2); }

hipError_t launch_density_groups(const double* part, int ngroups, long nr, double* rho, bool first, hipStream_t s) {
  hipLaunchKernelGGL(k_density_groups, dim3(stride_blocks(nr)), dim3(256), 0, s, part, ngroups, nr, rho, first ? 1 : 0);
  return hipGetLastError();
}

bool density128_supported(const GridDesc& g, int real_bytes) {
  return real_bytes == 4 && g.n1 == 128 && g.n2 == 128 && g.n1a <= 128;
}

hipError_t launch_density128(const float2* SB, const int* colstart, const GridDesc& g, const float2* tw,
                             const double* occ, int nbt, int ngroups, double* part, double* rho, bool first,
                             hipStream_t s) {
  if (nbt <= 0) return hipSuccess;
  const size_t lds = (size_t)(128 * 128 + 128) * sizeof(float2);
  if (!part || ngroups <= 1) {
    // one group per plane: its sum goes straight into rho
    hipLaunchKernelGGL(k_density128, dim3(g.n3, 1), dim3(512), lds, s, SB, colstart, g, tw, occ, nbt, nbt, rho,
                       first ? 0 : 1);
    return hipGetLastError();
  }
  if (ngroups > nbt) ngroups = nbt;
  const int per = (nbt + ngroups - 1) / ngroups;
  ngroups = (nbt + per - 1) / per;
  hipLaunchKernelGGL(k_density128, dim3(g.n3, ngroups), dim3(512), lds, s, SB, colstart, g, tw, occ, nbt, per, part,
                     0);
  const long nr = 128L * 128 * g.n3;
  hipLaunchKernelGGL(k_density_groups, dim3(stride_blocks(nr)), dim3(256), 0, s, part, ngroups, nr, rho,
                     first ? 1 : 0);
  return hipGetLastError();
}

// Inverse x pass of row y (as in xinv_row_acc); the row then holds psi(x) at word x ^ 8 (y & 1): eight columns of
// two neighbouring rows lie in different banks.
__device__ __forceinline__ void xinv_row_store(float2* plane, const float2* tw, int y, int t, int n1max) {
  constexpr int N = 128, A = 8, B = 16;
  const int sy = (((y >> 4) ^ y) & 1) << 3, py = (y & 1) << 3;
  float2* row = plane + y * N;
  float2 r1[2][A];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) {
      const int x = B * n1 + t + 8 * i;
      const int k = x < N / 2 ? x : x - N;
      r1[i][n1] = (!grid_empty(N, B, n1) && k <= n1max && -k <= n1max) ? row[(k + n1max) ^ sy] : make_float2(0.f, 0.f);
    }
  wave_sync();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int n2 = t + 8 * i;
    SmallDft<float, A, +1>::run(r1[i]);
#pragma unroll
    for (int k1 = 1; k1 < A; ++k1) {
      float2 w = tw[(n2 * k1) % N];
      w.y = -w.y;
      r1[i][k1] = cmul<float>(r1[i][k1], w);
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) row[B * k1 + (n2 ^ k1 ^ py)] = r1[i][k1];
  }
  wave_sync();
  float2 r2[B];
#pragma unroll
  for (int n2 = 0; n2 < B; ++n2) r2[n2] = row[B * t + (n2 ^ t ^ py)];
  SmallDft<float, B, +1>::run(r2);  // r2[k2] = psi at x = t + 8 k2
  wave_sync();
#pragma unroll
  for (int k2 = 0; k2 < B; ++k2) row[(t + A * k2) ^ py] = r2[k2];
}

// Inverse pass with the projections: a workgroup takes plane z of band b, transforms it inside LDS
// (inverse y on the active columns, inverse x on every row), then each wave takes entries of the
// plane (one atom each), sums g psi, g dx psi and g dy psi over the entry's points with its 64
// lanes (p_z = c1 dz g needs no sum of its own) and writes the four projector sums, reduced
// across the wave in a fixed order, to part[(b nent + e) 4 + m].
__global__ __launch_bounds__(1024) void k_rs_proj128(const float2* __restrict__ SB, const int* __restrict__ colstart,
                                                     GridDesc g, const float2* __restrict__ twg, RsDesc rd,
                                                     float2* __restrict__ part) {
  constexpr int N = 128, LPW = 8, NW = 16;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float2* plane = reinterpret_cast<float2*>(smem_raw);
  float2* tw = plane + N * N;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int l = lane >> 3, t = lane & 7;
  const int z = blockIdx.x, b = blockIdx.y;
  const int e0 = rd.zoff[z], e1 = rd.zoff[z + 1];
  if (e0 == e1) return;  // no atom within reach of this plane (uniform over the workgroup)
  const int n1a = g.n1a;
  const int ngrp = (n1a + LPW - 1) / LPW;
  for (int i = tid; i < N; i += 1024) tw[i] = twg[i];
  const float2* sb = SB + ((long)b * g.n3 + z) * g.nst;
  __syncthreads();
  for (int cg = wv; cg < ngrp; cg += NW) {
    float2 r[2][8];
    p128::yinv_load(sb, colstart, n1a, cg, l, t, r);
    p128::yinv_compute(plane, tw, n1a, cg, l, t, r);
  }
  __syncthreads();
  xinv_row_store(plane, tw, wv * LPW + l, t, g.n1max);
  __syncthreads();
  float2* pb = part + (long)b * rd.nent * 4;
  // this wave's entries e0 + wv + 16 k, their data loaded one entry per lane
  for (int base = e0 + __builtin_amdgcn_readfirstlane(wv); base < e1; base += NW * 64) {
    RsLaneEnt le = rs_empty();
    if (base + NW * lane < e1) le = rs_load(rd.zent[base + NW * lane]);
    const int cnt = min(64, (e1 - base + NW - 1) / NW);
    for (int k = 0; k < cnt; ++k) {
      const int e = base + NW * k;
      const RsEntry en = rs_entry(le, k);
      float s0x = 0.f, s0y = 0.f, sxx = 0.f, sxy = 0.f, syx = 0.f, syy = 0.f;
      if (en.nx <= 64 && en.ny <= 64) {
        // this lane's column t + 8 l
        const RsCol cw = rs_colpart(rd, en, t + 8 * l);
        const int swz = ((en.y0 + l) & 1) << 3;
        auto cols = [&](auto ncol, int c0) {
          constexpr int NC = decltype(ncol)::value;
          float d2[NC], gx[NC], gd[NC];
          int off[NC];
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const int a = 4 * t + 4 * c0 + 32 * c;
            const float dx = rs_from(cw.dx, a);
            gx[c] = rs_from(cw.gx, a);
            d2[c] = dx * dx;
            gd[c] = gx[c] * dx;
            off[c] = ((en.x0 + c0 + 8 * c + t) & (N - 1)) ^ swz;
          }
          int yo = (en.y0 + l) * N;
          float fq = (float)l;
          for (int q = 0; q < en.ny; q += 8, fq += 8.f, yo += 8 * N) {
            const RsRow rw = rs_rowpart(rd, fmaf(fq, rd.hy, en.by), en.dz2, true);
            const float2* row = plane + (yo & (N * N - 1));
            float2 v[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) v[c] = row[off[c]];
            float tx = 0.f, ty = 0.f, mx = 0.f, my = 0.f;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
              const bool in = d2[c] <= rw.lim;
              const float ga = in ? gx[c] : 0.f, gb = in ? gd[c] : 0.f;
              tx = fmaf(ga, v[c].x, tx);
              ty = fmaf(ga, v[c].y, ty);
              mx = fmaf(gb, v[c].x, mx);
              my = fmaf(gb, v[c].y, my);
            }
            const float gyz = rw.gyz, gdy = gyz * rw.dy;
            s0x = fmaf(gyz, tx, s0x);
            s0y = fmaf(gyz, ty, s0y);
            sxx = fmaf(gyz, mx, sxx);
            sxy = fmaf(gyz, my, sxy);
            syx = fmaf(gdy, tx, syx);
            syy = fmaf(gdy, ty, syy);
          }
        };
        for (int c0 = 0; c0 < en.nx; c0 += 32) {
          const int nx = en.nx - c0;
          if (nx > 24) cols(std::integral_constant<int, 4>{}, c0);
          else if (nx > 16) cols(std::integral_constant<int, 3>{}, c0);
          else if (nx > 8) cols(std::integral_constant<int, 2>{}, c0);
          else cols(std::integral_constant<int, 1>{}, c0);
        }
      } else {
        for (int xc = 0; xc < en.nx; xc += 64) {
          const int x = (en.x0 + xc + lane) & (N - 1);
          const RsCol cc = rs_colpart(rd, en, (x - en.x0) & (N - 1));
          const bool colok = xc + lane < en.nx;  // lanes past the range would alias its first columns
          for (int q = 0; q < en.ny; ++q) {
            const int y = (en.y0 + q) & (N - 1);
            const RsRow rw = rs_row(rd, en, y);
            const float gg = (colok && cc.dx2 <= rw.lim) ? cc.gx * rw.gyz : 0.f;
            const float2 v = plane[y * N + (x ^ ((y & 1) << 3))];
            const float gxv = gg * cc.dx, gyv = gg * rw.dy;
            s0x = fmaf(gg, v.x, s0x);
            s0y = fmaf(gg, v.y, s0y);
            sxx = fmaf(gxv, v.x, sxx);
            sxy = fmaf(gxv, v.y, sxy);
            syx = fmaf(gyv, v.x, syx);
            syy = fmaf(gyv, v.y, syy);
          }
        }
      }
      // rows of 16 lanes: u = sums of (s0x, sxx, s0y, sxy), v = (syx, syx, syy, syy)
      const float u = rs_row_sum(rs_half16(rs_half32(s0x, s0y), rs_half32(sxx, sxy)));
      const float h = rs_half32(syx, syy), v = rs_row_sum(rs_half16(h, h));
      if ((lane & 15) == 0) {
        const float c0 = rd.c0, c1 = rd.c1, c1z = rd.c1 * en.dz;
        float* o = reinterpret_cast<float*>(pb + (long)e * 4);
        const int im = lane >> 5;  // 0: real parts, 1: imaginary parts
        if (lane & 16) {
          o[2 + im] = c1 * u;
        } else {
          o[im] = c0 * u;
          o[4 + im] = c1 * v;
          o[6 + im] = c1z * u;
        }
      }
    }
  }
}

// dp[b nproj + 4a + m] = c_m dscale[m] inv_nr sum over atom a's entries (plane order) of part, in FP64
// (c_0 = c0, c_m = c1: the prefactor the addition would otherwise apply per point).
__global__ void k_rs_reduce(const float2* __restrict__ part, RsDesc rd, int nbt, const double* __restrict__ dscale,
                            double inv_nr, float2* __restrict__ dp, int nproj) {
  PW_GRID_STRIDE(idx, (long)nbt * rd.natoms) {
    const int j = (int)(idx / rd.natoms), a = (int)(idx - (long)j * rd.natoms);
    double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    // four entries in flight: the sums wait for nothing but their loads
    const int k1 = rd.aoff[a + 1];
    for (int k = rd.aoff[a]; k < k1; k += 4) {
      float4 u[4], v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4* q = reinterpret_cast<const float4*>(part + ((long)j * rd.nent + rd.aent[min(k + i, k1 - 1)]) * 4);
        u[i] = q[0];
        v[i] = q[1];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (k + i < k1) {
          s[0] += u[i].x;
          s[1] += u[i].y;
          s[2] += u[i].z;
          s[3] += u[i].w;
          s[4] += v[i].x;
          s[5] += v[i].y;
          s[6] += v[i].z;
          s[7] += v[i].w;
        }
      }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      // D P times the projector prefactor, as the addition uses it
      const double f = dscale[m] * inv_nr * (m == 0 ? (double)rd.c0 : (double)rd.c1);
      dp[(long)j * nproj + 4 * a + m] = make_float2((float)(s[2 * m] * f), (float)(s[2 * m + 1] * f));
    }
  }
}

hipError_t launch_rs_proj128(const float2* SB, const int* colstart, const GridDesc& g, const float2* tw,
                             const RsDesc& rd, int nbatch, float2* part, hipStream_t s) {
  if (nbatch <= 0 || rd.nent <= 0) return hipSuccess;
  if (g.n1 != 128 || g.n2 != 128 || !alias_free(g)) return hipErrorInvalidValue;
  const size_t lds = (size_t)(128 * 128 + 128) * sizeof(float2);
  hipLaunchKernelGGL(k_rs_proj128, dim3(g.n3, nbatch), dim3(1024), lds, s, SB, colstart, g, tw, rd, part);
  return hipGetLastError();
}

hipError_t launch_rs_reduce(const float2* part, const RsDesc& rd, int nbt, const double* dscale, double inv_nr,
                            float2* dp, int nproj, hipStream_t s) {
  if (nbt <= 0 || rd.natoms <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_rs_reduce, dim3(stride_blocks((long)nbt * rd.natoms)), dim3(256), 0, s, part, rd, nbt, dscale,
                     inv_nr, dp, nproj);
  return hipGetLastError();
}

hipError_t launch_plane128_nl(float2* SB, const float* V, int nbatch, const int* colstart, const GridDesc& g,
                              const float2* tw, float scale, const RsDesc& rd, const float2* dp, int nproj,
                              hipStream_t s) {
  if (nbatch <= 0) return hipSuccess;
  if (g.n1 != 128 || g.n2 != 128 || !alias_free(g)) return hipErrorInvalidValue;
  const size_t lds = (size_t)(128 * 128 + 128) * sizeof(float2);
  hipLaunchKernelGGL(k_plane128<true>, dim3(g.n3, nbatch), dim3(1024), lds, s, SB, V, colstart, g, tw, scale, rd, dp,
                     nproj);
  return hipGetLastError();
}

// ---- z transforms of the sticks with compile-time N = A B ---------------------------------
// gcd(A, B) threads share a stick; a block takes SPW sticks of one band (at most 256 threads and
// 48 KB of LDS).  Stick element i (0 <= i < len, h = (len - 1) / 2) sits at z = i - h mod N.
template <typename T, int A, int B>
struct StickShape {
  static constexpr int N = A * B, TT = cgcd(A, B);
  static constexpr int SPW0 = 256 / TT, SPWL = (48 * 1024) / (N * (int)sizeof(cplx<T>));
  static constexpr int SPW = SPW0 < SPWL ? SPW0 : SPWL;
  static constexpr int NT = SPW * TT;
  // LDS swizzle.  Lane = TT s + t: a half-wave (32 lanes, the unit in which the LDS serves a
  // 64-lane access of 8-byte elements) holds Gh = 32 / TT sticks, and its TT threads of one
  // stick touch TT positions at once, 1 or B apart, which in a plain [position][stick] layout
  // all fall in the same banks.  Stick s of position p is stored at column s ^ (Gh x(p)),
  // x(p) = (p + p / B) mod X with X = E / Gh slices of Gh sticks per 256-byte bank row (E
  // elements): the TT positions then occupy distinct slices (checked by enumeration for every
  // compiled size).  Used where the shapes allow it (32 % TT == 0, SPW a multiple of E).
  static constexpr int E = 256 / (int)sizeof(cplx<T>);
  static constexpr int Gh = 32 % TT == 0 ? 32 / TT : 0;
  static constexpr bool SWZ = Gh > 0 && E > Gh && SPW % E == 0;
  static constexpr int X = SWZ ? E / Gh : 1;
  __device__ __forceinline__ static int at(int p, int s) {
    if constexpr (SWZ) return p * SPW + (s ^ (Gh * ((p + p / B) % X)));
    else return p * SPW + s;
  }
};

__device__ __forceinline__ int stick_index(int z, int h, int N) {
  return z <= h ? z + h : (z >= N - h ? z - N + h : -1);
}

// sphere -> sticks, inverse FFT along z.  Grid (ceil(nst / SPW), nbatch).  SB layout [band][z][stick].
// TOP: largest |n3| carried, stick_top for a cutoff on a z shell, otherwise plane_top (points_empty).
template <typename T, int A, int B, int TOP>
__global__ __launch_bounds__(256) void k_sticks_inv_n(const cplx<T>* __restrict__ X, long ldx,
                                                      cplx<T>* __restrict__ SB, const Stick* __restrict__ st,
                                                      GridDesc g, const cplx<T>* __restrict__ twg) {
  using SS = StickShape<T, A, B>;
  constexpr int N = A * B, TT = SS::TT, SPW = SS::SPW, NT = SS::NT, I1 = B / TT, J2 = A / TT;
  __shared__ cplx<T> buf[N * SPW];  // [position][stick]
  __shared__ cplx<T> tw[N];
  const int tid = threadIdx.x, b = blockIdx.y;
  const int s = tid / TT, t = tid % TT;  // stick within the block, thread within the stick
  const int s0 = blockIdx.x * SPW;
  const bool act = s0 + s < g.nst;
  for (int i = tid; i < N; i += NT) tw[i] = twg[i];
  Stick sk{0, 0, 0, 0};
  if (act) sk = st[s0 + s];
  const int h = (sk.len - 1) >> 1;
  const cplx<T>* xs = X + (long)b * ldx + sk.off;
  // stage 1 input straight from the sphere: x[B n1 + n2], n2 = t + TT i
  cplx<T> r1[I1][A];
#pragma unroll
  for (int i = 0; i < I1; ++i)
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) {
      const int e = act && !points_empty(N, B, n1, TOP) ? stick_index(B * n1 + t + TT * i, h, N) : -1;
      r1[i][n1] = e >= 0 ? xs[e] : mk<T>(0, 0);
    }
  __syncthreads();  // twiddles
#pragma unroll
  for (int i = 0; i < I1; ++i) {
    const int n2 = t + TT * i;
    SmallDft<T, A, +1>::run(r1[i]);
#pragma unroll
    for (int k1 = 1; k1 < A; ++k1) {
      cplx<T> w = tw[(n2 * k1) % N];
      w.y = -w.y;
      r1[i][k1] = cmul<T>(r1[i][k1], w);
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) buf[SS::at(k1 * B + n2, s)] = r1[i][k1];
  }
  __syncthreads();
  cplx<T> r2[J2][B];
#pragma unroll
  for (int j = 0; j < J2; ++j) {
    const int k1 = t + TT * j;
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) r2[j][n2] = buf[SS::at(k1 * B + n2, s)];
    SmallDft<T, B, +1>::run(r2[j]);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < J2; ++j) {
    const int k1 = t + TT * j;
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) buf[SS::at(k1 + A * k2, s)] = r2[j][k2];
  }
  __syncthreads();
  // rows of SPW consecutive sticks per z
  const int ns = min(SPW, g.nst - s0);
  cplx<T>* sb = SB + (long)b * N * g.nst + s0;
  for (int i = tid; i < N * SPW; i += NT) {
    const int z = i / SPW, l = i - z * SPW;
    if (l < ns) sb[(long)z * g.nst + l] = buf[SS::at(z, l)];
  }
}

// sticks -> sphere, forward FFT along z.  UPD (FP32): the Chebyshev update of StickUpd is applied to
// each value as it is written (Z is then the updated block).
template <typename T, int A, int B, int TOP, bool UPD = false>
__global__ __launch_bounds__(256) void k_sticks_fwd_n(const cplx<T>* __restrict__ SB, cplx<T>* __restrict__ Z,
                                                      long ldz, const Stick* __restrict__ st, GridDesc g,
                                                      const cplx<T>* __restrict__ twg, StickUpd u) {
  using SS = StickShape<T, A, B>;
  constexpr int N = A * B, TT = SS::TT, SPW = SS::SPW, NT = SS::NT, I1 = B / TT, J2 = A / TT;
  __shared__ cplx<T> buf[N * SPW];
  __shared__ cplx<T> tw[N];
  const int tid = threadIdx.x, b = blockIdx.y;
  const int s = tid / TT, t = tid % TT;
  const int s0 = blockIdx.x * SPW;
  const int ns = min(SPW, g.nst - s0);
  const bool act = s < ns;
  for (int i = tid; i < N; i += NT) tw[i] = twg[i];
  const cplx<T>* sb = SB + (long)b * N * g.nst + s0;
  for (int i = tid; i < N * SPW; i += NT) {
    const int z = i / SPW, l = i - z * SPW;
    buf[SS::at(z, l)] = l < ns ? sb[(long)z * g.nst + l] : mk<T>(0, 0);
  }
  Stick sk{0, 0, 0, 0};
  if (act) sk = st[s0 + s];
  __syncthreads();
  cplx<T> r1[I1][A];
#pragma unroll
  for (int i = 0; i < I1; ++i)
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) r1[i][n1] = buf[SS::at(B * n1 + t + TT * i, s)];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < I1; ++i) {
    const int n2 = t + TT * i;
    SmallDft<T, A, -1>::run(r1[i]);
#pragma unroll
    for (int k1 = 1; k1 < A; ++k1) r1[i][k1] = cmul<T>(r1[i][k1], tw[(n2 * k1) % N]);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) buf[SS::at(k1 * B + n2, s)] = r1[i][k1];
  }
  __syncthreads();
  if (!act) return;
  const int h = (sk.len - 1) >> 1;
  cplx<T>* zs = Z + (long)b * ldz + sk.off;
#pragma unroll
  for (int j = 0; j < J2; ++j) {
    const int k1 = t + TT * j;
    cplx<T> r2[B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) r2[n2] = buf[SS::at(k1 * B + n2, s)];
    SmallDft<T, B, -1>::run(r2);
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) {
      const int e = stick_index(k1 + A * k2, h, N);
      if (!points_empty(N, A, k2, TOP) && e >= 0) {
        if constexpr (UPD) {
          const long i = (long)sk.off + e;
          const float2 y = u.Y[(long)b * u.ldy + i];
          const float kc = u.kin[i] - u.c;
          float2 v;
          v.x = u.alpha * (kc * y.x + r2[k2].x);
          v.y = u.alpha * (kc * y.y + r2[k2].y);
          if (u.Yp) {
            const float2 p = u.Yp[(long)b * u.ldp + i];
            v.x -= u.beta * p.x;
            v.y -= u.beta * p.y;
          }
          zs[e] = v;
        } else {
          zs[e] = r2[k2];
        }
      }
    }
  }
}

#define PW_STICK_SIZES(X) \
  X(24, 4, 6) X(27, 3, 9) X(32, 4, 8) X(48, 4, 12) X(54, 6, 9) X(64, 8, 8) X(81, 9, 9) X(96, 8, 12) X(128, 8, 16) \
  X(192, 12, 16)

bool sticks_n_supported(int n3) {
  switch (n3) {
#define PW_CASE(NN, AA, BB) case NN:
    PW_STICK_SIZES(PW_CASE)
#undef PW_CASE
    return true;
    default:
      return false;
  }
}

// The kernels for one length: the plan's largest |n3| decides what they leave out (always stick_top: a block of grid
// points more at some lengths, H X of 8 atoms on 24 points 36.6 us, 36.5 with plane_top).
#define PW_STICK_LAUNCH(KERNEL, TT, AA, BB, ...)                                                             \
  do {                                                                                                       \
    constexpr int lo = plane_top(AA * BB), hi = stick_top(AA * BB);                                          \
    const dim3 grid(ceil_div(g.nst, StickShape<TT, AA, BB>::SPW), nbatch), wg(StickShape<TT, AA, BB>::NT);   \
    if (g.n3max <= lo) hipLaunchKernelGGL((KERNEL(TT, AA, BB, lo)), grid, wg, 0, s, __VA_ARGS__);            \
    else if (g.n3max <= hi) hipLaunchKernelGGL((KERNEL(TT, AA, BB, hi)), grid, wg, 0, s, __VA_ARGS__);       \
    else return hipErrorInvalidValue;                                                                        \
  } while (0)
#define PW_STICKS_INV(TT, AA, BB, TOP) k_sticks_inv_n<TT, AA, BB, TOP>
#define PW_STICKS_FWD(TT, AA, BB, TOP) k_sticks_fwd_n<TT, AA, BB, TOP>
#define PW_STICKS_UPD(TT, AA, BB, TOP) k_sticks_fwd_n<TT, AA, BB, TOP, true>

template <typename T>
hipError_t launch_sticks_inv_n(const cplx<T>* X, long ldx, cplx<T>* SB, int nbatch, const Stick* st,
                               const GridDesc& g, const cplx<T>* tw3, hipStream_t s) {
  switch (g.n3) {
#define PW_CASE(NN, AA, BB)                                       \
  case NN:                                                        \
    PW_STICK_LAUNCH(PW_STICKS_INV, T, AA, BB, X, ldx, SB, st, g, tw3); \
    return hipGetLastError();
    PW_STICK_SIZES(PW_CASE)
#undef PW_CASE
    default:
      return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_sticks_fwd_n(const cplx<T>* SB, cplx<T>* Z, long ldz, int nbatch, const Stick* st,
                               const GridDesc& g, const cplx<T>* tw3, hipStream_t s) {
  switch (g.n3) {
#define PW_CASE(NN, AA, BB)                                       \
  case NN:                                                        \
    PW_STICK_LAUNCH(PW_STICKS_FWD, T, AA, BB, SB, Z, ldz, st, g, tw3, StickUpd{}); \
    return hipGetLastError();
    PW_STICK_SIZES(PW_CASE)
#undef PW_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_sticks_fwd_upd(const float2* SB, float2* out, long ldo, int nbatch, const Stick* st,
                                 const GridDesc& g, const float2* tw3, const StickUpd& u, hipStream_t s) {
  switch (g.n3) {
#define PW_CASE(NN, AA, BB)                                       \
  case NN:                                                        \
    PW_STICK_LAUNCH(PW_STICKS_UPD, float, AA, BB, SB, out, ldo, st, g, tw3, u); \
    return hipGetLastError();
    PW_STICK_SIZES(PW_CASE)
#undef PW_CASE
    default:
      return hipErrorInvalidValue;
  }
}
#undef PW_STICK_LAUNCH
#undef PW_STICKS_INV
#undef PW_STICKS_FWD
#undef PW_STICKS_UPD

template hipError_t launch_sticks_inv_n<float>(const cplx<float>*, long, cplx<float>*, int, const Stick*,
                                               const GridDesc&, const cplx<float>*, hipStream_t);
template hipError_t launch_sticks_inv_n<double>(const cplx<double>*, long, cplx<double>*, int, const Stick*,
                                                const GridDesc&, const cplx<double>*, hipStream_t);
template hipError_t launch_sticks_fwd_n<float>(const cplx<float>*, cplx<float>*, long, int, const Stick*,
                                               const GridDesc&, const cplx<float>*, hipStream_t);
template hipError_t launch_sticks_fwd_n<double>(const cplx<double>*, cplx<double>*, long, int, const Stick*,
                                                const GridDesc&, const cplx<double>*, hipStream_t);

// Sizes with a compile-time plane kernel, N = A B; 108 in FP32 only (its FP64 plane exceeds LDS).
#define PW_PLANE_SIZES(X) \
  X(24, 4, 6) X(27, 3, 9) X(32, 4, 8) X(48, 4, 12) X(54, 6, 9) X(64, 8, 8) X(81, 9, 9) X(96, 8, 12)

template <typename T, int A, int B>
static hipError_t launch_plane_w(cplx<T>* SB, const T* V, int nbatch, const int* colstart, const GridDesc& g,
                                 const cplx<T>* tw, T scale, hipStream_t s) {
  using S = PlaneShape<T, A, B>;
  // LOOP: two rounds of the workgroups a device holds (16 waves per CU at these register counts)
  const int per_cu = std::max(1, std::min((int)(160 * 1024 / S::LDS), 16 / S::NW));
  const int groups = S::LOOP ? std::max(1, std::min(nbatch, 2 * 256 * per_cu / g.n3)) : nbatch;
  hipLaunchKernelGGL((k_plane_w<T, A, B, false>), dim3(g.n3, groups), dim3(64 * S::NW), S::LDS, s, SB, V, colstart, g,
                     tw, scale, nbatch, (const double*)nullptr, 0, (double*)nullptr);
  return hipGetLastError();
}

template <typename T, int A, int B>
static hipError_t launch_density_w(const cplx<T>* SB, int nbatch, const int* colstart, const GridDesc& g,
                                   const cplx<T>* tw, const double* occ, int ngroups, double* part, hipStream_t s) {
  using S = PlaneShape<T, A, B>;
  hipLaunchKernelGGL((k_plane_w<T, A, B, true>), dim3(g.n3, ngroups), dim3(64 * S::NW), S::LDS, s,
                     const_cast<cplx<T>*>(SB), (const T*)nullptr, colstart, g, tw, (T)1, nbatch, occ,
                     ceil_div(nbatch, ngroups), part);
  return hipGetLastError();
}

bool plane_n_supported(int n1, int n2, int real_bytes, size_t max_lds) {
  if (n1 != n2) return false;
  size_t lds = 0;
  switch (n1) {
#define PW_CASE(NN, AA, BB)                                                                     \
  case NN:                                                                                      \
    lds = real_bytes == 4 ? PlaneShape<float, AA, BB>::LDS : PlaneShape<double, AA, BB>::LDS;   \
    break;
    PW_PLANE_SIZES(PW_CASE)
#undef PW_CASE
    case 108:
      if (real_bytes != 4) return false;
      lds = PlaneShape<float, 6, 18>::LDS;
      break;
    case 128:
      lds = (size_t)(128 * 128 + 128) * 2 * real_bytes;
      break;
    default:
      return false;
  }
  return lds <= max_lds;
}

template <typename T>
hipError_t launch_plane_n(cplx<T>* SB, const T* V, int nbatch, const int* colstart, const GridDesc& g,
                          const cplx<T>* tw, T scale, hipStream_t s) {
  if (!alias_free(g)) return hipErrorInvalidValue;
  if constexpr (std::is_same<T, float>::value) {
    if (g.n1 == 128) {
      const size_t lds = (size_t)(128 * 128 + 128) * sizeof(float2);
      hipLaunchKernelGGL(k_plane128<false>, dim3(g.n3, nbatch), dim3(1024), lds, s, SB, V, colstart, g, tw, scale,
                         RsDesc{}, (const float2*)nullptr, 0);
      return hipGetLastError();
    }
    if (g.n1 == 108) return launch_plane_w<T, 6, 18>(SB, V, nbatch, colstart, g, tw, scale, s);
  }
  switch (g.n1) {
#define PW_CASE(NN, AA, BB) \
  case NN:                  \
    return launch_plane_w<T, AA, BB>(SB, V, nbatch, colstart, g, tw, scale, s);
    PW_PLANE_SIZES(PW_CASE)
#undef PW_CASE
    default:
      return hipErrorInvalidValue;
  }
}

// Band groups of the density on planes inside LDS: two rounds of the workgroups that a device holds.
int density_plane_groups(const GridDesc& g, int real_bytes) {
  const size_t lds = (size_t)(g.n1 * g.n2 + g.n1) * 2 * real_bytes;  // a little under the kernel's own
  const int per_cu = std::max(1, std::min((int)(160 * 1024 / lds), 4));
  return std::max(1, 2 * 256 * per_cu / g.n3);
}

template <typename T>
hipError_t launch_density_plane_n(const cplx<T>* SB, int nbatch, const int* colstart, const GridDesc& g,
                                  const cplx<T>* tw, const double* occ, int ngroups, double* part, hipStream_t s) {
  if (!alias_free(g) || nbatch < 1 || ngroups < 1) return hipErrorInvalidValue;
  if constexpr (std::is_same<T, float>::value) {
    if (g.n1 == 108) return launch_density_w<T, 6, 18>(SB, nbatch, colstart, g, tw, occ, ngroups, part, s);
  }
  switch (g.n1) {
#define PW_CASE(NN, AA, BB) \
  case NN:                  \
    return launch_density_w<T, AA, BB>(SB, nbatch, colstart, g, tw, occ, ngroups, part, s);
    PW_PLANE_SIZES(PW_CASE)
#undef PW_CASE
    default:
      return hipErrorInvalidValue;
  }
}
template hipError_t launch_density_plane_n<float>(const cplx<float>*, int, const int*, const GridDesc&,
                                                  const cplx<float>*, const double*, int, double*, hipStream_t);
template hipError_t launch_density_plane_n<double>(const cplx<double>*, int, const int*, const GridDesc&,
                                                   const cplx<double>*, const double*, int, double*, hipStream_t);

void pw_allow_large_lds_plane_n() {
  const int bytes = (int)(160 * 1024);
  auto allow = [&](const void* k) {
    (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  };
#define PW_ALLOW(NN, AA, BB)                                     \
  allow(reinterpret_cast<const void*>(&k_plane_w<float, AA, BB, false>)); \
  allow(reinterpret_cast<const void*>(&k_plane_w<float, AA, BB, true>)); \
  allow(reinterpret_cast<const void*>(&k_plane_w<double, AA, BB, true>)); \
  allow(reinterpret_cast<const void*>(&k_plane_w<double, AA, BB, false>));
  PW_PLANE_SIZES(PW_ALLOW)
#undef PW_ALLOW
  allow(reinterpret_cast<const void*>(&k_plane_w<float, 6, 18, false>));
  allow(reinterpret_cast<const void*>(&k_plane_w<float, 6, 18, true>));
  allow(reinterpret_cast<const void*>(&k_plane128<false>));
  allow(reinterpret_cast<const void*>(&k_plane128<true>));
  allow(reinterpret_cast<const void*>(&k_rs_proj128));
  allow(reinterpret_cast<const void*>(&k_density128));
}

template hipError_t launch_plane_n<float>(cplx<float>*, const float*, int, const int*, const GridDesc&,
                                          const cplx<float>*, float, hipStream_t);
template hipError_t launch_plane_n<double>(cplx<double>*, const double*, int, const int*, const GridDesc&,
                                           const cplx<double>*, double, hipStream_t);

}  // namespace pw

// Pencil form of the plane stage with compile-time line lengths: y inverse (sticks -> G1), x rows
// (inverse, * V, forward, or the charge density), y forward (G1 -> sticks).  G1[band][z][y][xa] holds
// only the active x columns, xa = n1 + n1max, with a row pitch of `pitch` elements.
//
// A line of length N = A B belongs to TT = gcd(A, B) threads of one wave, which exchange between the
// two register stages through the wave's own LDS words: no workgroup barrier after the twiddle table
// is there, 64 / TT lines per wave, and any line length goes with any other.  Complex doubles exchange
// their real and imaginary parts one after the other, so that a wave needs 8 bytes per element in both
// precisions and eight waves of FP64 lines fit a compute unit.
// Bound by the traffic of G1 (written and read twice), which a batch keeps in the last-level cache.
// H X of 1,088 bands on 128^3 in FP64: the three passes take 38, 51 and 85 us per 6 bands (beside the
// projection's stream), the generic passes they replace took 327, 251 and 89 us per 6; 101 bands on
// 32 x 64 x 96 in FP32: 98 us (155 with rows of whole 128 bytes), the generic fused plane 297 us.
#pragma once

#include "fft_small.hpp"
#include "kernels.hpp"

namespace pw {

template <typename T, int A, int B>
struct PencilLine {
  static constexpr int N = A * B, TT = cgcd(A, B), I1 = B / TT, J2 = A / TT;
  static constexpr int LPW = 64 / TT;             // lines per wave
  static constexpr int BP = B % 2 == 0 ? B + 1 : B;  // row pitch of word (k1, n2): odd
  static constexpr int AP = A % 2 == 0 ? A + 1 : A;  // row pitch of word (q2, m1): odd
  static constexpr int W0 = A * BP > B * AP ? A * BP : B * AP;
  static constexpr int PL = (W0 + 23) / 32 * 32 + 8;  // words per line, 8 modulo 32: lines on distinct banks
  static_assert(PL >= W0, "line fits its words");
  static constexpr int WAVES = 4;
  using word = typename std::conditional<std::is_same<T, float>::value, float2, double>::type;

  // r1 (thread t: index a of B-major pairs) -> word (k1, n2); then r2 takes n2 = 0 .. B - 1 of k1 = t + TT j
  static __device__ __forceinline__ void first_to_second(word* w, int t, const cplx<T> (&r1)[I1][A],
                                                         cplx<T> (&r2)[J2][B]) {
    exchange(
        w, [&](int i, int k1) { return k1 * BP + t + TT * i; }, r1, [&](int j, int n2) { return (t + TT * j) * BP + n2; },
        r2);
  }
  // r2 (k1 = t + TT j: q2 = 0 .. B - 1) -> word (q2, m1); then r1 takes m1 = 0 .. A - 1 of q2 = t + TT i
  static __device__ __forceinline__ void second_to_first(word* w, int t, const cplx<T> (&r2)[J2][B],
                                                         cplx<T> (&r1)[I1][A]) {
    exchange(
        w, [&](int j, int q2) { return q2 * AP + t + TT * j; }, r2, [&](int i, int m1) { return (t + TT * i) * AP + m1; },
        r1);
  }
  template <class FW, class FR, int P, int Q, int R, int S>
  static __device__ __forceinline__ void exchange(word* w, FW at_w, const cplx<T> (&from)[P][Q], FR at_r,
                                                  cplx<T> (&to)[R][S]) {
    wave_sync();
    if constexpr (std::is_same<T, float>::value) {
#pragma unroll
      for (int i = 0; i < P; ++i)
#pragma unroll
        for (int k = 0; k < Q; ++k) w[at_w(i, k)] = from[i][k];
      wave_sync();
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int k = 0; k < S; ++k) to[j][k] = w[at_r(j, k)];
    } else {
#pragma unroll
      for (int i = 0; i < P; ++i)
#pragma unroll
        for (int k = 0; k < Q; ++k) w[at_w(i, k)] = from[i][k].x;
      wave_sync();
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int k = 0; k < S; ++k) to[j][k].x = w[at_r(j, k)];
      wave_sync();
#pragma unroll
      for (int i = 0; i < P; ++i)
#pragma unroll
        for (int k = 0; k < Q; ++k) w[at_w(i, k)] = from[i][k].y;
      wave_sync();
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int k = 0; k < S; ++k) to[j][k].y = w[at_r(j, k)];
    }
  }
  // stage 1 of a transform of sign SG: A-point DFTs over n1, then the twiddles W_N^{SG n2 k1}
  template <int SG>
  static __device__ __forceinline__ void stage1(cplx<T> (&r1)[I1][A], int t, const cplx<T>* tw) {
#pragma unroll
    for (int i = 0; i < I1; ++i) {
      const int n2 = t + TT * i;
      SmallDft<T, A, SG>::run(r1[i]);
#pragma unroll
      for (int k1 = 1; k1 < A; ++k1) {
        cplx<T> w = tw[(n2 * k1) % N];
        if (SG > 0) w.y = -w.y;
        r1[i][k1] = cmul<T>(r1[i][k1], w);
      }
    }
  }
};

// Lines of one launch: wave q of the grid takes lines LPW (q mod per) .. of plane z = (q / per) mod n3
// of band q / (per n3).
struct PencilTask {
  int per;     // waves per plane
  long waves;  // in all
};

// sticks -> y inverse -> G1
template <typename T, int A, int B>
__global__ __launch_bounds__(256) void k_pencil_yinv(const cplx<T>* __restrict__ SB, cplx<T>* __restrict__ G1,
                                                     const int* __restrict__ colstart, GridDesc g, int pitch,
                                                     const cplx<T>* __restrict__ twg, PencilTask q) {
  using PL = PencilLine<T, A, B>;
  constexpr int N = PL::N, TT = PL::TT;
  __shared__ cplx<T> tw[N];
  __shared__ typename PL::word ex[PL::WAVES * PL::LPW * PL::PL];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < N; i += 256) tw[i] = twg[i];
  __syncthreads();
  const long task = (long)blockIdx.x * PL::WAVES + wv;
  if (task >= q.waves) return;
  const int l = lane / TT, t = lane % TT;
  const int xa = (int)(task % q.per) * PL::LPW + l;
  const long bz = task / q.per;  // band n3 + z
  const bool act = l < PL::LPW && xa < g.n1a;
  typename PL::word* w = ex + (wv * PL::LPW + (l < PL::LPW ? l : 0)) * PL::PL;
  const cplx<T>* sb = SB + bz * g.nst;
  int cs = 0, m = -1;
  if (act) {
    cs = colstart[xa];
    m = (colstart[xa + 1] - cs - 1) >> 1;
  }
  cplx<T> r1[PL::I1][A], r2[PL::J2][B];
#pragma unroll
  for (int i = 0; i < PL::I1; ++i)
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) {
      const int y = B * n1 + t + TT * i;
      const int n2 = 2 * y < N ? y : y - N;
      r1[i][n1] = (!grid_empty(A * B, B, n1) && n2 <= m && -n2 <= m) ? sb[cs + n2 + m] : mk<T>(0, 0);
    }
  if (l >= PL::LPW) return;  // the lanes past the last line (TT does not divide 64)
  PL::template stage1<+1>(r1, t, tw);
  PL::first_to_second(w, t, r1, r2);
  if (!act) return;
  cplx<T>* out = G1 + bz * g.n2 * pitch + xa;
#pragma unroll
  for (int j = 0; j < PL::J2; ++j) {
    SmallDft<T, B, +1>::run(r2[j]);
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) out[(long)(t + TT * j + A * k2) * pitch] = r2[j][k2];
  }
}

// G1 -> y forward -> sticks * scale
template <typename T, int A, int B>
__global__ __launch_bounds__(256) void k_pencil_yfwd(cplx<T>* __restrict__ SB, const cplx<T>* __restrict__ G1,
                                                     const int* __restrict__ colstart, GridDesc g, int pitch,
                                                     const cplx<T>* __restrict__ twg, T scale, PencilTask q) {
  using PL = PencilLine<T, A, B>;
  constexpr int N = PL::N, TT = PL::TT;
  __shared__ cplx<T> tw[N];
  __shared__ typename PL::word ex[PL::WAVES * PL::LPW * PL::PL];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < N; i += 256) tw[i] = twg[i];
  __syncthreads();
  const long task = (long)blockIdx.x * PL::WAVES + wv;
  if (task >= q.waves) return;
  const int l = lane / TT, t = lane % TT;
  if (l >= PL::LPW) return;
  const int xa = (int)(task % q.per) * PL::LPW + l;
  const long bz = task / q.per;
  const bool act = xa < g.n1a;
  typename PL::word* w = ex + (wv * PL::LPW + l) * PL::PL;
  const cplx<T>* in = G1 + bz * g.n2 * pitch + xa;
  cplx<T> r1[PL::I1][A], r2[PL::J2][B];
#pragma unroll
  for (int i = 0; i < PL::I1; ++i)
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) r1[i][n1] = act ? in[(long)(B * n1 + t + TT * i) * pitch] : mk<T>(0, 0);
  PL::template stage1<-1>(r1, t, tw);
  PL::first_to_second(w, t, r1, r2);
  if (!act) return;
  const int cs = colstart[xa], m = (colstart[xa + 1] - cs - 1) >> 1;
  cplx<T>* sb = SB + bz * g.nst;
#pragma unroll
  for (int j = 0; j < PL::J2; ++j) {
    SmallDft<T, B, -1>::run(r2[j]);
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) {
      const int y = t + TT * j + A * k2;
      const int n2 = 2 * y < N ? y : y - N;
      if (!grid_empty(A * B, A, k2) && n2 <= m && -n2 <= m) sb[cs + n2 + m] = cscale<T>(r2[j][k2], scale);
    }
  }
}

// Inverse x transform of this thread's part of a row: r2[j][k2] = psi at x = t + TT j + A k2.
template <typename T, int A, int B>
__device__ __forceinline__ void pencil_x_inv(const cplx<T>* __restrict__ row, int n1max, bool act, int t,
                                             typename PencilLine<T, A, B>::word* w, const cplx<T>* tw,
                                             cplx<T> (&r1)[PencilLine<T, A, B>::I1][A],
                                             cplx<T> (&r2)[PencilLine<T, A, B>::J2][B]) {
  using PL = PencilLine<T, A, B>;
  constexpr int N = PL::N, TT = PL::TT;
#pragma unroll
  for (int i = 0; i < PL::I1; ++i)
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) {
      const int x = B * n1 + t + TT * i;
      const int k = 2 * x < N ? x : x - N;
      r1[i][n1] = (!grid_empty(A * B, B, n1) && act && k <= n1max && -k <= n1max) ? row[k + n1max] : mk<T>(0, 0);
    }
  PL::template stage1<+1>(r1, t, tw);
  PL::first_to_second(w, t, r1, r2);
#pragma unroll
  for (int j = 0; j < PL::J2; ++j) SmallDft<T, B, +1>::run(r2[j]);
}

// x rows of G1 in place: inverse, * V, forward.  A wave takes its rows of `bands` bands one after the
// other, with the rows of V in registers.
template <typename T, int A, int B>
__global__ __launch_bounds__(256) void k_pencil_x(cplx<T>* __restrict__ G1, const T* __restrict__ V, GridDesc g,
                                                  int pitch, const cplx<T>* __restrict__ twg, int nbatch, int bands,
                                                  PencilTask q) {
  using PL = PencilLine<T, A, B>;
  constexpr int N = PL::N, TT = PL::TT;
  __shared__ cplx<T> tw[N];
  __shared__ typename PL::word ex[PL::WAVES * PL::LPW * PL::PL];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < N; i += 256) tw[i] = twg[i];
  __syncthreads();
  const long task = (long)blockIdx.x * PL::WAVES + wv;
  if (task >= q.waves) return;
  const int l = lane / TT, t = lane % TT;
  if (l >= PL::LPW) return;
  const int y = (int)(task % q.per) * PL::LPW + l;
  const long gz = task / q.per;
  const int z = (int)(gz % g.n3), b0 = (int)(gz / g.n3) * bands, b1 = min(nbatch, b0 + bands);
  const bool act = y < g.n2;
  typename PL::word* w = ex + (wv * PL::LPW + l) * PL::PL;
  T vr[PL::J2][B];
  {
    const T* vz = V + ((long)z * g.n2 + (act ? y : 0)) * N + t;
#pragma unroll
    for (int j = 0; j < PL::J2; ++j)
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) vr[j][k2] = vz[TT * j + A * k2];
  }
  for (int b = b0; b < b1; ++b) {
    cplx<T>* row = G1 + (((long)b * g.n3 + z) * g.n2 + (act ? y : 0)) * pitch;
    cplx<T> r1[PL::I1][A], r2[PL::J2][B];
    pencil_x_inv<T, A, B>(row, g.n1max, act, t, w, tw, r1, r2);
#pragma unroll
    for (int j = 0; j < PL::J2; ++j) {
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) r2[j][k2] = cscale<T>(r2[j][k2], vr[j][k2]);
      SmallDft<T, B, -1>::run(r2[j]);  // over m2, output q2
#pragma unroll
      for (int q2 = 1; q2 < B; ++q2) r2[j][q2] = cmul<T>(r2[j][q2], tw[((t + TT * j) * q2) % N]);
    }
    PL::second_to_first(w, t, r2, r1);
#pragma unroll
    for (int i = 0; i < PL::I1; ++i) {
      SmallDft<T, A, -1>::run(r1[i]);  // r1[i][q1] = F[B q1 + q2]
#pragma unroll
      for (int q1 = 0; q1 < A; ++q1) {
        const int x = B * q1 + t + TT * i;
        const int k = 2 * x < N ? x : x - N;
        if (!grid_empty(A * B, B, q1) && act && k <= g.n1max && -k <= g.n1max) row[k + g.n1max] = r1[i][q1];
      }
    }
  }
}

// Charge density of the x rows: part[group][z][y][x] = sum over the group's bands, in order, of occ |psi|^2
// (FP64, |psi|^2 in the compute precision).  Group p takes bands p per_group ..
template <typename T, int A, int B>
__global__ __launch_bounds__(256) void k_pencil_density(const cplx<T>* __restrict__ G1, GridDesc g, int pitch,
                                                        const cplx<T>* __restrict__ twg, int nbatch, int per_group,
                                                        const double* __restrict__ occ, double* __restrict__ part,
                                                        PencilTask q) {
  using PL = PencilLine<T, A, B>;
  constexpr int N = PL::N, TT = PL::TT;
  __shared__ cplx<T> tw[N];
  __shared__ typename PL::word ex[PL::WAVES * PL::LPW * PL::PL];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < N; i += 256) tw[i] = twg[i];
  __syncthreads();
  const long task = (long)blockIdx.x * PL::WAVES + wv;
  if (task >= q.waves) return;
  const int l = lane / TT, t = lane % TT;
  if (l >= PL::LPW) return;
  const int y = (int)(task % q.per) * PL::LPW + l;
  const long gz = task / q.per;
  const int z = (int)(gz % g.n3), grp = (int)(gz / g.n3);
  const int b0 = grp * per_group, b1 = min(nbatch, b0 + per_group);
  const bool act = y < g.n2;
  typename PL::word* w = ex + (wv * PL::LPW + l) * PL::PL;
  double acc[PL::J2][B] = {};
  for (int b = b0; b < b1; ++b) {
    const cplx<T>* row = G1 + (((long)b * g.n3 + z) * g.n2 + (act ? y : 0)) * pitch;
    cplx<T> r1[PL::I1][A], r2[PL::J2][B];
    pencil_x_inv<T, A, B>(row, g.n1max, act, t, w, tw, r1, r2);
    const double o = occ[b];
#pragma unroll
    for (int j = 0; j < PL::J2; ++j)
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2)
        acc[j][k2] += o * (double)(r2[j][k2].x * r2[j][k2].x + r2[j][k2].y * r2[j][k2].y);
  }
  if (!act) return;
  double* dst = part + (((long)grp * g.n3 + z) * g.n2 + y) * N + t;
#pragma unroll
  for (int j = 0; j < PL::J2; ++j)
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) dst[TT * j + A * k2] = acc[j][k2];
}

// N, A, B: at most 24 elements per thread
#define PW_PENCIL_SIZES(X)                                                                                        \
  X(24, 4, 6) X(27, 3, 9) X(32, 4, 8) X(36, 6, 6) X(48, 4, 12) X(54, 6, 9) X(64, 8, 8) X(72, 6, 12) X(81, 9, 9)   \
  X(96, 8, 12) X(108, 6, 18) X(128, 8, 16) X(144, 12, 12) X(162, 9, 18) X(192, 8, 24)

template <typename T, int A, int B>
PencilTask pencil_tasks(int lines, long planes) {
  PencilTask q;
  q.per = ceil_div(lines, PencilLine<T, A, B>::LPW);
  q.waves = (long)q.per * planes;
  return q;
}

template <typename T>
hipError_t launch_pencil_yinv_n(const cplx<T>* SB, cplx<T>* G1, int nbatch, const int* colstart, const GridDesc& g,
                                int pitch, const cplx<T>* tw2, hipStream_t s) {
  if (g.n2max > plane_top(g.n2)) return hipErrorInvalidValue;
  switch (g.n2) {
#define PW_CASE(NN, AA, BB)                                                                                         \
  case NN: {                                                                                                        \
    const PencilTask q = pencil_tasks<T, AA, BB>(g.n1a, (long)g.n3 * nbatch);                                       \
    hipLaunchKernelGGL((k_pencil_yinv<T, AA, BB>), dim3(ceil_div(q.waves, 4)), dim3(256), 0, s, SB, G1, colstart, g, \
                       pitch, tw2, q);                                                                              \
    return hipGetLastError();                                                                                       \
  }
    PW_PENCIL_SIZES(PW_CASE)
#undef PW_CASE
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_pencil_yfwd_n(cplx<T>* SB, const cplx<T>* G1, int nbatch, const int* colstart, const GridDesc& g,
                                int pitch, const cplx<T>* tw2, T scale, hipStream_t s) {
  if (g.n2max > plane_top(g.n2)) return hipErrorInvalidValue;
  switch (g.n2) {
#define PW_CASE(NN, AA, BB)                                                                                         \
  case NN: {                                                                                                        \
    const PencilTask q = pencil_tasks<T, AA, BB>(g.n1a, (long)g.n3 * nbatch);                                       \
    hipLaunchKernelGGL((k_pencil_yfwd<T, AA, BB>), dim3(ceil_div(q.waves, 4)), dim3(256), 0, s, SB, G1, colstart, g, \
                       pitch, tw2, scale, q);                                                                       \
    return hipGetLastError();                                                                                       \
  }
    PW_PENCIL_SIZES(PW_CASE)
#undef PW_CASE
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_pencil_x_n(cplx<T>* G1, const T* V, int nbatch, const GridDesc& g, int pitch, const cplx<T>* tw1,
                             hipStream_t s) {
  if (g.n1max > plane_top(g.n1)) return hipErrorInvalidValue;
  switch (g.n1) {
#define PW_CASE(NN, AA, BB)                                                                                       \
  case NN: {                                                                                                      \
    /* bands per wave: V is read once for them; at least 4,096 waves (two per SIMD) stay in flight */             \
    const long one = pencil_tasks<T, AA, BB>(g.n2, (long)g.n3 * nbatch).waves;                                    \
    int bands = (int)(one / 4096);                                                                                \
    bands = bands < 1 ? 1 : bands > 4 ? 4 : bands;                                                                \
    const PencilTask q = pencil_tasks<T, AA, BB>(g.n2, (long)g.n3 * ceil_div(nbatch, bands));                     \
    hipLaunchKernelGGL((k_pencil_x<T, AA, BB>), dim3(ceil_div(q.waves, 4)), dim3(256), 0, s, G1, V, g, pitch, tw1, \
                       nbatch, bands, q);                                                                         \
    return hipGetLastError();                                                                                     \
  }
    PW_PENCIL_SIZES(PW_CASE)
#undef PW_CASE
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_pencil_density_n(const cplx<T>* G1, int nbatch, const GridDesc& g, int pitch, const cplx<T>* tw1,
                                   const double* occ, int ngroups, double* part, hipStream_t s) {
  const int per = ceil_div(nbatch, ngroups);
  if (g.n1max > plane_top(g.n1)) return hipErrorInvalidValue;
  switch (g.n1) {
#define PW_CASE(NN, AA, BB)                                                                                        \
  case NN: {                                                                                                       \
    const PencilTask q = pencil_tasks<T, AA, BB>(g.n2, (long)g.n3 * ngroups);                                      \
    hipLaunchKernelGGL((k_pencil_density<T, AA, BB>), dim3(ceil_div(q.waves, 4)), dim3(256), 0, s, G1, g, pitch, tw1, \
                       nbatch, per, occ, part, q);                                                                 \
    return hipGetLastError();                                                                                      \
  }
    PW_PENCIL_SIZES(PW_CASE)
#undef PW_CASE
  }
  return hipErrorInvalidValue;
}

#define PW_INST_PENCIL(T)                                                                                          \
  template hipError_t launch_pencil_yinv_n<T>(const cplx<T>*, cplx<T>*, int, const int*, const GridDesc&, int,     \
                                              const cplx<T>*, hipStream_t);                                        \
  template hipError_t launch_pencil_yfwd_n<T>(cplx<T>*, const cplx<T>*, int, const int*, const GridDesc&, int,     \
                                              const cplx<T>*, T, hipStream_t);                                     \
  template hipError_t launch_pencil_x_n<T>(cplx<T>*, const T*, int, const GridDesc&, int, const cplx<T>*,          \
                                           hipStream_t);                                                           \
  template hipError_t launch_pencil_density_n<T>(const cplx<T>*, int, const GridDesc&, int, const cplx<T>*,        \
                                                 const double*, int, double*, hipStream_t);

}  // namespace pw

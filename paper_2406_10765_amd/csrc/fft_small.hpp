// In-register DFTs of compile-time size with compile-time twiddles, shared by the sized FFT kernels
// (fft_plane.hip, fft_pencil.hpp).
#pragma once

#include <type_traits>
#include <utility>

#include "common.hpp"
#include "fft_trig.hpp"

namespace pw {

// static loop: f(std::integral_constant<int, i>) for i in [0, N)
template <typename F, int... I>
__device__ __forceinline__ void sfor_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void sfor(F&& f) {
  sfor_impl(f, std::make_integer_sequence<int, N>{});
}

// In-register DFT of compile-time size S with sign SG (+1 inverse, -1 forward), natural order.
template <typename T, int S, int SG>
struct SmallDft {
  static __device__ __forceinline__ void run(cplx<T>* v) {
    if constexpr (S == 1) {
      return;
    } else if constexpr (S == 2) {
      const cplx<T> a = v[0], b = v[1];
      v[0] = cadd<T>(a, b);
      v[1] = csub<T>(a, b);
    } else if constexpr (S == 3) {
      const T h = (T)0.86602540378443864676;
      const cplx<T> t1 = cadd<T>(v[1], v[2]), t2 = csub<T>(v[1], v[2]);
      const cplx<T> m = mk<T>(v[0].x - (T)0.5 * t1.x, v[0].y - (T)0.5 * t1.y);
      const cplx<T> r = cmuli<T>(cscale<T>(t2, h), SG);
      v[0] = cadd<T>(v[0], t1);
      v[1] = cadd<T>(m, r);
      v[2] = csub<T>(m, r);
    } else if constexpr (S == 4) {
      const cplx<T> s02 = cadd<T>(v[0], v[2]), d02 = csub<T>(v[0], v[2]);
      const cplx<T> s13 = cadd<T>(v[1], v[3]);
      const cplx<T> d13 = cmuli<T>(csub<T>(v[1], v[3]), SG);
      v[0] = cadd<T>(s02, s13);
      v[2] = csub<T>(s02, s13);
      v[1] = cadd<T>(d02, d13);
      v[3] = csub<T>(d02, d13);
    } else {
      // S = F * G with F the first radix (4, 2 or 3): n = G f + g, k = kf + F kg
      constexpr int F = (S % 4 == 0) ? 4 : (S % 2 == 0) ? 2 : 3;
      constexpr int G = S / F;
      cplx<T> t[G][F];
      sfor<G>([&](auto gi) {
        constexpr int g = decltype(gi)::value;
        cplx<T> u[F];
#pragma unroll
        for (int f = 0; f < F; ++f) u[f] = v[G * f + g];
        SmallDft<T, F, SG>::run(u);
        sfor<F>([&](auto ki) {
          constexpr int kf = decltype(ki)::value;
          if constexpr (g * kf != 0 && 4 * g * kf % S == 0) {  // a quarter, half or three quarter turn
            constexpr int q = 4 * g * kf / S % 4;
            u[kf] = q == 2 ? mk<T>(-u[kf].x, -u[kf].y) : cmuli<T>(u[kf], q == 1 ? SG : -SG);
          } else if constexpr (g * kf != 0) {
            constexpr T wc = (T)turn_cos(g * kf, S), ws = (T)turn_sin(SG * g * kf, S);
            static_assert(wc <= 1 && wc >= -1 && ws <= 1 && ws >= -1, "a constant for every angle");
            u[kf] = cmul<T>(u[kf], mk<T>(wc, ws));
          }
          t[g][kf] = u[kf];
        });
      });
#pragma unroll
      for (int kf = 0; kf < F; ++kf) {
        cplx<T> w[G];
#pragma unroll
        for (int g = 0; g < G; ++g) w[g] = t[g][kf];
        SmallDft<T, G, SG>::run(w);
#pragma unroll
        for (int kg = 0; kg < G; ++kg) v[kf + F * kg] = w[kg];
      }
    }
  }
};

// Largest |n| that the sized kernels carry on N points.  A plan has N >= 3 nmax + 1 points along each axis with
// nmax = floor(sqrt(2 ecut) L / 2 pi), rounded.  Across the planes no stick lies beyond nmax; along z a stick
// reaches nmax + 1 where the cutoff falls on a shell and rounding took nmax below it.
constexpr int plane_top(int N) { return (N - 1) / 3; }
constexpr int stick_top(int N) { return (N - 1) / 3 + 1; }
// Points top < e < N - top hold no plane wave: whether the points S block .. S block + S - 1 are all empty, whatever
// the sphere.  The sized kernels leave out the loads, terms and stores of such blocks; their launchers check the
// sphere against the top.
__device__ __host__ __forceinline__ constexpr bool points_empty(int N, int S, int block, int top) {
  return S * block > top && S * block + S - 1 < N - top;
}
__device__ __host__ __forceinline__ constexpr bool grid_empty(int N, int S, int block) {  // across the planes
  return points_empty(N, S, block, plane_top(N));
}

constexpr int cgcd(int a, int b) { return b == 0 ? a : cgcd(b, a % b); }

// Orders a wave's LDS accesses before and after it (lines whose threads sit in one wave exchange through
// LDS without a workgroup barrier).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
}  // namespace pw

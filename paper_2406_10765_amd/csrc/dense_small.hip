// Dense steps of the Rayleigh-Ritz problem H_s C = S C diag(lambda) for small blocks (up to kDenseMax bands):
// Cholesky factor, reduction to standard form, Householder tridiagonalisation and the way back.  The
// tridiagonal problem itself stays with the library.
//
// These are chains of n dependent steps on at most 331 KB: bound by the latency of a step.  The two
// factorisations run in one workgroup with the matrix in registers (12 waves: row 4 w + l / 16 + 48 a, column
// l % 16 + 16 b of lane l of wave w), so that a step costs one or two workgroup barriers and the sums over a row
// stay in sixteen neighbouring lanes.  The triangular solves and the reflectors act on each column by itself:
// a wave per column, its rows in registers, no barrier at all.
// 40 and 144 bands (us): Cholesky 28 and 205, reduction 20 and 72, tridiagonal form 69 and 518, reflectors and last
// solve 18 and 79; the library took 900 and 3,700 for the four (at 40 bands 41, 152, 207 and 500, the last in
// 118 launches).

#include "common.hpp"
#include "fft_small.hpp"
#include "kernels.hpp"

namespace pw {

namespace {

constexpr int kWaves = 12, kRows = 4 * kWaves, kDenseMax = 3 * kRows;

template <int CTRL>
__device__ __forceinline__ double ror_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
// sum over each row of 16 lanes, in all of them
__device__ __forceinline__ double row_sum(double v) {
  v = ror_add<0x128>(v);
  v = ror_add<0x124>(v);
  v = ror_add<0x122>(v);
  return ror_add<0x121>(v);
}
__device__ __forceinline__ double lane_of(double v, int k) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k),
                          __builtin_amdgcn_readlane(__double2loint(v), k));
}
__device__ __forceinline__ double wave_sum(double v) {
  v = row_sum(v);
  return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}
__device__ __forceinline__ double2 cz() { return make_double2(0.0, 0.0); }
// c + a b, c + a conj(b), c - a b, c - a conj(b)
__device__ __forceinline__ double2 fma_ab(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 fms_ab(double2 a, double2 b, double2 c) {
  return make_double2(fma(-a.x, b.x, fma(a.y, b.y, c.x)), fma(-a.x, b.y, fma(-a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 fms_abc(double2 a, double2 b, double2 c) {
  return make_double2(fma(-a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(-a.y, b.x, c.y)));
}

// S = L L^H in the lower triangle of S (n x n); info = 0, or 1 + the first column whose pivot is not positive.
template <int NA>
__global__ __launch_bounds__(64 * kWaves) void k_potrf_small(double2* __restrict__ S, int n, int* __restrict__ info) {
  constexpr int NB = 3 * NA;
  __shared__ double2 x[2][kDenseMax];  // column k, by parity of k
  const int tid = threadIdx.x, lane = tid & 63, r0 = 4 * (tid >> 6) + (lane >> 4), c0 = lane & 15;
  double2 m[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int r = r0 + kRows * a, c = c0 + 16 * b;
      m[a][b] = (r < n && c <= r) ? S[r + (long)c * n] : cz();
    }
  if (c0 == 0)
#pragma unroll
    for (int a = 0; a < NA; ++a) x[0][r0 + kRows * a] = m[a][0];
  __syncthreads();
  int bad = 0;
  for (int k = 0; k < n; ++k) {
    const double2* xk = x[k & 1];
    const double d = xk[k].x;
    if (!(d > 0.0)) {  // the same in every thread
      bad = k + 1;
      break;
    }
    const double rd = 1.0 / d;
    if (tid < n - k) {
      const double rt = sqrt(d);
      const double2 v = xk[k + tid];
      S[k + tid + (long)k * n] = tid == 0 ? make_double2(rt, 0.0) : make_double2(v.x / rt, v.y / rt);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (16 * b + 15 > k) {
        double2 xc = xk[c0 + 16 * b];
        xc.x *= rd;
        xc.y *= rd;
#pragma unroll
        for (int a = 0; a < NA; ++a)
          if (kRows * a + kRows - 1 > k && kRows * a + kRows > 16 * b)
            m[a][b] = fms_abc(xk[r0 + kRows * a], xc, m[a][b]);
      }
    }
    if (c0 == ((k + 1) & 15)) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b == ((k + 1) >> 4))
#pragma unroll
          for (int a = 0; a < NA; ++a) x[(k + 1) & 1][r0 + kRows * a] = m[a][b];
    }
    __syncthreads();
  }
  if (tid == 0) *info = bad;
}

// Q^H A Q = T, A Hermitian (lower triangle read), Q = H_0 H_1 .. H_{n-2}, H_k = I - tau_k v_k v_k^H with v_k zero up
// to row k and one in row k + 1 (the convention of LAPACK's zhetd2, lower): whole columns v_k to V, the diagonal
// and subdiagonal of T to D and E.
template <int NA>
__global__ __launch_bounds__(64 * kWaves) void k_hetrd_small(const double2* __restrict__ A, int n,
                                                            double2* __restrict__ V, double2* __restrict__ tau,
                                                            double* __restrict__ D, double* __restrict__ E) {
  constexpr int NB = 3 * NA, R = (kRows * NA + 63) / 64;
  __shared__ double2 x[64 * R], y[64 * R], v[64 * R], w[64 * R];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r0 = 4 * wave + (lane >> 4), c0 = lane & 15;
  double2 m[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int r = r0 + kRows * a, c = c0 + 16 * b;
      m[a][b] = cz();
      if (r < n && c < n) {
        m[a][b] = r >= c ? A[r + (long)c * n] : A[c + (long)r * n];
        if (r < c) m[a][b].y = -m[a][b].y;
        if (r == c) m[a][b].y = 0.0;
      }
    }
  for (int i = tid; i < 64 * R; i += 64 * kWaves) x[i] = y[i] = cz();
  __syncthreads();
  // column k below the diagonal to x, its diagonal entry to D
  auto column = [&](int k) {
    if (c0 == (k & 15)) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (b == (k >> 4))
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            const int r = r0 + kRows * a;
            x[r] = r > k ? m[a][b] : cz();
            if (r == k) D[k] = m[a][b].x;
          }
    }
  };
  column(0);
  __syncthreads();
  for (int k = 0; k + 1 < n; ++k) {
    // every wave makes the whole reflector: no barrier between its parts (all write the same values)
    double2 xv[R];
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      xv[j] = x[lane + 64 * j];
      if (lane + 64 * j > k + 1) s = fma(xv[j].x, xv[j].x, fma(xv[j].y, xv[j].y, s));
    }
    s = wave_sum(s);
    double2 al = x[k + 1];
    double down = 1.0;
    if (const double t = fma(al.x, al.x, fma(al.y, al.y, s)); !(t > 1e-270 && t < 1e270)) {
      // squares near or beyond the ends of the range (a zero column too): the same column times 2^600 or 2^-600
      const double up = t < 1.0 ? 0x1p600 : 0x1p-600;
      down = t < 1.0 ? 0x1p-600 : 0x1p600;
      al.x *= up;
      al.y *= up;
      s = 0.0;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        xv[j].x *= up;
        xv[j].y *= up;
        if (lane + 64 * j > k + 1) s = fma(xv[j].x, xv[j].x, fma(xv[j].y, xv[j].y, s));
      }
      s = wave_sum(s);
    }
    double beta = al.x;
    double2 tk = cz(), sc = cz();
    if (s != 0.0 || al.y != 0.0) {
      beta = -copysign(sqrt(fma(al.x, al.x, fma(al.y, al.y, s))), al.x);
      const double rb = 1.0 / beta, dx = al.x - beta, rn = 1.0 / fma(dx, dx, al.y * al.y);
      tk = make_double2((beta - al.x) * rb, -al.y * rb);
      sc = make_double2(dx * rn, -al.y * rn);  // 1 / (alpha - beta)
    }
    double2 vv[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int i = lane + 64 * j;
      vv[j] = fma_ab(xv[j], sc, cz());
      if (i == k + 1) vv[j] = make_double2(1.0, 0.0);
      v[i] = vv[j];
      if (wave == 0 && i < n) V[i + (long)k * n] = vv[j];
    }
    if (tid == 0) {
      tau[k] = tk;
      E[k] = beta * down;
    }
    wave_sync();
    // y = A v, rows below k
    double2 acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = cz();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (16 * b + 15 > k) {
        const double2 vc = v[c0 + 16 * b];
#pragma unroll
        for (int a = 0; a < NA; ++a)
          if (kRows * a + kRows - 1 > k) acc[a] = fma_ab(m[a][b], vc, acc[a]);
      }
    }
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      if (kRows * a + kRows - 1 > k) {
        acc[a].x = row_sum(acc[a].x);
        acc[a].y = row_sum(acc[a].y);
        const int r = r0 + kRows * a;
        if (c0 == 0) y[r] = r > k ? acc[a] : cz();
      }
    }
    __syncthreads();
    // w = tau y - (|tau|^2 / 2) (y^H v) v, y^H v real
    double2 yv[R];
    double dt = 0.0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      yv[j] = lane + 64 * j > k ? y[lane + 64 * j] : cz();
      dt = fma(yv[j].x, vv[j].x, fma(yv[j].y, vv[j].y, dt));
    }
    const double ah = -0.5 * fma(tk.x, tk.x, tk.y * tk.y) * wave_sum(dt);
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double2 wv = fma_ab(tk, yv[j], cz());
      wv.x = fma(ah, vv[j].x, wv.x);
      wv.y = fma(ah, vv[j].y, wv.y);
      w[lane + 64 * j] = wv;
    }
    wave_sync();
    // A -= v w^H + w v^H
    double2 vr[NA], wr[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      vr[a] = v[r0 + kRows * a];
      wr[a] = w[r0 + kRows * a];
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (16 * b + 15 > k) {
        const double2 vc = v[c0 + 16 * b], wc = w[c0 + 16 * b];
#pragma unroll
        for (int a = 0; a < NA; ++a)
          if (kRows * a + kRows - 1 > k) m[a][b] = fms_abc(wr[a], vc, fms_abc(vr[a], wc, m[a][b]));
      }
    }
    column(k + 1);
    __syncthreads();
  }
}

// out = L^{-1} B, or L^{-1} B^H (adj); a wave per column of out, lane l with rows l + 64 j.
template <int R>
__global__ __launch_bounds__(256) void k_lsolve_small(const double2* __restrict__ L, const double2* __restrict__ B,
                                                      int n, bool adj, double2* __restrict__ out) {
  const int lane = threadIdx.x & 63, c = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= n) return;
  double2 b[R];
  double rd[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int i = min(lane + 64 * j, n - 1);
    rd[j] = 1.0 / L[i + (long)i * n].x;
    b[j] = adj ? B[c + (long)i * n] : B[i + (long)c * n];
    if (adj) b[j].y = -b[j].y;
  }
#pragma unroll
  for (int jk = 0; jk < R; ++jk) {
    const int kn = min(64, n - 64 * jk);
#pragma unroll 4
    for (int kl = 0; kl < kn; ++kl) {
      const int k = 64 * jk + kl;
      double2 l[R];
#pragma unroll
      for (int j = jk; j < R; ++j) {
        const int i = lane + 64 * j;
        l[j] = (i > k && i < n) ? L[i + (long)k * n] : cz();
      }
      const double2 t = make_double2(b[jk].x * rd[jk], b[jk].y * rd[jk]);
      const double2 xk = make_double2(lane_of(t.x, kl), lane_of(t.y, kl));
      if (lane == kl) b[jk] = t;
#pragma unroll
      for (int j = jk; j < R; ++j) b[j] = fms_ab(l[j], xk, b[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < R; ++j)
    if (lane + 64 * j < n) out[lane + 64 * j + (long)c * n] = b[j];
}

// C = L^{-H} Q Z, Q as k_hetrd_small leaves it, Z real; a wave per column.
template <int R>
__global__ __launch_bounds__(256) void k_back_small(const double2* __restrict__ V, const double2* __restrict__ tau,
                                                    const double2* __restrict__ L, const double* __restrict__ Z, int n,
                                                    double2* __restrict__ C) {
  const int lane = threadIdx.x & 63, c = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= n) return;
  double2 z[R];
  double rd[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int i = lane + 64 * j;
    z[j] = i < n ? make_double2(Z[i + (long)c * n], 0.0) : cz();
    rd[j] = i < n ? 1.0 / L[i + (long)i * n].x : 0.0;
  }
  double2 vn[R];
  auto fetch = [&](int k) {
#pragma unroll
    for (int j = 0; j < R; ++j) vn[j] = lane + 64 * j < n ? V[lane + 64 * j + (long)k * n] : cz();
  };
  fetch(n - 2);
  double2 tn = tau[n - 2];
  for (int k = n - 2; k >= 0; --k) {
    double2 v[R];
#pragma unroll
    for (int j = 0; j < R; ++j) v[j] = vn[j];
    const double2 t = tn;
    if (k > 0) {
      fetch(k - 1);
      tn = tau[k - 1];
    }
    double sx = 0.0, sy = 0.0;  // v^H z
#pragma unroll
    for (int j = 0; j < R; ++j) {
      sx = fma(v[j].x, z[j].x, fma(v[j].y, z[j].y, sx));
      sy = fma(v[j].x, z[j].y, fma(-v[j].y, z[j].x, sy));
    }
    const double2 f = fma_ab(t, make_double2(wave_sum(sx), wave_sum(sy)), cz());
#pragma unroll
    for (int j = 0; j < R; ++j) z[j] = fms_ab(v[j], f, z[j]);
  }
#pragma unroll
  for (int jk = R - 1; jk >= 0; --jk) {
    const int kn = min(64, n - 64 * jk);
#pragma unroll 4
    for (int kl = kn - 1; kl >= 0; --kl) {
      const int k = 64 * jk + kl;
      double2 l[R];
#pragma unroll
      for (int j = 0; j <= jk; ++j) {
        const int i = lane + 64 * j;
        l[j] = i < k ? L[k + (long)i * n] : cz();
      }
      const double2 t = make_double2(z[jk].x * rd[jk], z[jk].y * rd[jk]);
      const double2 xk = make_double2(lane_of(t.x, kl), lane_of(t.y, kl));
      if (lane == kl) z[jk] = t;
#pragma unroll
      for (int j = 0; j <= jk; ++j) z[j] = fms_abc(xk, l[j], z[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < R; ++j)
    if (lane + 64 * j < n) C[lane + 64 * j + (long)c * n] = z[j];
}

}  // namespace

// From 4 bands (the library's own quick returns below) to what twelve waves hold in registers: at 144 bands these
// steps take 870 us, the library's 3,700.  More rows per wave or a blocked form beyond have not been measured.
bool dense_small_supported(int n) { return n >= 4 && n <= kDenseMax; }

hipError_t launch_potrf_small(double2* S, int n, int* info, hipStream_t s) {
  if (!dense_small_supported(n)) return hipErrorInvalidValue;
  if (n <= kRows) hipLaunchKernelGGL(k_potrf_small<1>, dim3(1), dim3(64 * kWaves), 0, s, S, n, info);
  else if (n <= 2 * kRows) hipLaunchKernelGGL(k_potrf_small<2>, dim3(1), dim3(64 * kWaves), 0, s, S, n, info);
  else hipLaunchKernelGGL(k_potrf_small<3>, dim3(1), dim3(64 * kWaves), 0, s, S, n, info);
  return hipGetLastError();
}

hipError_t launch_hetrd_small(const double2* A, int n, double2* V, double2* tau, double* D, double* E, hipStream_t s) {
  if (!dense_small_supported(n)) return hipErrorInvalidValue;
  if (n <= kRows) hipLaunchKernelGGL(k_hetrd_small<1>, dim3(1), dim3(64 * kWaves), 0, s, A, n, V, tau, D, E);
  else if (n <= 2 * kRows) hipLaunchKernelGGL(k_hetrd_small<2>, dim3(1), dim3(64 * kWaves), 0, s, A, n, V, tau, D, E);
  else hipLaunchKernelGGL(k_hetrd_small<3>, dim3(1), dim3(64 * kWaves), 0, s, A, n, V, tau, D, E);
  return hipGetLastError();
}

hipError_t launch_standard_small(const double2* L, double2* H, int n, double2* X, hipStream_t s) {
  if (!dense_small_supported(n)) return hipErrorInvalidValue;
  const dim3 grid(ceil_div(n, 4));
#define PW_LS(R)                                                                              \
  hipLaunchKernelGGL(k_lsolve_small<R>, grid, dim3(256), 0, s, L, (const double2*)H, n, false, X); \
  hipLaunchKernelGGL(k_lsolve_small<R>, grid, dim3(256), 0, s, L, (const double2*)X, n, true, H)
  if (n <= 64) {
    PW_LS(1);
  } else if (n <= 128) {
    PW_LS(2);
  } else {
    PW_LS(3);
  }
#undef PW_LS
  return hipGetLastError();
}

hipError_t launch_back_small(const double2* V, const double2* tau, const double2* L, const double* Z, int n, double2* C,
                             hipStream_t s) {
  if (!dense_small_supported(n)) return hipErrorInvalidValue;
  const dim3 grid(ceil_div(n, 4));
  if (n <= 64) hipLaunchKernelGGL(k_back_small<1>, grid, dim3(256), 0, s, V, tau, L, Z, n, C);
  else if (n <= 128) hipLaunchKernelGGL(k_back_small<2>, grid, dim3(256), 0, s, V, tau, L, Z, n, C);
  else hipLaunchKernelGGL(k_back_small<3>, grid, dim3(256), 0, s, V, tau, L, Z, n, C);
  return hipGetLastError();
}

}  // namespace pw

// GEMMs on the CDNA matrix cores (MFMA 16x16x4, fp64 or fp32).
//
// The dense contractions of the step (Section II-B: S = Psi^*(H Psi), and the
// per-atom pseudopotential application of Section III-A recast as projector
// GEMMs) reduce to two shapes of complex products and their forms on pairs
// (G, -G) for the projectors, which are real functions of position (below):
//   * "cn": C = A^H B with a very long inner dimension K = N_pw (Gram Y^H Y,
//     projected Hamiltonian Y^H W; projections beta^H Y).  Split over K; each
//     split writes complex-double partials that a second kernel sums in a
//     fixed order (deterministic, no atomics).  In fp32 the MFMA accumulators
//     are moved into fp64 registers every 256 K values, so the long sums keep
//     fp64-like accuracy.
//   * "nn": C = A B with K = N_b or N_proj and M = N_pw rows (rotation Y C;
//     beta (D P), whose epilogue assembles H Y or the Chebyshev update).
//
// Complex products run as four real MFMAs on the (re, im) planes:
//   conj(a) b: re += ar br + ai bi, im += ar bi - ai br
//   a b:       re += ar br - ai bi, im += ar bi + ai br
// MFMA 16x16x4 lane layout: operand A[i][k] comes from lane i + 16 k and
// operand B[k][j] from lane j + 16 k for both precisions; accumulator element r
// of lane l holds C[4 (l / 16) + r][l % 16] for f32 but C[l / 16 + 4 r][l % 16]
// for f64 (measured with one-hot operands on gfx950).
//
// The complex products and the nonlocal product on pairs read their operands from global memory
// straight into the lanes' MFMA layout, a wave per tile, with no LDS and no barrier between waves
// (below); the projection on pairs goes through two LDS buffers, so each K tile costs one barrier,
// with the next one's global loads in registers meanwhile.  Tiles are handed out XCD by XCD: consecutive
// tiles, which share operand panels, run on the same L2.

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace pw {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <typename T> struct MF;
template <> struct MF<double> {
  using acc = v4d;
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <> struct MF<float> {
  using acc = v4f;
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

constexpr int kXcd = 8;  // XCDs per MI355X

// Tile index -> (tm, tn, split) with the tiles of one XCD contiguous.  Launch order
// sends workgroup w to XCD w % 8.
__device__ __forceinline__ int xcd_tile(int w, int total) {
  const int per = total / kXcd, rem = total % kXcd;
  const int x = w % kXcd, i = w / kXcd;
  // XCDs 0..rem-1 get per + 1 tiles, the others per
  return x < rem ? x * (per + 1) + i : rem * (per + 1) + (x - rem) * per + i;
}

// K value u of lane group q (0..3) among the eight of a step: whole 64-byte pieces of a column per load in
// fp64, 16-byte loads in fp32
template <typename T>
__device__ __forceinline__ constexpr int koff(int q, int u) {
  return std::is_same<T, double>::value ? 4 * u + q : 2 * q + u;
}

// ------------------------------------------------------------------------------------------
// Complex products, one wave per tile of 16 WA x 16 WB: each lane loads its own operands of eight K values
// (two of each column or row, so 128-byte lines in fp64) from global memory and the next eight are in flight
// under the products of the present ones.  Bound by the matrix cores (64 cycles per fp64 instruction, two
// waves on a SIMD): no barrier stops a wave, narrow tiles leave little padding and fill the last round, and
// the loads (13 bytes a cycle and compute unit at 2 x 3 blocks) stay far below what the caches give.
// ------------------------------------------------------------------------------------------
template <typename T, int WA, int WB, bool CONJ>
__device__ __forceinline__ void mma_step(const cplx<T> (&av)[WA][2], const cplx<T> (&bv)[WB][2],
                                         typename MF<T>::acc (&cr)[WA][WB], typename MF<T>::acc (&ci)[WA][WB]) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int a = 0; a < WA; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b) {
        cr[a][b] = MF<T>::mma(av[a][u].x, bv[b][u].x, cr[a][b]);
        ci[a][b] = MF<T>::mma(av[a][u].x, bv[b][u].y, ci[a][b]);
      }
#pragma unroll
    for (int a = 0; a < WA; ++a) {
      const T y = CONJ ? av[a][u].y : -av[a][u].y;
#pragma unroll
      for (int b = 0; b < WB; ++b) {
        cr[a][b] = MF<T>::mma(y, bv[b][u].y, cr[a][b]);
        ci[a][b] = MF<T>::mma(-y, bv[b][u].x, ci[a][b]);
      }
    }
  }
}

// cn: part[s] = A^H B over K chunk s, a quarter of the chunk per wave, the four waves' tiles summed in LDS.
// herm > 0: the first herm columns of B are A itself; tiles of that Gram block wholly below its diagonal are
// left out.  [S | H_s] of 144 bands over 37,073 plane waves in fp64: 160 us; 64 x 64 tiles through LDS
// took 377 us.
template <typename T, int WA, int WB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_cn(
    const cplx<T>* __restrict__ A, long lda, const cplx<T>* __restrict__ B, long ldb, const cplx<T>* __restrict__ B2,
    long ldb2, int ncol1, int M, int N, int K, int kchunk, int tiles_m, int tiles_n, double2* __restrict__ part,
    int herm) {
  constexpr bool F32 = std::is_same<T, float>::value;
  constexpr int FLUSH = 32;  // fp32: steps of eight K values per move into fp64 registers
  using acc_t = typename MF<T>::acc;
  __shared__ double2 red[2][4][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, q = lane >> 4;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  // tiles of one split are contiguous; inside a split, n fastest
  const int sp = t / (tiles_m * tiles_n);
  const int tr = t - sp * tiles_m * tiles_n;
  const int tm = tr / tiles_n, tn = tr - tm * tiles_n;
  const int i0 = tm * 16 * WA, j0 = tn * 16 * WB;
  if (j0 + 16 * WB <= herm && i0 >= j0 + 16 * WB) return;
  const int kb = sp * kchunk + wave * (kchunk / 4), ke = min(K, kb + kchunk / 4);
  const cplx<T>*pa[WA], *pb[WB];
#pragma unroll
  for (int a = 0; a < WA; ++a) pa[a] = A + (long)min(i0 + a * 16 + i, M - 1) * lda + kb + koff<T>(q, 0);
#pragma unroll
  for (int b = 0; b < WB; ++b) {
    const int c = min(j0 + b * 16 + i, N - 1);
    pb[b] = (c < ncol1 ? B + (long)c * ldb : B2 + (long)(c - ncol1) * ldb2) + kb + koff<T>(q, 0);
  }
  acc_t cr[WA][WB], ci[WA][WB];
  double dr[F32 ? WA : 1][F32 ? WB : 1][4] = {}, di[F32 ? WA : 1][F32 ? WB : 1][4] = {};
#pragma unroll
  for (int a = 0; a < WA; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b) cr[a][b] = ci[a][b] = acc_t{0, 0, 0, 0};
  cplx<T> a0[WA][2], b0[WB][2], a1[WA][2], b1[WB][2];
  auto load = [&](cplx<T>(&av)[WA][2], cplx<T>(&bv)[WB][2], int s) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int a = 0; a < WA; ++a) av[a][u] = pa[a][8 * (long)s + koff<T>(0, u)];
#pragma unroll
      for (int b = 0; b < WB; ++b) bv[b][u] = pb[b][8 * (long)s + koff<T>(0, u)];
    }
  };
  auto flush = [&]() {
    if constexpr (F32) {
#pragma unroll
      for (int a = 0; a < WA; ++a)
#pragma unroll
        for (int b = 0; b < WB; ++b) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            dr[a][b][r] += (double)cr[a][b][r];
            di[a][b][r] += (double)ci[a][b][r];
          }
          cr[a][b] = ci[a][b] = acc_t{0, 0, 0, 0};
        }
    }
  };
  const int full = ke > kb ? (ke - kb) / 8 : 0;
  if (full > 0) load(a0, b0, 0);
  int s = 0;
  for (; s + 1 < full; s += 2) {
    load(a1, b1, s + 1);
    mma_step<T, WA, WB, true>(a0, b0, cr, ci);
    load(a0, b0, min(s + 2, full - 1));
    mma_step<T, WA, WB, true>(a1, b1, cr, ci);
    if (F32 && (s % FLUSH) == FLUSH - 2) flush();
  }
  if (s < full) mma_step<T, WA, WB, true>(a0, b0, cr, ci);
  if (kb + 8 * full < ke) {  // the last K values, zeros behind them
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bool in = kb + 8 * full + koff<T>(q, u) < ke;
#pragma unroll
      for (int a = 0; a < WA; ++a) a1[a][u] = in ? pa[a][8 * (long)full + koff<T>(0, u)] : mk<T>(0, 0);
#pragma unroll
      for (int b = 0; b < WB; ++b) b1[b][u] = in ? pb[b][8 * (long)full + koff<T>(0, u)] : mk<T>(0, 0);
    }
    mma_step<T, WA, WB, true>(a1, b1, cr, ci);
  }
  // thread (row, column) of a block: accumulator element and lane that hold it
  const int row = tid & 15, col = tid >> 4;
  const int slot = F32 ? (row & 3) * 64 + (row >> 2) * 16 + col : (row >> 2) * 64 + (row & 3) * 16 + col;
#pragma unroll
  for (int a = 0; a < WA; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b) {
      const int buf = (a * WB + b) & 1;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double2 v = make_double2((double)cr[a][b][r], (double)ci[a][b][r]);
        if constexpr (F32) {
          v.x += dr[a][b][r];
          v.y += di[a][b][r];
        }
        red[buf][wave][r * 64 + lane] = v;
      }
      __syncthreads();
      double2 v = red[buf][0][slot];
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        v.x += red[buf][w][slot].x;
        v.y += red[buf][w][slot].y;
      }
      const int gi = i0 + a * 16 + row, gj = j0 + b * 16 + col;
      if (gi < M && gj < N) part[((long)sp * N + gj) * M + gi] = v;
    }
}

template <typename T>
__global__ void k_reduce_parts(const double2* __restrict__ part, int nsplit, int M, int N,
                               const double* __restrict__ dscale, int dper, double2* __restrict__ out64,
                               long ldo64, cplx<T>* __restrict__ outT, long ldoT) {
  PW_GRID_STRIDE(idx, (long)M * N) {
    const int j = (int)(idx / M), i = (int)(idx - (long)j * M);
    double2 s = sum_splits(part + idx, nsplit, (long)M * N);
    if (dscale) {
      const double d = dscale[i % dper];
      s.x *= d;
      s.y *= d;
    }
    if (out64) out64[(long)j * ldo64 + i] = s;
    if (outT) outT[(long)j * ldoT + i] = mk<T>((T)s.x, (T)s.y);
  }
}

// nn: out = A B (+ Zl in mode 2).  A: M x K (m contiguous), B: K x N (k contiguous).  The four waves of a
// workgroup share their columns.  The product is formed transposed, so that sixteen lanes hold consecutive
// rows and the stores are whole lines.  37,073 x 144 x 144 in fp64: 100 us; 128 x 64 tiles through LDS,
// one workgroup per compute unit, took 212 us.
template <typename T, int WA, int WB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_nn(
    const cplx<T>* __restrict__ A, long lda, const cplx<T>* __restrict__ B, long ldb, int M, int N, int K, int tiles_n,
    cplx<T>* out, long ldo, EpiH e) {
  using acc_t = typename MF<T>::acc;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, q = lane >> 4;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int tm = t / tiles_n, tn = t - tm * tiles_n;  // n fastest: workgroups sharing an A panel are adjacent
  const int i0 = (tm * 4 + wave) * 16 * WA, j0 = tn * 16 * WB;
  if (i0 >= M) return;
  const cplx<T>*pa[WA], *pb[WB];
#pragma unroll
  for (int a = 0; a < WA; ++a) pa[a] = A + koff<T>(q, 0) * lda + min(i0 + a * 16 + i, M - 1);
#pragma unroll
  for (int b = 0; b < WB; ++b) pb[b] = B + (long)min(j0 + b * 16 + i, N - 1) * ldb + koff<T>(q, 0);
  acc_t cr[WB][WA], ci[WB][WA];
#pragma unroll
  for (int b = 0; b < WB; ++b)
#pragma unroll
    for (int a = 0; a < WA; ++a) cr[b][a] = ci[b][a] = acc_t{0, 0, 0, 0};
  cplx<T> a0[WA][2], b0[WB][2], a1[WA][2], b1[WB][2];
  auto load = [&](cplx<T>(&av)[WA][2], cplx<T>(&bv)[WB][2], int s) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int a = 0; a < WA; ++a) av[a][u] = pa[a][(8 * (long)s + koff<T>(0, u)) * lda];
#pragma unroll
      for (int b = 0; b < WB; ++b) bv[b][u] = pb[b][8 * (long)s + koff<T>(0, u)];
    }
  };
  const int full = K / 8;
  if (full > 0) load(a0, b0, 0);
  int s = 0;
  for (; s + 1 < full; s += 2) {
    load(a1, b1, s + 1);
    mma_step<T, WB, WA, false>(b0, a0, cr, ci);
    load(a0, b0, min(s + 2, full - 1));
    mma_step<T, WB, WA, false>(b1, a1, cr, ci);
  }
  if (s < full) mma_step<T, WB, WA, false>(b0, a0, cr, ci);
  if (8 * full < K) {  // the last K values, zeros behind them
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bool in = 8 * full + koff<T>(q, u) < K;
#pragma unroll
      for (int a = 0; a < WA; ++a) a1[a][u] = in ? pa[a][(8 * (long)full + koff<T>(0, u)) * lda] : mk<T>(0, 0);
#pragma unroll
      for (int b = 0; b < WB; ++b) b1[b][u] = in ? pb[b][8 * (long)full + koff<T>(0, u)] : mk<T>(0, 0);
    }
    mma_step<T, WB, WA, false>(b1, a1, cr, ci);
  }
  const cplx<T>* Zl = static_cast<const cplx<T>*>(e.Zl);
#pragma unroll
  for (int b = 0; b < WB; ++b)
#pragma unroll
    for (int a = 0; a < WA; ++a) {
      const int row = i0 + a * 16 + i;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = j0 + b * 16 + MF<T>::row(lane, r);
        if (row < M && col < N) {
          cplx<T> v = mk<T>(cr[b][a][r], ci[b][a][r]);
          if (e.mode == 2) {
            const auto z = Zl[(long)col * e.ldz + row];
            v.x += z.x;
            v.y += z.y;
          }
          out[(long)col * ldo + row] = v;
        }
      }
    }
}

// ------------------------------------------------------------------------------------------
// Projector products on pairs (G, -G).  Every projector column is the transform of a real function,
// beta(-G) = conj beta(G) (its l = 1 columns times i where needed, which V_NL does not see), and a
// band is f + i g with f, g real, so the sums run over half of the sphere's rows (nh = (npw + 1) / 2;
// row npw - 1 - g is -G of row g, row nh - 1 is G = 0) with real products:
//   F = (p.x + m.x, p.y - m.y), G = (p.y + m.y, m.x - p.x),  p = y[h], m = y[npw - 1 - h]
//   (G = 0: F = (p.x, 0), G = (p.y, 0))
//   projection  p_f += beta.x F.x + beta.y F.y, p_g the same with G
//   nonlocal    zf = sum_k beta q_f[k], zg = sum_k beta q_g[k] (q real),
//               V_NL y[h] = zf + i zg, V_NL y[npw - 1 - h] = conj(zf) + i conj(zg)
// half the multiplications and half the table of the complex products over the whole sphere.
//
// The projection runs four waves along M, all columns of the tile in each, through LDS (every column needs two
// loads, which the four waves share).  Bound by the matrix cores (64 cycles per fp64 instruction): what counts
// is two workgroups per compute unit, so that one's barriers and loads run under the other's products, and a
// split whose last round is full.  2,048 projectors x 1,088 bands x 147,834 half rows in fp64: projection
// 41.6 ms, nonlocal product 35.2 ms (63 and 75 TFLOP/s; 41.6 ms through LDS); the complex products over the
// whole sphere took 95.1 and 98.2 ms.
// ------------------------------------------------------------------------------------------
template <typename T> struct PairCfg;  // K tile of the projection
template <> struct PairCfg<double> {
  static constexpr int BK = 8;
};
template <> struct PairCfg<float> {
  static constexpr int BK = 16;
};

// The four projectors of an atom at one half row: radial factors r, phase e.
template <typename T>
__device__ __forceinline__ void beta_four(const double4& r, const double2& e, cplx<T> (&v)[4]) {
  v[0] = mk<T>((T)(r.x * e.x), (T)(r.x * e.y));
  v[1] = mk<T>((T)(-r.y * e.y), (T)(r.y * e.x));
  v[2] = mk<T>((T)(-r.z * e.y), (T)(r.z * e.x));
  v[3] = mk<T>((T)(-r.w * e.y), (T)(r.w * e.x));
}
// The four projectors of atom a at half row g (zero past the half sphere / the atoms).
template <typename T>
__device__ __forceinline__ void beta_gen4(const BetaGen& bg, int g, int a, cplx<T> (&v)[4]) {
  if (g >= bg.nh || a >= bg.natoms) {
#pragma unroll
    for (int m = 0; m < 4; ++m) v[m] = mk<T>(0, 0);
    return;
  }
  const int n1 = bg.miller[3 * g], n2 = bg.miller[3 * g + 1], n3 = bg.miller[3 * g + 2];
  const double2* p = bg.ph + (long)a * bg.w;
  const double2 e1 = p[n1 + bg.h1], e2 = p[bg.o2 + n2 + bg.h2], e3 = p[bg.o3 + n3 + bg.h3];
  const double2 e12 = make_double2(e1.x * e2.x - e1.y * e2.y, e1.x * e2.y + e1.y * e2.x);
  const double2 e = make_double2(e12.x * e3.x - e12.y * e3.y, e12.x * e3.y + e12.y * e3.x);
  beta_four<T>(*reinterpret_cast<const double4*>(bg.rad + 4 * (long)g), e, v);
}

// Projector panels: COLS projectors x ROWS half rows, element (row, column) to S[row * LDS_LD + column].  From
// the table (row-contiguous columns) or generated, four projectors of an atom per unit.
template <typename T, int COLS, int ROWS, bool OTF>
struct BetaPanel {
  static constexpr int W = OTF ? 4 : 1;  // projectors per unit
  static constexpr int UNITS = ROWS * COLS / W, PER = (UNITS + 255) / 256;
  cplx<T> r[PER][W];
  __device__ __forceinline__ void load(const cplx<T>* __restrict__ A, long lda, const BetaGen& bg, int nh, int ncols,
                                       int r0, int c0, int tid) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256, row = r0 + idx % ROWS, col = c0 + W * (idx / ROWS);
      const bool in = idx < UNITS && row < nh && col < ncols;
      if constexpr (OTF) {
        beta_gen4<T>(bg, in ? row : bg.nh, col / 4, r[q]);
      } else {
        r[q][0] = in ? A[(long)col * lda + row] : mk<T>(0, 0);
      }
    }
  }
  template <int LDS_LD>
  __device__ __forceinline__ void store(cplx<T>* S, int tid) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256, row = idx % ROWS, col = W * (idx / ROWS);
      if (idx < UNITS) {
#pragma unroll
        for (int m = 0; m < W; ++m) S[row * LDS_LD + col + m] = r[q][m];
      }
    }
  }
};

// Pair sums of NC bands at BK half rows.
template <typename T, int NC, int BK>
struct PairPanel {
  static constexpr int UNITS = BK * NC, PER = (UNITS + 255) / 256;
  cplx<T> p[PER], m[PER];
  __device__ __forceinline__ void load(const cplx<T>* __restrict__ Y, long ld, int npw, int nh, int ncols, int c0,
                                       int k0, int tid) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256, h = k0 + idx % BK, c = c0 + idx / BK;
      p[q] = m[q] = mk<T>(0, 0);
      if (idx < UNITS && h < nh && c < ncols) {
        p[q] = Y[(long)c * ld + h];
        m[q] = Y[(long)c * ld + (npw - 1 - h)];
      }
    }
  }
  template <int LDS_LD>
  __device__ __forceinline__ void store(cplx<T>* SF, cplx<T>* SG, int nh, int k0, int tid) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256, k = idx % BK, c = idx / BK;
      if (idx < UNITS) {
        const bool zero = k0 + k == nh - 1;  // G = 0
        SF[k * LDS_LD + c] = zero ? mk<T>(p[q].x, 0) : mk<T>(p[q].x + m[q].x, p[q].y - m[q].y);
        SG[k * LDS_LD + c] = zero ? mk<T>(p[q].y, 0) : mk<T>(p[q].y + m[q].y, m[q].x - p[q].x);
      }
    }
  }
};

// part[s][band][projector] = (p_f, p_g) over half rows [s kchunk, (s + 1) kchunk).  Tile 64 WBM projectors x
// 16 NBN bands.
template <typename T, int WBM, int NBN, bool OTF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_pairs_cn(
    const cplx<T>* __restrict__ A, long lda, BetaGen bg, const cplx<T>* __restrict__ Y, long ldy, int M, int N, int npw,
    int nh, int kchunk, int tiles_m, int tiles_n, double2* __restrict__ part) {
  constexpr int BK = PairCfg<T>::BK, BM = 64 * WBM, BN = 16 * NBN, LA = BM + 1, LB = BN + 1;
  constexpr int FLUSH = 256 / BK;  // fp32: K tiles per move into fp64 registers
  constexpr bool F32 = std::is_same<T, float>::value;
  using acc_t = typename MF<T>::acc;
  __shared__ cplx<T> sA[2][BK * LA];
  __shared__ cplx<T> sF[2][BK * LB], sG[2][BK * LB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int sp = t / (tiles_m * tiles_n);
  const int tr = t - sp * tiles_m * tiles_n;
  const int tm = tr / tiles_n, tn = tr - tm * tiles_n;
  const int i0 = tm * BM, j0 = tn * BN;
  const int kb = sp * kchunk, ke = min(nh, kb + kchunk);
  const int mo = wave * 16 * WBM;
  acc_t cf[WBM][NBN], cg[WBM][NBN];
  double df[F32 ? WBM : 1][F32 ? NBN : 1][4] = {}, dg[F32 ? WBM : 1][F32 ? NBN : 1][4] = {};
#pragma unroll
  for (int a = 0; a < WBM; ++a)
#pragma unroll
    for (int b = 0; b < NBN; ++b) cf[a][b] = cg[a][b] = acc_t{0, 0, 0, 0};
  BetaPanel<T, BM, BK, OTF> la;
  PairPanel<T, BN, BK> lb;
  const int ntiles = ke > kb ? (ke - kb + BK - 1) / BK : 0;
  if (ntiles > 0) {
    la.load(A, lda, bg, ke, M, kb, i0, tid);
    lb.load(Y, ldy, npw, ke, N, j0, kb, tid);
    la.template store<LA>(sA[0], tid);
    lb.template store<LB>(sF[0], sG[0], nh, kb, tid);
  }
  __syncthreads();
  for (int it = 0; it < ntiles; ++it) {
    const int cur = it & 1, kn = kb + (it + 1) * BK;
    const bool more = it + 1 < ntiles;
    if (more) {
      la.load(A, lda, bg, ke, M, kn, i0, tid);
      lb.load(Y, ldy, npw, ke, N, j0, kn, tid);
    }
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const int kr = kk + (lane >> 4);
      cplx<T> av[WBM], fv[NBN], gv[NBN];
#pragma unroll
      for (int a = 0; a < WBM; ++a) av[a] = sA[cur][kr * LA + mo + a * 16 + (lane & 15)];
#pragma unroll
      for (int b = 0; b < NBN; ++b) {
        fv[b] = sF[cur][kr * LB + b * 16 + (lane & 15)];
        gv[b] = sG[cur][kr * LB + b * 16 + (lane & 15)];
      }
#pragma unroll
      for (int a = 0; a < WBM; ++a)
#pragma unroll
        for (int b = 0; b < NBN; ++b) {
          cf[a][b] = MF<T>::mma(av[a].x, fv[b].x, cf[a][b]);
          cg[a][b] = MF<T>::mma(av[a].x, gv[b].x, cg[a][b]);
        }
#pragma unroll
      for (int a = 0; a < WBM; ++a)
#pragma unroll
        for (int b = 0; b < NBN; ++b) {
          cf[a][b] = MF<T>::mma(av[a].y, fv[b].y, cf[a][b]);
          cg[a][b] = MF<T>::mma(av[a].y, gv[b].y, cg[a][b]);
        }
    }
    if constexpr (F32) {
      if ((it % FLUSH) == FLUSH - 1) {
#pragma unroll
        for (int a = 0; a < WBM; ++a)
#pragma unroll
          for (int b = 0; b < NBN; ++b) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              df[a][b][r] += (double)cf[a][b][r];
              dg[a][b][r] += (double)cg[a][b][r];
            }
            cf[a][b] = cg[a][b] = acc_t{0, 0, 0, 0};
          }
      }
    }
    if (more) {
      la.template store<LA>(sA[cur ^ 1], tid);
      lb.template store<LB>(sF[cur ^ 1], sG[cur ^ 1], nh, kn, tid);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < WBM; ++a)
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
      const int col = j0 + b * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = i0 + mo + a * 16 + MF<T>::row(lane, r);
        if (row < M && col < N) {
          double2 v = make_double2((double)cf[a][b][r], (double)cg[a][b][r]);
          if constexpr (F32) {
            v.x += df[a][b][r];
            v.y += dg[a][b][r];
          }
          part[((long)sp * N + col) * M + row] = v;
        }
      }
    }
}

// out = EpiH(mode 1) with V_NL psi = beta q over K projectors, a wave per tile of 16 WA half rows x 16 WB bands
// like the complex products (operands straight from memory, the four waves of a workgroup on the same
// bands, the product transposed so that sixteen lanes hold consecutive rows).  Generated projectors: a lane
// makes the four of one atom for its row, whose radial factors stay in registers.
// The epilogue moves three times the block's bytes: 256 projectors x 144 bands, 18,537 half rows in fp64 138 us
// (65 at the matrix cores' rate, 54 for the bytes; 170 us through LDS), generated 112 us (162 through LDS).
template <typename T, int WA, int WB, bool OTF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_pairs_nn(
    const cplx<T>* __restrict__ A, long lda, BetaGen bg, const cplx<T>* __restrict__ Q, long ldq, int npw, int nh, int N,
    int K, int tiles_n, cplx<T>* out, long ldo, EpiH e) {
  constexpr int U = OTF ? 4 : 2, STEP = 4 * U;  // projectors per lane and step, per step
  using acc_t = typename MF<T>::acc;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, q = lane >> 4;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int tm = t / tiles_n, tn = t - tm * tiles_n;  // n fastest: workgroups sharing an A panel are adjacent
  const int i0 = (tm * 4 + wave) * 16 * WA, j0 = tn * 16 * WB;
  if (i0 >= nh) return;
  auto ko = [](int g, int u) { return OTF ? 4 * g + u : koff<T>(g, u); };
  const cplx<T>*pa[WA], *pb[WB];
  int m1[OTF ? WA : 1], m2[OTF ? WA : 1], m3[OTF ? WA : 1];
  double4 rad[OTF ? WA : 1];
#pragma unroll
  for (int a = 0; a < WA; ++a) {
    const int h = min(i0 + a * 16 + i, nh - 1);
    if constexpr (OTF) {
      m1[a] = bg.miller[3 * h] + bg.h1;
      m2[a] = bg.o2 + bg.miller[3 * h + 1] + bg.h2;
      m3[a] = bg.o3 + bg.miller[3 * h + 2] + bg.h3;
      rad[a] = *reinterpret_cast<const double4*>(bg.rad + 4 * (long)h);
      pa[a] = nullptr;
    } else {
      pa[a] = A + ko(q, 0) * lda + h;
    }
  }
#pragma unroll
  for (int b = 0; b < WB; ++b) pb[b] = Q + (long)min(j0 + b * 16 + i, N - 1) * ldq + ko(q, 0);
  acc_t fx[WB][WA], fy[WB][WA], gx[WB][WA], gy[WB][WA];
#pragma unroll
  for (int b = 0; b < WB; ++b)
#pragma unroll
    for (int a = 0; a < WA; ++a) fx[b][a] = fy[b][a] = gx[b][a] = gy[b][a] = acc_t{0, 0, 0, 0};
  auto load = [&](cplx<T>(&av)[WA][U], cplx<T>(&bv)[WB][U], int s) {
    if constexpr (OTF) {
      const double2* p = bg.ph + (long)(4 * s + q) * bg.w;
#pragma unroll
      for (int a = 0; a < WA; ++a) {
        const double2 e1 = p[m1[a]], e2 = p[m2[a]], e3 = p[m3[a]];
        const double2 e12 = make_double2(e1.x * e2.x - e1.y * e2.y, e1.x * e2.y + e1.y * e2.x);
        beta_four<T>(rad[a], make_double2(e12.x * e3.x - e12.y * e3.y, e12.x * e3.y + e12.y * e3.x), av[a]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int a = 0; a < WA; ++a) av[a][u] = pa[a][(STEP * (long)s + ko(0, u)) * lda];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int b = 0; b < WB; ++b) bv[b][u] = pb[b][STEP * (long)s + ko(0, u)];
  };
  auto mma = [&](const cplx<T>(&av)[WA][U], const cplx<T>(&bv)[WB][U]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int a = 0; a < WA; ++a) {
          fx[b][a] = MF<T>::mma(bv[b][u].x, av[a][u].x, fx[b][a]);
          fy[b][a] = MF<T>::mma(bv[b][u].x, av[a][u].y, fy[b][a]);
          gx[b][a] = MF<T>::mma(bv[b][u].y, av[a][u].x, gx[b][a]);
          gy[b][a] = MF<T>::mma(bv[b][u].y, av[a][u].y, gy[b][a]);
        }
  };
  const int full = K / STEP;
  cplx<T> a0[WA][U], b0[WB][U], a1[WA][U], b1[WB][U];
  if (full > 0) load(a0, b0, 0);
  int s = 0;
  for (; s + 1 < full; s += 2) {
    load(a1, b1, s + 1);
    mma(a0, b0);
    load(a0, b0, min(s + 2, full - 1));
    mma(a1, b1);
  }
  if (s < full) mma(a0, b0);
  if (STEP * full < K) {  // the last projectors, zeros behind them
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = STEP * full + ko(q, u) < K;
#pragma unroll
      for (int a = 0; a < WA; ++a)
        if constexpr (!OTF) a1[a][u] = in ? pa[a][(STEP * (long)full + ko(0, u)) * lda] : mk<T>(0, 0);
#pragma unroll
      for (int b = 0; b < WB; ++b) b1[b][u] = in ? pb[b][STEP * (long)full + ko(0, u)] : mk<T>(0, 0);
    }
    if constexpr (OTF) {
#pragma unroll
      for (int a = 0; a < WA; ++a) beta_gen4<T>(bg, min(i0 + a * 16 + i, nh - 1), 4 * full + q, a1[a]);
    }
    mma(a1, b1);
  }
  const T* kin = static_cast<const T*>(e.kin);
  const T alpha = (T)e.alpha, cc = (T)e.c, beta = (T)e.beta;
#pragma unroll
  for (int b = 0; b < WB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      __builtin_amdgcn_sched_barrier(0);  // one column at a time: bounded register use
      const int col = j0 + b * 16 + MF<T>::row(lane, r);
      if (col >= N) continue;
      const cplx<T>* Y = static_cast<const cplx<T>*>(e.Y) + (long)col * e.ldy;
      const cplx<T>* Zl = static_cast<const cplx<T>*>(e.Zl) + (long)col * e.ldz;
      const cplx<T>* Yp = e.Yp ? static_cast<const cplx<T>*>(e.Yp) + (long)col * e.ldp : nullptr;
      cplx<T>* o = out + (long)col * ldo;
#pragma unroll
      for (int a = 0; a < WA; ++a) {
        const int h = i0 + a * 16 + i;
        if (h >= nh) continue;
        const int g = npw - 1 - h;  // == h at G = 0
        const T kc = kin[h] - cc;
        const cplx<T> yp = Y[h], ym = Y[g], zp = Zl[h], zm = Zl[g];
        cplx<T> p = mk<T>(alpha * (kc * yp.x + zp.x + (fx[b][a][r] - gy[b][a][r])),
                          alpha * (kc * yp.y + zp.y + (fy[b][a][r] + gx[b][a][r])));
        cplx<T> m = mk<T>(alpha * (kc * ym.x + zm.x + (fx[b][a][r] + gy[b][a][r])),
                          alpha * (kc * ym.y + zm.y + (gx[b][a][r] - fy[b][a][r])));
        if (Yp) {
          const cplx<T> qp = Yp[h], qm = Yp[g];
          p.x -= beta * qp.x;
          p.y -= beta * qp.y;
          m.x -= beta * qm.x;
          m.y -= beta * qm.y;
        }
        if (g != h) o[g] = m;
        o[h] = p;
      }
    }
}

// ------------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------------
// Blocks of a wave's tile (cn: 16 wa x 16 wb) and K splits from smin to smax, by the time of the busiest
// compute unit: its steps of eight K values at the matrix cores' rate or at that of the loads (72 cycles per
// 64-lane load of fp64 measured, half of that per value pair in fp32), whichever is longer, no step shorter
// than the latency of its loads (a quarter longer with one wave per SIMD), + start and end of a round + the
// partials' traffic.  [S | H_s] in fp64 without the tiles left out, in 3 x 2, 2 x 2 and 1 x 1 blocks: 480 bands x
// 124,289 6.6, 7.3 and 13.4 ms (52, 47 and 26 TFLOP/s of what is computed); 1,088 x 295,667 80, 95 and 171 ms;
// 144 x 37,073 162, 159 and 265 us (2 x 2 fills the last round best); 40 x 5,891 14.6, 10.7 and 7.7 us, where 11
// splits of 64 x 64 tiles took 92 us on 22 compute units.
struct CnShape {
  int wa, wb, splits;
};
static CnShape cn_shape(int M, int N, int K, bool fp64, int herm, int smin, int smax) {
  static constexpr int kShapes[][2] = {{3, 2}, {2, 3}, {2, 2}, {1, 2}, {1, 1}};
  CnShape best{2, 2, smin};
  if (M <= 0 || N <= 0 || K <= 0) return best;
  const int steps = ceil_div(K, 32);  // of the four waves
  double cost = 1e300;
  for (const auto& w : kShapes) {
    const int tm = ceil_div(M, 16 * w[0]);
    long tiles = (long)tm * ceil_div(N, 16 * w[1]);
    for (int j = 1; 16 * w[1] * j <= herm; ++j) tiles -= std::max(0, tm - ceil_div(w[1] * j, w[0]));  // left out
    const double step = std::max(w[0] * w[1] * 8 * 70, (w[0] + w[1]) * 8 * 72) * (fp64 ? 1.0 : 0.5) / 2400.0;
    for (int n = smin; n <= smax; ++n) {
      const int chunk = ceil_div(steps, n);
      if (n > smin && (ceil_div(steps, chunk) != n || chunk < 2)) continue;
      const long wg = tiles * n, r2 = (wg + 511) / 512;
      const double c = std::max((double)((wg + 255) / 256) * chunk * step, r2 * chunk * 0.6) * (wg > 256 ? 1.0 : 1.25) + 3.0 * r2 + 0.1 * n +
                       n * (double)M * N * 32.0 / 4.5e6;
      if (c < cost) {
        cost = c;
        best = CnShape{w[0], w[1], n};
      }
    }
  }
  return best;
}
int gemm_cn_splits(int M, int N, int K, bool fp64, int herm_cols) {
  return cn_shape(M, N, K, fp64, herm_cols, 1, 64).splits;
}

template <typename T>
hipError_t launch_gemm_cn(const cplx<T>* A, long lda, const cplx<T>* B, long ldb, const cplx<T>* B2, long ldb2,
                          int ncol1, int M, int N, int K, int nsplit, double2* part, hipStream_t s, int herm_cols) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const CnShape c = cn_shape(M, N, K, sizeof(T) == 8, herm_cols, nsplit, nsplit);
  const int kchunk = std::max(1, ceil_div(ceil_div(K, 32), nsplit)) * 32;
  const int tm = ceil_div(M, 16 * c.wa), tn = ceil_div(N, 16 * c.wb);
  const cplx<T>* b2 = B2 ? B2 : B;
  const long l2 = B2 ? ldb2 : ldb;
  const dim3 grid(tm * tn * nsplit);
#define PW_CN(WA, WB)                                                                                              \
  case 4 * WA + WB:                                                                                                \
    hipLaunchKernelGGL((k_gemm_cn<T, WA, WB>), grid, dim3(256), 0, s, A, lda, B, ldb, b2, l2, ncol1, M, N, K, kchunk, \
                       tm, tn, part, herm_cols);                                                                   \
    break
  switch (4 * c.wa + c.wb) {
    PW_CN(3, 2);
    PW_CN(2, 3);
    PW_CN(2, 2);
    PW_CN(1, 2);
    PW_CN(1, 1);
    default: return hipErrorInvalidValue;
  }
#undef PW_CN
  return hipGetLastError();
}

template <typename T>
hipError_t launch_reduce_parts(const double2* part, int nsplit, int M, int N, const double* dscale, int dper,
                               double2* out64, long ldo64, cplx<T>* outT, long ldoT, hipStream_t s) {
  const long n = (long)M * N;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_parts<T>, dim3(stride_blocks(n)), dim3(256), 0, s, part, nsplit, M, N, dscale,
                     dper > 0 ? dper : 1, out64, ldo64, outT, ldoT);
  return hipGetLastError();
}

// Blocks of a wave's tile of an nn product (16 wa rows x 16 wb columns, four waves along the rows): the shape that
// leaves the fewest block products to the busiest compute unit, the wider one among equals (fewer loads).
// 37,073 x 144: 1 x 3 leaves 7 tiles of 3 blocks to a SIMD and takes 100 us, 2 x 3 leaves 4 of 6 and takes
// 109 us, 1 x 1 has no idle SIMD but three times the loads: 114 us.
struct NnShape {
  int wa, wb;
};
static NnShape nn_shape(int M, int N, int max_blocks) {
  static constexpr int kShapes[][2] = {{2, 3}, {2, 2}, {1, 3}, {1, 2}, {1, 1}};
  NnShape best{1, 1};
  long cost = 1L << 60;
  for (const auto& w : kShapes) {
    const long c = ((long)ceil_div(M, 64 * w[0]) * ceil_div(N, 16 * w[1]) + 255) / 256 * (w[0] * w[1] * 16 + 4);
    if (w[0] * w[1] <= max_blocks && c < cost) {
      cost = c;
      best = NnShape{w[0], w[1]};
    }
  }
  return best;
}

template <typename T>
hipError_t launch_gemm_nn(const cplx<T>* A, long lda, const cplx<T>* B, long ldb, int M, int N, int K,
                          cplx<T>* out, long ldo, const EpiH& e, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const NnShape w = nn_shape(M, N, 6);
  const int tm = ceil_div(M, 64 * w.wa), tn = ceil_div(N, 16 * w.wb);
  const dim3 grid(tm * tn);
#define PW_NN(WA, WB)                                                                                              \
  case 4 * WA + WB:                                                                                                \
    hipLaunchKernelGGL((k_gemm_nn<T, WA, WB>), grid, dim3(256), 0, s, A, lda, B, ldb, M, N, K, tn, out, ldo, e);   \
    break
  switch (4 * w.wa + w.wb) {
    PW_NN(2, 3);
    PW_NN(2, 2);
    PW_NN(1, 3);
    PW_NN(1, 2);
    PW_NN(1, 1);
    default: return hipErrorInvalidValue;
  }
#undef PW_NN
  return hipGetLastError();
}

// Projectors per tile: 128, but 64 for few projectors, and in fp32 at the full width, whose fp64 sums of 128
// rows would not fit in registers.
static int pair_rows(int M, int w, bool fp64) { return M > 64 && (fp64 || w < 64) ? 128 : 64; }

// Bands per tile (16 .. 64) and K splits of the projection: those that minimise rounds of two workgroups per
// compute unit x (matrix-core cycles of a workgroup's K tiles, two sharing a SIMD, + their start and end)
// plus the partials' traffic, with at most cap and 64 splits.  2,048 projectors x 1,088 bands in fp64 (272
// tiles): 15 splits fill 4,080 of 4,096 places; 4 splits of the complex product's 64 x 64 tiles filled
// 2,176 of 2,560.  144 bands take 3 tiles of 48, not 3 of 64.
PairsCn pairs_cn_plan(int M, int nb, int nh, bool fp64, long cap) {
  PairsCn best{64, 1};
  if (M <= 0 || nb <= 0 || nh <= 0) return best;
  const int bk = fp64 ? PairCfg<double>::BK : PairCfg<float>::BK, ktiles = ceil_div(nh, bk);
  double cost = 1e300;
  for (int w = 64; w >= 16; w -= 16) {
    const int rows = pair_rows(M, w, fp64);
    const long tiles = (long)ceil_div(M, rows) * ceil_div(nb, w);
    const double us = (bk / 4) * (rows / 64) * (w / 16) * 4 * (fp64 ? 64 : 32) * 2 / 2400.0 * 1.15 + 0.3;
    for (int n = 1; n <= 64 && n <= ktiles && (n == 1 || n <= cap); ++n) {
      const int chunk = ceil_div(ktiles, n);
      if (ceil_div(ktiles, chunk) != n) continue;
      const double rounds = (double)((tiles * n + 511) / 512);
      const double c = rounds * (chunk * us + 5.0) + 0.04 * n + n * (double)M * nb * 32.0 / 4.5e6;
      if (c < cost) {
        cost = c;
        best = PairsCn{w, n};
      }
    }
  }
  return best;
}
template <typename T>
hipError_t launch_pairs_cn(const cplx<T>* A, long lda, const BetaGen* bg, const cplx<T>* Y, long ldy, int M, int nb,
                           int npw, const PairsCn& c, double2* part, hipStream_t s) {
  if (M <= 0 || nb <= 0) return hipSuccess;
  constexpr int BK = PairCfg<T>::BK;
  const int nh = (npw + 1) / 2, kchunk = ceil_div(ceil_div(nh, BK), c.splits) * BK;
  const int w = c.width, rows = pair_rows(M, w, sizeof(T) == 8), tm = ceil_div(M, rows), tn = ceil_div(nb, w);
  const dim3 grid(tm * tn * c.splits);
  const BetaGen g = bg ? *bg : BetaGen{};
#define PW_PCN(WBM, NBN, OTF)                                                                                       \
  hipLaunchKernelGGL((k_pairs_cn<T, WBM, NBN, OTF>), grid, dim3(256), 0, s, A, lda, g, Y, ldy, M, nb, npw, nh, kchunk, \
                     tm, tn, part)
#define PW_PCN_W(NBN)                                                       \
  case 16 * NBN:                                                            \
    if (rows == 128) {                                                      \
      constexpr int WB = NBN < 4 || sizeof(T) == 8 ? 2 : 1;                 \
      if (bg) PW_PCN(WB, NBN, true); else PW_PCN(WB, NBN, false);           \
    } else {                                                                \
      if (bg) PW_PCN(1, NBN, true); else PW_PCN(1, NBN, false);             \
    }                                                                       \
    break
  switch (w) {
    PW_PCN_W(1);
    PW_PCN_W(2);
    PW_PCN_W(3);
    PW_PCN_W(4);
    default: return hipErrorInvalidValue;
  }
#undef PW_PCN_W
#undef PW_PCN
  return hipGetLastError();
}

template <typename T>
hipError_t launch_pairs_nn(const cplx<T>* A, long lda, const BetaGen* bg, const cplx<T>* Q, long ldq, int npw, int nb,
                           int K, cplx<T>* out, long ldo, const EpiH& e, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  const int nh = (npw + 1) / 2;
  // Blocks at most: few projectors leave more waves to hide the epilogue (256 x 144 bands, 18,537 half rows, fp64:
  // 1 x 3 139 us, 2 x 2 155; generated 1 x 1 112, 1 x 2 121), many want fewer loads (2,048 x 1,088: 2 x 2 35.2 ms,
  // 1 x 3 39.0; generated, 864 x 480: 1 x 2 3.41 ms, 1 x 1 3.52); the line lies between 256 and 512 projectors
  // (512 x 256: 2 x 2 634 us, 1 x 2 742; generated 1 x 2 709, 1 x 1 722).
  const NnShape w = nn_shape(nh, nb, bg ? (K < 512 ? 1 : 2) : (K < 512 ? 3 : 4));
  const int tm = ceil_div(nh, 64 * w.wa), tn = ceil_div(nb, 16 * w.wb);
  const dim3 grid(tm * tn);
  const BetaGen g = bg ? *bg : BetaGen{};
#define PW_PNN(WA, WB, OTF)                                                                                          \
  hipLaunchKernelGGL((k_pairs_nn<T, WA, WB, OTF>), grid, dim3(256), 0, s, A, lda, g, Q, ldq, npw, nh, nb, K, tn, out, \
                     ldo, e)
  switch (4 * w.wa + w.wb) {
    case 10: PW_PNN(2, 2, false); break;
    case 7: PW_PNN(1, 3, false); break;
    case 6:
      if (bg) PW_PNN(1, 2, true); else PW_PNN(1, 2, false);
      break;
    default:
      if (bg) PW_PNN(1, 1, true); else PW_PNN(1, 1, false);
  }
#undef PW_PNN
  return hipGetLastError();
}

#define PW_INST_GEMM(T)                                                                                      \
  template hipError_t launch_gemm_cn<T>(const cplx<T>*, long, const cplx<T>*, long, const cplx<T>*, long,   \
                                        int, int, int, int, int, double2*, hipStream_t, int);                \
  template hipError_t launch_reduce_parts<T>(const double2*, int, int, int, const double*, int, double2*,   \
                                             long, cplx<T>*, long, hipStream_t);                             \
  template hipError_t launch_gemm_nn<T>(const cplx<T>*, long, const cplx<T>*, long, int, int, int, cplx<T>*, \
                                        long, const EpiH&, hipStream_t);                                     \
  template hipError_t launch_pairs_cn<T>(const cplx<T>*, long, const BetaGen*, const cplx<T>*, long, int,    \
                                         int, int, const PairsCn&, double2*, hipStream_t);                   \
  template hipError_t launch_pairs_nn<T>(const cplx<T>*, long, const BetaGen*, const cplx<T>*, long, int,    \
                                         int, int, cplx<T>*, long, const EpiH&, hipStream_t);
PW_INST_GEMM(float)
PW_INST_GEMM(double)

}  // namespace pw

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
// Structure of one workgroup (4 waves in a 2 x 2 arrangement): global loads of
// the next K tile go to registers (16-byte loads where the leading dimension
// allows) while the MFMAs run on the current tile; the tiles live in two LDS
// buffers, so each K tile costs one barrier.  Tiles are handed out XCD by XCD:
// consecutive tiles, which share operand panels, run on the same L2.

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

constexpr int kBK = 16;     // K per tile (complex elements)
constexpr int kFlush = 16;  // fp32 cn: K tiles per move into fp64 registers
constexpr int kXcd = 8;     // XCDs per MI355X

// 16 bytes = U complex elements (U = 2 for fp32, 1 for fp64)
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  using type = float4;
  static constexpr int U = 2;
};
template <> struct Vec16<double> {
  using type = double2;
  static constexpr int U = 1;
};

// Tile index -> (tm, tn, split) with the tiles of one XCD contiguous.  Launch order
// sends workgroup w to XCD w % 8.
__device__ __forceinline__ int xcd_tile(int w, int total) {
  const int per = total / kXcd, rem = total % kXcd;
  const int x = w % kXcd, i = w / kXcd;
  // XCDs 0..rem-1 get per + 1 tiles, the others per
  return x < rem ? x * (per + 1) + i : rem * (per + 1) + (x - rem) * per + i;
}

// Loader of a K-contiguous operand panel: kBK values of NC columns starting at (k0, c0).
// Element (k, c) goes to S[k * LDS_LD + c].
template <typename T, int NC, bool VEC>
struct KcLoader {
  static constexpr int U = VEC ? Vec16<T>::U : 1;
  static constexpr int UNITS = kBK / U * NC;  // loads per tile
  static constexpr int PER = (UNITS + 255) / 256;
  cplx<T> r[PER][U];
  __device__ __forceinline__ void load(const cplx<T>* __restrict__ P, long ld, const cplx<T>* __restrict__ P2, long ld2,
                                       int ncol1, int ncols, int c0, int k0, int kend, int tid) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256;
      const int ku = idx % (kBK / U), c = idx / (kBK / U);
      const int gc = c0 + c, gk = k0 + ku * U;
#pragma unroll
      for (int u = 0; u < U; ++u) r[q][u] = mk<T>(0, 0);
      if (idx < UNITS && gc < ncols) {
        const cplx<T>* col = gc < ncol1 ? P + (long)gc * ld : P2 + (long)(gc - ncol1) * ld2;
        if (VEC && gk + U <= kend) {
          const typename Vec16<T>::type v = *reinterpret_cast<const typename Vec16<T>::type*>(col + gk);
          if constexpr (std::is_same<T, float>::value) {
            r[q][0] = mk<T>(v.x, v.y);
            r[q][U - 1] = mk<T>(v.z, v.w);
          } else {
            r[q][0] = mk<T>(v.x, v.y);
          }
        } else {
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (gk + u < kend) r[q][u] = col[gk + u];
        }
      }
    }
  }
  template <int LDS_LD>
  __device__ __forceinline__ void store(cplx<T>* S, int tid) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256;
      if (idx < UNITS) {
        const int ku = idx % (kBK / U), c = idx / (kBK / U);
#pragma unroll
        for (int u = 0; u < U; ++u) S[(ku * U + u) * LDS_LD + c] = r[q][u];
      }
    }
  }
};

// Loader of an M-contiguous operand panel (nn A): NR rows x kBK columns of a column-major matrix.
template <typename T, int NR, bool VEC>
struct McLoader {
  static constexpr int U = VEC ? Vec16<T>::U : 1;
  static constexpr int UNITS = NR / U * kBK;
  static constexpr int PER = (UNITS + 255) / 256;
  cplx<T> r[PER][U];
  __device__ __forceinline__ void load(const cplx<T>* __restrict__ P, long ld, int nrows, int r0, int k0, int kend,
                                       int tid) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256;
      const int mu = idx % (NR / U), k = idx / (NR / U);
      const int gm = r0 + mu * U, gk = k0 + k;
#pragma unroll
      for (int u = 0; u < U; ++u) r[q][u] = mk<T>(0, 0);
      if (idx < UNITS && gk < kend) {
        const cplx<T>* col = P + (long)gk * ld;
        if (VEC && gm + U <= nrows) {
          const typename Vec16<T>::type v = *reinterpret_cast<const typename Vec16<T>::type*>(col + gm);
          if constexpr (std::is_same<T, float>::value) {
            r[q][0] = mk<T>(v.x, v.y);
            r[q][U - 1] = mk<T>(v.z, v.w);
          } else {
            r[q][0] = mk<T>(v.x, v.y);
          }
        } else {
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (gm + u < nrows) r[q][u] = col[gm + u];
        }
      }
    }
  }
  template <int LDS_LD>
  __device__ __forceinline__ void store(cplx<T>* S, int tid) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256;
      if (idx < UNITS) {
        const int mu = idx % (NR / U), k = idx / (NR / U);
#pragma unroll
        for (int u = 0; u < U; ++u) S[k * LDS_LD + mu * U + u] = r[q][u];
      }
    }
  }
};

// Wave-level MFMA accumulation over one K tile held in LDS.
// sA: kBK x (BM + 1) (m contiguous), sB: kBK x (BN + 1) (n contiguous).
template <typename T, int WBM, int WBN, bool CONJ_A>
__device__ __forceinline__ void mma_tile(const cplx<T>* sA, const cplx<T>* sB, int lda_s, int ldb_s, int mo, int no,
                                         int lane, typename MF<T>::acc (&cr)[WBM][WBN],
                                         typename MF<T>::acc (&ci)[WBM][WBN]) {
#pragma unroll
  for (int kk = 0; kk < kBK; kk += 4) {
    cplx<T> av[WBM], bv[WBN];
    const int kr = kk + (lane >> 4);
#pragma unroll
    for (int a = 0; a < WBM; ++a) av[a] = sA[kr * lda_s + mo + a * 16 + (lane & 15)];
#pragma unroll
    for (int b = 0; b < WBN; ++b) bv[b] = sB[kr * ldb_s + no + b * 16 + (lane & 15)];
#pragma unroll
    for (int a = 0; a < WBM; ++a)
#pragma unroll
      for (int b = 0; b < WBN; ++b) cr[a][b] = MF<T>::mma(av[a].x, bv[b].x, cr[a][b]);
#pragma unroll
    for (int a = 0; a < WBM; ++a)
#pragma unroll
      for (int b = 0; b < WBN; ++b) ci[a][b] = MF<T>::mma(av[a].x, bv[b].y, ci[a][b]);
#pragma unroll
    for (int a = 0; a < WBM; ++a) {
      const T ai = CONJ_A ? av[a].y : -av[a].y;
#pragma unroll
      for (int b = 0; b < WBN; ++b) cr[a][b] = MF<T>::mma(ai, bv[b].y, cr[a][b]);
    }
#pragma unroll
    for (int a = 0; a < WBM; ++a) {
      const T ai = CONJ_A ? -av[a].y : av[a].y;
#pragma unroll
      for (int b = 0; b < WBN; ++b) ci[a][b] = MF<T>::mma(ai, bv[b].x, ci[a][b]);
    }
  }
}

// ------------------------------------------------------------------------------------------
// cn: part[s] = A^H B over K chunk s.  Workgroup tile BM x BN (waves 2 x 2).
// ------------------------------------------------------------------------------------------
template <typename T, int BM, int BN, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_cn(const cplx<T>* __restrict__ A, long lda,
                                                 const cplx<T>* __restrict__ B, long ldb,
                                                 const cplx<T>* __restrict__ B2, long ldb2, int ncol1, int M, int N,
                                                 int K, int kchunk, int tiles_m, int tiles_n,
                                                 double2* __restrict__ part) {
  constexpr int WBM = BM / 32, WBN = BN / 32;  // 16x16 blocks per wave
  constexpr int LA = BM + 1, LB = BN + 1;
  using acc_t = typename MF<T>::acc;
  __shared__ cplx<T> sA[2][kBK * LA];
  __shared__ cplx<T> sB[2][kBK * LB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nsplit = gridDim.x / (tiles_m * tiles_n);
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  // tiles of one split are contiguous; inside a split, n fastest
  const int sp = t / (tiles_m * tiles_n);
  const int tr = t - sp * tiles_m * tiles_n;
  const int tm = tr / tiles_n, tn = tr - tm * tiles_n;
  (void)nsplit;
  const int i0 = tm * BM, j0 = tn * BN;
  const int kb = sp * kchunk, ke = min(K, kb + kchunk);
  const int mo = (wave & 1) * (BM / 2), no = (wave >> 1) * (BN / 2);
  acc_t cr[WBM][WBN], ci[WBM][WBN];
  double dr[WBM][WBN][4], di[WBM][WBN][4];
#pragma unroll
  for (int a = 0; a < WBM; ++a)
#pragma unroll
    for (int b = 0; b < WBN; ++b) {
      cr[a][b] = acc_t{0, 0, 0, 0};
      ci[a][b] = acc_t{0, 0, 0, 0};
#pragma unroll
      for (int r = 0; r < 4; ++r) dr[a][b][r] = di[a][b][r] = 0.0;
    }
  KcLoader<T, BM, VEC> la;
  KcLoader<T, BN, VEC> lb;
  const int ntiles = ke > kb ? (ke - kb + kBK - 1) / kBK : 0;
  if (ntiles > 0) {
    la.load(A, lda, A, lda, M, M, i0, kb, ke, tid);
    lb.load(B, ldb, B2, ldb2, ncol1, N, j0, kb, ke, tid);
    la.template store<LA>(sA[0], tid);
    lb.template store<LB>(sB[0], tid);
  }
  __syncthreads();
  for (int it = 0; it < ntiles; ++it) {
    const int cur = it & 1;
    const bool more = it + 1 < ntiles;
    if (more) {
      const int kn = kb + (it + 1) * kBK;
      la.load(A, lda, A, lda, M, M, i0, kn, ke, tid);
      lb.load(B, ldb, B2, ldb2, ncol1, N, j0, kn, ke, tid);
    }
    mma_tile<T, WBM, WBN, true>(sA[cur], sB[cur], LA, LB, mo, no, lane, cr, ci);
    if constexpr (std::is_same<T, float>::value) {
      if ((it % kFlush) == kFlush - 1) {
#pragma unroll
        for (int a = 0; a < WBM; ++a)
#pragma unroll
          for (int b = 0; b < WBN; ++b) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              dr[a][b][r] += (double)cr[a][b][r];
              di[a][b][r] += (double)ci[a][b][r];
            }
            cr[a][b] = acc_t{0, 0, 0, 0};
            ci[a][b] = acc_t{0, 0, 0, 0};
          }
      }
    }
    if (more) {
      la.template store<LA>(sA[cur ^ 1], tid);
      lb.template store<LB>(sB[cur ^ 1], tid);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < WBM; ++a)
#pragma unroll
    for (int b = 0; b < WBN; ++b) {
      const int col = j0 + no + b * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = i0 + mo + a * 16 + MF<T>::row(lane, r);
        if (row < M && col < N) {
          double2 v;
          v.x = dr[a][b][r] + (double)cr[a][b][r];
          v.y = di[a][b][r] + (double)ci[a][b][r];
          part[((long)sp * N + col) * M + row] = v;
        }
      }
    }
}

template <typename T>
__global__ void k_reduce_parts(const double2* __restrict__ part, int nsplit, int M, int N,
                               const double* __restrict__ dscale, int dper, double2* __restrict__ out64,
                               long ldo64, cplx<T>* __restrict__ outT, long ldoT) {
  PW_GRID_STRIDE(idx, (long)M * N) {
    const int j = (int)(idx / M), i = (int)(idx - (long)j * M);
    double2 s = part[idx];
    for (int p = 1; p < nsplit; ++p) {
      const double2 v = part[(long)p * M * N + idx];
      s.x += v.x;
      s.y += v.y;
    }
    if (dscale) {
      const double d = dscale[i % dper];
      s.x *= d;
      s.y *= d;
    }
    if (out64) out64[(long)j * ldo64 + i] = s;
    if (outT) outT[(long)j * ldoT + i] = mk<T>((T)s.x, (T)s.y);
  }
}

// ------------------------------------------------------------------------------------------
// nn: out = epilogue(A B).  A: M x K (m contiguous), B: K x N (k contiguous).
// ------------------------------------------------------------------------------------------
template <typename T, int BM, int BN, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_nn(const cplx<T>* __restrict__ A, long lda,
                                                 const cplx<T>* __restrict__ B, long ldb, int M, int N, int K,
                                                 int tiles_n, cplx<T>* out, long ldo, EpiH e) {
  constexpr int WBM = BM / 32, WBN = BN / 32;
  constexpr int LA = BM + 1, LB = BN + 1;
  using acc_t = typename MF<T>::acc;
  __shared__ cplx<T> sA[2][kBK * LA];
  __shared__ cplx<T> sB[2][kBK * LB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int tm = t / tiles_n, tn = t - tm * tiles_n;  // n fastest: workgroups sharing an A panel are adjacent
  const int i0 = tm * BM, j0 = tn * BN;
  const int mo = (wave & 1) * (BM / 2), no = (wave >> 1) * (BN / 2);
  acc_t cr[WBM][WBN], ci[WBM][WBN];
#pragma unroll
  for (int a = 0; a < WBM; ++a)
#pragma unroll
    for (int b = 0; b < WBN; ++b) {
      cr[a][b] = acc_t{0, 0, 0, 0};
      ci[a][b] = acc_t{0, 0, 0, 0};
    }
  McLoader<T, BM, VEC> la;
  KcLoader<T, BN, VEC> lb;
  const int ntiles = (K + kBK - 1) / kBK;
  if (ntiles > 0) {
    la.load(A, lda, M, i0, 0, K, tid);
    lb.load(B, ldb, B, ldb, N, N, j0, 0, K, tid);
    la.template store<LA>(sA[0], tid);
    lb.template store<LB>(sB[0], tid);
  }
  __syncthreads();
  for (int it = 0; it < ntiles; ++it) {
    const int cur = it & 1;
    const bool more = it + 1 < ntiles;
    if (more) {
      const int kn = (it + 1) * kBK;
      la.load(A, lda, M, i0, kn, K, tid);
      lb.load(B, ldb, B, ldb, N, N, j0, kn, K, tid);
    }
    mma_tile<T, WBM, WBN, false>(sA[cur], sB[cur], LA, LB, mo, no, lane, cr, ci);
    if (more) {
      la.template store<LA>(sA[cur ^ 1], tid);
      lb.template store<LB>(sB[cur ^ 1], tid);
    }
    __syncthreads();
  }
  const cplx<T>* Zl = static_cast<const cplx<T>*>(e.Zl);
#pragma unroll
  for (int a = 0; a < WBM; ++a)
#pragma unroll
    for (int b = 0; b < WBN; ++b) {
      const int col = j0 + no + b * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = i0 + mo + a * 16 + MF<T>::row(lane, r);
        if (row < M && col < N) {
          cplx<T> v = mk<T>(cr[a][b][r], ci[a][b][r]);
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
// Four waves along M, all columns of the tile in each; the tile's width is the multiple of 16 up to 64
// that pads the band count least.  Bound by the matrix cores (64 cycles per fp64 instruction): what
// counts is two workgroups per compute unit, so that one's barriers and loads run under the other's
// products, and a split whose last round is full.  2,048 projectors x 1,088 bands x 147,834 half rows
// in fp64: projection 44.7 ms and nonlocal product 42.3 ms (59 and 62 TFLOP/s); the complex products
// over the whole sphere, one or two workgroups per compute unit, took 95.1 and 98.2 ms.
// ------------------------------------------------------------------------------------------
template <typename T> struct PairCfg;
template <> struct PairCfg<double> {
  static constexpr int BKC = 8, HB = 1, CYC = 64;  // K tile of the projection, row blocks per wave (nonlocal)
};
template <> struct PairCfg<float> {
  static constexpr int BKC = 16, HB = 2, CYC = 32;
};

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
  const double4 r = *reinterpret_cast<const double4*>(bg.rad + 4 * (long)g);
  v[0] = mk<T>((T)(r.x * e.x), (T)(r.x * e.y));
  v[1] = mk<T>((T)(-r.y * e.y), (T)(r.y * e.x));
  v[2] = mk<T>((T)(-r.z * e.y), (T)(r.z * e.x));
  v[3] = mk<T>((T)(-r.w * e.y), (T)(r.w * e.x));
}

// Projector panels: COLS projectors x ROWS half rows, element (row, column) to S[row * LDS_LD + column]
// (projection, ROWS = K) or S[column * LDS_LD + row] (nonlocal, ROWS = M).  From the table (row-contiguous
// columns) or generated, four projectors of an atom per unit.
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
  template <int LDS_LD, bool ROWMAJOR>
  __device__ __forceinline__ void store(cplx<T>* S, int tid) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int idx = tid + q * 256, row = idx % ROWS, col = W * (idx / ROWS);
      if (idx < UNITS) {
#pragma unroll
        for (int m = 0; m < W; ++m) S[ROWMAJOR ? row * LDS_LD + col + m : (col + m) * LDS_LD + row] = r[q][m];
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
  constexpr int BK = PairCfg<T>::BKC, BM = 64 * WBM, BN = 16 * NBN, LA = BM + 1, LB = BN + 1;
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
    la.template store<LA, true>(sA[0], tid);
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
      la.template store<LA, true>(sA[cur ^ 1], tid);
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

// out = EpiH(mode 1) with V_NL psi = beta q over K projectors.  Tile 64 HB half rows x 16 NBN bands.
template <typename T, int NBN, bool OTF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_pairs_nn(
    const cplx<T>* __restrict__ A, long lda, BetaGen bg, const cplx<T>* __restrict__ Q, long ldq, int npw, int nh, int N,
    int K, int tiles_n, cplx<T>* out, long ldo, EpiH e) {
  constexpr int HB = PairCfg<T>::HB, BM = 64 * HB, BN = 16 * NBN, LA = BM + 1, LB = BN + 1;
  using acc_t = typename MF<T>::acc;
  __shared__ cplx<T> sA[2][kBK * LA];
  __shared__ cplx<T> sB[2][kBK * LB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int tm = t / tiles_n, tn = t - tm * tiles_n;  // n fastest: workgroups sharing an A panel are adjacent
  const int i0 = tm * BM, j0 = tn * BN, mo = wave * 16 * HB;
  acc_t fx[HB][NBN], fy[HB][NBN], gx[HB][NBN], gy[HB][NBN];
#pragma unroll
  for (int a = 0; a < HB; ++a)
#pragma unroll
    for (int b = 0; b < NBN; ++b) fx[a][b] = fy[a][b] = gx[a][b] = gy[a][b] = acc_t{0, 0, 0, 0};
  BetaPanel<T, kBK, BM, OTF> la;
  KcLoader<T, BN, false> lb;
  const int ntiles = (K + kBK - 1) / kBK;
  if (ntiles > 0) {
    la.load(A, lda, bg, nh, K, i0, 0, tid);
    lb.load(Q, ldq, Q, ldq, N, N, j0, 0, K, tid);
    la.template store<LA, false>(sA[0], tid);
    lb.template store<LB>(sB[0], tid);
  }
  __syncthreads();
  for (int it = 0; it < ntiles; ++it) {
    const int cur = it & 1, kn = (it + 1) * kBK;
    const bool more = it + 1 < ntiles;
    if (more) {
      la.load(A, lda, bg, nh, K, i0, kn, tid);
      lb.load(Q, ldq, Q, ldq, N, N, j0, kn, K, tid);
    }
#pragma unroll
    for (int kk = 0; kk < kBK; kk += 4) {
      const int kr = kk + (lane >> 4);
      cplx<T> av[HB], bv[NBN];
#pragma unroll
      for (int a = 0; a < HB; ++a) av[a] = sA[cur][kr * LA + mo + a * 16 + (lane & 15)];
#pragma unroll
      for (int b = 0; b < NBN; ++b) bv[b] = sB[cur][kr * LB + b * 16 + (lane & 15)];
#pragma unroll
      for (int a = 0; a < HB; ++a)
#pragma unroll
        for (int b = 0; b < NBN; ++b) {
          fx[a][b] = MF<T>::mma(av[a].x, bv[b].x, fx[a][b]);
          fy[a][b] = MF<T>::mma(av[a].y, bv[b].x, fy[a][b]);
          gx[a][b] = MF<T>::mma(av[a].x, bv[b].y, gx[a][b]);
          gy[a][b] = MF<T>::mma(av[a].y, bv[b].y, gy[a][b]);
        }
    }
    if (more) {
      la.template store<LA, false>(sA[cur ^ 1], tid);
      lb.template store<LB>(sB[cur ^ 1], tid);
    }
    __syncthreads();
  }
  const T* kin = static_cast<const T*>(e.kin);
  const T alpha = (T)e.alpha, cc = (T)e.c, beta = (T)e.beta;
#pragma unroll
  for (int a = 0; a < HB; ++a)
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
      __builtin_amdgcn_sched_barrier(0);  // one block at a time: bounded register use
      const int col = j0 + b * 16 + (lane & 15);
      if (col >= N) continue;
      const cplx<T>* Y = static_cast<const cplx<T>*>(e.Y) + (long)col * e.ldy;
      const cplx<T>* Zl = static_cast<const cplx<T>*>(e.Zl) + (long)col * e.ldz;
      const cplx<T>* Yp = e.Yp ? static_cast<const cplx<T>*>(e.Yp) + (long)col * e.ldp : nullptr;
      cplx<T>* o = out + (long)col * ldo;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int h = i0 + mo + a * 16 + MF<T>::row(lane, r);
        if (h >= nh) continue;
        const int g = npw - 1 - h;  // == h at G = 0
        const T kc = kin[h] - cc;
        const cplx<T> yp = Y[h], ym = Y[g], zp = Zl[h], zm = Zl[g];
        cplx<T> p = mk<T>(alpha * (kc * yp.x + zp.x + (fx[a][b][r] - gy[a][b][r])),
                          alpha * (kc * yp.y + zp.y + (fy[a][b][r] + gx[a][b][r])));
        cplx<T> m = mk<T>(alpha * (kc * ym.x + zm.x + (fx[a][b][r] + gy[a][b][r])),
                          alpha * (kc * ym.y + zm.y + (gx[a][b][r] - fy[a][b][r])));
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
template <typename T> struct CnShape;
template <> struct CnShape<float> {
  static constexpr int BM = 128, BN = 64;
};
template <> struct CnShape<double> {
  static constexpr int BM = 64, BN = 64;
};
template <typename T> struct NnShape;
template <> struct NnShape<float> {
  static constexpr int BM = 128, BN = 128;
};
template <> struct NnShape<double> {
  static constexpr int BM = 128, BN = 64;
};

static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <typename T>
static bool vec_ok(const void* p, long ld) {
  return aligned16(p) && (sizeof(T) == 8 || (ld % 2) == 0);
}

int gemm_cn_tiles(int M, int N, bool fp64) {
  const int bm = fp64 ? CnShape<double>::BM : CnShape<float>::BM;
  const int bn = fp64 ? CnShape<double>::BN : CnShape<float>::BN;
  return ceil_div(M, bm) * ceil_div(N, bn);
}

template <typename T>
hipError_t launch_gemm_cn(const cplx<T>* A, long lda, const cplx<T>* B, long ldb, const cplx<T>* B2, long ldb2,
                          int ncol1, int M, int N, int K, int nsplit, double2* part, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  constexpr int BM = CnShape<T>::BM, BN = CnShape<T>::BN;
  int kchunk = ceil_div(K, nsplit);
  kchunk = ceil_div(kchunk, kBK) * kBK;
  if (kchunk <= 0) kchunk = kBK;
  const int tm = ceil_div(M, BM), tn = ceil_div(N, BN);
  const cplx<T>* b2 = B2 ? B2 : B;
  const long l2 = B2 ? ldb2 : ldb;
  const bool vec = vec_ok<T>(A, lda) && vec_ok<T>(B, ldb) && vec_ok<T>(b2, l2);
  dim3 grid(tm * tn * nsplit);
  if (vec)
    hipLaunchKernelGGL((k_gemm_cn<T, BM, BN, true>), grid, dim3(256), 0, s, A, lda, B, ldb, b2,
                       l2, ncol1, M, N, K, kchunk, tm, tn, part);
  else
    hipLaunchKernelGGL((k_gemm_cn<T, BM, BN, false>), grid, dim3(256), 0, s, A, lda, B, ldb,
                       b2, l2, ncol1, M, N, K, kchunk, tm, tn, part);
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

template <typename T>
hipError_t launch_gemm_nn(const cplx<T>* A, long lda, const cplx<T>* B, long ldb, int M, int N, int K,
                          cplx<T>* out, long ldo, const EpiH& e, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  constexpr int BM = NnShape<T>::BM, BN = NnShape<T>::BN;
  const int tm = ceil_div(M, BM), tn = ceil_div(N, BN);
  const bool vec = vec_ok<T>(A, lda) && vec_ok<T>(B, ldb);
  dim3 grid(tm * tn);
  if (vec)
    hipLaunchKernelGGL((k_gemm_nn<T, BM, BN, true>), grid, dim3(256), 0, s, A, lda, B, ldb, M,
                       N, K, tn, out, ldo, e);
  else
    hipLaunchKernelGGL((k_gemm_nn<T, BM, BN, false>), grid, dim3(256), 0, s, A, lda, B, ldb,
                       M, N, K, tn, out, ldo, e);
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
  const int bk = fp64 ? PairCfg<double>::BKC : PairCfg<float>::BKC, ktiles = ceil_div(nh, bk);
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
// Bands per tile of the nonlocal product: rounds of two workgroups per compute unit x (columns + what a
// tile costs whatever its width).  Narrow tiles fill the chip for small cells (85 row tiles x 101 bands: 4 of
// 32), wide ones read the projector panel less often.
static int pairs_nn_width(int row_tiles, int nb) {
  int best = 64;
  long cost = 1L << 60;
  for (int w = 64; w >= 16; w -= 16) {
    const long c = ((long)row_tiles * ceil_div(nb, w) + 511) / 512 * (w + 16);
    if (c < cost) {
      cost = c;
      best = w;
    }
  }
  return best;
}

template <typename T>
hipError_t launch_pairs_cn(const cplx<T>* A, long lda, const BetaGen* bg, const cplx<T>* Y, long ldy, int M, int nb,
                           int npw, const PairsCn& c, double2* part, hipStream_t s) {
  if (M <= 0 || nb <= 0) return hipSuccess;
  constexpr int BK = PairCfg<T>::BKC;
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
  const int nh = (npw + 1) / 2, tm = ceil_div(nh, 64 * PairCfg<T>::HB), w = pairs_nn_width(tm, nb), tn = ceil_div(nb, w);
  const dim3 grid(tm * tn);
  const BetaGen g = bg ? *bg : BetaGen{};
#define PW_PNN(NBN)                                                                                                  \
  case 16 * NBN:                                                                                                     \
    if (bg)                                                                                                          \
      hipLaunchKernelGGL((k_pairs_nn<T, NBN, true>), grid, dim3(256), 0, s, A, lda, g, Q, ldq, npw, nh, nb, K, tn, out, \
                         ldo, e);                                                                                    \
    else                                                                                                             \
      hipLaunchKernelGGL((k_pairs_nn<T, NBN, false>), grid, dim3(256), 0, s, A, lda, g, Q, ldq, npw, nh, nb, K, tn, out, \
                         ldo, e);                                                                                    \
    break
  switch (w) {
    PW_PNN(1);
    PW_PNN(2);
    PW_PNN(3);
    PW_PNN(4);
  }
#undef PW_PNN
  return hipGetLastError();
}

#define PW_INST_GEMM(T)                                                                                      \
  template hipError_t launch_gemm_cn<T>(const cplx<T>*, long, const cplx<T>*, long, const cplx<T>*, long,   \
                                        int, int, int, int, int, double2*, hipStream_t);                     \
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

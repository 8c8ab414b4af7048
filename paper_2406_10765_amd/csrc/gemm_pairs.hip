// Projector products on pairs (G, -G), split-precision (MFMA 16x16x32 bf16, fp32 accumulation).
//
// The projectors are real functions of position (times a constant phase), so beta(-G) = conj
// beta(G) up to that phase, which D B B^H does not see.  A band psi = f + i g (f, g real functions)
// then has the projections p = <beta|f> + i <beta|g>, each a sum of real products over half of the
// sphere, and V_NL psi = sum_k d_k p_k beta_k needs beta on that half only.  Against the complex
// products over the whole sphere this halves the multiplications, the projector table and its
// traffic.  The sphere's rows are ordered so that -G of row g is row npw - 1 - g: the half is rows
// 0 .. nh - 1, nh = (npw + 1) / 2, its last row is G = 0.
//
//   pair sums of a band y, words (re, im) per half row h with p = y[h], m = y[npw - 1 - h]:
//     F = (p.x + m.x, p.y - m.y)   G = (p.y + m.y, m.x - p.x)   (h < nh - 1)
//     F = (p.x, 0)                 G = (p.y, 0)                 (h = nh - 1, G = 0)
//   projection    p_f = sum_h beta_r F_r + beta_i F_i, p_g the same with G
//   nonlocal      Z_f[h] = sum_k beta[h, k] q_f[k] (q = d p, real), Z_g the same with q_g
//     V_NL y[h] = (Z_f.x - Z_g.y, Z_f.y + Z_g.x),  V_NL y[npw - 1 - h] = (Z_f.x + Z_g.y, Z_g.x - Z_f.y)
//
// Every operand is a pair of bf16 planes (hi, lo) and every product three terms, as in gemm16.hip.
// The block's planes hold columns 0 .. nb - 1 = F, nb .. 2 nb - 1 = G; a tile's groups of 16 real
// columns alternate F and G of the same 16 bands, so that one lane ends up with both parts of a
// band and the complex results leave in the layout of the complex products.
#include <type_traits>

#include "bf16mma.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace pw {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));

// Workgroup barrier the compiler moves no memory access across.
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// K-contiguous tile of 16 NG real columns x 16 words, hi and lo planes, one load of 1 KB per plane
// and group.  PAIR: group g holds the F (g even) or G (g odd) columns of bands c0 + 16 (g / 2) ..;
// otherwise columns c0 + 16 g .. of one matrix.
template <int NG, int NW, bool PAIR>
struct PkTile {
  static constexpr int L = 2 * NG, Q = (L + NW - 1) / NW;
  static_assert(L % NW == 0, "the same number of loads for every wave");
  unsigned int off[Q];
  __device__ __forceinline__ void offsets(long ld, int c0, int ncols, int wave, int lane) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int g = (wave + NW * q) % NG;
      off[q] = pipe_koff_bytes(c0, PAIR ? g >> 1 : g, ncols, ld, lane);
    }
  }
  __device__ __forceinline__ void load(const unsigned int* __restrict__ H, const unsigned int* __restrict__ Lo, long ld,
                                       int c0, int ncols, int k0, unsigned char* dst, int wave) const {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int j = wave + NW * q, pl = j / NG, g = j % NG;
      const int col = PAIR ? (g & 1) * ncols + pipe_kbase_col(c0, g >> 1, ncols) : pipe_kbase_col(c0, g, ncols);
      dma16(at_off((pl ? Lo : H) + (long)col * ld + k0, off[q]), dst + j * 1024);
    }
  }
};

// ------------------------------------------------------------------------------------------
// Projection: part[s][col][row] = (p_f, p_g) of row (projector) and band col over K chunk s.
// ------------------------------------------------------------------------------------------
// Tile 16 AT WM projectors x 16 BT WN real columns, WM x WN waves, NS stages in LDS; every wave
// holds its B fragments and streams the A ones.  Bound by the matrix cores where both dimensions
// fill a tile: 256 x 256 real, two stages of 64 KB (a stage's loads have one stage of MFMAs,
// 3,072 cycles, to arrive in).  2,048 projectors x 1,088 bands x 147,834 half rows: 8.4 ms beside
// the FFTs' stream, 15.8 ms as complex products over the whole sphere.  The K range is whole tiles
// of 16 words: the words of each column from nh to the leading dimension are zero in both operands.
template <int WM, int WN, int AT, int BT, int NS, int WPE>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void k_pairs_proj(
    const unsigned int* __restrict__ Ah, const unsigned int* __restrict__ Al, long lda,
    const unsigned int* __restrict__ Bh, const unsigned int* __restrict__ Bl, long ldb, int M, int N, int ktiles,
    int kchunk, int tiles_m, int tiles_n, double2* __restrict__ part) {
  constexpr int NW = WM * WN, GA = WM * AT, GB = WN * BT;  // groups of 16 rows / real columns
  constexpr int PA = GA * 1024, PB = GB * 1024;            // bytes per plane
  constexpr int SB = 2 * (PA + PB);
  using TA = PkTile<GA, NW, false>;
  using TB = PkTile<GB, NW, true>;
  constexpr int LPW = TA::Q + TB::Q;
  static_assert(BT % 2 == 0, "a wave's columns are whole (F, G) pairs");
  __shared__ __align__(16) unsigned char smem[NS * SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = xcd_tile16(blockIdx.x, gridDim.x);
  const int sp = t / (tiles_m * tiles_n);
  const int tr = t - sp * tiles_m * tiles_n;
  const int tm = tr / tiles_n, tn = tr - tm * tiles_n;
  const int i0 = tm * GA * 16, j0 = tn * GB * 8;
  const int wm = wave % WM, wn = wave / WM;
  const int kt0 = sp * kchunk, ntiles = min(kchunk, ktiles - kt0);  // >= 1
  TA ta;
  TB tb;
  ta.offsets(lda, i0, M, wave, lane);
  tb.offsets(ldb, j0, N, wave, lane);
  auto issue = [&](int kt) {
    unsigned char* st = smem + (kt % NS) * SB;
    const int k0 = (kt0 + kt) * hBK;
    ta.load(Ah, Al, lda, i0, M, k0, st, wave);
    tb.load(Bh, Bl, ldb, j0, N, k0, st + 2 * PA, wave);
  };
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < ntiles) issue(p);
  v4f16 acc[AT][BT];
  bool stored = false;
  int it = 0;
  do {
    const int fend = min(ntiles, it + hFlush);
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
      for (int b = 0; b < BT; ++b) acc[a][b] = v4f16{0, 0, 0, 0};
    for (; it < fend; ++it) {
      // tile it has landed (the next NS - 2 may be in flight); every wave is done with tile it - 1,
      // whose stage receives tile it + NS - 1
      if (NS > 2 && it + NS - 2 < ntiles) wait_vm<(NS - 2) * LPW>();
      else wait_vm<0>();
      wait_lds();
      wg_barrier();
      if (it + NS - 1 < ntiles) issue(it + NS - 1);
      const uint4* st = reinterpret_cast<const uint4*>(smem + (it % NS) * SB);
      const uint4 *Ah_s = st, *Al_s = st + GA * 64, *Bh_s = st + 2 * GA * 64, *Bl_s = Bh_s + GB * 64;
      v8bf bh[BT], bl[BT];
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        bh[b] = frag(Bh_s, (wn * BT + b) * 16, lane);
        bl[b] = frag(Bl_s, (wn * BT + b) * 16, lane);
      }
#pragma unroll
      for (int a = 0; a < AT; ++a) {
        const v8bf ah = frag(Ah_s, (wm * AT + a) * 16, lane);
        const v8bf al = frag(Al_s, (wm * AT + a) * 16, lane);
#pragma unroll
        for (int b = 0; b < BT; ++b) acc[a][b] = mma16(ah, bh[b], acc[a][b]);
#pragma unroll
        for (int b = 0; b < BT; ++b) acc[a][b] = mma16(ah, bl[b], acc[a][b]);
#pragma unroll
        for (int b = 0; b < BT; ++b) acc[a][b] = mma16(al, bh[b], acc[a][b]);
      }
    }
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
      for (int b = 0; b < BT; b += 2) {
        const int col = j0 + (wn * BT + b) * 8 + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = i0 + (wm * AT + a) * 16 + 4 * (lane >> 4) + r;
          if (row < M && col < N) {
            double2* dst = part + ((long)sp * N + col) * M + row;
            double2 v = make_double2((double)acc[a][b][r], (double)acc[a][b + 1][r]);
            if (stored) {
              const double2 o = *dst;
              v.x += o.x;
              v.y += o.y;
            }
            *dst = v;
          }
        }
      }
    stored = true;
  } while (it < ntiles);
}

// ------------------------------------------------------------------------------------------
// Nonlocal product with the H / Chebyshev update as its epilogue.
// ------------------------------------------------------------------------------------------
// A tile: TH half rows (2 TH real rows re, im) of 32 projectors, M-contiguous words, read as MFMA
// fragments by the transposing LDS reads (four 16-bit values of consecutive k per lane).  LDS image of
// one plane: row k of TH words; the 16-byte chunk c of row k sits at chunk c ^ f(k), f(k) = 4
// ((k ^ k / 8) % 4), so that the sixteen rows one read touches fall on four bank windows evenly.
template <int TH, int NW>
struct PmTile {
  static constexpr int R = 256 / TH, LP = 32 / R;  // rows per load of 1 KB, loads per plane
  static constexpr int Q = 2 * LP / NW;
  static_assert(2 * LP % NW == 0, "the same number of loads for every wave");
  unsigned int off[Q];
  // cols: the operand's columns where they are fewer than 32 (then k0 = 0), otherwise 32
  __device__ __forceinline__ void offsets(long ld, int r0, int wave, int lane, int cols) {
#pragma unroll
    for (int q = 0; q < Q; ++q) off[q] = pairs_moff_bytes(TH, ld, r0, (wave + NW * q) % LP, lane, cols);
  }
  __device__ __forceinline__ void load(const unsigned int* __restrict__ H, const unsigned int* __restrict__ Lo, long ld,
                                       int r0, int k0, unsigned char* dst, int wave, int cols) const {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int j = wave + NW * q, pl = j / LP, i = j % LP;
      dma16(at_off((pl ? Lo : H) + (long)(k0 + pairs_mbase_col(TH, i, cols)) * ld + r0, off[q]), dst + j * 1024);
    }
  }
};

__device__ __forceinline__ v8bf frag_tr(const unsigned char* lo_k, const unsigned char* hi_k) {
  typedef __attribute__((address_space(3))) v4s* lp;
  const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(lo_k));
  const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(hi_k));
  return __builtin_bit_cast(v8bf, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// 16 bytes at an 8-byte (float2 pair) or 4-byte (word quad) boundary
struct __attribute__((aligned(8))) F4u {
  float x, y, z, w;
};
struct __attribute__((aligned(4))) U4u {
  unsigned int x, y, z, w;
};

// Four consecutive complex rows of a column, ascending from p: aligned to 16 bytes, or to 8.
template <bool AL>
__device__ __forceinline__ void ld4(const float2* p, float2 (&v)[4]) {
  if constexpr (AL) {
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    v[0] = make_float2(a.x, a.y);
    v[1] = make_float2(a.z, a.w);
    v[2] = make_float2(b.x, b.y);
    v[3] = make_float2(b.z, b.w);
  } else {
    const F4u a = reinterpret_cast<const F4u*>(p)[0], b = reinterpret_cast<const F4u*>(p)[1];
    v[0] = make_float2(a.x, a.y);
    v[1] = make_float2(a.z, a.w);
    v[2] = make_float2(b.x, b.y);
    v[3] = make_float2(b.z, b.w);
  }
}
template <bool AL>
__device__ __forceinline__ void st4(float2* p, const float2 (&v)[4]) {
  if constexpr (AL) {
    reinterpret_cast<float4*>(p)[0] = make_float4(v[0].x, v[0].y, v[1].x, v[1].y);
    reinterpret_cast<float4*>(p)[1] = make_float4(v[2].x, v[2].y, v[3].x, v[3].y);
  } else {
    reinterpret_cast<F4u*>(p)[0] = F4u{v[0].x, v[0].y, v[1].x, v[1].y};
    reinterpret_cast<F4u*>(p)[1] = F4u{v[2].x, v[2].y, v[3].x, v[3].y};
  }
}

// Pair sums of rows g and -g (see the head of this file).
__device__ __forceinline__ float2 pair_f(float2 p, float2 m) { return make_float2(p.x + m.x, p.y - m.y); }
__device__ __forceinline__ float2 pair_g(float2 p, float2 m) { return make_float2(p.y + m.y, m.x - p.x); }
__device__ __forceinline__ void split_word(float2 v, unsigned int& h, unsigned int& l) {
  const Split2 a = split(v.x), b = split(v.y);
  h = pack(a.h, b.h);
  l = pack(a.l, b.l);
}

// The update of four half rows h0 .. h0 + 3 of one band from their accumulators zf, zg.
struct PairEpi {
  const EpiH& e;
  int npw, nh, nb;
  float2* out;
  long ldo;
  float alpha, cc, beta;
  __device__ __forceinline__ PairEpi(const EpiH& e_, int npw_, int nh_, int nb_, float2* out_, long ldo_)
      : e(e_), npw(npw_), nh(nh_), nb(nb_), out(out_), ldo(ldo_), alpha((float)e_.alpha), cc((float)e_.c),
        beta((float)e_.beta) {}
  __device__ __forceinline__ float2 update(float2 v, float kr, float2 y, float2 z, float2 p) const {
    const float kc = kr - cc;
    v.x = alpha * (kc * y.x + z.x + v.x);
    v.y = alpha * (kc * y.y + z.y + v.y);
    if (e.Yp) {
      v.x -= beta * p.x;
      v.y -= beta * p.y;
    }
    return v;
  }
  __device__ __forceinline__ void quad(int h0, int col, const float2 (&zf)[4], const float2 (&zg)[4]) const {
    const float* kin = static_cast<const float*>(e.kin);
    const float2* Y = static_cast<const float2*>(e.Y) + (long)col * e.ldy;
    const float2* Zl = static_cast<const float2*>(e.Zl) + (long)col * e.ldz;
    const float2* Yp = e.Yp ? static_cast<const float2*>(e.Yp) + (long)col * e.ldp : nullptr;
    float2* o = out + (long)col * ldo;
    unsigned int *fh = static_cast<unsigned int*>(e.ph), *fl = static_cast<unsigned int*>(e.pl);
    unsigned int *ch = static_cast<unsigned int*>(e.ch), *cl = static_cast<unsigned int*>(e.cl);
    const long of = (long)col * e.ldpl + h0, og = (long)(nb + col) * e.ldpl + h0, oc = (long)col * e.ldcl;
    if (e.vec4 && h0 + 4 < nh) {
      const int m0 = npw - 4 - h0;  // row of -(h0 + 3)
      float2 p[4], m[4], y[4], z[4], q[4] = {};
      const float4 k4 = *reinterpret_cast<const float4*>(kin + h0);
      const float kr[4] = {k4.x, k4.y, k4.z, k4.w};
      ld4<true>(Y + h0, y);
      ld4<true>(Zl + h0, z);
      if (Yp) ld4<true>(Yp + h0, q);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        p[r] = update(make_float2(zf[r].x - zg[r].y, zf[r].y + zg[r].x), kr[r], y[r], z[r], q[r]);
      ld4<false>(Y + m0, y);
      ld4<false>(Zl + m0, z);
      if (Yp) ld4<false>(Yp + m0, q);
#pragma unroll
      for (int r = 0; r < 4; ++r)  // m[i] is row m0 + i, the partner of h0 + 3 - i
        m[r] = update(make_float2(zf[3 - r].x + zg[3 - r].y, zg[3 - r].x - zf[3 - r].y), kr[3 - r], y[r], z[r], q[r]);
      st4<true>(o + h0, p);
      st4<false>(o + m0, m);
      if (fh) {
        unsigned int wh[4], wl[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) split_word(pair_f(p[r], m[3 - r]), wh[r], wl[r]);
        *reinterpret_cast<uint4*>(fh + of) = uint4{wh[0], wh[1], wh[2], wh[3]};
        *reinterpret_cast<uint4*>(fl + of) = uint4{wl[0], wl[1], wl[2], wl[3]};
#pragma unroll
        for (int r = 0; r < 4; ++r) split_word(pair_g(p[r], m[3 - r]), wh[r], wl[r]);
        *reinterpret_cast<uint4*>(fh + og) = uint4{wh[0], wh[1], wh[2], wh[3]};
        *reinterpret_cast<uint4*>(fl + og) = uint4{wl[0], wl[1], wl[2], wl[3]};
      }
      if (ch) {
        unsigned int wh[4], wl[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) split_word(p[r], wh[r], wl[r]);
        *reinterpret_cast<uint4*>(ch + oc + h0) = uint4{wh[0], wh[1], wh[2], wh[3]};
        *reinterpret_cast<uint4*>(cl + oc + h0) = uint4{wl[0], wl[1], wl[2], wl[3]};
#pragma unroll
        for (int r = 0; r < 4; ++r) split_word(m[r], wh[r], wl[r]);
        *reinterpret_cast<U4u*>(ch + oc + m0) = U4u{wh[0], wh[1], wh[2], wh[3]};
        *reinterpret_cast<U4u*>(cl + oc + m0) = U4u{wl[0], wl[1], wl[2], wl[3]};
      }
      return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int h = h0 + r;
      float2 F = make_float2(0.f, 0.f), G = F;  // words past the half sphere are zero
      if (h < nh) {
        const int g = npw - 1 - h;
        const float2 zero = make_float2(0.f, 0.f);
        const float2 p = update(make_float2(zf[r].x - zg[r].y, zf[r].y + zg[r].x), kin[h], Y[h], Zl[h],
                                Yp ? Yp[h] : zero);
        float2 m = zero;
        if (h < nh - 1)
          m = update(make_float2(zf[r].x + zg[r].y, zg[r].x - zf[r].y), kin[h], Y[g], Zl[g], Yp ? Yp[g] : zero);
        o[h] = p;
        if (h < nh - 1) o[g] = m;
        F = h < nh - 1 ? pair_f(p, m) : make_float2(p.x, 0.f);
        G = h < nh - 1 ? pair_g(p, m) : make_float2(p.y, 0.f);
        if (ch) {
          split_word(p, ch[oc + h], cl[oc + h]);
          if (h < nh - 1) split_word(m, ch[oc + g], cl[oc + g]);
        }
      }
      if (fh && h < e.ldpl) {
        split_word(F, fh[of + r], fl[of + r]);
        split_word(G, fh[og + r], fl[og + r]);
      }
    }
  }
};

// Tile 16 HB WM half rows x 8 CB WN bands.  K tile of 32 projectors; B planes hold q as words of
// two projectors (K-contiguous, zero past nproj: the table holds whole K tiles, or the projectors alone where
// they are fewer than 32).  Bound by the matrix cores, then by the update's
// traffic (three blocks read, one block and its planes written): at the size above 9.1 ms, 14.4 ms
// as complex products.
template <int WM, int WN, int HB, int CB, int NS, int WPE>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void k_pairs_nl(
    const unsigned int* __restrict__ Ah, const unsigned int* __restrict__ Al, long lda,
    const unsigned int* __restrict__ Bh, const unsigned int* __restrict__ Bl, long ldb, int npw, int nh, int nb,
    int ktiles, int cols, int tiles_n, float2* out, long ldo, EpiH e) {
  constexpr int NW = WM * WN, TH = 16 * HB * WM, GB = WN * CB;
  constexpr int PA = 32 * TH * 4, PB = GB * 1024;  // bytes per plane
  constexpr int SB = 2 * (PA + PB);
  using TA = PmTile<TH, NW>;
  using TB = PkTile<GB, NW, true>;
  constexpr int LPW = TA::Q + TB::Q;
  static_assert(CB % 2 == 0, "a wave's columns are whole (F, G) pairs");
  __shared__ __align__(16) unsigned char smem[NS * SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = xcd_tile16(blockIdx.x, gridDim.x);
  const int tm = t / tiles_n, tn = t - tm * tiles_n;
  const int r0 = tm * TH, j0 = tn * GB * 8;
  const int wm = wave % WM, wn = wave / WM;
  TA ta;
  TB tb;
  ta.offsets(lda, r0, wave, lane, cols);
  tb.offsets(ldb, j0, nb, wave, lane);
  auto issue = [&](int kt) {
    unsigned char* st = smem + (kt % NS) * SB;
    ta.load(Ah, Al, lda, r0, kt * 32, st, wave, cols);
    tb.load(Bh, Bl, ldb, j0, nb, kt * hBK, st + 2 * PA, wave);
  };
  // this lane's part of the transposing reads: row k = 8 (l / 16) + 4 u + (l % 16) / 4, chunk l % 4 of
  // the 16-row block's four
  const int kg = lane >> 4, ks = (lane & 15) >> 2;
  const int arow = ((8 * kg + ks) * TH + 4 * (lane & 3)) * 4, win = (ks ^ kg) & 3;
  v4f16 acc[HB][2][CB];
#pragma unroll
  for (int a = 0; a < HB; ++a)
#pragma unroll
    for (int b = 0; b < CB; ++b) acc[a][0][b] = acc[a][1][b] = v4f16{0, 0, 0, 0};
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < ktiles) issue(p);
  for (int it = 0; it < ktiles; ++it) {
    if (NS > 2 && it + NS - 2 < ktiles) wait_vm<(NS - 2) * LPW>();
    else wait_vm<0>();
    wait_lds();
    wg_barrier();
    if (it + NS - 1 < ktiles) issue(it + NS - 1);
    const unsigned char* st = smem + (it % NS) * SB;
    const uint4* Bh_s = reinterpret_cast<const uint4*>(st + 2 * PA);
    const uint4* Bl_s = Bh_s + GB * 64;
    v8bf bh[CB], bl[CB];
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      bh[b] = frag(Bh_s, (wn * CB + b) * 16, lane);
      bl[b] = frag(Bl_s, (wn * CB + b) * 16, lane);
    }
#pragma unroll
    for (int a = 0; a < HB; ++a) {
      const unsigned char* pa = st + arow + ((wm * HB + a) ^ win) * 64;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const v8bf ah = frag_tr(pa + 8 * q, pa + 8 * q + 16 * TH);
        const v8bf al = frag_tr(pa + 8 * q + PA, pa + 8 * q + PA + 16 * TH);
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[a][q][b] = mma16(ah, bh[b], acc[a][q][b]);
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[a][q][b] = mma16(ah, bl[b], acc[a][q][b]);
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[a][q][b] = mma16(al, bh[b], acc[a][q][b]);
      }
    }
  }
  const PairEpi epi(e, npw, nh, nb, out, ldo);
#pragma unroll
  for (int a = 0; a < HB; ++a)
#pragma unroll
    for (int b = 0; b < CB; b += 2) {
      __builtin_amdgcn_sched_barrier(0);  // one block at a time: bounded register use
      const int col = j0 + (wn * CB + b) * 8 + (lane & 15);
      const int h0 = r0 + (wm * HB + a) * 16 + 4 * (lane >> 4);
      if (col >= nb) continue;
      float2 zf[4], zg[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        zf[r] = make_float2(acc[a][r >> 1][b][2 * (r & 1)], acc[a][r >> 1][b][2 * (r & 1) + 1]);
        zg[r] = make_float2(acc[a][r >> 1][b + 1][2 * (r & 1)], acc[a][r >> 1][b + 1][2 * (r & 1) + 1]);
      }
      epi.quad(h0, col, zf, zg);
    }
}

// ------------------------------------------------------------------------------------------
// Operand preparation
// ------------------------------------------------------------------------------------------
// Pair planes of nb fp32 columns: four half rows per thread, zero words from nh to ldp.
template <bool VEC>
__global__ __launch_bounds__(256) void k_pair_planes(const float2* __restrict__ X, long ldx, int npw, int nh, int nb,
                                                     unsigned int* __restrict__ H, unsigned int* __restrict__ L,
                                                     long ldp) {
  const long per = ldp / 4;
  PW_GRID_STRIDE(idx, per * nb) {
    const int j = (int)(idx / per), h0 = 4 * (int)(idx - (long)j * per);
    const float2* x = X + (long)j * ldx;
    float2 p[4], m[4];
    unsigned int fh[4], fl[4], gh[4], gl[4];
    if (VEC && h0 + 4 < nh) {
      ld4<true>(x + h0, p);
      ld4<false>(x + (npw - 4 - h0), m);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        split_word(pair_f(p[r], m[3 - r]), fh[r], fl[r]);
        split_word(pair_g(p[r], m[3 - r]), gh[r], gl[r]);
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int h = h0 + r;
        float2 F = make_float2(0.f, 0.f), G = F;
        if (h < nh) {
          const float2 a = x[h];
          const float2 b = x[npw - 1 - h];
          F = h < nh - 1 ? pair_f(a, b) : make_float2(a.x, 0.f);
          G = h < nh - 1 ? pair_g(a, b) : make_float2(a.y, 0.f);
        }
        split_word(F, fh[r], fl[r]);
        split_word(G, gh[r], gl[r]);
      }
    }
    const long of = (long)j * ldp + h0, og = (long)(nb + j) * ldp + h0;
    *reinterpret_cast<uint4*>(H + of) = uint4{fh[0], fh[1], fh[2], fh[3]};
    *reinterpret_cast<uint4*>(L + of) = uint4{fl[0], fl[1], fl[2], fl[3]};
    *reinterpret_cast<uint4*>(H + og) = uint4{gh[0], gh[1], gh[2], gh[3]};
    *reinterpret_cast<uint4*>(L + og) = uint4{gl[0], gl[1], gl[2], gl[3]};
  }
}

// Sum of the projection's partials in split order, times d, rounded to fp32 and split: words of two
// consecutive projectors, columns 0 .. nb - 1 the f parts, nb .. 2 nb - 1 the g parts, zero from nproj
// to 2 ldp projectors.
__global__ __launch_bounds__(256) void k_pair_reduce(const double2* __restrict__ part, int nsplit, int M, int nb,
                                                     const double* __restrict__ dscale, unsigned int* __restrict__ H,
                                                     unsigned int* __restrict__ L, long ldp) {
  PW_GRID_STRIDE(idx, ldp * nb) {
    const int j = (int)(idx / ldp), w = (int)(idx - (long)j * ldp);
    unsigned int fh = 0, fl = 0, gh = 0, gl = 0;
    if (2 * w < M) {  // M is a multiple of 4
      const double2* src = part + (long)j * M + 2 * w;
      const double2 a = sum_splits(src, nsplit, (long)M * nb), b = sum_splits(src + 1, nsplit, (long)M * nb);
      const double d0 = dscale[(2 * w) & 3], d1 = dscale[(2 * w + 1) & 3];
      split_word(make_float2((float)(a.x * d0), (float)(b.x * d1)), fh, fl);
      split_word(make_float2((float)(a.y * d0), (float)(b.y * d1)), gh, gl);
    }
    H[(long)j * ldp + w] = fh;
    L[(long)j * ldp + w] = fl;
    H[(long)(nb + j) * ldp + w] = gh;
    L[(long)(nb + j) * ldp + w] = gl;
  }
}

// ------------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------------
namespace {

// Tile shapes of the projection, by what a K tile costs a compute unit that runs `per_cu` of them.
struct ProjShape {
  int rows, bands, per_cu;
  double us, lat;  // per K tile of 16 words: of a full compute unit's time, and from its loads to its products
};
constexpr ProjShape kProj[4] = {
    {256, 128, 1, 1.7, 1.7}, {128, 64, 2, 0.55, 0.9}, {64, 32, 3, 0.3, 0.3}, {256, 16, 1, 2.0, 2.0}};

// The largest tile that the product fills.  Below 65,536 outputs 64 x 32, from there 128 x 64, at 18,537 half rows
// (us in the one and the other): 256 projectors x 144 bands 38.5 and 44.5, 256 x 256 54.2 and 60.2, 256 x 300 71.9
// and 65.1, 512 x 240 103 and 89; at 40,363 they cross sooner: 256 x 160 76.7 and 76.9, 256 x 240 111 and 103, 256 x 300
// 179 and 144.  From 2^17 outputs 256 x 128 (128 x 64 and 256 x 128): 18,537 half rows 512 x 256 90 and 117, 864 x 200
// 128 and 148; 40,363: 512 x 160 151 and 157, 512 x 256 214 and 190, 864 x 200 294 and 266, 864 x 440 534 and 467: the
// line lies between the two lengths' own.  Up to 16 bands (a Lanczos vector) the table's one read is the cost and the
// narrow tile keeps three stages of it in flight (one band, 2,048 projectors: 0.48 ms, 5.0 TB/s of a 2.4 GB table;
// 1.65 ms as complex products in 256 x 128 tiles).
int proj_shape(int M, int nb) {
  if (nb <= 16 && M >= 256) return 3;
  if (M >= 256 && nb >= 96 && (long)M * nb >= (1L << 17)) return 0;
  if (M >= 128 && nb >= 48 && (long)M * nb >= (1L << 16)) return 1;
  return 2;
}

}  // namespace

// K splits: the number that minimises the busiest compute unit's K tiles + the start and end of each round + the
// partials' traffic, at most cap (what the partials' buffer holds) and 64.  With 72 tiles (2,048 projectors,
// 1,088 bands) 7 splits fill 504 of 512 places in two rounds; their partials are an eighth of those of the
// 57 short chunks the complex products balanced their tail with (reduction 0.41 ms there).  With one tile
// (32 projectors, 20 bands, 52 K tiles) 52 splits of one tile each take 4 us, 3 splits took 51.
int pairs_proj_splits(int M, int nb, int ktiles, long cap) {
  if (M <= 0 || nb <= 0 || ktiles <= 0) return 1;
  const ProjShape& s = kProj[proj_shape(M, nb)];
  const long tiles = (long)ceil_div(M, s.rows) * ceil_div(nb, s.bands), slots = 256L * s.per_cu;
  int best = 1;
  double cost = 1e300;
  for (int n = 1; n <= 64 && n <= ktiles && (n == 1 || n <= cap); ++n) {
    const int chunk = ceil_div(ktiles, n);
    if (ceil_div(ktiles, chunk) != n) continue;
    const double rounds = (double)((tiles * n + slots - 1) / slots), per_cu = (double)((tiles * n + 255) / 256);
    const double c = std::max(per_cu * s.us, rounds * s.lat) * chunk + 6.0 * rounds + 0.02 * n +
                     n * (double)M * nb * 32.0 / 4.5e6;
    if (c < cost) {
      cost = c;
      best = n;
    }
  }
  return best;
}

hipError_t launch_pairs_proj(const unsigned int* Ah, const unsigned int* Al, long lda, const unsigned int* Bh,
                             const unsigned int* Bl, long ldb, int M, int nb, int ktiles, int nsplit, double2* part,
                             hipStream_t s) {
  if (M <= 0 || nb <= 0) return hipSuccess;
  const int shape = proj_shape(M, nb);
  const int tm = ceil_div(M, kProj[shape].rows), tn = ceil_div(nb, kProj[shape].bands);
  const int kchunk = ceil_div(ktiles, nsplit);
  if ((long)kchunk * (nsplit - 1) >= ktiles) return hipErrorInvalidValue;  // every split has work
  const dim3 grid(tm * tn * nsplit);
#define PW_PROJ(WM, WN, AT, BT, NS, WPE)                                                                             \
  hipLaunchKernelGGL((k_pairs_proj<WM, WN, AT, BT, NS, WPE>), grid, dim3(64 * WM * WN), 0, s, Ah, Al, lda, Bh, Bl, ldb, \
                     M, nb, ktiles, kchunk, tm, tn, part)
  switch (shape) {
    case 0: PW_PROJ(2, 4, 8, 4, 2, 2); break;
    case 1: PW_PROJ(2, 2, 4, 4, 2, 2); break;
    case 2: PW_PROJ(2, 2, 2, 2, 3, 3); break;
    default: PW_PROJ(4, 1, 4, 2, 4, 1); break;
  }
#undef PW_PROJ
  return hipGetLastError();
}

hipError_t launch_pairs_nl(const unsigned int* Ah, const unsigned int* Al, long lda, const unsigned int* Bh,
                           const unsigned int* Bl, long ldb, int npw, int nb, int acols, float2* out, long ldo,
                           const EpiH& e0, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  const int nh = (npw + 1) / 2, ktiles = ceil_div(acols, 32), cols = std::min(acols, 32);
  if (acols > 32 && acols % 32 != 0) return hipErrorInvalidValue;  // whole K tiles
  EpiH e = e0;
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  e.vec4 = al(out) && ldo % 2 == 0 && al(e.Zl) && e.ldz % 2 == 0 && al(e.kin) && al(e.Y) && e.ldy % 2 == 0 &&
           (!e.Yp || (al(e.Yp) && e.ldp % 2 == 0));
#define PW_NL(WM, WN, HB, CB, NS, WPE)                                                                              \
  do {                                                                                                              \
    const int tn = ceil_div(nb, 8 * CB * WN);                                                                       \
    hipLaunchKernelGGL((k_pairs_nl<WM, WN, HB, CB, NS, WPE>), dim3(ceil_div(nh, 16 * HB * WM) * tn),                \
                       dim3(64 * WM * WN), 0, s, Ah, Al, lda, Bh, Bl, ldb, npw, nh, nb, ktiles, cols, tn, out, ldo,  \
                       e);                                                                                          \
  } while (0)
  // 128 half rows x 128 bands when that leaves several tiles per compute unit and pads the bands by at most a
  // tenth more than 64 would (1,088 bands: 8.64 ms, 9.45 in 64 x 64; 440 bands, 40,363 half rows: 616 us and 563);
  // 64 x 64 (two workgroups per compute unit) below, 64 x 48 where it pads less (144 bands, 18,537 half rows:
  // 43.6 us, 48.7 in 64 x 64; at equal padding they are equal); 128 x 16 for few bands, where the table's read is
  // the cost (one band, 2,048 projectors: 0.56 ms; 2.1 ms as complex products in 128 x 128 tiles)
  if (nb <= 16 && ktiles >= 8) PW_NL(4, 1, 2, 2, 3, 1);
  else if (nb >= 96 && (long)ceil_div(nh, 128) * ceil_div(nb, 128) >= 512 && 20 * ceil_div(nb, 128) <= 11 * ceil_div(nb, 64))
    PW_NL(2, 4, 4, 4, 2, 2);
  else if (48 * ceil_div(nb, 48) < 64 * ceil_div(nb, 64)) PW_NL(4, 1, 1, 6, 2, 2);
  else PW_NL(2, 2, 2, 4, 2, 2);
#undef PW_NL
  return hipGetLastError();
}

hipError_t launch_pair_planes(const float2* X, long ldx, int npw, int nb, unsigned int* H, unsigned int* L, long ldp,
                              hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  const int nh = (npw + 1) / 2;
  const dim3 grid(stride_blocks(ldp / 4 * nb));
  if ((reinterpret_cast<uintptr_t>(X) & 15) == 0 && ldx % 2 == 0)
    hipLaunchKernelGGL(k_pair_planes<true>, grid, dim3(256), 0, s, X, ldx, npw, nh, nb, H, L, ldp);
  else
    hipLaunchKernelGGL(k_pair_planes<false>, grid, dim3(256), 0, s, X, ldx, npw, nh, nb, H, L, ldp);
  return hipGetLastError();
}

hipError_t launch_pair_reduce(const double2* part, int nsplit, int M, int nb, const double* dscale, unsigned int* H,
                              unsigned int* L, long ldp, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pair_reduce, dim3(stride_blocks(ldp * nb)), dim3(256), 0, s, part, nsplit, M, nb, dscale, H, L,
                     ldp);
  return hipGetLastError();
}

}  // namespace pw

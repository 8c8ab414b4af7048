// Host planner: plane-wave sphere, sticks, grid, radix plans and arena layout.
#pragma once

#include <string>
#include <vector>

#include "../../include/pw.h"
#include "common.hpp"
#include "kernels.hpp"

namespace pw {

constexpr size_t kArenaAlign = 256;
constexpr size_t kDefaultMaxLds = 160 * 1024;  // LDS per workgroup on gfx950
constexpr int kLanczosChunk = 64;  // Lanczos steps whose (alpha, beta) stay on the device between host reads

struct ArenaLayout {
  size_t miller, sticks, colstart, kin, tw1, tw2, tw3, vr, frac, mmil, mamp, mpha, vg, dscale;
  size_t beta, brad, bph, yp, u0, u1, zb, wf, sb, g1, pparts, pt, parts, sh, ct, ct2, eig, ework, resid, info, scal, lanc,
      occ, lz;
  size_t rsat, rszo, rsze, rsbo, rsbe, rsao, rsae, rsp;  // real-space projector tables and partials
  size_t total;
};

struct Plan {
  // copy of the description
  double L[3];
  double ecut;
  int natoms;
  std::vector<double> tau;  // 3 * natoms, Cartesian
  std::vector<double> frac; // 3 * natoms, fractional (tau / L)
  int nbands;
  double zval, rc, gauss_c, beta_sigma, d0, d1;
  std::vector<int> mode_miller;
  std::vector<double> mode_amp, mode_phase;
  int prec;
  unsigned flags;
  int real_bytes;  // 8 (FP64) or 4 (mixed)
  // basis
  int nmax[3];
  int n[3];
  int npw, nst, nproj;
  long ldw;  // internal leading dimension (npw rounded up to 16)
  // half of the sphere, rows 0 .. nh - 1 (row npw - 1 - g is -G of row g; row nh - 1 is G = 0), and
  // its leading dimension (a multiple of 16)
  int nh;
  long ldh;
  int nproj32;  // nproj rounded up to 32 (the split-precision products' K tile)
  int bcols;    // projector columns of the split-precision table: nproj32, or nproj where that is below 32
  std::vector<int> miller;     // 3 * npw, stick order
  std::vector<Stick> sticks;   // nst
  std::vector<int> colstart;   // n1a + 1: first stick of each active x column
  std::vector<double> kin;     // npw: |G|^2 / 2
  GridDesc g;
  FftLaunch fl;
  int fft_batch;               // bands per FFT launch group
  int nbb;                     // bands per filter block (== nbands: unblocked step)
  int nsplit_proj, nsplit_gram;
  int nsplit_lob;  // K splits of the LOBPCG basis Gram product (PW_FLAG_LOBPCG), else 0
  size_t gram_bytes;   // partials of the Gram products
  size_t fft_budget;   // bytes of the stick and pencil buffers of one batch
  int pencil_pitch;    // row pitch of the sized pencil form, 0: none for this grid
  // bf16 plane columns held per plane, of ldy words: nbb (the pair planes of the block entering the
  // projection, 2 nb columns of ldh words), or 2 nbb when the unblocked step also keeps the planes of
  // Y and H Y for the Gram product: Y's in the first nb columns, and in the nb columns after them the
  // pair planes until the projection of H Y has read them, then the planes of H Y
  int yp_cols;
  long ldy;  // max(ldw, 2 ldh)
  int hmax[3];                 // max |n_d| over the sphere (projector generator tables)
  int bwidth;                  // per-atom axis-factor table length
  int proj_form;               // PW_PROJ_GSPACE or PW_PROJ_LOCALIZED
  // real-space projectors (PW_FLAG_RSPACE_KB): per-atom positions, the (atom, plane) entries per
  // plane and per (plane, 8-row band), and each atom's per-plane entries; see RsDesc
  bool rspace;
  double rs_radius;
  std::vector<float> rs_atoms;  // 4 per atom
  std::vector<int> rs_zoff, rs_boff, rs_aoff, rs_aent;
  std::vector<RsEnt> rs_zent, rs_bent;
  ArenaLayout lay;
  // Whether an H application on nb bands may run its local part (memory bound) on the second stream beside the
  // projection (matrix cores): the buffers of the two are then in use together.
  bool overlaps(int nb) const { return !rspace && (double)npw * nb >= (double)(1 << 26); }
};

// Fills `p` from `d`; returns PW_OK or PW_EINVAL with a message.
pw_status make_plan(const pw_cell_desc* d, size_t max_lds, Plan* p, std::string* err);
// Arena bytes up to which widen_plan enlarges the FFT batches, at least lay.total (the footprint).
size_t plan_useful_bytes(const Plan& p);
// Larger FFT batches where an arena beyond lay.total holds them; the other buffers stay in place.
void widen_plan(Plan* p, size_t arena_bytes);

// 2^p 3^q test and radix plan
bool is_23_smooth(int n);
FftPlan radix_plan(int n);

}  // namespace pw

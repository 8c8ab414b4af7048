// Host-side bounds test of the direct global-to-LDS loads of the projector products on pairs, with the
// kernels' own address arithmetic (pipe_addr.hpp): every load of the first and last K tile of every
// workgroup tile lies inside its operand, and the 16-byte chunks of an A tile fill its LDS image once.
// Usage: pairs_bounds npw nproj nb
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#define __host__
#define __device__
#include "../paper_2406_10765_amd/csrc/pipe_addr.hpp"

using namespace pw;

static long bad = 0, checked = 0;

static void check(long word, long lo, long hi) {
  ++checked;
  if (word < lo || word + 3 >= hi) ++bad;
}

// groups of 16 columns; pair: F and G alternate
static void kgroups(int ng, bool pair, int c0, int ncols, long ld, int k0) {
  for (int g = 0; g < ng; ++g)
    for (int lane = 0; lane < 64; ++lane) {
      const int gi = pair ? g >> 1 : g;
      const long col = (pair ? (g & 1) * (long)ncols : 0) + pipe_kbase_col(c0, gi, ncols);
      const long word = col * ld + k0 + pipe_koff_bytes(c0, gi, ncols, ld, lane) / 4;
      const long lo = pair ? (g & 1) * (long)ncols * ld : 0;
      check(word, lo, lo + (long)ncols * ld);
      check(word % ld, 0, ld);
    }
}

int main(int argc, char** argv) {
  if (argc < 4) return 2;
  const int npw = std::atoi(argv[1]), M = std::atoi(argv[2]), nb = std::atoi(argv[3]);
  const int nh = (npw + 1) / 2, ldh = (nh + 15) / 16 * 16, m32 = (M + 31) / 32 * 32;
  const int rows[4] = {256, 128, 64, 256}, bands[4] = {128, 64, 32, 16};
  for (int s = 0; s < 4; ++s)
    for (int i0 = 0; i0 < M; i0 += rows[s])
      for (int j0 = 0; j0 < nb; j0 += bands[s])
        for (int k0 : {0, ldh - 16}) {
          kgroups(rows[s] / 16, false, i0, M, ldh, k0);
          kgroups(bands[s] / 8, true, j0, nb, ldh, k0);
        }
  for (int th : {64, 128}) {
    const int R = 256 / th;
    for (int r0 = 0; r0 < nh; r0 += th)
      for (int kt : {0, m32 / 32 - 1})
        for (int i = 0; i < 32 / R; ++i)
          for (int lane = 0; lane < 64; ++lane)
            check((long)(kt * 32 + i * R) * ldh + r0 + pairs_moff_bytes(th, ldh, r0, i, lane) / 4, 0, (long)ldh * m32);
    // an unclamped tile: each chunk of each row exactly once
    for (int i = 0; i < 32 / R; ++i)
      for (int kk = 0; kk < R; ++kk) {
        std::vector<long> c;
        for (int l = 0; l < th / 4; ++l) c.push_back(pairs_moff_bytes(th, 4096, 0, i, kk * (th / 4) + l) / 4 - kk * 4096L);
        std::sort(c.begin(), c.end());
        for (int l = 0; l < th / 4; ++l) {
          ++checked;
          if (c[l] != 4 * l) ++bad;
        }
      }
  }
  for (int j0 = 0; j0 < nb; j0 += 64)
    for (int k0 : {0, m32 / 2 - 16}) kgroups(8, true, j0, nb, m32 / 2, k0);
  for (int j0 = 0; j0 < nb; j0 += 48)
    for (int k0 : {0, m32 / 2 - 16}) kgroups(6, true, j0, nb, m32 / 2, k0);
  for (int j0 = 0; j0 < nb; j0 += 128)
    for (int k0 : {0, m32 / 2 - 16}) kgroups(16, true, j0, nb, m32 / 2, k0);
  std::printf("npw=%d nproj=%d nb=%d: %ld checked, %ld wrong\n", npw, M, nb, checked, bad);
  return bad ? 1 : 0;
}

// Twiddle constants of the in-register DFTs (fft_small.hpp): sin and cos of whole fractions of a turn, reduced in
// integers and taken from decimals, so that each is the nearest double (a power series of the angle in double was
// off by up to 1.7e-16, the same way in every transform, which a density does not average out).  No GPU code: the
// host checks it.
#pragma once

namespace pw {

struct SinCos {
  double s, c;
};
// sin and cos of k / 144 of a turn (2.5 k degrees), 0 <= k <= 18, for the angles of 2^p 3^q points that occur
constexpr SinCos octant(int k) {
  switch (k) {
    case 0: return {0.0, 1.0};
    case 4: return {0.17364817766693034885171662676931, 0.98480775301220805936674302458952};   // 10 degrees
    case 6: return {0.25881904510252076234889883762405, 0.96592582628906828674974319972890};   // 15
    case 8: return {0.34202014332566873304409961468226, 0.93969262078590838405410927732473};   // 20
    case 9: return {0.38268343236508977172845998403040, 0.92387953251128675612818318939679};   // 22.5
    case 12: return {0.5, 0.86602540378443864676372317075294};                                 // 30
    case 16: return {0.64278760968653932632264340990726, 0.76604444311897803520239265055542};  // 40
    case 18: return {0.70710678118654752440084436210485, 0.70710678118654752440084436210485};  // 45
  }
  return {2.0, 2.0};  // an angle without a constant: refused where it is used
}
// sin(2 pi t / S)
constexpr double turn_sin(int t, int S) {
  t = (t % S + S) % S;
  if (2 * t > S) return -turn_sin(S - t, S);
  if (4 * t > S) return turn_sin(S - 2 * t, 2 * S);
  const int k = 8 * t > S ? 36 * (S - 4 * t) : 144 * t;
  const SinCos v = octant(k % S == 0 ? k / S : -1);
  return 8 * t > S ? v.c : v.s;
}
constexpr double turn_cos(int t, int S) { return turn_sin(4 * t + S, 4 * S); }

}  // namespace pw

// Tile geometry of the odd-p passes (odd.hip): the plan of a transform, the
// tile shapes the kernels are compiled for, and their register digits.  Plain
// C++, so that the whole of it can be checked on the host.
#pragma once

#include <stdint.h>

#include <vector>

namespace fdwt {

// One pass of a plan: digits [d0, d0 + r), rows of p^wdig elements; le: the
// tile exponent of an odd-p pass (wdig + r).
struct PassGeom {
  int d0, r, wdig, le;
};

// Tiles as small as two passes allow, by measurement, with rows of at least 40
// bytes: more workgroups at few points, and several per CU, whose loads,
// arithmetic and stores overlap.
inline std::vector<PassGeom> odd_plan(int p, int m, bool f64) {
  std::vector<PassGeom> out;
  auto first = [&](int le) { out.push_back({0, le, 0, le}); };
  auto strided = [&](int le, int r) {
    const int d0 = out.back().d0 + out.back().r;
    out.push_back({d0, r, le - r, le});
  };
  // The largest net of one tile, and the exponent of every tile beyond it.
  // Forward + inverse pairs, this choice (us) against the generic passes
  // before it, and against the next tile: p = 3 double m = 9 20 / 30, m = 12
  // 33 / 46, m = 14 114 / 153 (3^7 and three passes: 139); p = 3 float m = 14
  // 60 (3^7: 81); p = 5 float m = 8 25 / 55, m = 10 140 / 226 (5^5 and three
  // passes: 154), m = 11 846 / 1268 (5^5: 932); p = 5 double m = 10 302 / 519;
  // p = 7 float m = 5 20 / 23, m = 8 103 / 154, m = 9 802 / 1118 (two passes
  // of 7^5, a CU each: 818); double m = 8 172 / 250.
  // p = 3 float, a pair with tiles of 3^7 / 3^8: 3^12 points 21.5 / 24.6; 3^9
  // 15.5 / 15.9, 3^10 14.7 / 17.7, 3^11 15.5 / 20.2.  The last three stay at
  // 3^8: tiles of 3^7 take the digits in another order, which changes the last
  // bits of the coefficients.
  int single, le;
  if (p == 3) {
    single = 8;
    le = f64 ? (m <= 12 || m > 14 ? 7 : 8) : (m == 12 ? 7 : 8);
  } else if (p == 5) {
    single = f64 ? 5 : 6;
    le = f64 ? (m <= 6 ? 4 : 5) : (m <= 9 ? 5 : 6);
  } else {
    single = 4;
    le = m <= 5 ? 3 : 4;
  }
  if (m <= single) {
    first(m);
    return out;
  }
  first(le);
  const int rest = m - le;
  // Digits of a strided pass: rows of 9 (p = 3), 5 or 25 (p = 5) and 7
  // (p = 7) elements at least.
  const int cap = p == 3 ? le - 2 : le - 1;
  if (p == 3 && rest == 1) le = 7;  // 3^9 points, float: one digit needs rows of 3^6
  const int n = (rest + cap - 1) / cap;
  for (int i = 0, done = 0; i < n; ++i) {
    const int r = (rest - done + (n - i) - 1) / (n - i);
    strided(le, r);
    done += r;
  }
  return out;
}

// The tile shapes (p^le elements, rd digits) of the plans above: what the pass
// kernels are compiled for.
constexpr bool odd_has_shape(int p, bool f64, int le, int rd) {
  const int single = p == 3 ? 8 : (p == 5 ? (f64 ? 5 : 6) : 4);
  if (rd == le) return le >= 1 && le <= single;
  if (p == 3 && f64) return (le == 7 && rd >= 2 && rd <= 5) || (le == 8 && (rd == 5 || rd == 6));
  if (p == 3) return (le == 7 && (rd == 1 || rd == 5)) || (le == 8 && rd >= 2 && rd <= 6);
  if (p == 5 && f64) return (le == 4 && rd == 2) || (le == 5 && rd >= 2 && rd <= 4);
  if (p == 5) return (le == 5 && rd >= 2 && rd <= 4) || (le == 6 && (rd == 4 || rd == 5));
  return (le == 3 && rd == 2) || (le == 4 && (rd == 2 || rd == 3));
}

// Register digits of a shape: two where the tile's p^(le - 2) threads still
// fill waves (p = 5 float, m = 9: 43 against 46 us a pair with one), but one
// for p = 5 in double (25 complex values and as many prefetched leave few
// waves: eff_dim at m = 9, s = 20 823 against 729 us).
constexpr int odd_kt(int p, int le, int rd, bool f64) { return rd >= 2 && le >= 5 && !(p == 5 && f64) ? 2 : 1; }

// Three register digits for the p = 3 float tiles of 3^8 elements (243
// threads, three workgroups per CU; with two digits 729 threads, two per CU)
// where they let every tile run in one round and two digits do not: 512 to 768
// tiles on 256 CUs, which 3^14 points make (729 tiles, 58.3 against 62.5 us a
// pair).  The digits' order depends on it, so the rule counts the CUs of the
// whole chip, not those that a device has: a result does not depend on the
// partition that computes it.
constexpr bool odd_kt3(int p, bool f64, int le, int64_t tiles) {
  return p == 3 && !f64 && le == 8 && tiles > 2 * 256 && tiles <= 3 * 256;
}
// ... which only the passes of that plan need: 8 digits, then 6.
constexpr bool odd_kt3_shape(int le, int rd) { return le == 8 && (rd == 8 || rd == 6); }

}  // namespace fdwt

// Interpolant evaluation by table rows: Sf(q) = sum_n c_n K(q, x_n) (Section
// 3.2) for nets whose points come in blocks that share their lookups.
//
// The p^K points n = h p^K + r of a block (K = 2 for p = 2, 1 for p odd) have
// X_j(n) = X_j(h p^K) (+) X_j(r) (digit-wise mod p).  When the first K columns
// of every C_j are zero below a non-singular K x K block (as in every
// non-singular upper triangular C_j), the X_j(r) have no digits but their
// first K, and those take all p^K values, so of the differences
// q_j (-) X_j(n) of one block exactly one starts with K zero digits, and the
// digits after the first K are the same in all.  With z = q_j (-) X_j(h p^K), b its
// first K digits and t the index of its first non-zero digit after them, the
// block's p^K factors 1 + gamma_j K'(.) depend on (b, t) only: a row of p^K
// floats in LDS.  One XOR, one leading-zero count and one address serve p^K
// evaluations, each of which then costs one multiplication and 4 bytes of
// LDS reads, against four operations and a 4-byte read of its own in
// k_spline_eval (spline.hip), which takes the nets outside this rule.
// Measured on MI355X, k_spline_eval before and this after: p = 2, N = 2^14,
// s = 20, 4096 queries 167 -> 58 us (2.3e13 evaluations/s); p = 3, N = 3^12,
// s = 10, 15001 queries 8.3 -> 4.7 ms (1.7e13/s); p = 5, N = 5^8, s = 10,
// 10000 queries 4.1 -> 2.1 ms (1.9e13/s); p = 7, N = 7^6, s = 10, 20000
// queries 2.5 -> 1.05 ms (2.2e13/s).  What bounds it is the issue of vector
// operations (an integer operation takes a SIMD 4 cycles per wave, a float
// multiplication 2: measured), then bank conflicts of the row reads.
#include "coords.h"
#include "dev_math.h"

#include <algorithm>
#include <cstring>

namespace fdwt {

// Geometry of the rows for one prime.
//   A point word (one per block and coordinate, wave-uniform) holds the ND
//   digits after the first K at the top, DB bits each; p = 2 puts b's share
//   at bits 5..4 (the row's byte offset) and a one at bit 0; p odd puts
//   1 + (first digit), 1..p, in the low bits.  FMASK covers these low bits
//   alone: the ND digits end right above (p = 3: the 16th digit of 3^16 points
//   lies at bits 3..2).  The low bits keep z non-zero, so its leading-zero
//   count is at most 31 and no row index is out of range.
//   Counts of ND DB or more mean that all ND digits agree.
//   A row is 16 bytes (the factors r = 0..3); for p = 5, 7 the factors from
//   r = 4 on lie in a second region of the coordinate (R2 bytes per row).
//   NT groups of RPT rows: one group per count (p = 2) or per digit.  The
//   rows of a coordinate's frequent digits should lie in distinct LDS banks:
//   16 rows do, so merging the counts of one digit pays for its operation
//   (p = 5: 2.48 -> 2.11 ms, p = 7: 1.58 -> 1.06 ms at the sizes above), and
//   8-byte parts instead of 16-byte rows cost more reads than they save
//   conflicts (p = 5: 4.0 ms).
//   U: blocks taken together in the loop (p = 3: 4.85 against 5.1 ms for one;
//   three, or two for the other primes, were no faster).
template <int P>
struct RowCfg;
template <>
struct RowCfg<2> {
  static constexpr int K = 2, B = 4, ND = 26, DB = 1, NT = 32, RPT = 4, R2 = 0, U = 1;
  static constexpr uint32_t FMASK = 63;
};
template <>
struct RowCfg<3> {
  static constexpr int K = 1, B = 3, ND = 15, DB = 2, NT = 16, RPT = 3, R2 = 0, U = 2;
  static constexpr uint32_t FMASK = 3;
};
template <>
struct RowCfg<5> {
  static constexpr int K = 1, B = 5, ND = 9, DB = 3, NT = 16, RPT = 5, R2 = 4, U = 1;
  static constexpr uint32_t FMASK = 7;
};
template <>
struct RowCfg<7> {
  static constexpr int K = 1, B = 7, ND = 9, DB = 3, NT = 16, RPT = 7, R2 = 16, U = 1;
  static constexpr uint32_t FMASK = 7;
};
template <int P>
constexpr bool low_bits_apart() {
  return RowCfg<P>::FMASK >= P && RowCfg<P>::FMASK >> (32 - RowCfg<P>::ND * RowCfg<P>::DB) == 0;
}
static_assert(low_bits_apart<2>() && low_bits_apart<3>() && low_bits_apart<5>() && low_bits_apart<7>(),
              "the low bits of a point word hold no digit after the first K");
template <int P>
constexpr int row_bytes() { return RowCfg<P>::NT * RowCfg<P>::RPT * (16 + RowCfg<P>::R2); }  // LDS per coordinate

// Values of one coordinate's factor in LDS after the rows, kRowT floats each:
// entry k < D for first differing digit k, entry D when all D digits agree.
// The first K digits of X_j(1) and X_j(2) (p = 2: bits 1..0 and 3..2 of
// kt.ix[j], first digit in the higher bit) or of X_j(1) (p odd: kt.ix[j]).
constexpr int kRowT = kTab;

// Leading zero digits of b (-) (first K digits of X_j(r)), K if all are zero.
template <int P>
__device__ __forceinline__ int lead_of_row(int pf, int b, int r) {
  if constexpr (P == 2) {
    const int z = b ^ ((r & 1 ? pf & 3 : 0) ^ (r & 2 ? (pf >> 2) & 3 : 0));
    return z == 0 ? 2 : (z & 2 ? 0 : 1);
  } else {
    return (b + r * (P - pf)) % P == 0 ? 1 : 0;
  }
}

// ------------------------------------------------------------ point words
__device__ __forceinline__ uint32_t row_word_p2(uint32_t q32) {
  return ((q32 << 2) & ~63u) | ((q32 >> 30) << 4);
}

__global__ void __launch_bounds__(256) k_row_words_p2(const uint32_t* __restrict__ xtab, int nbytes, int s, int m,
                                                      int64_t nblk, uint32_t* __restrict__ out) {
  const int64_t total = nblk * s;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t h = (uint32_t)(i / s), j = (uint32_t)(i - (int64_t)h * s), n = h * 4;
    const uint32_t* t = xtab + (size_t)j * nbytes * 256;
    uint32_t x = 0;
    for (int b = 0; b < nbytes; ++b) x ^= t[b * 256 + ((n >> (8 * b)) & 255)];
    out[i] = row_word_p2(x << (32 - m)) | 1u;
  }
}

template <int P>
__global__ void __launch_bounds__(256) k_row_words_odd(const uint64_t* __restrict__ ptab, int s, int m, int64_t nblk,
                                                       uint32_t* __restrict__ out) {
  using R = RowCfg<P>;
  using O = OddCoords<P>;
  const int64_t total = nblk * s;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t h = (uint32_t)(i / s), n = h * P;
    const int j = (int)(i - (int64_t)h * s);
    const uint64_t x = addmod_packed<P>(ptab[(int64_t)j * O::groups(m) * O::PK + n % O::PK],
                                        O::upper(ptab, m, j, n / O::PK));
    // digit r + 1 of X_j at bits 4(m - 1 - r)
    uint32_t w = 1u + (uint32_t)((x >> (4 * (m - 1))) & 15u);
    for (int f = 1; f < m && f <= R::ND; ++f) w |= (uint32_t)((x >> (4 * (m - 1 - f))) & 15u) << (32 - R::DB * f);
    out[i] = w;
  }
}

// ----------------------------------------------------------- query words
// (hi, lo) of a query: hi the ND digits after the first K in the point words'
// layout; lo = first digit (p odd) and, at bits 15..8, the index of the first
// non-zero digit after those ND (D if there is none): the first differing
// digit of a query and a point that agree on all the digits before, since
// points have no more than K + ND digits (eval_rows_ok).
__device__ __forceinline__ uint2 row_query_p2(uint32_t v) {
  const uint32_t low = v & 15u;
  return make_uint2(row_word_p2(v), (low ? (uint32_t)__clz(low) : 32u) << 8);
}

template <int P>
__global__ void __launch_bounds__(256) k_row_queries(const uint32_t* __restrict__ q, int64_t nq, int s, int D,
                                                     uint2* __restrict__ out) {
  using R = RowCfg<P>;
  const int64_t total = (int64_t)s * nq;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    uint32_t v = q[i], hi = 0;
    int keq = D;
    for (int f = D - 1; f >= 1; --f) {
      const uint32_t dg = v % P;
      v /= P;
      if (f <= R::ND) hi |= dg << (32 - R::DB * f);
      else if (dg) keq = f;
    }
    out[i] = make_uint2(hi, v % P | ((uint32_t)keq << 8));
  }
}

// ------------------------------------------------------------- evaluation
// The rows start at LDS address 0 (the kernel has no other shared arrays), so
// row addresses are plain LDS byte addresses.
using lds_cf = const float __attribute__((address_space(3)))*;

// Multiplies pr by the row at byte address a of the coordinate region at off.
template <int P>
__device__ __forceinline__ void mul_row(float* pr, uint32_t a, uint32_t off) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  using l4 = const f4 __attribute__((address_space(3)))*;
  const f4 v = *(l4)(a + off);
  if constexpr (P == 2) {
    pr[0] *= v.x;
    pr[1] *= v.y;
    pr[2] *= v.z;
    pr[3] *= v.w;
  } else if constexpr (P == 3) {
    pr[0] *= v.x;
    pr[1] *= v.y;
    pr[2] *= v.z;
  } else {
    constexpr uint32_t second = RowCfg<P>::NT * RowCfg<P>::RPT * 16;
    pr[0] *= v.x;
    pr[1] *= v.y;
    pr[2] *= v.z;
    pr[3] *= v.w;
    if constexpr (P == 5) {
      pr[4] *= *(lds_cf)((a >> 2) + (off + second));
    } else {
      const f4 w = *(l4)(a + (off + second));
      pr[4] *= w.x;
      pr[5] *= w.y;
      pr[6] *= w.z;
    }
  }
}

// Workgroups of TH threads: tqw waves' worth of queries (64 tqw) and
// TH / (64 tqw) sub-chunks of points, so that the table of a workgroup serves
// 16 waves whatever the number of queries.  Sub-chunk y of all takes blocks
// [y bpc, (y + 1) bpc); a workgroup adds its sub-chunks' sums in order and
// writes one partial sum per query.  SG: coordinates rounded up to 4.
// Point words, c and the first digits are wave-uniform: scalar loads.
// Factors are multiplied in the order of the coordinates; the float sums are
// closed every 64 points (at multiples of 64 where a sub-chunk has more than
// 128 points) and then added as float pairs, as in k_spline_eval.
// Two workgroups of 1024 threads share a CU while a wave needs at most 64
// vector and 80 scalar registers: asked of the compiler where the query words
// leave room (p = 3, s = 10 without it: 86 scalar registers, 6.9 against
// 4.75 ms).
constexpr int row_waves(int p, int sg, int th) {
  return sg <= (p == 2 ? 36 : (p == 3 ? 20 : 12)) ? 8 : th / 256;
}
template <int P, int SG, int TH>
__global__ void __launch_bounds__(TH, row_waves(P, SG, TH)) k_eval_rows(const uint32_t* __restrict__ xw, const float* __restrict__ c, int nblk,
                                                  int s, const void* __restrict__ qv, int64_t nq,
                                                  KernTab kt, int tqw, int bpc, df* __restrict__ partial) {
  using R = RowCfg<P>;
  constexpr int B = R::B, NT = R::NT, JB = row_bytes<P>();
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x;
  float* tt = reinterpret_cast<float*>(smem + (size_t)s * JB);  // [s][kRowT]
  int* pfx = reinterpret_cast<int*>(tt + s * kRowT);           // [s]
  {
#pragma clang fp contract(off)
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    double kv = 0.0;
#pragma unroll
    for (int t = 0; t < kTab; ++t)
      if (lane == t) kv = kt.kp[t];
    for (int j = w; j < s; j += TH / 64) {
      const double g = kt.gamma[j];
      if (lane < kTab) tt[j * kRowT + lane] = (float)(1.0 + g * kv);
      if (lane == kTab) pfx[j] = kt.ix[j];
    }
  }
  __syncthreads();
  // Rows: entry r of row (t, b) of coordinate j.
  for (int i = tid; i < s * NT * R::RPT; i += TH) {
    const int j = i / (NT * R::RPT), e = i - j * (NT * R::RPT), t = e / R::RPT, b = e - t * R::RPT;
    const float* T = tt + j * kRowT;
    const int pf = pfx[j];
    const int dg = R::NT < 32 ? t : t / R::DB;  // first non-zero digit: K + dg (K + ND or more: see exact())
    float* row = reinterpret_cast<float*>(smem + (size_t)j * JB + e * 16);
    float* row2 = reinterpret_cast<float*>(smem + (size_t)j * JB + NT * R::RPT * 16 + e * R::R2);
#pragma unroll
    for (int r = 0; r < B; ++r) {
      int k = lead_of_row<P>(pf, b, r);
      if (k == R::K) k = dg < R::ND ? R::K + dg : -1;
      (r < 4 ? row[r] : row2[r - 4]) = k < 0 ? __int_as_float(0x7fc00000) : T[k];
    }
  }
  __syncthreads();
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nsub = (TH / 64) / tqw, sub = wv / tqw;
  const int ql = (wv - sub * tqw) * 64 + (tid & 63);
  const int64_t qi = (int64_t)blockIdx.x * (64 * tqw) + ql;
  const int64_t qq = qi < nq ? qi : nq - 1;
  // Words of query i, coordinate j (p = 2: made here from the query itself).
  auto query = [&](int j, int64_t i) -> uint2 {
    if constexpr (P == 2) return row_query_p2(((const uint32_t*)qv)[(int64_t)j * nq + i]);
    else return ((const uint2*)qv)[(int64_t)j * nq + i];
  };
  uint32_t qh[SG];
  uint32_t m0[P == 2 ? 1 : SG], m1[P >= 5 ? SG : 1];
#pragma unroll
  for (int j = 0; j < SG; ++j) {
    if (j >= SG - 3 && j >= s) continue;
    const uint2 v = query(j, qq);
    qh[j] = v.x;
    if constexpr (P != 2) {
      // Byte 1 + x0 of (m1, m0): byte offset of row b = (q0 - x0) mod p.
      const uint32_t q0 = v.y & 255u;
      uint32_t lo = 0, hi = 0;
#pragma unroll
      for (int x0 = 0; x0 < P; ++x0) {
        const uint32_t b = (q0 >= (uint32_t)x0 ? q0 - x0 : q0 + P - x0) * 16;
        if (x0 < 3) lo |= b << (8 * (x0 + 1));
        else hi |= b << (8 * (x0 - 3));
      }
      m0[j] = lo;
      if constexpr (P >= 5) m1[j] = hi;
    }
  }
  using cu32 = const uint32_t __attribute__((address_space(4)))*;
  using cf32 = const float __attribute__((address_space(4)))*;
  const cu32 xs = (cu32)xw;
  const cf32 cs = (cf32)c;
  // Row address of coordinate j for point word x.
  auto addr = [&](uint32_t x, uint32_t qw, uint32_t a0, uint32_t a1) -> uint32_t {
    const uint32_t z = qw ^ x;
    uint32_t t;
    asm("v_ffbh_u32 %0, %1" : "=v"(t) : "v"(z));
    if constexpr (P == 2) return (t << 6) | (z & 48u);
    const uint32_t sel = (x & R::FMASK) | 0x0c0c0c00u;
    const uint32_t w = __builtin_amdgcn_perm(a1, a0, sel);
    if constexpr (P == 3) return __umul24(t & 30u, 24) + w;
    return __umul24(__umul24(t, 43) >> 7, R::RPT * 16) + w;  // t / 3
  };
  const int y = blockIdx.y * nsub + sub;
  const int h0 = (int)min((int64_t)y * bpc, (int64_t)nblk), h1 = (int)min((int64_t)h0 + bpc, (int64_t)nblk);
  df acc = {0.0f, 0.0f};
  // Products of the points of U consecutive blocks from block h on.
  auto products = [&](int h, auto& pr) {
    constexpr int U = sizeof(pr) / sizeof(float) / B;
    const cu32 xp = xs + (int64_t)h * s;
#pragma unroll
    for (int u = 0; u < U * B; ++u) pr[u] = 1.0f;
#pragma unroll
    for (int j = 0; j < SG; ++j) {
      if (j >= SG - 3 && j >= s) continue;
#pragma unroll
      for (int v = 0; v < U; ++v)
        mul_row<P>(pr + v * B,
                   addr(xp[v * s + j], qh[j], P == 2 ? 0u : m0[P == 2 ? 0 : j], P >= 5 ? m1[P >= 5 ? j : 0] : 0u),
                   (uint32_t)(j * JB));
    }
  };
  // The points of block h exactly, where all ND digits of some coordinate
  // agree with a point of the block: that factor depends on the query's
  // remaining digits only.
  auto exact = [&](int h, float* pr) {
    const cu32 xp = xs + (int64_t)h * s;
    int64_t qo = qq;
    asm volatile("" : "+v"(qo));
#pragma unroll
    for (int u = 0; u < B; ++u) pr[u] = 1.0f;
    for (int j = 0; j < s; ++j) {
      const uint2 v = query(j, qo);
      const uint32_t x = xp[j], z = v.x ^ x;
      const int t = __clz(z), dg = t / R::DB;
      const float* T = tt + j * kRowT;
      const int pf = pfx[j];
      int b;
      if constexpr (P == 2) b = (int)((z >> 4) & 3u);
      else b = ((int)(v.y & 255u) + P - (int)((x & R::FMASK) - 1u)) % P;
#pragma unroll
      for (int u = 0; u < B; ++u) {
        int k = lead_of_row<P>(pf, b, u);
        if (k == R::K) k = dg < R::ND ? R::K + dg : (int)(v.y >> 8);
        pr[u] *= T[k];
      }
    }
  };
  // Points whose factors may need the exact path (NaN products).
  auto mend = [&](int h, auto& pr) {
    constexpr int U = sizeof(pr) / sizeof(float) / B;
#pragma unroll
    for (int v = 0; v < U; ++v) {
      bool rare = false;
#pragma unroll
      for (int u = 0; u < B; ++u) rare |= __builtin_isnan(pr[v * B + u]);
      if (rare) exact(h + v, pr + v * B);
    }
  };
  int left = 64;  // points until the float sum is closed (wave-uniform)
  float sum = 0.0f;
  for (int h = h0; h < h1;) {
    const int he = h + min((left - 1) / (R::U * B), (h1 - h) / R::U) * R::U;
    left -= (he - h) * B;
    for (; h < he; h += R::U) {
      float pr[R::U * B];
      products(h, pr);
      float next = sum;
#pragma unroll
      for (int u = 0; u < R::U * B; ++u) next += cs[(int64_t)h * B + u] * pr[u];
      if (__builtin_isnan(next)) {
        mend(h, pr);
        next = sum;
#pragma unroll
        for (int u = 0; u < R::U * B; ++u) next += cs[(int64_t)h * B + u] * pr[u];
      }
      sum = next;
    }
    if (h < h1) {  // one block, in which the sum may be closed
      float pr[B];
      products(h, pr);
      mend(h, pr);
#pragma unroll
      for (int u = 0; u < B; ++u) {
        sum += cs[(int64_t)h * B + u] * pr[u];
        if (u + 1 == left) {
          acc = add(acc, df{sum, 0.0f});
          sum = 0.0f;
        }
      }
      left -= B;
      if (left <= 0) left += 64;
      ++h;
    }
  }
  acc = add(acc, df{sum, 0.0f});
  // Sub-chunks of the workgroup in order (the rows are no longer needed).
  __syncthreads();
  df* red = reinterpret_cast<df*>(smem);
  red[sub * 64 * tqw + ql] = acc;
  __syncthreads();
  if (sub == 0 && qi < nq) {
    for (int i = 1; i < nsub; ++i) acc = add(acc, red[i * 64 * tqw + ql]);
    partial[(int64_t)blockIdx.y * nq + qi] = acc;
  }
}

// =============================================================== host side
static int row_k(int p) { return p == 2 ? 2 : 1; }
static int row_bytes_of(int p) { return p == 2 ? row_bytes<2>() : p == 3 ? row_bytes<3>() : p == 5 ? row_bytes<5>() : row_bytes<7>(); }

static size_t rows_lds(int p, int s) { return (size_t)s * (row_bytes_of(p) + kRowT * 4 + 4); }

// Prefixes of coordinate j (see kRowT), or -1 when the first K columns
// of C_j are not a non-singular K x K block over zeros.
static int row_prefix(const Net& net, int j) {
  auto C = [&](int r, int c) { return (int)net.C[((size_t)j * net.m + r) * net.m + c]; };
  for (int c = 0; c < row_k(net.p); ++c)
    for (int r = row_k(net.p); r < net.m; ++r)
      if (C(r, c)) return -1;
  if (net.p != 2) return C(0, 0) ? C(0, 0) : -1;
  const int x1 = C(0, 0) * 2 + C(1, 0), x2 = C(0, 1) * 2 + C(1, 1);
  return x1 && x2 && x1 != x2 ? x1 | x2 << 2 : -1;
}

// Nets the rows serve: the first K columns of every generator matrix as
// above, the points have no digits
// beyond the words' K + ND (p = 5: m <= 10; the other primes' largest nets
// fit), and the rows of all coordinates fit a CU's LDS (p = 7: s <= 44).
bool eval_rows_ok(const Net& net) {
  if (net.m < row_k(net.p) || (net.p == 5 && net.m > 10) || rows_lds(net.p, net.s) > 160 * 1024) return false;
  for (int j = 0; j < net.s; ++j)
    if (row_prefix(net, j) < 0) return false;
  return true;
}

// Threads of a workgroup: 1024 while the query words (p = 2: one, p = 3: two,
// p = 5, 7: three registers per coordinate) leave the loop its registers.
constexpr int row_threads(int p, int sg) { return (p == 2 ? 1 : (p == 3 ? 2 : 3)) * sg > 80 ? 512 : 1024; }

// Query groups of 64 tqw queries x gy workgroups, bpc blocks per sub-chunk; a
// function of the shape alone, so that a result does not depend on where it
// runs.  Of the divisions into up to eight rounds of workgroups, the one with
// the least work on the busiest slot (a workgroup's start counted as 12
// blocks); sub-chunks of 128 points or more end at multiples of 64.
// No more partial sums per query than k_spline_eval makes of the shape
// (eval_grid), so that the workspace does not depend on the kernel: where 256
// queries a workgroup would need more, fewer queries share it, and more of
// its waves divide the points.
void eval_rows_grid(int p, int s, int64_t N, int64_t nq, int* tqw_out, int* gy_out, int* bpc_out) {
  const int sg = (s + 3) / 4 * 4, th = row_threads(p, sg);
  const int64_t slots = 256 * (row_waves(p, sg, th) * 256 / th);
  const int64_t nblk = N / (p == 2 ? 4 : p);
  const int unit = p == 2 ? 16 : 64;  // blocks that end at a multiple of 64 points
  int gy_most;
  int64_t ppc, best = -1;
  eval_grid(N, nq, &gy_most, &ppc);
  auto consider = [&](int tqw, int64_t most) {
    const int nsub = th / 64 / tqw;
    const int64_t qg = (nq + 64 * tqw - 1) / (64 * tqw);
    for (int rounds = 1; rounds <= 8; ++rounds) {
      int64_t gy = std::max<int64_t>(1, std::min({rounds * slots / qg, nblk / (8 * nsub), most}));
      int64_t bpc = std::max<int64_t>(1, (nblk + gy * nsub - 1) / (gy * nsub));
      if (bpc >= 2 * unit) bpc = (bpc + unit - 1) / unit * unit;
      gy = std::max<int64_t>(1, (nblk + bpc * nsub - 1) / (bpc * nsub));
      // (One round of long workgroups ends unevenly: p = 7, N = 7^6, 20000
      // queries 1.18 ms in one, 1.03 ms in more.)
      const int64_t cost = (gy * qg + slots - 1) / slots * (bpc + 12) + (rounds == 1 && bpc >= 256 ? bpc / 4 : 0);
      if (best >= 0 && cost >= best) continue;
      best = cost;
      *tqw_out = tqw;
      *gy_out = (int)gy;
      *bpc_out = (int)bpc;
    }
  };
  const int tqw = nq <= 64 ? 1 : (nq <= 128 ? 2 : 4);
  consider(tqw, nblk);
  if (*gy_out <= gy_most) return;
  best = -1;
  for (int t = tqw; t >= 1; t /= 2) consider(t, gy_most);
}

// The prefixes of every coordinate into kt.ix.
void eval_rows_prefixes(const Net& net, KernTab& kt) {
  for (int j = 0; j < net.s; ++j) kt.ix[j] = row_prefix(net, j);
}

static unsigned rows_grid1(int64_t n) { return (unsigned)std::min<int64_t>((n + 255) / 256, 4096); }

// Point words of every block, [N / p^K][s] (within packed_bytes(net)).
int launch_row_words(const Net& net, uint32_t* out, hipStream_t st) {
  const int64_t nblk = net.N / (net.p == 2 ? 4 : net.p);
  const unsigned g = rows_grid1(nblk * net.s);
  if (net.p == 2) {
    hipLaunchKernelGGL(k_row_words_p2, dim3(g), dim3(256), 0, st, net.d_xtab, net.nbytes, net.s, net.m, nblk, out);
  } else if (net.p == 3) {
    hipLaunchKernelGGL(k_row_words_odd<3>, dim3(g), dim3(256), 0, st, net.d_ptab, net.s, net.m, nblk, out);
  } else if (net.p == 5) {
    hipLaunchKernelGGL(k_row_words_odd<5>, dim3(g), dim3(256), 0, st, net.d_ptab, net.s, net.m, nblk, out);
  } else {
    hipLaunchKernelGGL(k_row_words_odd<7>, dim3(g), dim3(256), 0, st, net.d_ptab, net.s, net.m, nblk, out);
  }
  FDWT_HIP(hipGetLastError());
  return FDWT_OK;
}

// p odd: the query words [s][nq].
int launch_row_queries(const Net& net, const uint32_t* q, int64_t nq, void* out, hipStream_t st) {
  const unsigned g = rows_grid1(nq * net.s);
  const int D = query_depth(net.p);
  uint2* o = (uint2*)out;
  if (net.p == 3) hipLaunchKernelGGL(k_row_queries<3>, dim3(g), dim3(256), 0, st, q, nq, net.s, D, o);
  else if (net.p == 5) hipLaunchKernelGGL(k_row_queries<5>, dim3(g), dim3(256), 0, st, q, nq, net.s, D, o);
  else hipLaunchKernelGGL(k_row_queries<7>, dim3(g), dim3(256), 0, st, q, nq, net.s, D, o);
  FDWT_HIP(hipGetLastError());
  return FDWT_OK;
}

template <int P, int SG>
static int launch_rows_sg(const Net& net, const uint32_t* xw, const float* c, int64_t nq, const void* qv,
                          const KernTab& kt, df* partial, int tqw, int gy, int bpc, hipStream_t st) {
  if constexpr ((SG - 3) * row_bytes<P>() > 160 * 1024) {
    return fail(FDWT_EINVAL, "evaluation rows exceed the LDS");
  } else {
    constexpr int TH = row_threads(P, SG);
    auto fn = k_eval_rows<P, SG, TH>;
    const size_t lds = std::max<size_t>(rows_lds(P, net.s), (size_t)TH * sizeof(df));
    if (int rc = allow_lds((const void*)fn, lds)) return rc;
    const dim3 grid((unsigned)((nq + 64 * tqw - 1) / (64 * tqw)), (unsigned)gy);
    const int nblk = (int)(net.N / RowCfg<P>::B);
    hipLaunchKernelGGL(fn, grid, dim3(TH), lds, st, xw, c, nblk, net.s, qv, nq, kt, tqw, bpc, partial);
    FDWT_HIP(hipGetLastError());
    return FDWT_OK;
  }
}

template <int P>
static int launch_rows_p(const Net& net, const uint32_t* xw, const float* c, int64_t nq, const void* qv,
                         const KernTab& kt, df* partial, int tqw, int gy, int bpc, hipStream_t st) {
  switch ((net.s + 3) / 4) {
#define FDWT_ROWS(G) \
  case G: return launch_rows_sg<P, 4 * G>(net, xw, c, nq, qv, kt, partial, tqw, gy, bpc, st)
    FDWT_ROWS(1); FDWT_ROWS(2); FDWT_ROWS(3); FDWT_ROWS(4); FDWT_ROWS(5); FDWT_ROWS(6); FDWT_ROWS(7); FDWT_ROWS(8);
    FDWT_ROWS(9); FDWT_ROWS(10); FDWT_ROWS(11); FDWT_ROWS(12); FDWT_ROWS(13); FDWT_ROWS(14); FDWT_ROWS(15);
    FDWT_ROWS(16);
#undef FDWT_ROWS
  }
  return fail(FDWT_EINVAL, "s must be in 1..64");
}

// Partial sums [gy][nq] of Sf at nq queries (p = 2: the queries themselves, p
// odd: their words from launch_row_queries).
int launch_eval_rows(const Net& net, const uint32_t* xw, const float* c, int64_t nq, const void* qv, const KernTab& kt,
                     df* partial, hipStream_t st) {
  int tqw, gy, bpc;
  eval_rows_grid(net.p, net.s, net.N, nq, &tqw, &gy, &bpc);
  switch (net.p) {
    case 2: return launch_rows_p<2>(net, xw, c, nq, qv, kt, partial, tqw, gy, bpc, st);
    case 3: return launch_rows_p<3>(net, xw, c, nq, qv, kt, partial, tqw, gy, bpc, st);
    case 5: return launch_rows_p<5>(net, xw, c, nq, qv, kt, partial, tqw, gy, bpc, st);
  }
  return launch_rows_p<7>(net, xw, c, nq, qv, kt, partial, tqw, gy, bpc, st);
}

}  // namespace fdwt

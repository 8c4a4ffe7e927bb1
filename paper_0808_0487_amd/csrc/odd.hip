// Passes of the transforms over Z_p, p = 3, 5, 7, with the tile geometry
// fixed at compile time (see fwt.hip for the split of a transform into
// passes).  A tile holds p^LE elements: p^RD rows (the RD digits of the pass)
// of W = p^(LE - RD) contiguous elements (the lowest digits).  Each of
// TH = p^(LE - KT) threads takes p^KT elements: element e = tid + k TH lies in
// row tid / W + k p^(RD - KT), so the values a thread loads differ exactly in
// the KT top digits of the pass (k = j0 + p j1 + ...), whose radix-p stages
// run in registers; the other digits go through LDS in groups of up to KT
// digits, with compile-time strides from a per-thread base.  The strides W p^q
// are odd multiples of the row length, so the tile needs no padding.  The
// stages run in ascending order of the digits (the top digits on the values
// read back for the store), so a transform's rounding does not depend on how
// it is split into passes; the p = 3 float tiles of 3^8 elements take the KT
// top digits first, on the values as loaded.  Tile sizes and KT follow from
// p, m, the type and the number of columns alone (pass_geom.h).
#include "pass_core.h"

#include <algorithm>
#include <type_traits>

namespace fdwt {

template <int P, int LE, int RD, int KT>
struct OddShape {
  static constexpr int E = PowC<P, LE>::v;
  static constexpr int EPT = PowC<P, KT>::v;  // elements per thread
  static constexpr int TH = E / EPT;
  static constexpr int W = PowC<P, LE - RD>::v;
  static constexpr int RSTEP = PowC<P, RD - KT>::v;  // rows between a thread's elements
  static_assert(RD >= KT && RD <= LE && TH % W == 0 && TH <= 1024, "unsupported odd-p shape");
};

// Radix-p stages over the digits 0..KG-1 of the index of x (p^KG values).
template <int P, int KG, bool INV, class T, int N>
__device__ __forceinline__ void dft_digits(T (&x)[N]) {
  static_assert(PowC<P, KG>::v == N, "p^KG values");
#pragma unroll
  for (int t = 0, st = 1; t < KG; ++t, st *= P) {
#pragma unroll
    for (int j0 = 0; j0 < N; ++j0)
      if ((j0 / st) % P == 0) Dft<P, INV>::run(x + j0, st);
  }
}

// Register groups over row digits [Q, Q + KG) for Q < RD - KT, then the next.
template <int P, int LE, int RD, int KT, int Q, bool INV, class T, bool DONE = (Q >= RD - KT)>
struct OddGroups {
  static __device__ __forceinline__ void run(T* lds, int tid) {
    using S = OddShape<P, LE, RD, KT>;
    constexpr int KG = (RD - KT - Q) >= KT ? KT : (RD - KT - Q);
    constexpr int R = PowC<P, KG>::v;
    constexpr int PQ = PowC<P, Q>::v;
    constexpr int STQ = S::W * PQ;          // element stride of digit Q
    constexpr int GPT = S::E / R / S::TH;   // groups per thread
    const int c = tid % S::W;
    const int u0 = tid / S::W;
#pragma unroll
    for (int g = 0; g < GPT; ++g) {
      // group tid + g TH: rows u = lo + PQ (j + R hi), lo < PQ
      const int u = u0 + g * S::RSTEP;
      const int lo = u % PQ, hi = u / PQ;
      T* base = lds + c + S::W * (lo + PQ * R * hi);
      T x[R];
#pragma unroll
      for (int j = 0; j < R; ++j) x[j] = base[j * STQ];
      dft_digits<P, KG, INV>(x);
#pragma unroll
      for (int j = 0; j < R; ++j) base[j * STQ] = x[j];
    }
    lds_barrier();
    OddGroups<P, LE, RD, KT, Q + KG, INV, T>::run(lds, tid);
  }
};
template <int P, int LE, int RD, int KT, int Q, bool INV, class T>
struct OddGroups<P, LE, RD, KT, Q, INV, T, true> {
  static __device__ __forceinline__ void run(T*, int) {}
};

// The KT top digits of a pass that come first, on the values as loaded.
template <int P, int LE, int RD, int KT, class T>
struct OddOrder {
  static constexpr bool top_first = RD == KT || (P == 3 && LE == 8 && std::is_same<T, float2>::value);
};

// A tile's values from the loaded ones: the stages of the pass.  `between`
// runs after the tile went to LDS (the wide tiles' prefetch).
template <int P, int LE, int RD, int KT, bool INV, class T, int N, class F>
__device__ __forceinline__ void odd_tile(T (&v)[N], T* lds, int tid, F between) {
  using S = OddShape<P, LE, RD, KT>;
  constexpr bool TOP_FIRST = OddOrder<P, LE, RD, KT, T>::top_first;
  if constexpr (TOP_FIRST) dft_digits<P, KT, INV>(v);
  if constexpr (RD > KT) {
#pragma unroll
    for (int k = 0; k < N; ++k) lds[tid + k * S::TH] = v[k];
    lds_barrier();
    between();
    OddGroups<P, LE, RD, KT, 0, INV, T>::run(lds, tid);
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = lds[tid + k * S::TH];
  }
  if constexpr (!TOP_FIRST) dft_digits<P, KT, INV>(v);
}

// Grouped sums of a tile (complex double: a pair of real columns carried as
// one complex column, the imaginary one scaled by 2^pexp): the terms of the
// thread's values, then the threads' sums in a fixed order.
template <int TH, int N>
__device__ __forceinline__ void odd_sums(const double2 (&v)[N], double2* red, const PassDesc& d, int col, int tile,
                                         int64_t base, uint32_t gstep, int tid) {
  const double us = ldexp(1.0, -d.pexp[col]);
  double2 acc = make_double2(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const float2 wt = d.wts[base + (int64_t)k * gstep];
    const double2 y = v[k];
    const double ra = fmin(fmax(y.x * (double)wt.y, 0.0), 1.0);
    const double rb = fmin(fmax(y.y * us * (double)wt.y, 0.0), 1.0);
    const double ta = (double)wt.x * ra, tb = (double)wt.x * rb;
    acc.x += ta;
    acc.y += tb;
    if (base + (int64_t)k * gstep == 0) {
      if (2 * col == d.h0_col) *d.h0_out = ta;
      if (2 * col + 1 == d.h0_col) *d.h0_out = tb;
    }
  }
  lds_barrier();
  red[tid] = acc;
  lds_barrier();
  if (tid < 64) {
    double2 t = red[tid];
    for (int i = tid + 64; i < TH; i += 64) t = add(t, red[i]);
    if constexpr (TH >= 64) {
      for (int off = 32; off > 0; off >>= 1) {
        t.x += __shfl_xor(t.x, off);
        t.y += __shfl_xor(t.y, off);
      }
    } else if (tid == 0) {
      for (int i = 1; i < TH; ++i) t = add(t, red[i]);
    }
    if (tid == 0) {
      d.partial[(int64_t)(2 * col) * d.ntiles + tile] = t.x;
      if (2 * col + 1 < d.ncols) d.partial[(int64_t)(2 * col + 1) * d.ntiles + tile] = t.y;
    }
  }
}

template <int W>
__device__ __forceinline__ int64_t odd_base(const PassDesc& d, int tile) {
  return (int64_t)(tile % d.nlo) * W + (int64_t)(tile / d.nlo) * d.shi;
}

// A tile that leaves room for a second one on its CU: a workgroup per tile,
// so that the hardware overlaps one tile's arithmetic with the others' loads
// and stores; bound by memory.  Forward + inverse against the persistent form
// below (us): p = 3 float 3^13 35.4 / 37.6, 3^14 59.9 / 63.6, 3^15 210 / 245,
// double 3^15 422 / 459; p = 5 double 5^10 302 / 326; p = 7 float 7^8
// 102.6 / 106.5, double 7^8 172 / 206.
template <int P, int LE, int RD, int KT, bool INV, class Tin, class T, class Tout, int EPI>
__global__ void __launch_bounds__((OddShape<P, LE, RD, KT>::TH))
    fwt_odd(const Tin* __restrict__ in, Tout* out, PassDesc d) {
  using S = OddShape<P, LE, RD, KT>;
  constexpr int EPT = S::EPT;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* lds = reinterpret_cast<T*>(smem_raw);
  const int lb = d.xcd ? xcd_first(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  // Sums: neighbours share a tile's weights.
  const int col = EPI == EPI_REDUCE ? lb % d.batch : lb / d.ntiles;
  const int tile = EPI == EPI_REDUCE ? lb / d.batch : lb % d.ntiles;
  const int tid = threadIdx.x;
  // Global offset of element tid + k TH: goff0 + k gstep.
  const uint32_t sd0 = (uint32_t)d.sd0;
  const uint32_t goff0 = (uint32_t)(tid % S::W) + (uint32_t)(tid / S::W) * sd0;
  const uint32_t gstep = (uint32_t)S::RSTEP * sd0;
  const int64_t base = odd_base<S::W>(d, tile);
  const Tin* src = in + (int64_t)col * d.col_in + base;
  Tin pre[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) pre[k] = src[goff0 + k * gstep];
  T v[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) v[k] = cvt_in<Tin, T>(pre[k]);
  odd_tile<P, LE, RD, KT, INV>(v, lds, tid, [] {});
  if constexpr (EPI == EPI_STORE) {
    Tout* dst = out + (int64_t)col * d.col_out + base;
#pragma unroll
    for (int k = 0; k < EPT; ++k) dst[goff0 + k * gstep] = cvt_out<T, Tout>(v[k], d.scale, d.scale64);
  } else {
    odd_sums<S::TH>(v, reinterpret_cast<double2*>(smem_raw), d, col, tile, base + goff0, gstep, tid);
  }
}

// A tile that takes its CU alone (3^8 elements in double, 5^6 in float):
// persistent workgroups, the next tile prefetched into registers while this
// one goes through LDS (a workgroup per tile: p = 5 float 5^10 152 against
// 140 us a pair, 5^11 945 against 846; p = 3 double 3^14 131 against 114).
template <int P, int LE, int RD, int KT, bool INV, class Tin, class T, class Tout, int EPI>
__global__ void __launch_bounds__((OddShape<P, LE, RD, KT>::TH))
    fwt_odd_wide(const Tin* __restrict__ in, Tout* out, PassDesc d) {
  using S = OddShape<P, LE, RD, KT>;
  constexpr int EPT = S::EPT;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* lds = reinterpret_cast<T*>(smem_raw);
  const int G = gridDim.x;
  const int nb = d.ntiles * d.batch;
  const int hw = blockIdx.x;
  int lb = d.xcd ? xcd_first(hw, G) : hw;
  const int tid = threadIdx.x;
  const uint32_t sd0 = (uint32_t)d.sd0;
  const uint32_t goff0 = (uint32_t)(tid % S::W) + (uint32_t)(tid / S::W) * sd0;
  const uint32_t gstep = (uint32_t)S::RSTEP * sd0;
  auto locate = [&](int l, int& col, int& tile) {
    col = EPI == EPI_REDUCE ? l % d.batch : l / d.ntiles;
    tile = EPI == EPI_REDUCE ? l / d.batch : l % d.ntiles;
  };
  Tin pre[EPT];
  // live false: every load reads the tile's first element (one cache line), a
  // stand-in that keeps the loads unconditional when there is no next tile.
  auto prefetch = [&](int l, bool live) {
    int col, tile;
    locate(l, col, tile);
    const Tin* src = in + (int64_t)col * d.col_in + odd_base<S::W>(d, tile) + (live ? goff0 : 0u);
    const uint32_t st = live ? gstep : 0u;
#pragma unroll
    for (int k = 0; k < EPT; ++k) pre[k] = src[k * st];
  };
  if (lb < nb) prefetch(lb, true);
  for (; lb < nb; lb += G) {
    T v[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) v[k] = cvt_in<Tin, T>(pre[k]);
    int col, tile;
    locate(lb, col, tile);
    const int64_t base = odd_base<S::W>(d, tile) + goff0;
    odd_tile<P, LE, RD, KT, INV>(v, lds, tid, [&] {
      prefetch(lb + G < nb ? lb + G : lb, lb + G < nb);  // unconditional: exact wait counts
    });
    if constexpr (EPI == EPI_STORE) {
      Tout* dst = out + (int64_t)col * d.col_out + base;
#pragma unroll
      for (int k = 0; k < EPT; ++k) dst[k * gstep] = cvt_out<T, Tout>(v[k], d.scale, d.scale64);
    } else {
      odd_sums<S::TH>(v, reinterpret_cast<double2*>(smem_raw), d, col, tile, base, gstep, tid);
    }
    lds_barrier();
  }
}

// ----------------------------------------------------------------- launch
template <int P, int LE, int RD, int KT, bool INV, class Tin, class T, class Tout, int EPI>
static int launch_odd(const void* in, void* out, const PassGeom& g, int m, int batch, double scale,
                      const ReduceArgs* red, hipStream_t st) {
  using S = OddShape<P, LE, RD, KT>;
  constexpr bool wide = RD > KT && 2 * S::E * sizeof(T) > 160 * 1024;  // one tile per CU
  const void* fn;
  if constexpr (wide) fn = (const void*)fwt_odd_wide<P, LE, RD, KT, INV, Tin, T, Tout, EPI>;
  else fn = (const void*)fwt_odd<P, LE, RD, KT, INV, Tin, T, Tout, EPI>;
  const int64_t N = ipow(P, m);
  PassDesc d{};
  d.col_in = N;
  d.col_out = N;
  d.sd0 = ipow(P, g.d0);
  d.shi = ipow(P, g.d0 + g.r);
  d.r = g.r;
  d.wdig = g.wdig;
  d.w = S::W;
  d.nlo = (int)(ipow(P, g.d0) / S::W);
  d.E = S::E;
  d.scale = (float)scale;
  d.scale64 = scale;
  const int64_t ntiles = N / S::E;
  const int64_t nb = ntiles * batch;
  d.ntiles = (int)ntiles;
  d.batch = batch;
  d.h0_col = -1;
  if (red) {
    d.wts = red->wts;
    d.partial = red->partial;
    d.h0_out = red->h0_out;
    d.h0_col = red->h0_col;
    d.ncols = red->ncols;
    for (int i = 0; i < batch; ++i) d.pexp[i] = (int16_t)red->pexp[i];
  }
  const size_t lds = std::max<size_t>(RD > KT ? (size_t)S::E * sizeof(T) : 0, EPI == EPI_REDUCE ? S::TH * sizeof(double2) : 0);
  if (int rc = allow_lds(fn, lds)) return rc;
  const int64_t G = wide ? std::min(nb, (int64_t)occupancy(fn, S::TH, lds) * device_cus()) : nb;
  d.xcd = G >= 64 ? 1 : 0;
  const Tin* inp = (const Tin*)in;
  Tout* outp = (Tout*)out;
  void* args[] = {(void*)&inp, (void*)&outp, (void*)&d};
  const double work = red ? (double)N * (batch * sizeof(Tin) + sizeof(float2))
                          : (double)N * batch * (sizeof(Tin) + sizeof(Tout));
  return launch_timed(fn, dim3((unsigned)G), dim3(S::TH), args, lds, st,
                      std::is_same<T, double2>::value ? FDWT_TC_PASS_F64 : FDWT_TC_PASS_CF32, work);
}

// Kinds of one shape.  Real input and, for the inverse, real output occur in
// contiguous first passes and last passes; the grouped sums in last passes of
// forward double transforms.
template <int P, int LE, int RD, int KT, class R, class C>
static int odd_kinds(bool inv, bool in_real, bool out_real, const void* in, void* out, const PassGeom& g, int m,
                     int batch, double scale, const ReduceArgs* red, hipStream_t st) {
  if (red) {
    if constexpr (std::is_same<C, double2>::value)
      return launch_odd<P, LE, RD, KT, false, C, C, C, EPI_REDUCE>(in, out, g, m, batch, scale, red, st);
    else return fail(FDWT_EINVAL, "grouped sums are computed in double");
  }
  if (!inv) {
    if (out_real) return fail(FDWT_EINVAL, "unsupported transform element types");
    if constexpr (RD == LE) {
      if (in_real) return launch_odd<P, LE, RD, KT, false, R, C, C, EPI_STORE>(in, out, g, m, batch, scale, red, st);
    }
    if (!in_real) return launch_odd<P, LE, RD, KT, false, C, C, C, EPI_STORE>(in, out, g, m, batch, scale, red, st);
  } else if (!in_real) {
    if (out_real) return launch_odd<P, LE, RD, KT, true, C, C, R, EPI_STORE>(in, out, g, m, batch, scale, red, st);
    return launch_odd<P, LE, RD, KT, true, C, C, C, EPI_STORE>(in, out, g, m, batch, scale, red, st);
  }
  return fail(FDWT_EINVAL, "unsupported transform element types");
}

template <int P, class R, class C>
static int odd_shape(bool inv, bool in_real, bool out_real, const void* in, void* out, const PassGeom& g, int m,
                     int batch, double scale, const ReduceArgs* red, hipStream_t st) {
  constexpr bool D = std::is_same<C, double2>::value;
  if (g.le < 1 || g.r > g.le || g.wdig != g.le - g.r || g.d0 < g.wdig || (g.d0 == 0) != (g.r == g.le))
    return fail(FDWT_EINVAL, "not an odd-p pass shape");
  const bool kt3 = odd_kt3(P, D, g.le, ipow(P, m - g.le) * batch);
#define FDWT_ODD(LE, RD)                                                                                       \
  if constexpr (odd_has_shape(P, D, LE, RD)) {                                                                 \
    if (g.le == LE && g.r == RD) {                                                                             \
      if constexpr (P == 3 && !D && odd_kt3_shape(LE, RD)) {                                                   \
        if (kt3) return odd_kinds<P, LE, RD, 3, R, C>(inv, in_real, out_real, in, out, g, m, batch, scale, red, st); \
      }                                                                                                        \
      return odd_kinds<P, LE, RD, odd_kt(P, LE, RD, D), R, C>(inv, in_real, out_real, in, out, g, m, batch, scale, red, st); \
    }                                                                                                          \
  }
#define FDWT_ODD_LE(LE) \
  FDWT_ODD(LE, 1) FDWT_ODD(LE, 2) FDWT_ODD(LE, 3) FDWT_ODD(LE, 4) FDWT_ODD(LE, 5) FDWT_ODD(LE, 6) FDWT_ODD(LE, 7) FDWT_ODD(LE, 8)
  FDWT_ODD_LE(1) FDWT_ODD_LE(2) FDWT_ODD_LE(3) FDWT_ODD_LE(4) FDWT_ODD_LE(5) FDWT_ODD_LE(6) FDWT_ODD_LE(7) FDWT_ODD_LE(8)
#undef FDWT_ODD_LE
#undef FDWT_ODD
  return fail(FDWT_EINVAL, "not an odd-p pass shape");
}

// One pass of a p = 3, 5, 7 transform in working type `work` (K_CF32, K_CF64).
int odd_pass(int p, bool inv, Kind ik, Kind work, Kind ok, const void* in, void* out, const PassGeom& g, int m,
             int batch, double scale, const ReduceArgs* red, hipStream_t st) {
  if (work == K_CF32) {
    const bool ir = ik == K_F32, orl = ok == K_F32;
    if ((!ir && ik != K_CF32) || (!orl && ok != K_CF32)) return fail(FDWT_EINVAL, "unsupported transform element types");
    if (p == 3) return odd_shape<3, float, float2>(inv, ir, orl, in, out, g, m, batch, scale, red, st);
    if (p == 5) return odd_shape<5, float, float2>(inv, ir, orl, in, out, g, m, batch, scale, red, st);
    if (p == 7) return odd_shape<7, float, float2>(inv, ir, orl, in, out, g, m, batch, scale, red, st);
  } else if (work == K_CF64) {
    const bool ir = ik == K_F64, orl = ok == K_F64;
    if ((!ir && ik != K_CF64) || (!orl && ok != K_CF64)) return fail(FDWT_EINVAL, "unsupported transform element types");
    if (p == 3) return odd_shape<3, double, double2>(inv, ir, orl, in, out, g, m, batch, scale, red, st);
    if (p == 5) return odd_shape<5, double, double2>(inv, ir, orl, in, out, g, m, batch, scale, red, st);
    if (p == 7) return odd_shape<7, double, double2>(inv, ir, orl, in, out, g, m, batch, scale, red, st);
  }
  return fail(FDWT_EUNSUPPORTED, "p must be 3, 5 or 7");
}

}  // namespace fdwt

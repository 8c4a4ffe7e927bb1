// Radix-p butterfly passes of the fast discrete Walsh transform and its
// inverse (Algorithm 1 of Section 2.2, Algorithm 2 of Section 3.3).
//
// Stage r of Algorithm 1 replaces index digit n_{r-1} by h_{r-1} through a
// p-point DFT with weights omega^(-n h); stages act on different digits and
// commute, so the m stages are grouped into passes over HBM.  A pass
// transforms r consecutive digits [d0, d0+r) of every column: a workgroup
// loads a tile of p^r rows (the r digits) by w contiguous elements (the lowest
// digits, so that HBM reads and writes come in full segments), stages it in
// LDS, runs the r stages in groups of k digits held in registers (p^k values
// per thread, one LDS round trip per group), and writes the tile back in
// place.  This file has the passes of p = 2 and the plans of every p, odd.hip
// the passes of p = 3, 5, 7.  The output is in natural order
// (h = sum h_i p^i), as in Algorithm 1.
#include "coords.h"
#include "family.h"
#include "p2_stages.h"
#include "pass_core.h"

#include <algorithm>
#include <cmath>
#include <map>
#include <type_traits>
#include <mutex>

namespace fdwt {

size_t kind_bytes(Kind k) {
  switch (k) {
    case K_F32: return 4;
    case K_U32: return 4;
    case K_CF32: return 8;
    case K_F64: return 8;
    case K_CF64: return 16;
  }
  return 0;
}

// ------------------------------------------------- p = 2, up to 2^6 points
// A wave per column, a point per lane, the stages between the lanes (too few
// points for the tiles below).  The grouped sums (double) as in fwt_p2_sums.
template <class T, int EPI>
__global__ void __launch_bounds__(64) fwt_p2_small(const T* in, T* out, PassDesc d) {
  const int e = threadIdx.x, col = blockIdx.x;
  const bool on = e < d.E;
  T v = on ? in[(int64_t)col * d.col_in + e] : T(0);
  for (int b = 0; b < d.r; ++b) {
    const T o = __shfl_xor(v, 1 << b);
    v = (e >> b) & 1 ? sub(o, v) : add(v, o);
  }
  if constexpr (EPI == EPI_STORE) {
    if (on) out[(int64_t)col * d.col_out + e] = cvt_out<T, T>(v, d.scale, d.scale64);
  } else {
    double acc = 0.0;
    if (on) {
      const float2 wt = d.wts[e];
      const double rho = fmin(fmax(v * (double)wt.y, 0.0), 1.0);
      acc = (double)wt.x * rho;
      if (e == 0 && col == d.h0_col) *d.h0_out = acc;
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (e == 0) d.partial[col] = acc;
  }
}

// -------------------------------------------- p = 2 passes, static shape
// (tile geometry, register groups and stages: p2_stages.h)

// One pass that stores its coefficients: a workgroup per tile, so that the
// hardware overlaps one tile's arithmetic with its neighbours' loads and
// stores.  The pass is bound by memory (or the last-level cache), and at one
// tile a workgroup the kernel needs 36 registers (float), so LDS alone limits
// it: two 2^14-element float tiles per CU.  A persistent form that prefetched
// the next tile into registers had one (its 100 scalar registers allow 7 waves
// a SIMD), loads and stores of the whole device in step.  Forward + inverse, a
// workgroup per tile against that form (us): float m = 20 20.0 / 22.6, m = 21
// 28.7 / 36.6, m = 22 33.6 / 36.9, m = 24 95.4 / 106.2, m = 25 256 / 296, m =
// 26 550 / 583; double m = 20 29.6 / 33.1, m = 23 103 / 115, m = 24 221 / 232;
// with the stages between lanes (p2_stages.h) float m = 24 then 93.2.
template <class T, int LOGE, int WDIG>
__global__ void __launch_bounds__((P2Shape<LOGE, WDIG>::THREADS), (sizeof(T) == 4 ? 8 : 4))
    fwt_p2(const T* __restrict__ in, T* out, PassDesc d) {
  using S = P2Shape<LOGE, WDIG>;
  constexpr int EPT = S::EPT, TH = S::THREADS;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* lds = reinterpret_cast<T*>(smem_raw);
  const int lb = d.xcd ? xcd_first(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int col = lb / d.ntiles, tile = lb % d.ntiles;
  const int64_t base = (int64_t)(tile % d.nlo) * S::W + (int64_t)(tile / d.nlo) * d.shi;
  const int tid = threadIdx.x;
  // Element e = tid + k*TH of the tile: row i = e >> WDIG, column e & (W-1);
  // global offset goff0 + k*gstep, LDS index pad(tid) + pad(k*TH).
  const uint32_t sd0 = (uint32_t)d.sd0;
  const uint32_t goff0 = (uint32_t)(tid & (S::W - 1)) + (uint32_t)(tid >> WDIG) * sd0;
  const uint32_t gstep = (uint32_t)(TH >> WDIG) * sd0;
  const gptr<const T> src =
      to_global((d.in_tab ? col_ptr<const T>(d.in_tab, col) : in + (int64_t)col * d.col_in) + base);
  T v[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) v[k] = src[goff0 + k * gstep];
  T* lrow = lds + cpad(tid);
  if constexpr (LOGE >= 10) {
    // Three stage groups.  The 16 elements a thread loads (e = tid + k TH)
    // differ in the top 4 bits of e: those stages run in registers before the
    // tile goes to LDS.  The stages of bits [WDIG, 6): of a strided tile,
    // between the lanes (as its rows take the lower lane bits); of a
    // contiguous tile, p2_low6.  The store mapping e = lane + 64 k + 1024 w
    // (still coalesced) puts bits 6..9 in the register index: the remaining
    // stages run in registers after reading the tile back.
    constexpr int NS = (LOGE - 10) < 4 ? (LOGE - 10) : 4;
    // The wave index is uniform in a wave: read as a scalar, the addresses
    // derived from it stay in scalar registers.
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t goffS = (uint32_t)(lane & (S::W - 1)) + (uint32_t)((lane >> WDIG) + (1024 >> WDIG) * wv) * sd0;
    const uint32_t gstepS = (uint32_t)(64 >> WDIG) * sd0;
    const T* lrowS = lds + cpad(lane + 1024 * wv);
    reg_bfly<4>(v);
    // Strided tiles: their digits below 6 are lane bits 4 and 5 (rows of 32: 5).
    if constexpr (WDIG == 4) lane_bfly<16>(v);
    if constexpr (WDIG > 0) lane_bfly<32>(v);
#pragma unroll
    for (int k = 0; k < EPT; ++k) lrow[cpad(k * TH)] = v[k];
    lds_barrier();
    if constexpr (WDIG == 0) p2_low6<LOGE>(lds, tid);
#pragma unroll
    for (int k = 0; k < EPT; ++k) v[k] = lrowS[66 * k];
    reg_bfly<NS>(v);
    if (WDIG == 0 && d.oblk) {
      // Blocked layout: e = lane + 64 k + 1024 w has row e >> 4 and column e & 15.
      const int64_t rs = d.oblk;
      const gptr<T> dst = to_global(out + (int64_t)col * d.col_out + ((lane >> 4) + 64 * wv) * rs +
                                    (int64_t)tile * 16 + (lane & 15));
#pragma unroll
      for (int k = 0; k < EPT; ++k) dst[k * 4 * rs] = cvt_out<T, T>(v[k], d.scale, d.scale64);
    } else {
      const gptr<T> dst = to_global((d.out_tab ? col_ptr<T>(d.out_tab, col) : out + (int64_t)col * d.col_out) + base);
#pragma unroll
      for (int k = 0; k < EPT; ++k) dst[goffS + k * gstepS] = cvt_out<T, T>(v[k], d.scale, d.scale64);
    }
  } else {
#pragma unroll
    for (int k = 0; k < EPT; ++k) lrow[cpad(k * TH)] = v[k];
    lds_barrier();
    P2Groups<LOGE, WDIG, 0, T>::run(lds, tid);
    const gptr<T> dst = to_global((d.out_tab ? col_ptr<T>(d.out_tab, col) : out + (int64_t)col * d.col_out) + base);
#pragma unroll
    for (int k = 0; k < EPT; ++k) dst[goff0 + k * gstep] = cvt_out<T, T>(lrow[cpad(k * TH)], d.scale, d.scale64);
  }
}

// Last pass of the variance columns (double): the grouped sums instead of a
// store.  Persistent, with the next tile prefetched: with wkeep a workgroup
// takes every column of one tile and keeps the tile's weights in registers.
template <int LOGE, int WDIG>
__global__ void __launch_bounds__((P2Shape<LOGE, WDIG>::THREADS))
    fwt_p2_sums(const double* __restrict__ in, PassDesc d) {
  using S = P2Shape<LOGE, WDIG>;
  constexpr int EPT = S::EPT, TH = S::THREADS;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* lds = reinterpret_cast<double*>(smem_raw);
  const int G = gridDim.x;
  const int nb = d.ntiles * d.batch;
  const int hw = blockIdx.x;
  int lb = d.xcd ? xcd_first(hw, G) : hw;
  const int tid = threadIdx.x;
  const uint32_t sd0 = (uint32_t)d.sd0;
  const uint32_t goff0 = (uint32_t)(tid & (S::W - 1)) + (uint32_t)(tid >> WDIG) * sd0;
  const uint32_t gstep = (uint32_t)(TH >> WDIG) * sd0;
  double* lrow = lds + cpad(tid);
  auto locate = [&](int l, int& col, int& tile) {
    if (d.wkeep) {
      const int r = l / G;
      col = r % d.batch;
      tile = (r / d.batch) * G + l % G;
    } else {
      col = l % d.batch;
      tile = l / d.batch;
    }
  };
  auto tile_base = [&](int tile) {
    const int lo = tile % d.nlo;
    const int hi = tile / d.nlo;
    return (int64_t)lo * S::W + (int64_t)hi * d.shi;
  };
  double pre[EPT];
  // Moves the prefetched elements into the tile registers.  The empty asm is
  // a use of each register, so the wait for the prefetch sits here: a pass
  // takes the next tile before it stores the current one's partial sum.
  auto take = [&](double (&v)[EPT]) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      v[k] = pre[k];
      asm volatile("" : "+v"(v[k]));
    }
  };
  auto prefetch = [&](int l) {
    int col, tile;
    locate(l, col, tile);
    // The scalar pointer runs along, its step opaque per tile: otherwise the
    // 16 multiples stay in scalar registers across the loop (105 spilled).
    const double* src = in + (int64_t)col * d.col_in + tile_base(tile);
    uint32_t gs = gstep;
    asm volatile("" : "+s"(gs));
#pragma unroll
    for (int k = 0; k < EPT; ++k, src += gs) pre[k] = to_global(src)[goff0];
  };
  if (lb < nb) prefetch(lb);
  if constexpr (LOGE >= 10) {
    // The stage groups and the store mapping of fwt_p2.
    constexpr int NS = (LOGE - 10) < 4 ? (LOGE - 10) : 4;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t goffS = (uint32_t)(lane & (S::W - 1)) + (uint32_t)((lane >> WDIG) + (1024 >> WDIG) * wv) * sd0;
    const uint32_t gstepS = (uint32_t)(64 >> WDIG) * sd0;
    double* lrowS = lds + cpad(lane + 1024 * wv);
    double v[EPT];
    if (lb < nb) take(v);
    float2 wcur[EPT];  // the weights of the tile
    for (; lb < nb; lb += G) {
      reg_bfly<4>(v);
      if constexpr (WDIG == 4) {
        lane_bfly<16>(v);
        lane_bfly<32>(v);
      }
#pragma unroll
      for (int k = 0; k < EPT; ++k) lrow[cpad(k * TH)] = v[k];
      lds_barrier();
      int col, tile;
      locate(lb, col, tile);
      const int64_t base = tile_base(tile);
      if (!d.wkeep || col == 0) {  // with wkeep, column 0 starts a new tile
        const float2* wt = d.wts + base;
        uint32_t gs = gstepS;
        asm volatile("" : "+s"(gs));
#pragma unroll
        for (int k = 0; k < EPT; ++k, wt += gs) wcur[k] = wt[goffS];
      }
      prefetch(lb + G < nb ? lb + G : lb);  // unconditional: exact wait counts
      // 2-digit register groups: with the weights and the next tile live they
      // keep the kernel within 128 registers.
      if constexpr (WDIG == 0) P2Groups<LOGE, 0, 0, double, 2, 6>::run(lds, tid);
      double y[EPT];
#pragma unroll
      for (int k = 0; k < EPT; ++k) y[k] = lrowS[66 * k];
      reg_bfly<NS>(y);
      double acc = 0.0;
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const double rho = fmin(fmax(y[k] * (double)wcur[k].y, 0.0), 1.0);
        const double term = (double)wcur[k].x * rho;
        acc += term;
        if (col == d.h0_col && base + goffS + (int64_t)k * gstepS == 0) *d.h0_out = term;
      }
      for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
      take(v);
      if (lane == 0) d.partial[((int64_t)col * d.ntiles + tile) * (TH / 64) + wv] = acc;
      lds_barrier();
    }
    return;
  }
  double v[EPT];
  if (lb < nb) take(v);
  for (; lb < nb; lb += G) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) lrow[cpad(k * TH)] = v[k];
    lds_barrier();
    int col, tile;
    locate(lb, col, tile);
    const int64_t base = tile_base(tile);
    // The tile's weights: loaded now, used after the butterflies.
    float2 wcur[EPT];
    const float2* wt = d.wts + base + goff0;
#pragma unroll
    for (int k = 0; k < EPT; ++k) wcur[k] = wt[k * gstep];
    // Unconditional (the last round re-reads its own block): with no branch
    // around the loads the compiler's wait counts stay exact, so waiting for
    // this tile's weights does not wait for the next tile's elements.
    prefetch(lb + G < nb ? lb + G : lb);
    P2Groups<LOGE, WDIG, 0, double, 2>::run(lds, tid);
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const float2 w2 = wcur[k];
      const double rho = fmin(fmax(lrow[cpad(k * TH)] * (double)w2.y, 0.0), 1.0);
      const double term = (double)w2.x * rho;
      acc += term;
      if (col == d.h0_col && base + goff0 + (int64_t)k * gstep == 0) *d.h0_out = term;
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    take(v);
    if ((tid & 63) == 0) d.partial[((int64_t)col * d.ntiles + tile) * (TH / 64) + (tid >> 6)] = acc;
    lds_barrier();
  }
}

// First (contiguous) pass of float64 transforms whose input columns are
// generated in registers instead of read from memory (p = 2, Section 4):
//  * truncation columns (KCOL false): U_d = prod_{j<=d} (1 + a_j) - 1,
//    d = 1..s, with a_j = gamma_j^2 R'(x_{n,j}) = tab[j][t];
//  * kernel column (KCOL true): K(x_n, 0) = prod_j rl[j][t] with
//    rl[j][t] = 1 + gamma_j K'(x_{n,j}, 0).
// t is the index of the first non-zero digit of x_{n,j} (the leading-zero
// count of X_j(n) in m bits; t = m for X = 0).  Each workgroup takes whole
// tiles and runs j = 1..s in order; a thread keeps the running value for its
// 16 points (n = tile E + tid + k TH) in registers (for U: U_j = U_{j-1} +
// a_j (1 + U_{j-1}), one column stored per j).  X_j(n) is the XOR of the
// generator columns of the set bits of n (Definition of a digital net,
// p = 2); the columns and the tables are staged in LDS, so the loop's only
// memory accesses are its stores.  With few tiles the columns of a tile are
// divided among nch workgroups, each of which runs the products from d = 1
// but transforms and stores its own columns only.
struct ColGen {
  const uint32_t* xtab;  // [s][nbytes][256]: X_j of byte value v at byte b
  int nbytes, s, m;
  int d0, d1;            // truncation columns U_{d0+1}..U_{d1} are stored (out column d - 1 - d0)
  int nch, per;          // ... by nch workgroups a tile, `per` columns each
};

template <int LOGE, bool KCOL>
__global__ void __launch_bounds__((P2Shape<LOGE, 0>::THREADS)) fwt_p2_gen(ColGen g, double* out, PassDesc d, KernTab kt) {
  using S = P2Shape<LOGE, 0>;
  constexpr int EPT = S::EPT, TH = S::THREADS, TB = LOGE - 4;  // tid has TB bits
  static_assert(LOGE >= 10 && EPT == 16, "16 elements per thread");
  constexpr int NS = (LOGE - 10) < 4 ? (LOGE - 10) : 4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* lds = reinterpret_cast<double*>(smem_raw);
  const int m = g.m, s = g.s;
  double* rl = lds + ((cpad(S::E) + 1) & ~1);                    // [s][m + 1]
  uint32_t* cl = reinterpret_cast<uint32_t*>(rl + s * (m + 1));   // [s][m]: generator columns
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  stage_kern_tables(kt, s, m + 1, KCOL ? rl : nullptr, KCOL ? nullptr : rl);
  for (int i = tid; i < s * m; i += TH) {
    const int j = i / m, c = i % m;
    cl[i] = g.xtab[((size_t)j * g.nbytes + (c >> 3)) * 256 + (1 << (c & 7))];
  }
  __syncthreads();
  const int G = gridDim.x, hw = blockIdx.x;
  int lb = d.xcd ? xcd_first(hw, G) : hw;
  double* lrow = lds + cpad(tid);
  double* lrowS = lds + cpad(lane + 1024 * wv);
  const uint32_t goffS = (uint32_t)(lane + 1024 * wv);
  const int sh = 32 - m;
  int tile = 0;
  // Pass over one generated column of the tile: the same stage groups as
  // fwt_p2's first pass, then a coalesced store.
  auto transform_store = [&](const double (&u)[EPT], int col) {
    double v[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) v[k] = u[k];
    reg_bfly<4>(v);
#pragma unroll
    for (int k = 0; k < EPT; ++k) lrow[cpad(k * TH)] = v[k];
    lds_barrier();
    p2_low6<LOGE>(lds, tid);
#pragma unroll
    for (int k = 0; k < EPT; ++k) v[k] = lrowS[66 * k];
    reg_bfly<NS>(v);
    if (d.oblk) {  // blocked layout (PassDesc::oblk)
      const int64_t rs = d.oblk;
      const gptr<double> dst =
          to_global(out + (int64_t)col * d.col_out + ((lane >> 4) + 64 * wv) * rs + (int64_t)tile * 16 + (lane & 15));
#pragma unroll
      for (int k = 0; k < EPT; ++k) dst[k * 4 * rs] = v[k];
    } else {
      const gptr<double> dst = to_global(out + (int64_t)col * d.col_out + ((int64_t)tile << LOGE) + goffS);
#pragma unroll
      for (int k = 0; k < EPT; ++k) dst[k * 64] = v[k];
    }
    lds_barrier();
  };
  for (; lb < d.ntiles * g.nch; lb += G) {
    tile = lb / g.nch;
    const int jfirst = g.d0 + (lb - tile * g.nch) * g.per;
    const uint32_t n0 = (uint32_t)tile << LOGE;
    double u[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) u[k] = KCOL ? 1.0 : 0.0;
    const int jend = KCOL ? s : min(g.d1, jfirst + g.per);
    for (int j = 0; j < jend; ++j) {
      const uint32_t* cj = cl + j * m;
      uint32_t xt = 0;  // X_j(tid) ^ X_j(n0)
#pragma unroll
      for (int c = 0; c < TB; ++c) xt ^= cj[c] & (0u - (((uint32_t)tid >> c) & 1u));
      for (int c = LOGE; c < m; ++c)
        if ((n0 >> c) & 1) xt ^= cj[c];
      uint32_t kx[EPT];  // X_j(k TH): the XOR of the columns of k's bits
      kx[0] = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint32_t cb = cj[TB + b];
#pragma unroll
        for (int k = 0; k < (1 << b); ++k) kx[k + (1 << b)] = kx[k] ^ cb;
      }
      const double* rj = rl + j * (m + 1);
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const double a = rj[(int)__clz(xt ^ kx[k]) - sh];
        u[k] = KCOL ? u[k] * a : fma(a, 1.0 + u[k], u[k]);
      }
      if constexpr (!KCOL) {
        if (j >= jfirst) transform_store(u, j - g.d0);
      }
    }
    if constexpr (KCOL) transform_store(u, 0);
  }
}


// One evaluation of the split cost (Section 5.1, run_split_cost) for a first
// half of 2^LOGE points, by one workgroup: K and G generated as fwt_p2_gen
// generates K, transformed in the tile (the stages of a single fwt_p2 tile),
// combined to f~ G / K_u, transformed back, compared with the second half.
// z = (X_j(n) << 1) ^ delta_j has m + 1 digits (delta 0: the first half).
// A search makes 100 to 200 of these calls one after another, so what counts
// is their latency: one launch (about 20 us for 2^13 points) instead of nine
// of 2 to 8 us and the gaps between them.
struct SplitTile {
  const uint32_t* xtab;
  int nbytes, s, m;
  const float *ft, *fval;
  double* ku;        // K_u in passing, N
  float* sf;         // nullable
  double* cost;      // pinned host memory
};

template <int LOGE>
__global__ void __launch_bounds__((P2Shape<LOGE, 0>::THREADS)) fwt_p2_split(SplitTile g, KernTab kt) {
  using S = P2Shape<LOGE, 0>;
  constexpr int EPT = S::EPT, TH = S::THREADS, TB = LOGE - 4;
  static_assert(LOGE >= 10 && EPT == 16, "16 elements per thread");
  constexpr int NS = (LOGE - 10) < 4 ? (LOGE - 10) : 4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* lds = reinterpret_cast<double*>(smem_raw);
  const int s = g.s, m2 = LOGE + 1;
  double* rl = lds + ((cpad(S::E) + 1) & ~1);                     // [s][m2 + 1]
  uint32_t* cl = reinterpret_cast<uint32_t*>(rl + s * (m2 + 1));  // [s][LOGE]: generator columns
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  stage_kern_tables(kt, s, m2 + 1, rl, nullptr);
  for (int i = tid; i < s * LOGE; i += TH) {
    const int j = i / LOGE, c = i % LOGE;
    cl[i] = g.xtab[((size_t)j * g.nbytes + (c >> 3)) * 256 + (1 << (c & 7))];
  }
  double* lrow = lds + cpad(tid);
  double* lrowS = lds + cpad(lane + 1024 * wv);
  const int e0 = lane + 1024 * wv;  // stored element k: e0 + 64 k
  __syncthreads();
  auto generate = [&](bool shifted, double (&u)[EPT]) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) u[k] = 1.0;
    for (int j = 0; j < s; ++j) {
      const uint32_t* cj = cl + j * LOGE;
      uint32_t xt = 0;
#pragma unroll
      for (int c = 0; c < TB; ++c) xt ^= cj[c] & (0u - (((uint32_t)tid >> c) & 1u));
      xt = (xt << 1) ^ (shifted ? (uint32_t)kt.ix[j] : 0u);
      uint32_t kx[EPT];
      kx[0] = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint32_t cb = cj[TB + b] << 1;
#pragma unroll
        for (int k = 0; k < (1 << b); ++k) kx[k + (1 << b)] = kx[k] ^ cb;
      }
      const double* rj = rl + j * (m2 + 1);
#pragma unroll
      for (int k = 0; k < EPT; ++k) u[k] *= rj[(int)__clz(xt ^ kx[k]) - (32 - m2)];
    }
  };
  // In: element tid + k TH in v[k]; out: element e0 + 64 k.
  auto transform = [&](double (&v)[EPT]) {
    reg_bfly<4>(v);
#pragma unroll
    for (int k = 0; k < EPT; ++k) lrow[cpad(k * TH)] = v[k];
    lds_barrier();
    p2_low6<LOGE>(lds, tid);
#pragma unroll
    for (int k = 0; k < EPT; ++k) v[k] = lrowS[66 * k];
    reg_bfly<NS>(v);
    lds_barrier();
  };
  double v[EPT];
  generate(false, v);
  transform(v);
#pragma unroll
  for (int k = 0; k < EPT; ++k) g.ku[e0 + 64 * k] = v[k];  // read back by this thread
  generate(true, v);
  transform(v);
#pragma unroll
  for (int k = 0; k < EPT; ++k)
    lrowS[66 * k] = (double)g.ft[e0 + 64 * k] * v[k] / fmax(g.ku[e0 + 64 * k], 1e-300);
  lds_barrier();
#pragma unroll
  for (int k = 0; k < EPT; ++k) v[k] = lrow[cpad(k * TH)];
  lds_barrier();
  transform(v);
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const double d = (double)g.fval[e0 + 64 * k] - v[k];
    acc += d * d;
    if (g.sf) g.sf[e0 + 64 * k] = (float)v[k];
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) lds[wv] = acc;
  lds_barrier();
  if (tid == 0) {
    for (int w = 1; w < TH / 64; ++w) acc += lds[w];
    *g.cost = acc;
  }
}


// First pass of the forward transform of a test function sampled at the
// net (p = 2, fdwt_dwt_forward_family): the 16 values each thread would load
// are generated instead, f(x_n) at n = tile E + tid + k TH, with the sampling
// kernel's arithmetic (family.h, the same operations in the same order), then
// transformed and stored exactly as fwt_p2's first pass does, so the result
// equals sampling then transforming bit for bit while the samples never
// cross HBM.  X_j(n) is linear over Z_2 in the bits of n, which split into
// the tid part (a vector lookup in the net's byte tables), the 16 k parts
// (built by doubling from four generator columns) and the tile part; the
// last two are the same for the whole workgroup and come from scalar loads.
struct FamGen {
  const uint32_t* xtab;  // [s][nbytes][256]: X_j of byte value v at byte b
  int nbytes, m;
  FamilyArgs fa;
};

template <int LOGE, int FAM>
__global__ void __launch_bounds__((P2Shape<LOGE, 0>::THREADS)) fwt_p2_fam(FamGen g, float* out, PassDesc d) {
  using S = P2Shape<LOGE, 0>;
  constexpr int EPT = S::EPT, TH = S::THREADS, TB = LOGE - 4;  // tid has TB bits
  static_assert(LOGE >= 10 && EPT == 16, "16 elements per thread");
  constexpr int NS = (LOGE - 10) < 4 ? (LOGE - 10) : 4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float* lds = reinterpret_cast<float*>(smem_raw);
  using ctab = const uint32_t __attribute__((address_space(4)))*;
  const ctab tc = (ctab)g.xtab;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = g.fa.s, nby = g.nbytes;
  const float inv = 1.0f / (float)(1u << g.m);  // exact power of two, as the sampling kernel's
  float* lrow = lds + cpad(tid);
  float* lrowS = lds + cpad(lane + 1024 * wv);
  const uint32_t goffS = (uint32_t)(lane + 1024 * wv);
  const int G = gridDim.x, hw = blockIdx.x;
  int lb = d.xcd ? xcd_first(hw, G) : hw;
  for (; lb < d.ntiles; lb += G) {
    const uint32_t n0 = (uint32_t)lb << LOGE;
    typename FamState<FAM>::T acc[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) acc[k] = fam_init<FAM>(g.fa);
    for (int j = 0; j < s; ++j) {
      const uint32_t* tj = g.xtab + (size_t)j * nby * 256;
      uint32_t xt = tj[tid & 255];
      if constexpr (TB > 8) xt ^= tj[256 + (tid >> 8)];
      uint32_t tp = 0;  // X_j(n0)
      for (int b = 1; b < nby; ++b) tp ^= tc[(j * nby + b) * 256 + ((n0 >> (8 * b)) & 255)];
      xt ^= tp;
      uint32_t kx[EPT];  // X_j(k TH)
      kx[0] = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int bit = TB + b;
        const uint32_t cb = tc[(j * nby + (bit >> 3)) * 256 + (1 << (bit & 7))];
#pragma unroll
        for (int k = 0; k < (1 << b); ++k) kx[k + (1 << b)] = kx[k] ^ cb;
      }
      const float a = g.fa.a[j], ia = g.fa.inv1a[j];
#pragma unroll
      for (int k = 0; k < EPT; ++k) fam_step<FAM, false>(acc[k], g.fa, a, ia, xt ^ kx[k], inv, (double)inv);
    }
    float v[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) v[k] = fam_final<FAM>(acc[k], g.fa);
    reg_bfly<4>(v);
#pragma unroll
    for (int k = 0; k < EPT; ++k) lrow[cpad(k * TH)] = v[k];
    lds_barrier();
    p2_low6<LOGE>(lds, tid);
    float y[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) y[k] = lrowS[66 * k];
    reg_bfly<NS>(y);
    const gptr<float> dst = to_global(out + ((int64_t)lb << LOGE) + goffS);
#pragma unroll
    for (int k = 0; k < EPT; ++k) dst[k * 64] = cvt_out<float, float>(y[k], d.scale, d.scale64);
    lds_barrier();
  }
}


// ----------------------------------------------------------------- planner
// LDS of a float64 tile: a whole CU, so that m = 24 still needs only two
// passes (measured faster than three passes with two workgroups per CU);
// FDWT_LDS_KB_WIDE overrides that budget (KiB).
static size_t wide_lds_budget() {
  static const size_t wide = [] {
    const char* e = getenv("FDWT_LDS_KB_WIDE");
    const long v = e ? atol(e) : 160;
    return (size_t)std::max(16L, std::min(160L, v)) * 1024;
  }();
  return wide;
}

// Compute units of the current device (cached per device).
int device_cus() {
  static std::mutex mu;
  static std::vector<int> cache;
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::lock_guard<std::mutex> g(mu);
  if ((int)cache.size() <= dev) cache.resize(dev + 1, 0);
  if (!cache[dev]) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cache[dev] = n;
  }
  return cache[dev];
}

template <class T>
static int launch_small(const void* in, void* out, int m, int batch, double scale, const ReduceArgs* red,
                        hipStream_t st) {
  PassDesc d{};
  const int E = 1 << m;
  d.col_in = E;
  d.col_out = E;
  d.r = m;
  d.E = E;
  d.ntiles = 1;
  d.batch = batch;
  d.scale = (float)scale;
  d.scale64 = scale;
  d.h0_col = -1;
  const void* fn = (const void*)fwt_p2_small<T, EPI_STORE>;
  if (red) {
    if constexpr (std::is_same<T, double>::value) fn = (const void*)fwt_p2_small<T, EPI_REDUCE>;
    else return fail(FDWT_EINVAL, "grouped sums are computed in double");
    d.wts = red->wts;
    d.partial = red->partial;
    d.h0_out = red->h0_out;
    d.h0_col = red->h0_col;
    d.ncols = red->ncols;
  }
  void* args[] = {(void*)&in, (void*)&out, (void*)&d};
  const double elems = (double)E * batch;
  const double work = red ? elems * sizeof(T) + (double)E * sizeof(float2) : elems * 2 * sizeof(T);
  return launch_timed(fn, dim3((unsigned)batch), dim3(64), args, 0, st, sizeof(T) == 8 ? FDWT_TC_PASS_F64 : FDWT_TC_PASS_F32, work);
}

static int run_small(int m, Kind k, const void* in, void* out, int batch, double scale, const ReduceArgs* red,
                     hipStream_t st) {
  if (k == K_F32) return launch_small<float>(in, out, m, batch, scale, red, st);
  if (k == K_U32) return launch_small<uint32_t>(in, out, m, batch, scale, red, st);
  if (k == K_F64) return launch_small<double>(in, out, m, batch, scale, red, st);
  return fail(FDWT_EINVAL, "unsupported transform element types");
}

// ---------------------------------------------- p = 2 static-shape passes
struct P2Pass {
  int d0, loge, wdig;
};

// Two passes cover m <= 24: a contiguous first pass of up to 2^14 elements,
// then strided passes over the remaining digits with rows of 2^wd elements,
// split evenly (>= 2^7 elements per tile).  Rows of 16 doubles or 32 floats
// are 128 bytes, the cache line: a row never shares a line with another tile
// (tiles of one column are not neighbours in time) and each DRAM access
// moves a whole line.  4-byte elements take rows of 32 when that does not
// add a pass (every m <= 23); m = 24 keeps rows of 16 (64 bytes) and two
// passes.
static std::vector<P2Pass> plan_p2_w(int m, int emax, int wd) {
  std::vector<P2Pass> out;
  if (m <= emax) {
    out.push_back({0, m, 0});
    return out;
  }
  const int rem = m - emax;
  const int cap = emax - wd;
  const int nstr = (rem + cap - 1) / cap;
  const int rd = std::max((rem + nstr - 1) / nstr, 7 - wd);
  const int first = m - nstr * rd;
  out.push_back({0, first, 0});
  for (int i = 0; i < nstr; ++i) out.push_back({first + i * rd, rd + wd, wd});
  return out;
}

static std::vector<P2Pass> plan_p2_e(int m, int emax, size_t bytes = 4) {
  std::vector<P2Pass> v = plan_p2_w(m, emax, 4);
  if (bytes <= 4) {
    std::vector<P2Pass> w = plan_p2_w(m, emax, 5);
    if (w.size() <= v.size()) return w;
  }
  return v;
}

// First-pass bound of a plain transform: the largest tile (2^14) where the
// transform fits one tile or needs it to stay at two passes, and smaller
// tiles where two passes hold anyway: their workgroups are more than the CUs
// at fewer points, and several share a CU (a 2^14-element float64 tile takes
// a whole one).  Forward + inverse pairs (us), 2^14 / this bound: float
// m = 18 15.0 / 14.6, m = 19 16.2 / 15.0 (2^12: 14.7), m = 20 20.2 / 18.8
// (2^12: 20.1), m = 22 32.3 / 32.0 (m = 23 47.6, with 2^13 three passes and
// 62.6; m = 15 to 17 within 0.4 for every bound); float64 m = 16 15.8 / 14.6,
// m = 17 21.8 / 14.7, m = 19 27.4 / 20.2, m = 20 35.5 / 28.4, m = 21
// 37.0 / 33.6 with 2^13 (2^12: three passes, 43.9), m = 22 53.5 with 2^14
// (2^13: 48.9, not taken yet).
static int p2_emax(int m, size_t bytes) {
  if (bytes < 8) return m >= 18 && m <= 22 ? 13 : 14;
  if (m <= 14) return 14;
  return m <= 20 ? 12 : (m <= 21 ? 13 : 14);
}

static std::vector<P2Pass> plan_p2(int m, size_t bytes) {
  const int e = p2_emax(m, bytes);
  return plan_p2_e(m, (bytes >= 8 && wide_lds_budget() < 136 * 1024) ? std::min(e, 13) : e, bytes);
}

// Plan of the kernel spectrum and of the variance columns (float64): 2^14
// first-pass tiles at every size.  The spectra's small bins are differences
// of large sums, so their last digits follow the order of the stages, which
// a plan fixes; many columns fill the device with any tile.
static std::vector<P2Pass> plan_p2_cols(int m) { return plan_p2_e(m, wide_lds_budget() < 136 * 1024 ? 13 : 14, 8); }

template <class T, int WDIG>
static const void* p2_store_kernel(int loge) {
  switch (loge) {
    case 7: return (const void*)fwt_p2<T, 7, WDIG>;
    case 8: return (const void*)fwt_p2<T, 8, WDIG>;
    case 9: return (const void*)fwt_p2<T, 9, WDIG>;
    case 10: return (const void*)fwt_p2<T, 10, WDIG>;
    case 11: return (const void*)fwt_p2<T, 11, WDIG>;
    case 12: return (const void*)fwt_p2<T, 12, WDIG>;
    case 13: return (const void*)fwt_p2<T, 13, WDIG>;
    case 14: return (const void*)fwt_p2<T, 14, WDIG>;
  }
  return nullptr;
}

template <int WDIG>
static const void* p2_sums_kernel(int loge) {
  switch (loge) {
    case 7: return (const void*)fwt_p2_sums<7, WDIG>;
    case 8: return (const void*)fwt_p2_sums<8, WDIG>;
    case 9: return (const void*)fwt_p2_sums<9, WDIG>;
    case 10: return (const void*)fwt_p2_sums<10, WDIG>;
    case 11: return (const void*)fwt_p2_sums<11, WDIG>;
    case 12: return (const void*)fwt_p2_sums<12, WDIG>;
    case 13: return (const void*)fwt_p2_sums<13, WDIG>;
    case 14: return (const void*)fwt_p2_sums<14, WDIG>;
  }
  return nullptr;
}

// Workgroups per CU for (kernel, LDS), cached.
int occupancy(const void* fn, int threads, size_t lds) {
  static std::mutex mu;
  static std::map<std::pair<const void*, size_t>, int> cache;
  std::lock_guard<std::mutex> g(mu);
  auto key = std::make_pair(fn, lds);
  auto it = cache.find(key);
  if (it != cache.end()) return it->second;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, threads, lds) != hipSuccess || n < 1) n = 1;
  cache[key] = n;
  return n;
}

// Partial sums per column written by a reducing static pass: one per wave of
// every tile.
static int64_t p2_reduce_parts(int m, const P2Pass& g) {
  const int threads = std::max(64, std::min(1024, (1 << g.loge) / 16));
  return ((int64_t(1) << m) >> g.loge) * (threads / 64);
}

// FDWT_REDUCE_WKEEP = 0 turns the grouped-sum weight reuse off (the sums are
// bit-identical either way: each partial sum covers the same elements).
// Read at each launch.
static bool wkeep_enabled() {
  const char* e = getenv("FDWT_REDUCE_WKEEP");
  return !(e && atoi(e) == 0);
}

// layout: 0 natural; 1 the (contiguous first) pass stores in the blocked
// layout of PassDesc::oblk; 2 the (strided) pass reads and writes that
// blocked layout, where each of its tiles is one contiguous block.
template <class T>
static int launch_p2(const void* in, void* out, const P2Pass& g, int m, int batch, double scale,
                     const ReduceArgs* red, hipStream_t st, const void* const* in_tab = nullptr,
                     void* const* out_tab = nullptr, int layout = 0) {
  constexpr bool wide = sizeof(T) >= 8;
  const void* fn = nullptr;
  if (red) {
    if constexpr (wide) fn = g.wdig ? p2_sums_kernel<4>(g.loge) : p2_sums_kernel<0>(g.loge);
  } else {
    if (g.wdig == 5) {
      if constexpr (!wide) fn = p2_store_kernel<T, 5>(g.loge);
    } else {
      fn = g.wdig ? p2_store_kernel<T, 4>(g.loge) : p2_store_kernel<T, 0>(g.loge);
    }
  }
  if (!fn || (g.wdig != 0 && g.wdig != 4 && g.wdig != 5)) return fail(FDWT_EINVAL, "no static pass shape");
  const int64_t N = int64_t(1) << m;
  const int E = 1 << g.loge;
  const int threads = std::max(64, std::min(1024, E / 16));
  PassDesc d{};
  d.col_in = N;
  d.col_out = N;
  d.sd0 = int64_t(1) << g.d0;
  d.shi = int64_t(1) << (g.d0 + g.loge - g.wdig);
  d.r = g.loge - g.wdig;
  d.wdig = g.wdig;
  d.w = 1 << g.wdig;
  d.nlo = (int)(int64_t(1) << (g.d0 - g.wdig));
  d.E = E;
  d.scale = (float)scale;
  d.scale64 = scale;
  const int64_t ntiles = N / E;
  const int64_t nb = ntiles * batch;
  d.ntiles = (int)ntiles;
  d.batch = batch;
  if (red) {
    d.wts = red->wts;
    d.partial = red->partial;
    d.h0_out = red->h0_out;
    d.h0_col = red->h0_col;
    d.ncols = red->ncols;
  } else {
    d.h0_col = -1;
  }
  d.in_tab = in_tab;
  d.out_tab = out_tab;
  if (layout == 1) {
    if (g.wdig != 0 || g.loge < 10 || in_tab || out_tab) return fail(FDWT_EINVAL, "blocked store needs a first pass");
    d.oblk = ntiles * 16;
  } else if (layout == 2) {
    if (g.wdig != 4 || g.d0 + g.loge - g.wdig != m) return fail(FDWT_EINVAL, "blocked read needs the last pass");
    d.sd0 = 16;
    d.nlo = 1;
    d.shi = E;
  }
  const size_t lds = ((size_t)cpad(E) * sizeof(T) + 15) / 16 * 16;
  if (int rc = allow_lds(fn, lds)) return rc;
  int64_t G = nb;
  if (red) G = std::min(nb, (int64_t)occupancy(fn, threads, lds) * device_cus());
  // Neighbouring tiles of a strided pass share 128-byte lines when its rows
  // are shorter: they go to one XCD.  Rows of whole lines do better on the
  // order of dispatch (float m = 21 28.7 against 31.3 us a pair, m = 23 49.7
  // against 54.6; with short rows, m = 24, 120 against 95), contiguous tiles
  // on one XCD (m = 24 95 against 97).
  const bool lines = !red && g.wdig && layout == 0 && ((size_t)sizeof(T) << g.wdig) >= 128;
  d.xcd = G >= 64 && !lines ? 1 : 0;
  // Grouped sums over several columns: a workgroup keeps one tile's weights
  // for all its columns when the tiles split evenly over the grid.
  d.wkeep = (red && g.loge >= 10 && batch > 1 && ntiles % G == 0 && wkeep_enabled()) ? 1 : 0;
  void* args[] = {(void*)&in, (void*)&out, (void*)&d};
  void* sargs[] = {(void*)&in, (void*)&d};
  const double elems = (double)N * batch;
  const double work = red ? elems * sizeof(T) + (double)N * sizeof(float2) : elems * 2 * sizeof(T);
  return launch_timed(fn, dim3((unsigned)G), dim3(threads), red ? sargs : args, lds, st, wide ? FDWT_TC_PASS_F64 : FDWT_TC_PASS_F32,
                      work);
}

static int p2_pass(Kind k, const void* in, void* out, const P2Pass& g, int m, int batch, double scale,
                   const ReduceArgs* red, hipStream_t st, int layout = 0) {
  if (k == K_F32 && !red) return launch_p2<float>(in, out, g, m, batch, scale, nullptr, st);
  if (k == K_U32 && !red) return launch_p2<uint32_t>(in, out, g, m, batch, scale, nullptr, st);
  if (k == K_F64) return launch_p2<double>(in, out, g, m, batch, scale, red, st, nullptr, nullptr, layout);
  return fail(FDWT_EINVAL, "unsupported p = 2 element type");
}

// p = 2: forward and inverse coincide up to the scale.
static int run_p2(int m, Kind k, const void* in, void* out, void* tmp, int batch, double scale,
                  const ReduceArgs* red, hipStream_t st) {
  if (m < 7) return run_small(m, k, in, out, batch, scale, red, st);
  const std::vector<P2Pass> passes = red ? plan_p2_cols(m) : plan_p2(m, kind_bytes(k));
  const size_t np = passes.size();
  if (np == 1) return p2_pass(k, in, out, passes[0], m, batch, scale, red, st);
  void* mid = red ? tmp : out;
  if (!mid) return fail(FDWT_EINVAL, "transform needs a workspace for its intermediate passes");
  int rc = p2_pass(k, in, mid, passes[0], m, batch, 1.0f, nullptr, st);
  for (size_t i = 1; !rc && i + 1 < np; ++i) rc = p2_pass(k, mid, mid, passes[i], m, batch, 1.0f, nullptr, st);
  if (rc) return rc;
  return p2_pass(k, mid, out, passes[np - 1], m, batch, scale, red, st);
}

static int run_passes(int p, int m, bool inverse, Kind in_kind, const void* in, Kind work_kind,
                      Kind out_kind, void* out, void* tmp, int batch, double scale, const ReduceArgs* red,
                      hipStream_t st) {
  if (p == 2) {
    if (in_kind != work_kind || out_kind != work_kind) return fail(FDWT_EINVAL, "unsupported transform element types");
    return run_p2(m, work_kind, in, out, tmp, batch, scale, red, st);
  }
  const std::vector<PassGeom> passes = odd_plan(p, m, work_kind == K_CF64);
  const size_t np = passes.size();
  auto one = [&](Kind ik, Kind ok, const void* src, void* dst, const PassGeom& g, double sc, const ReduceArgs* rd) {
    return odd_pass(p, inverse, ik, work_kind, ok, src, dst, g, m, batch, sc, rd, st);
  };
  if (np == 1) return one(in_kind, out_kind, in, out, passes[0], scale, red);
  // Intermediate buffer: the output itself when it holds the working type.
  void* mid = (!red && kind_bytes(out_kind) == kind_bytes(work_kind)) ? out : tmp;
  if (!mid) return fail(FDWT_EINVAL, "transform needs a workspace for its intermediate passes");
  int rc = one(in_kind, work_kind, in, mid, passes[0], 1.0, nullptr);
  if (rc) return rc;
  for (size_t i = 1; i + 1 < np; ++i) {
    rc = one(work_kind, work_kind, mid, mid, passes[i], 1.0, nullptr);
    if (rc) return rc;
  }
  return one(work_kind, out_kind, mid, out, passes[np - 1], scale, red);
}

int fwt_run_tmp(int p, int m, bool inverse, Kind in_kind, const void* in, Kind work_kind,
                Kind out_kind, void* out, void* tmp, int batch, double scale, hipStream_t st) {
  return run_passes(p, m, inverse, in_kind, in, work_kind, out_kind, out, tmp, batch, scale, nullptr, st);
}

int fwt_run(int p, int m, bool inverse, Kind in_kind, const void* in, Kind work_kind,
            Kind out_kind, void* out, int batch, double scale, hipStream_t st) {
  return fwt_run_tmp(p, m, inverse, in_kind, in, work_kind, out_kind, out, nullptr, batch, scale, st);
}

// Unnormalised forward transform of ncols real float64 columns with the
// grouped-sum epilogue in its last pass (no output stored).  p = 2: `in` holds
// the columns and tmp the intermediate passes.  p odd: `in` holds pairs of
// columns as complex ones, column 2 i as the real part and column 2 i + 1
// times 2^pexp[i] as the imaginary part (both spectra are real: the
// kernel columns are even functions of the point index), and is overwritten;
// tmp is not used.  partial receives [ncols][fwt_reduce_parts] partial sums.
int fwt_reduce_f64(int p, int m, void* in, void* tmp, int ncols, const float2* wts, const int32_t* pexp,
                   double* partial, double* h0_out, int h0_col, hipStream_t st) {
  ReduceArgs red{wts, partial, h0_out, h0_col, pexp, ncols};
  if (p == 2) return run_passes(p, m, false, K_F64, in, K_F64, K_F64, tmp, tmp, ncols, 1.0, &red, st);
  return run_passes(p, m, false, K_CF64, in, K_CF64, K_CF64, in, in, (ncols + 1) / 2, 1.0, &red, st);
}

// Plans of p = 2 float transforms for the batch tuner: the first pass takes
// up to 2^emax elements (emax in 7..14), then strided passes of rows of 16.
int p2_plan_passes(int m, int emax) { return (int)plan_p2_e(m, emax).size(); }
// Plans for two values of emax are the same pass list.
bool p2_plans_equal(int m, int e1, int e2) {
  const std::vector<P2Pass> a = plan_p2_e(m, e1), b = plan_p2_e(m, e2);
  if (a.size() != b.size()) return false;
  for (size_t i = 0; i < a.size(); ++i)
    if (a[i].d0 != b[i].d0 || a[i].loge != b[i].loge || a[i].wdig != b[i].wdig) return false;
  return true;
}

// Pass `level` of the plan (m, emax) for a group of njobs float jobs of 2^m
// points each: column c reads in_tab[c] (level 0) or out_tab[c] and writes
// out_tab[c]; the last pass scales by 2^-m (Eq. (eq_dwalshcoeff)).
int fwt_p2_group_pass(int m, int emax, int level, const void* const* in_tab, void* const* out_tab, int njobs,
                      hipStream_t st) {
  const std::vector<P2Pass> passes = plan_p2_e(m, emax);
  if (level < 0 || level >= (int)passes.size()) return fail(FDWT_EINVAL, "no such pass");
  const bool last = level + 1 == (int)passes.size();
  const double scale = last ? std::ldexp(1.0, -m) : 1.0;
  const void* const* src = level == 0 ? in_tab : (const void* const*)out_tab;
  return launch_p2<float>(nullptr, nullptr, passes[level], m, njobs, scale, nullptr, st, src, out_tab);
}

// The p = 2 float64 transform of a batch of columns split after its first
// pass, for callers that produce part of the first pass's output with
// fwt_p2_gen_first: whether the plan for m has that shape (two or more
// passes, the first contiguous with 2^12..2^14-element tiles), the first pass
// alone (in -> out), and the remaining passes in place with the grouped-sum
// epilogue in the last (partial as for fwt_reduce_f64).
bool fwt_p2_split_ok(int m) {
  if (m < 7) return false;
  const std::vector<P2Pass> v = plan_p2_cols(m);
  return v.size() >= 2 && v[0].d0 == 0 && v[0].wdig == 0 && v[0].loge >= 12 && v[0].loge <= 14;
}

// Two-pass plans can keep the intermediate in the blocked layout of
// PassDesc::oblk (the first pass stores blocks, the grouped-sum pass reads
// each tile as one contiguous block; its weights then come in the same
// layout, fwt_p2_blocked_index).
bool fwt_p2_blocked_ok(int m) { return fwt_p2_split_ok(m) && plan_p2_cols(m).size() == 2; }

// The whole transform is one tile that can generate its own column.
bool fwt_p2_single_ok(int m) { return m >= 10 && plan_p2_cols(m).size() == 1; }

// Digits of the first pass of the float64 plan for m.
int fwt_p2_first_loge(int m) { return plan_p2_cols(m)[0].loge; }

int fwt_p2_f64_first(int m, const double* in, double* out, int batch, bool blocked, hipStream_t st) {
  if (!fwt_p2_split_ok(m) || (blocked && !fwt_p2_blocked_ok(m))) return fail(FDWT_EINVAL, "no split plan for this m");
  return p2_pass(K_F64, in, out, plan_p2_cols(m)[0], m, batch, 1.0, nullptr, st, blocked ? 1 : 0);
}

int fwt_p2_f64_reduce_rest(int m, double* data, int batch, const float2* wts, double* partial, double* h0_out,
                           int h0_col, bool blocked, hipStream_t st) {
  if (!fwt_p2_split_ok(m) || (blocked && !fwt_p2_blocked_ok(m))) return fail(FDWT_EINVAL, "no split plan for this m");
  const std::vector<P2Pass> v = plan_p2_cols(m);
  const ReduceArgs red{wts, partial, h0_out, h0_col, nullptr, batch};
  int rc = FDWT_OK;
  for (size_t i = 1; !rc && i + 1 < v.size(); ++i) rc = p2_pass(K_F64, data, data, v[i], m, batch, 1.0, nullptr, st);
  if (rc) return rc;
  return p2_pass(K_F64, data, data, v.back(), m, batch, 1.0, &red, st, blocked ? 2 : 0);
}

// First pass of the transforms of generated columns (fwt_p2_gen): the
// truncation columns U_{d0+1}..U_{d1} from the R' table (kcol false: out
// receives d1 - d0 columns), or the kernel column K from the K' table (kcol
// true: one column; d0, d1 unused; a net of one tile gets its whole spectrum).
int fwt_p2_gen_first(int m, int s, const uint32_t* xtab, int nbytes, const KernTab& kt, bool kcol,
                     int d0, int d1, double* out, bool blocked, hipStream_t st) {
  const bool single = kcol && fwt_p2_single_ok(m);
  if ((!single && !fwt_p2_split_ok(m)) || s < 1 || s > 64 || kTab <= m) return fail(FDWT_EINVAL, "bad generated-column pass");
  if (!kcol && (d0 < 0 || d1 > s || d0 >= d1)) return fail(FDWT_EINVAL, "bad generated-column range");
  const P2Pass g = plan_p2_cols(m)[0];
  const void* fn = nullptr;
  if (kcol) fn = g.loge == 14   ? (const void*)fwt_p2_gen<14, true>
                 : g.loge == 13 ? (const void*)fwt_p2_gen<13, true>
                 : g.loge == 12 ? (const void*)fwt_p2_gen<12, true>
                 : g.loge == 11 ? (const void*)fwt_p2_gen<11, true>
                                : (const void*)fwt_p2_gen<10, true>;
  else fn = g.loge == 14 ? (const void*)fwt_p2_gen<14, false>
            : g.loge == 13 ? (const void*)fwt_p2_gen<13, false> : (const void*)fwt_p2_gen<12, false>;
  const int64_t N = int64_t(1) << m;
  const int E = 1 << g.loge;
  const int threads = E / 16;
  const int ncol = kcol ? 1 : d1 - d0;
  PassDesc d{};
  d.col_in = N;
  d.col_out = N;
  d.ntiles = (int)(N / E);
  d.batch = ncol;
  d.h0_col = -1;
  if (blocked) {
    if (!fwt_p2_blocked_ok(m)) return fail(FDWT_EINVAL, "no blocked plan for this m");
    d.oblk = (int64_t)d.ntiles * 16;
  }
  const size_t lds = (size_t)((cpad(E) + 1) & ~1) * sizeof(double) + (size_t)s * (m + 1) * sizeof(double) +
                     (size_t)s * m * sizeof(uint32_t);
  if (int rc = allow_lds(fn, lds)) return rc;
  int64_t G = (int64_t)occupancy(fn, threads, lds) * device_cus();
  // Columns of a tile divided so that the workgroups fill the device once.
  const int nch0 = (int)std::max<int64_t>(1, std::min<int64_t>(ncol, G / d.ntiles));
  const int per = (ncol + nch0 - 1) / nch0, nch = (ncol + per - 1) / per;
  if (G >= (int64_t)d.ntiles * nch) G = (int64_t)d.ntiles * nch;
  d.xcd = G >= 64 ? 1 : 0;
  ColGen cg{xtab, nbytes, s, m, kcol ? 0 : d0, kcol ? s : d1, nch, per};
  void* args[] = {(void*)&cg, (void*)&out, (void*)&d, (void*)&kt};
  return launch_timed(fn, dim3((unsigned)G), dim3(threads), args, lds, st, FDWT_TC_PASS_F64,
                      (double)N * ncol * sizeof(double));
}

// The split cost in one launch (fwt_p2_split): first halves of 2^10..2^14
// points.
bool fwt_p2_split_tile_ok(int m) { return m >= 10 && m <= 14; }

int fwt_p2_split_tile(const Net& tr, const KernTab& kt, const float* ft, const float* fval, double* ku, float* sf,
                      double* cost, hipStream_t st) {
  const int m = tr.m, E = 1 << m;
  const void* fn = m == 10   ? (const void*)fwt_p2_split<10>
                   : m == 11 ? (const void*)fwt_p2_split<11>
                   : m == 12 ? (const void*)fwt_p2_split<12>
                   : m == 13 ? (const void*)fwt_p2_split<13>
                   : m == 14 ? (const void*)fwt_p2_split<14>
                             : nullptr;
  if (!fn) return fail(FDWT_EINVAL, "no one-launch split cost for this m");
  const size_t lds = (size_t)((cpad(E) + 1) & ~1) * sizeof(double) + (size_t)tr.s * (m + 2) * sizeof(double) +
                     (size_t)tr.s * m * sizeof(uint32_t);
  if (int rc = allow_lds(fn, lds)) return rc;
  SplitTile g{tr.d_xtab, tr.nbytes, tr.s, m, ft, fval, ku, sf, cost};
  KernTab k = kt;
  void* args[] = {(void*)&g, (void*)&k};
  // f~ and the second half read, K_u (and Sf) written.
  return launch_timed(fn, dim3(1), dim3(E / 16), args, lds, st, FDWT_TC_PASS_F64, (double)E * (sf ? 20 : 16));
}

// The passes after the first of an unnormalised p = 2 float64 transform, in
// place (the first pass's output already in data).
int fwt_p2_f64_rest(int m, double* data, int batch, hipStream_t st) {
  if (!fwt_p2_split_ok(m)) return fail(FDWT_EINVAL, "no split plan for this m");
  const std::vector<P2Pass> v = plan_p2_cols(m);
  int rc = FDWT_OK;
  for (size_t i = 1; !rc && i < v.size(); ++i) rc = p2_pass(K_F64, data, data, v[i], m, batch, 1.0, nullptr, st);
  return rc;
}

// fdwt_dwt_forward_family for p = 2: the first pass samples its own input
// (fwt_p2_fam), the remaining passes run in place on out.  Returns
// FDWT_EUNSUPPORTED (nothing enqueued) when the plan's first pass has fewer
// than 2^10 elements; the caller then samples and transforms separately.
template <int FAM>
static const void* fam_kernel(int loge) {
  switch (loge) {
    case 10: return (const void*)fwt_p2_fam<10, FAM>;
    case 11: return (const void*)fwt_p2_fam<11, FAM>;
    case 12: return (const void*)fwt_p2_fam<12, FAM>;
    case 13: return (const void*)fwt_p2_fam<13, FAM>;
    case 14: return (const void*)fwt_p2_fam<14, FAM>;
  }
  return nullptr;
}

int fwt_p2_forward_family(const Net& net, int family, const FamilyArgs& fa, float* out, hipStream_t st) {
  const std::vector<P2Pass> passes = plan_p2(net.m, 4);
  const P2Pass& g0 = passes[0];
  if (net.p != 2 || net.m < 10 || g0.d0 != 0 || g0.wdig != 0 || g0.loge < 10 || g0.loge > 14)
    return FDWT_EUNSUPPORTED;
  const void* fn = family == FDWT_FAMILY_PRODUCT ? fam_kernel<FDWT_FAMILY_PRODUCT>(g0.loge)
                   : family == FDWT_FAMILY_EXP   ? fam_kernel<FDWT_FAMILY_EXP>(g0.loge)
                   : family == FDWT_FAMILY_ASIAN ? fam_kernel<FDWT_FAMILY_ASIAN>(g0.loge)
                                                 : fam_kernel<FDWT_FAMILY_WANGFANG>(g0.loge);
  if (!fn) return fail(FDWT_EINVAL, "no fused sampling pass for this shape");
  const int64_t N = int64_t(1) << net.m;
  const int E = 1 << g0.loge;
  const int threads = E / 16;
  const double scale = std::ldexp(1.0, -net.m);  // Eq. (eq_dwalshcoeff), applied by the last pass
  PassDesc d{};
  d.ntiles = (int)(N / E);
  d.batch = 1;
  d.h0_col = -1;
  d.scale = passes.size() == 1 ? (float)scale : 1.0f;
  d.scale64 = passes.size() == 1 ? scale : 1.0;
  const size_t lds = ((size_t)cpad(E) * sizeof(float) + 15) / 16 * 16;
  if (int rc = allow_lds(fn, lds)) return rc;
  int64_t G = (int64_t)occupancy(fn, threads, lds) * device_cus();
  if (G >= d.ntiles) G = d.ntiles;
  d.xcd = G >= 64 ? 1 : 0;
  FamGen fg{net.d_xtab, net.nbytes, net.m, fa};
  void* args[] = {(void*)&fg, (void*)&out, (void*)&d};
  if (int rc = launch_timed(fn, dim3((unsigned)G), dim3(threads), args, lds, st, FDWT_TC_SAMPLE, 4.0 * (double)N))
    return rc;
  for (size_t i = 1; i < passes.size(); ++i) {
    const bool last = i + 1 == passes.size();
    if (int rc = p2_pass(K_F32, out, out, passes[i], net.m, 1, last ? scale : 1.0, nullptr, st)) return rc;
  }
  return FDWT_OK;
}

// Partial sums per column of fwt_reduce_f64 and fwt_p2_f64_reduce_rest.
int64_t fwt_reduce_parts(int p, int m) {
  if (p == 2) return m < 7 ? 1 : p2_reduce_parts(m, plan_p2_cols(m).back());
  return ipow(p, m - odd_plan(p, m, true).back().le);
}

}  // namespace fdwt

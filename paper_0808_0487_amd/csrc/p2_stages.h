// Building blocks of the static-shape p = 2 passes (fwt.hip: fwt_p2,
// fwt_p2_gen, fwt_p2_fam; batch.hip: the one-launch batch tiles).
#pragma once

#include "pass_core.h"

#include <type_traits>

namespace fdwt {

// -------------------------------------------- p = 2 passes, static shape
// For p = 2 the tile shape (2^LOGE elements, rows of 2^WDIG contiguous
// elements) is a template parameter, so every LDS and global offset inside a
// tile is a compile-time constant added to a per-thread base: the per-element
// work is the butterfly itself.  Padded LDS index pad(e) = e + e/32; for the
// element sets used here pad(e0 + j*stride) = pad(e0) + pad(j*stride) holds
// exactly (checked exhaustively for every shape), so the offsets fold.
__host__ __device__ constexpr int cpad(int e) { return e + (e >> 5); }
__host__ __device__ constexpr int cilog2(int v) { return v <= 1 ? 0 : 1 + cilog2(v >> 1); }
__host__ __device__ constexpr int cmin(int a, int b) { return a < b ? a : b; }

template <int LOGE, int WDIG>
struct P2Shape {
  static constexpr int E = 1 << LOGE;
  static constexpr int W = 1 << WDIG;
  static constexpr int RD = LOGE - WDIG;                 // digits transformed
  static constexpr int THREADS = E / 16 < 64 ? 64 : (E / 16 > 1024 ? 1024 : E / 16);
  static constexpr int EPT = E / THREADS;                // elements per thread
  static constexpr int KGMAX = cmin(4, cilog2(EPT));     // digits per register group
  static_assert(EPT >= 2 && THREADS % W == 0, "unsupported shape");
};

// Register groups over row digits [Q, Q+KG), then the next group.  KGM caps
// the group size (fewer live registers when other values must stay live).
template <int LOGE, int WDIG, int Q, class T, int KGM = 4, int RDL = P2Shape<LOGE, WDIG>::RD,
          bool DONE = (Q >= RDL)>
struct P2Groups {
  static __device__ __forceinline__ void run(T* lds, int tid) {
    using S = P2Shape<LOGE, WDIG>;
    constexpr int KG = cmin(cmin(S::KGMAX, KGM), RDL - Q);
    constexpr int R = 1 << KG;
    constexpr int STQ = S::W << Q;                      // element stride of digit Q
    constexpr int GPT = (S::E >> KG) / S::THREADS;      // groups per thread
#pragma unroll
    for (int t = 0; t < GPT; ++t) {
      const int g = tid + t * S::THREADS;
      const int c = g & (S::W - 1);
      const int rem = g >> WDIG;
      const int il = rem & ((1 << Q) - 1);
      const int ih = rem >> Q;
      const int e0 = c + S::W * (il + (ih << (Q + KG)));
      T* base = lds + cpad(e0);
      T x[R];
#pragma unroll
      for (int j = 0; j < R; ++j) x[j] = base[cpad(j * STQ)];
#pragma unroll
      for (int b = 0; b < KG; ++b) {
#pragma unroll
        for (int j0 = 0; j0 < R; ++j0) {
          if (((j0 >> b) & 1) == 0) {
            const T u = x[j0], v = x[j0 + (1 << b)];
            x[j0] = add(u, v);
            x[j0 + (1 << b)] = sub(u, v);
          }
        }
      }
#pragma unroll
      for (int j = 0; j < R; ++j) base[cpad(j * STQ)] = x[j];
    }
    lds_barrier();
    P2Groups<LOGE, WDIG, Q + KG, T, KGM, RDL>::run(lds, tid);
  }
};
template <int LOGE, int WDIG, int Q, class T, int KGM, int RDL>
struct P2Groups<LOGE, WDIG, Q, T, KGM, RDL, true> {
  static __device__ __forceinline__ void run(T*, int) {}
};

// Radix-2 stages over register-index bits [0, NB) of v.
template <int NB, class T, int N>
__device__ __forceinline__ void reg_bfly(T (&v)[N]) {
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int j0 = 0; j0 < N; ++j0) {
      if (((j0 >> b) & 1) == 0) {
        const T u = v[j0], w = v[j0 + (1 << b)];
        v[j0] = add(u, w);
        v[j0 + (1 << b)] = sub(u, w);
      }
    }
  }
}

// Radix-2 stages over register-index bits [LO, HI) of v.
template <int LO, int HI, class T, int N>
__device__ __forceinline__ void reg_bfly_bits(T (&v)[N]) {
#pragma unroll
  for (int b = LO; b < HI; ++b) {
#pragma unroll
    for (int j0 = 0; j0 < N; ++j0) {
      if (((j0 >> b) & 1) == 0) {
        const T u = v[j0], w = v[j0 + (1 << b)];
        v[j0] = add(u, w);
        v[j0 + (1 << b)] = sub(u, w);
      }
    }
  }
}

// The value of the lane whose index differs in bit B (0 or 1): a move inside
// the four lanes of a quad.
template <int B>
__device__ __forceinline__ int quad_other(int v) {
  constexpr int ctrl = B == 0 ? 0xB1 : 0x4E;  // quad_perm [1,0,3,2] / [2,3,0,1]
  return __builtin_amdgcn_mov_dpp(v, ctrl, 0xF, 0xF, true);
}
template <int B>
__device__ __forceinline__ float quad_other(float v) {
  return __int_as_float(quad_other<B>(__float_as_int(v)));
}
template <int B>
__device__ __forceinline__ uint32_t quad_other(uint32_t v) {
  return (uint32_t)quad_other<B>((int)v);
}
template <int B>
__device__ __forceinline__ double quad_other(double v) {
  return __hiloint2double(quad_other<B>(__double2hiint(v)), quad_other<B>(__double2loint(v)));
}
// A butterfly's half in each lane: own + other, or other - own where the
// lane's bit is set (sg = -1): the same sum, rounded once, as in registers.
__device__ __forceinline__ float half_bfly(float own, float other, float sg) { return fmaf(own, sg, other); }
__device__ __forceinline__ double half_bfly(double own, double other, double sg) { return fma(own, sg, other); }
__device__ __forceinline__ uint32_t half_bfly(uint32_t own, uint32_t other, int sg) {
  const uint32_t neg = (uint32_t)(sg >> 1);  // -1: all ones, 1: 0
  return (own ^ neg) + other - neg;
}

// Stages of the digits 0..5 of a contiguous tile of LOGE >= 10 digits held in
// LDS: 0..3 in registers (a thread's 16 consecutive elements), then 4 and 5,
// which are bits 0 and 1 of the lane, between the lanes of a quad: one round
// trip through LDS and one barrier less than with a second register group
// (float 2^24 forward + inverse 94.7 -> 92.9 us, a split cost 41.6 -> 40.2).
template <int LOGE, class T>
__device__ __forceinline__ void p2_low6(T* lds, int tid) {
  static_assert(LOGE >= 10 && P2Shape<LOGE, 0>::THREADS * 16 == P2Shape<LOGE, 0>::E, "16 elements a thread");
  using Sg = typename std::conditional<std::is_same<T, uint32_t>::value, int, T>::type;
  T* base = lds + cpad(16 * tid);
  T x[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) x[j] = base[cpad(j)];
  reg_bfly<4>(x);
  const Sg s0 = (tid & 1) ? (Sg)-1 : (Sg)1, s1 = (tid & 2) ? (Sg)-1 : (Sg)1;
#pragma unroll
  for (int j = 0; j < 16; ++j) x[j] = half_bfly(x[j], quad_other<0>(x[j]), s0);
#pragma unroll
  for (int j = 0; j < 16; ++j) x[j] = half_bfly(x[j], quad_other<1>(x[j]), s1);
#pragma unroll
  for (int j = 0; j < 16; ++j) base[cpad(j)] = x[j];
  lds_barrier();
}

// Swaps of registers between lane halves (H = 32) or odd and even rows of 16
// (H = 16): a's lanes with bit H set and b's lanes with it clear.
template <int H>
__device__ __forceinline__ void lane_swap(uint32_t& a, uint32_t& b) {
  if constexpr (H == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  }
}
template <int H>
__device__ __forceinline__ void lane_swap(float& a, float& b) {
  uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
  lane_swap<H>(x, y);
  a = __uint_as_float(x);
  b = __uint_as_float(y);
}
template <int H>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
  uint32_t xl = (uint32_t)__double2loint(a), xh = (uint32_t)__double2hiint(a);
  uint32_t yl = (uint32_t)__double2loint(b), yh = (uint32_t)__double2hiint(b);
  lane_swap<H>(xl, yl);
  lane_swap<H>(xh, yh);
  a = __hiloint2double((int)xh, (int)xl);
  b = __hiloint2double((int)yh, (int)yl);
}
// The butterfly stage of lane bit H on every value: a pair of registers is
// swapped so that both halves of each butterfly meet in one lane, and back.
// In place of a round trip through LDS (float 2^24 forward + inverse 94.0 ->
// 93.2 us, a step at 2^24, s = 20 3653 -> 3630).
template <int H, class T, int N>
__device__ __forceinline__ void lane_bfly(T (&v)[N]) {
#pragma unroll
  for (int j = 0; j < N; j += 2) {
    lane_swap<H>(v[j], v[j + 1]);
    const T u = v[j], w = v[j + 1];
    v[j] = add(u, w);
    v[j + 1] = sub(u, w);
    lane_swap<H>(v[j], v[j + 1]);
  }
}

}  // namespace fdwt

// Point operations spread over four lanes, for calls too small to fill the
// device with one request per lane.
//
// A point in XYZZ coordinates lies across a quad of lanes, one coordinate each
// (lane 0: X, 1: Y, 2: ZZ, 3: ZZZ), and every lane computes one product of each
// level of a formula: an addition takes 4 levels instead of 14 products, a
// doubling 3 instead of 9.  With the coordinates laid out so, the operands of
// most products are in place or one quad permutation (a DPP move) away.
// Moves and selections cost about a third of the products: an addition on
// BLS12-381 issues 2,400 instructions per lane against 7,000 on one lane, so
// a chain runs 2 to 2.9 times as fast as long as lanes are free, and costs 1.3
// times the work when they are not.
//
// Infinity is a flag, the same in all four lanes; branches on it and on the
// exceptional cases are uniform in the quad.  Values and limbs are bounded as
// in lazy.h, but for Y3: the difference of two products that are reduced on
// their own, it lies in (-1.1, 1.1) p with limbs within 2^B, and may be below
// -p.  The formulas take that, as factor and as subtrahend; a stored sum's Y is
// back in (-0.2, 1.2) p (qz_store: one masked addition there; a product in the
// reduction instead took 308 -> 335 us of k_reduce_a_xz, by its registers).
#pragma once
#include "lazy.h"

namespace eccmi {

// lane l of each quad <- lane (SEL >> 2 l) & 3
template <int SEL>
__device__ __forceinline__ int32_t quad32(int32_t v) {
  return __builtin_amdgcn_mov_dpp(v, SEL, 0xf, 0xf, true);
}
constexpr int quad_sel(int l0, int l1, int l2, int l3) { return l0 | (l1 << 2) | (l2 << 4) | (l3 << 6); }
constexpr int QUAD_ALL(int l) { return quad_sel(l, l, l, l); }
constexpr int QUAD_SWAP2 = quad_sel(2, 3, 0, 1);

template <class F, int SEL>
__device__ __forceinline__ Lz<F> quad_perm(const Lz<F>& a) {
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = quad32<SEL>(a.w[i]);
  return r;
}

__device__ __forceinline__ int quad_lane() { return int(threadIdx.x & 3u); }

// the point's coordinate of this lane
template <class C>
using Qz = Lz<typename C::F>;

// A <- 2 A (not O): dbl-2008-s-1 in three levels,
// [X^2 or (X - ZZ)(X + ZZ), U^2] -> [S = X V, W = U V, V ZZ, M^2]
//   -> [M (S - X3), W Y, -, W ZZZ]
template <class C>
__device__ __forceinline__ void qz_dbl(Qz<C>& A) {
  using F = typename C::F;
  const int q = quad_lane();
  Lz<F> x, y;
  {
    const Lz<F> U = lz_carry_if29<F>(lz_shl<F>(A, 1));
    if constexpr (C::A_IS_MINUS3) {
      const Lz<F> ZZ = quad_perm<F, QUAD_ALL(2)>(A);
      x = lz_select<F>(q == 0, lz_sub<F>(A, ZZ), U);
      y = lz_select<F>(q == 0, lz_add<F>(A, ZZ), U);
    } else {
      x = y = lz_select<F>(q == 0, A, U);
    }
  }
  const Lz<F> r1 = lz_mul<F>(x, y);                             // lane 0: t, lane 1: V
  const Lz<F> V = quad_perm<F, QUAD_ALL(1)>(r1);
  const Lz<F> t = quad_perm<F, QUAD_ALL(0)>(r1);
  const Lz<F> M = lz_carry<F>(lz_add<F>(lz_shl<F>(t, 1), t));   // every lane
  // lanes 0, 2: A V; lane 1: U V; lane 3: M M
#pragma unroll
  for (int i = 0; i < F::NL; i++) {
    x.w[i] = q == 3 ? M.w[i] : int32_t(uint32_t(A.w[i]) << (q == 1 ? 1 : 0));
    y.w[i] = q == 3 ? M.w[i] : V.w[i];
  }
  const Lz<F> r2 = lz_mul<F>(x, y);                             // S, W, ZZ3, M^2
  const Lz<F> X3 = lz_carry<F>(lz_sub<F>(quad_perm<F, QUAD_ALL(3)>(r2), lz_shl<F>(r2, 1)));  // in lane 0
  const Lz<F> W = quad_perm<F, QUAD_ALL(1)>(r2);
  x = lz_select<F>(q == 0, M, W);
  y = lz_select<F>(q == 0, lz_sub<F>(r2, X3), A);
  const Lz<F> r3 = lz_mul<F>(x, y);                             // M (S - X3), W Y, -, ZZZ3
  const Lz<F> Y3 = lz_sub<F>(quad_perm<F, QUAD_ALL(0)>(r3), r3);  // in lane 1
#pragma unroll
  for (int i = 0; i < F::NL; i++)
    A.w[i] = q == 0 ? X3.w[i] : q == 1 ? Y3.w[i] : q == 2 ? r2.w[i] : r3.w[i];
  A = lz_carry_if29<F>(A);
}

// levels 2 to 4 of an addition.  d: P in lane 0 and R in lane 1; r1: U1 in
// lane 0 and S1 in lane 1; zx zy: the product Zf in lane 2 and Zzf in lane 3
// (the second point's ZZ, ZZZ: 1 in an addition of an affine point).
template <class C>
__device__ __forceinline__ void qz_add_tail(Qz<C>& A, const Lz<typename C::F>& d, const Lz<typename C::F>& r1,
                                            const Lz<typename C::F>& B) {
  using F = typename C::F;
  const int q = quad_lane();
  Lz<F> x = lz_select<F>(q < 2, d, A), y = lz_select<F>(q < 2, d, B);
  const Lz<F> r2 = lz_mul<F>(x, y);                             // PP, RR, Zf, Zzf
  const Lz<F> U1 = quad_perm<F, QUAD_ALL(0)>(r1);
  y = quad_perm<F, QUAD_ALL(0)>(r2);                            // PP
#pragma unroll
  for (int i = 0; i < F::NL; i++) x.w[i] = q == 0 ? d.w[i] : q == 1 ? U1.w[i] : r2.w[i];
  const Lz<F> r3 = lz_mul<F>(x, y);                             // PPP, Q, ZZ3, -
  const Lz<F> PPP = quad_perm<F, QUAD_ALL(0)>(r3);
  const Lz<F> X3 = lz_carry<F>(lz_sub<F>(lz_sub<F>(r2, PPP), lz_shl<F>(r3, 1)));  // in lane 1
  const Lz<F> S1 = quad_perm<F, QUAD_ALL(1)>(r1);
#pragma unroll
  for (int i = 0; i < F::NL; i++) {
    x.w[i] = q == 0 ? S1.w[i] : q == 1 ? d.w[i] : r2.w[i];
    y.w[i] = q == 1 ? r3.w[i] - X3.w[i] : PPP.w[i];
  }
  const Lz<F> r4 = lz_mul<F>(x, y);                             // S1 PPP, R (Q - X3), -, ZZZ3
  const Lz<F> Y3 = lz_sub<F>(r4, quad_perm<F, QUAD_ALL(0)>(r4));  // in lane 1
  const Lz<F> X3l0 = quad_perm<F, QUAD_ALL(1)>(X3);
#pragma unroll
  for (int i = 0; i < F::NL; i++)
    A.w[i] = q == 0 ? X3l0.w[i] : q == 1 ? Y3.w[i] : q == 2 ? r3.w[i] : r4.w[i];
  A = lz_carry_if29<F>(A);
}

// whether the P in lane 0 (|P| < K p) is 0 mod p, and the R in lane 1
template <class F, int K>
__device__ __forceinline__ bool quad_equal_x(const Lz<F>& d, bool& equal_y) {
  if (quad32<QUAD_ALL(0)>(lz_maybe_zero<F, K>(d)) == 0) return false;
  const int z = lz_is_zero<F>(d);
  equal_y = quad32<QUAD_ALL(1)>(z) != 0;
  return quad32<QUAD_ALL(0)>(z) != 0;
}

// add-2008-s, every case
template <class C>
__device__ __forceinline__ void qz_add(Qz<C>& A, bool& inf, const Qz<C>& B, bool binf) {
  using F = typename C::F;
  if (binf) return;
  if (inf) {
    A = B;
    inf = false;
    return;
  }
  const Lz<F> r1 = lz_mul<F>(A, quad_perm<F, QUAD_SWAP2>(B));   // U1, S1, U2, S2
  const Lz<F> d = lz_sub<F>(quad_perm<F, QUAD_SWAP2>(r1), r1);  // P, R, -, -
  bool equal_y;
  if (quad_equal_x<F, 4>(d, equal_y)) {
    if (equal_y) qz_dbl<C>(A);
    else inf = true;
    return;
  }
  qz_add_tail<C>(A, d, r1, B);
}

// an affine point across the quad: x, y, 1, 1
template <class C>
__device__ __forceinline__ Qz<C> qz_affine(const Lz<typename C::F>& x, const Lz<typename C::F>& y) {
  using F = typename C::F;
  constexpr Words<F::NL> one = F::ONE;
  const int q = quad_lane();
  Qz<C> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = q == 0 ? x.w[i] : q == 1 ? y.w[i] : int32_t(one.w[i]);
  return r;
}

// madd-2008-s, every case: B = qz_affine(x, y).  [x ZZ, y ZZZ] -> levels 2-4
// with ZZ2 = ZZZ2 = 1: as an addition but for U1 = X1, S1 = Y1, whose
// products with 1 are not taken
template <class C>
__device__ __forceinline__ void qz_madd(Qz<C>& A, bool& inf, const Qz<C>& B) {
  using F = typename C::F;
  if (inf) {
    A = B;
    inf = false;
    return;
  }
  const Lz<F> r = lz_mul<F>(quad_perm<F, QUAD_SWAP2>(A), B);    // U2, S2 in lanes 0, 1
  const Lz<F> d = lz_sub<F>(r, A);                              // P, R
  bool equal_y;
  if (quad_equal_x<F, 8>(d, equal_y)) {
    if (equal_y) qz_dbl<C>(A);
    else inf = true;
    return;
  }
  qz_add_tail<C>(A, d, A, B);
}

// the whole point in every lane
template <class C>
__device__ __forceinline__ Xz<C> qz_gather(const Qz<C>& A) {
  using F = typename C::F;
  Xz<C> r;
  r.X = quad_perm<F, QUAD_ALL(0)>(A);
  r.Y = quad_perm<F, QUAD_ALL(1)>(A);
  r.ZZ = quad_perm<F, QUAD_ALL(2)>(A);
  r.ZZZ = quad_perm<F, QUAD_ALL(3)>(A);
  return r;
}

// lane SRC's own point (each lane holds one) across the quad
template <class C, int SRC>
__device__ __forceinline__ Qz<C> qz_spread(const Xz<C>& P) {
  const int q = quad_lane();
  Qz<C> r;
#pragma unroll
  for (int i = 0; i < C::F::NL; i++) {
    const int32_t x = quad32<QUAD_ALL(SRC)>(P.X.w[i]), y = quad32<QUAD_ALL(SRC)>(P.Y.w[i]);
    const int32_t zz = quad32<QUAD_ALL(SRC)>(P.ZZ.w[i]), zzz = quad32<QUAD_ALL(SRC)>(P.ZZZ.w[i]);
    r.w[i] = q == 0 ? x : q == 1 ? y : q == 2 ? zz : zzz;
  }
  return r;
}

// a point stored by xz_store, one coordinate per lane, and back
template <class C>
__device__ __forceinline__ void qz_load(const uint32_t* __restrict__ p, Qz<C>& A, bool& inf) {
  using F = typename C::F;
  A = lz_load<F>(p + quad_lane() * F::CW);
  inf = quad32<QUAD_ALL(0)>(A.w[0]) < 0;
}
template <class C>
__device__ __forceinline__ void qz_store(uint32_t* __restrict__ p, const Qz<C>& A, bool inf) {
  using F = typename C::F;
  constexpr Words<F::NL> P = F::P;
  const int q = quad_lane();
  // Y + p where Y is negative (its top limb decides but for values within
  // p / 2^16 of 0, which may go either way)
  const int32_t neg = q == 1 ? A.w[F::NL - 1] >> 31 : 0;
  Lz<F> a;
#pragma unroll
  for (int i = 0; i < F::NL; i++) a.w[i] = A.w[i] + (int32_t(P.w[i]) & neg);
  a = lz_carry_if29<F>(a);
  if (inf && q == 0) a.w[0] = -1;
  lz_store<F>(p + q * F::CW, a);
}

}  // namespace eccmi

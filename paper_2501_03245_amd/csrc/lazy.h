// Signed lazy field arithmetic and the point formulas built on it, one
// element per lane.
//
// The limbs of field.h (radix 2^B, Montgomery R = 2^(B NL)) as signed 32-bit
// words.  A sum or difference is NL word operations with no carry, no
// comparison and no multiple of p: a product takes signed limbs of up to about
// B + 1 bits (v_mad_i64_i32 issues at the rate of v_mad_u64_u32) and any value
// small against R, and its reduction brings both back.  A modular subtraction
// of field.h costs about 9 NL instructions, a canonical form 5 NL; in a point
// addition they were a third of all instructions.  Two products whose sum or
// difference is wanted (Y3 of every formula) share one reduction (lz_mul2).
//
// Bounds.  Write u = p 2^0 for the modulus and rho = R / p (BN254: 169,
// BLS12-381: 2^11.3, the 256-bit ECDSA primes: 2^24).
//   lz_mul(a, b)      : value in (-e, 1 + e) p with e = |a b| / (rho p^2);
//                       limbs in [0, 2^B) below the signed top one;
//   columns           : NL max|a_i| max|b_j| (summed over the products that
//                       share a reduction) + NL 2^(2B) must stay below 2^63,
//                       that is, with limbs counted in units of 2^B: the sum
//                       of the unit products plus one is at most 14 for
//                       BN254 (9 limbs of 29 bits: 2^63 / (9 2^58) = 3.5, so
//                       at most 3.5 there), 9.1 for BLS12-381 (14 of 28 bits)
//                       and 12.8 for the 256-bit primes (10 of 28 bits);
//   lz_carry(a)       : one parallel carry pass: limbs in [-k, 2^B + k) for
//                       limbs below k 2^B, the same value.
// The formulas state the values they keep: X in (-3.5, 1.2) p, Y, Z, ZZ, ZZZ
// product outputs in (-0.2, 1.2) p.
#pragma once
#include "point.h"

namespace eccmi {

template <class F>
struct Lz {
  int32_t w[F::NL];
};

template <class F>
__device__ __forceinline__ Lz<F> lz_of(const Fp<F>& a) {
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = int32_t(a.w[i]);
  return r;
}

template <class F>
__device__ __forceinline__ Lz<F> lz_zero() {
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = 0;
  return r;
}

template <class F>
__device__ __forceinline__ Lz<F> lz_one() {
  return lz_of<F>(fp_one<F>());
}

template <class F>
__device__ __forceinline__ Lz<F> lz_add(const Lz<F>& a, const Lz<F>& b) {
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = a.w[i] + b.w[i];
  return r;
}

template <class F>
__device__ __forceinline__ Lz<F> lz_sub(const Lz<F>& a, const Lz<F>& b) {
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = a.w[i] - b.w[i];
  return r;
}

// a 2^s
template <class F>
__device__ __forceinline__ Lz<F> lz_shl(const Lz<F>& a, int s) {
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = int32_t(uint32_t(a.w[i]) << s);
  return r;
}

template <class F>
__device__ __forceinline__ Lz<F> lz_neg(const Lz<F>& a) {
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = -a.w[i];
  return r;
}

// -a where neg, else a
template <class F>
__device__ __forceinline__ Lz<F> lz_neg_if(const Lz<F>& a, bool neg) {
  const int32_t m = neg ? -1 : 0;
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = (a.w[i] ^ m) - m;
  return r;
}

template <class F>
__device__ __forceinline__ Lz<F> lz_select(bool c, const Lz<F>& a, const Lz<F>& b) {
  Lz<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = c ? a.w[i] : b.w[i];
  return r;
}

// one carry pass, every limb at once: no chain through the limbs
template <class F>
__device__ __forceinline__ Lz<F> lz_carry(const Lz<F>& a) {
  Lz<F> r;
  r.w[0] = a.w[0] & int32_t(F::MASK);
#pragma unroll
  for (int i = 1; i < F::NL - 1; i++) r.w[i] = (a.w[i] & int32_t(F::MASK)) + (a.w[i - 1] >> F::B);
  r.w[F::NL - 1] = a.w[F::NL - 1] + (a.w[F::NL - 2] >> F::B);
  return r;
}

// the same where the 29-bit limbs of BN254 leave no room for wider operands
template <class F>
__device__ __forceinline__ Lz<F> lz_carry_if29(const Lz<F>& a) {
  if constexpr (F::B > 28) return lz_carry<F>(a);
  else return a;
}

// ---- Montgomery products ---------------------------------------------------
// Algorithm 2 column by column as in field.h, with the columns of the integer
// product supplied by col(acc, k) and every carry shifted arithmetically.
template <class F, class Col>
__device__ __forceinline__ Lz<F> lz_montgomery(Col col) {
  constexpr int NL = F::NL;
  constexpr int B = F::B;
  uint32_t m[NL];
  Lz<F> r;
  uint64_t acc = 0;
  if constexpr (F::SPARSE) {
    int32_t dq[NL];
    sparse_digits<F>(dq);
#pragma unroll
    for (int k = 0; k < 2 * NL - 1; k++) {
      col(acc, k);
      sparse_terms<F>(acc, m, dq, k, k < NL ? 0 : k - NL + 1, k < NL ? k : NL);
      const uint32_t low = uint32_t(acc) & F::MASK;
      if (k < NL) m[k] = low;
      else r.w[k - NL] = int32_t(low);
      acc = uint64_t(int64_t(acc) >> B);
    }
  } else {
    constexpr Words<NL> qc = F::P;
    // modulus limbs and q_inv in scalar registers (see fp_mul)
    uint32_t q[NL];
#pragma unroll
    for (int j = 0; j < NL; j++) {
      q[j] = qc.w[j];
      asm("" : "+s"(q[j]));
    }
    uint32_t qinv = F::QINV;
    asm("" : "+s"(qinv));
#pragma unroll
    for (int k = 0; k < 2 * NL - 1; k++) {
      col(acc, k);
#pragma unroll
      for (int i = k < NL ? 0 : k - NL + 1; i < (k < NL ? k : NL); i++) acc += uint64_t(m[i]) * q[k - i];
      if (k < NL) {
        m[k] = (uint32_t(acc) * qinv) & F::MASK;
        acc += uint64_t(m[k]) * q[0];  // clears the low B bits
      } else {
        r.w[k - NL] = int32_t(uint32_t(acc) & F::MASK);
      }
      acc = uint64_t(int64_t(acc) >> B);
    }
  }
  r.w[NL - 1] = int32_t(uint32_t(acc));
  return r;
}

// column k of a b
template <class F>
__device__ __forceinline__ void lz_col(uint64_t& acc, const Lz<F>& a, const Lz<F>& b, int k) {
#pragma unroll
  for (int i = k < F::NL ? 0 : k - F::NL + 1; i < (k < F::NL ? k + 1 : F::NL); i++)
    acc += uint64_t(int64_t(a.w[i]) * int64_t(b.w[k - i]));
}

// column k of a^2, a2 = 2 a
template <class F>
__device__ __forceinline__ void lz_col_sqr(uint64_t& acc, const Lz<F>& a, const Lz<F>& a2, int k) {
#pragma unroll
  for (int i = k < F::NL ? 0 : k - F::NL + 1; 2 * i < k; i++)
    acc += uint64_t(int64_t(a.w[i]) * int64_t(a2.w[k - i]));
  if ((k & 1) == 0) acc += uint64_t(int64_t(a.w[k / 2]) * int64_t(a.w[k / 2]));
}

template <class F>
__device__ __forceinline__ Lz<F> lz_mul(const Lz<F>& a, const Lz<F>& b) {
  return lz_montgomery<F>([&](uint64_t& acc, int k) __attribute__((always_inline)) { lz_col<F>(acc, a, b, k); });
}

template <class F>
__device__ __forceinline__ Lz<F> lz_sqr(const Lz<F>& a) {
  const Lz<F> a2 = lz_shl<F>(a, 1);
  return lz_montgomery<F>([&](uint64_t& acc, int k) __attribute__((always_inline)) { lz_col_sqr<F>(acc, a, a2, k); });
}

// a b + c d with one reduction
template <class F>
__device__ __forceinline__ Lz<F> lz_mul2(const Lz<F>& a, const Lz<F>& b, const Lz<F>& c, const Lz<F>& d) {
  return lz_montgomery<F>([&](uint64_t& acc, int k) __attribute__((always_inline)) {
    lz_col<F>(acc, a, b, k);
    lz_col<F>(acc, c, d, k);
  });
}

// ---- back to the forms of field.h --------------------------------------------

// a in (-p, 2p), limbs below 2^(B+2) in magnitude: normalised, in [0, 2p)
template <class F>
__device__ __forceinline__ Fp<F> lz_semi(const Lz<F>& a) {
  constexpr Words<F::NL> p = F::P;
  int32_t d[F::NL];
  int32_t c = 0;
#pragma unroll
  for (int i = 0; i < F::NL; i++) {
    int32_t v = a.w[i] + c;
    if (i < F::NL - 1) {
      c = v >> F::B;
      v &= int32_t(F::MASK);
    }
    d[i] = v;
  }
  const int32_t neg = d[F::NL - 1] >> 31;
  Fp<F> r;
  c = 0;
#pragma unroll
  for (int i = 0; i < F::NL; i++) {
    int32_t v = d[i] + (int32_t(p.w[i]) & neg) + c;
    if (i < F::NL - 1) {
      c = v >> F::B;
      v &= int32_t(F::MASK);
    }
    r.w[i] = uint32_t(v);
  }
  return r;
}

// the same, canonical
template <class F>
__device__ __forceinline__ Fp<F> lz_canonical(const Lz<F>& a) {
  return fp_canonical<F>(lz_semi<F>(a));
}

// Whether a (|a| < K p, any limbs) may be 0 mod p: the multiples of p in that
// range differ in their low B bits, so the test is right but for one value in
// about 2^(B-1) / K; callers confirm with lz_is_zero.
template <class F, int K>
__device__ __forceinline__ bool lz_maybe_zero(const Lz<F>& a) {
  constexpr uint32_t pinv = (0u - F::QINV) & F::MASK;  // p^-1 mod 2^B
  const uint32_t t = uint32_t(a.w[0]) * pinv;          // a = k p gives k mod 2^B
  return ((t + uint32_t(K)) & F::MASK) <= 2u * K;
}

template <class F>
__device__ __forceinline__ bool lz_is_zero(const Lz<F>& a) {
  const Lz<F> v = lz_mul<F>(lz_carry<F>(a), lz_one<F>());  // a mod p, in (-p, 2p) with normalised limbs
  constexpr Words<F::NL> p = F::P;
  uint32_t z = 0, e = 0;
#pragma unroll
  for (int i = 0; i < F::NL; i++) {
    z |= uint32_t(v.w[i]);
    e |= uint32_t(v.w[i]) ^ p.w[i];
  }
  return z == 0 || e == 0;
}

// ---- points in XYZZ coordinates -----------------------------------------------
// (X, Y, ZZ, ZZZ) of point.h with lazy coordinates; infinity is a flag kept
// beside the point, so that no operation tests ZZ.

template <class C>
struct Xz {
  Lz<typename C::F> X, Y, ZZ, ZZZ;
};

template <class C>
__device__ __forceinline__ void xz_set(Xz<C>& A, const Lz<typename C::F>& x, const Lz<typename C::F>& y) {
  A.X = x;
  A.Y = y;
  A.ZZ = A.ZZZ = lz_one<typename C::F>();
}

// 2 (x, y) of an affine point (dbl-2008-s-1 with ZZ = ZZZ = 1): x in (-1, 1) p
// with limbs below 2^B in magnitude, y likewise
template <class C>
__device__ __forceinline__ void xz_mdbl(Xz<C>& A, const Lz<typename C::F>& x, const Lz<typename C::F>& y) {
  using F = typename C::F;
  const Lz<F> U = lz_carry<F>(lz_shl<F>(y, 1));
  const Lz<F> V = lz_sqr<F>(U);
  const Lz<F> W = lz_mul<F>(U, V);
  const Lz<F> S = lz_mul<F>(x, V);
  Lz<F> t = lz_sqr<F>(x);
  if constexpr (C::A_IS_MINUS3) t = lz_sub<F>(t, lz_one<F>());
  const Lz<F> M = lz_carry<F>(lz_add<F>(lz_add<F>(t, t), t));
  A.X = lz_carry<F>(lz_sub<F>(lz_sqr<F>(M), lz_shl<F>(S, 1)));
  A.Y = lz_mul2<F>(M, lz_sub<F>(S, A.X), lz_neg<F>(W), y);
  A.ZZ = V;
  A.ZZZ = W;
}

// madd-2008-s: A += (bx, by), every case.  |bx|, |by| < 1.1 p with limbs
// below 2^B in magnitude (a canonical or product-form coordinate, or the
// negative of one).
template <class C>
__device__ __forceinline__ void xz_madd(Xz<C>& A, bool& inf, const Lz<typename C::F>& bx,
                                        const Lz<typename C::F>& by) {
  using F = typename C::F;
  if (inf) {
    xz_set<C>(A, bx, by);
    inf = false;
    return;
  }
  const Lz<F> P = lz_sub<F>(lz_mul<F>(bx, A.ZZ), A.X);   // |P| < 5p
  const Lz<F> R = lz_sub<F>(lz_mul<F>(by, A.ZZZ), A.Y);  // |R| < 2.5p
  if (lz_maybe_zero<F, 8>(P)) {
    if (lz_is_zero<F>(P)) {
      if (lz_is_zero<F>(R)) xz_mdbl<C>(A, bx, by);
      else inf = true;
      return;
    }
  }
  const Lz<F> PP = lz_sqr<F>(P);
  const Lz<F> PPP = lz_mul<F>(P, PP);
  const Lz<F> Q = lz_mul<F>(A.X, PP);
  A.X = lz_carry<F>(lz_sub<F>(lz_sub<F>(lz_sqr<F>(R), PPP), lz_shl<F>(Q, 1)));
  A.Y = lz_mul2<F>(R, lz_sub<F>(Q, A.X), lz_neg<F>(A.Y), PPP);
  A.ZZ = lz_mul<F>(A.ZZ, PP);
  A.ZZZ = lz_mul<F>(A.ZZZ, PPP);
}

// ---- points in Jacobian coordinates ---------------------------------------------
// x = X / Z^2, y = Y / Z^3: where doublings outnumber additions.  A doubling
// takes 4 products, 4 squarings and 7 reductions (a = 0: 3, 4 and 6) against
// 7, 2 and 8 in XYZZ; a mixed addition one squaring and one reduction more.

template <class C>
struct Jz {
  Lz<typename C::F> X, Y, Z;
};

// dbl-2001-b (a = -3) and dbl-2009-l (a = 0) of the Explicit-Formulas
// Database, arranged so that Y3 = alpha (4 beta - X3) - 8 gamma^2 takes one
// reduction.  A point at infinity (kept as a flag beside the point) may be
// passed through: its coordinates stay within the bounds.
template <class C>
__device__ __forceinline__ void jz_dbl(Jz<C>& A) {
  using F = typename C::F;
  const Lz<F> G = lz_sqr<F>(A.Y);                       // gamma
  const Lz<F> V = lz_carry<F>(lz_shl<F>(G, 2));         // 4 gamma
  const Lz<F> S = lz_mul<F>(A.X, V);                    // 4 beta
  Lz<F> t;
  if constexpr (C::A_IS_MINUS3) {
    const Lz<F> D = lz_sqr<F>(A.Z);
    t = lz_mul<F>(lz_sub<F>(A.X, D), lz_add<F>(A.X, D));
  } else {
    t = lz_sqr<F>(A.X);
  }
  const Lz<F> M = lz_carry<F>(lz_add<F>(lz_shl<F>(t, 1), t));  // alpha
  A.Z = lz_mul<F>(lz_shl<F>(A.Y, 1), A.Z);
  A.X = lz_carry<F>(lz_sub<F>(lz_sqr<F>(M), lz_shl<F>(S, 1)));
  A.Y = lz_mul2<F>(M, lz_sub<F>(S, A.X), V, lz_neg<F>(lz_carry_if29<F>(lz_shl<F>(G, 1))));
}

// 2 (x, y) of an affine point
template <class C>
__device__ __forceinline__ void jz_mdbl(Jz<C>& A, const Lz<typename C::F>& x, const Lz<typename C::F>& y) {
  A.X = x;
  A.Y = y;
  A.Z = lz_one<typename C::F>();
  jz_dbl<C>(A);
}

// A += (bx, by), every case; operands as for xz_madd
template <class C>
__device__ __forceinline__ void jz_madd(Jz<C>& A, bool& inf, const Lz<typename C::F>& bx,
                                        const Lz<typename C::F>& by) {
  using F = typename C::F;
  if (inf) {
    A.X = bx;
    A.Y = by;
    A.Z = lz_one<F>();
    inf = false;
    return;
  }
  const Lz<F> ZZ = lz_sqr<F>(A.Z);
  const Lz<F> H = lz_sub<F>(lz_mul<F>(bx, ZZ), A.X);
  const Lz<F> R = lz_sub<F>(lz_mul<F>(by, lz_mul<F>(A.Z, ZZ)), A.Y);
  if (lz_maybe_zero<F, 8>(H)) {
    if (lz_is_zero<F>(H)) {
      if (lz_is_zero<F>(R)) jz_mdbl<C>(A, bx, by);
      else inf = true;
      return;
    }
  }
  const Lz<F> HH = lz_sqr<F>(H);
  const Lz<F> HHH = lz_mul<F>(H, HH);
  const Lz<F> V = lz_mul<F>(A.X, HH);
  A.X = lz_carry<F>(lz_sub<F>(lz_sub<F>(lz_sqr<F>(R), HHH), lz_shl<F>(V, 1)));
  A.Y = lz_mul2<F>(R, lz_sub<F>(V, A.X), lz_neg<F>(A.Y), HHH);
  A.Z = lz_mul<F>(A.Z, H);
}

}  // namespace eccmi

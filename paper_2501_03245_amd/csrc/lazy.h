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
// Bounds, with rho = R / p (BN254: 169,
// BLS12-381: 2^11.3, the 256-bit ECDSA primes: 2^24).
//   lz_mul(a, b)      : value in (-e, 1 + e) p with e = |a b| / (rho p^2);
//                       limbs in [0, 2^B) below the signed top one;
//   columns           : NL max|a_i| max|b_j| (summed over the products that
//                       share a reduction) + NL 2^(2B) must stay below 2^63:
//                       with limbs counted in units of 2^B, the sum of the
//                       unit products plus one is at most 2^63 / (NL 2^(2B)),
//                       which is 3.5 for BN254 (9 limbs of 29 bits), 9.1 for
//                       BLS12-381 (14 of 28) and 12.8 for the 256-bit primes
//                       (10 of 28);
//   lz_carry(a)       : one parallel carry pass: limbs in [-k, 2^B + k) for
//                       limbs below k 2^B, the same value.
// The formulas state the values they keep: X in (-3.5, 1.2) p, Y, Z, ZZ, ZZZ
// product outputs in (-0.2, 1.2) p, but for the Y of a sum that a quad has not
// stored yet (quad.h), the difference of two, in (-1.1, 1.1) p.
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
    constexpr Digits<NL> sd = F::SD;
    int32_t dq[NL];
    sparse_digits<F>(dq);
#pragma unroll
    for (int k = 0; k < 2 * NL - 1; k++) {
      col(acc, k);
#pragma unroll
      for (int i = k < NL ? 0 : k - NL + 1; i < (k < NL ? k : NL); i++) {
        const int32_t d = sd.d[k - i];
        if (d > 0) acc += uint64_t(m[i]) * uint32_t(dq[k - i]);
        if (d < 0) acc += uint64_t(int64_t(int32_t(m[i])) * int64_t(dq[k - i]));
      }
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
      for (int i = k < NL ? 0 : k - NL + 1; i < (k < NL ? k : NL); i++) {
        acc += uint64_t(m[i]) * q[k - i];
      }
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
  for (int i = k < F::NL ? 0 : k - F::NL + 1; i < (k < F::NL ? k + 1 : F::NL); i++) {
    acc += uint64_t(int64_t(a.w[i]) * int64_t(b.w[k - i]));
  }
}

// column k of a^2, a2 = 2 a
template <class F>
__device__ __forceinline__ void lz_col_sqr(uint64_t& acc, const Lz<F>& a, const Lz<F>& a2, int k) {
#pragma unroll
  for (int i = k < F::NL ? 0 : k - F::NL + 1; 2 * i < k; i++) {
    acc += uint64_t(int64_t(a.w[i]) * int64_t(a2.w[k - i]));
  }
  if ((k & 1) == 0) {
    acc += uint64_t(int64_t(a.w[k / 2]) * int64_t(a.w[k / 2]));
  }
}

// Columns of products as lists of terms, so that two products can be taken
// term by term in turn.
template <class F>
struct ColMul {
  const Lz<F>&a, &b;
  static constexpr int len(int k) { return k < F::NL ? k + 1 : 2 * F::NL - 1 - k; }
  __device__ __forceinline__ void term(uint64_t& acc, int k, int s) const {
    const int i = (k < F::NL ? 0 : k - F::NL + 1) + s;
    acc += uint64_t(int64_t(a.w[i]) * int64_t(b.w[k - i]));
  }
};
template <class F>
struct ColSqr {
  const Lz<F>&a, &a2;
  static constexpr int len(int k) { return k < F::NL ? k / 2 + 1 : F::NL - (k + 1) / 2; }
  __device__ __forceinline__ void term(uint64_t& acc, int k, int s) const {
    const int i = (k < F::NL ? 0 : k - F::NL + 1) + s;
    acc += uint64_t(int64_t(a.w[i]) * int64_t((2 * i < k ? a2 : a).w[k - i]));
  }
};

// Two independent products, term by term and column by column together (the
// fence keeps the scheduler to a column).  A wave that has only one chain of
// multiply-adds to issue stalls on their latency between its neighbours'
// issues; two chains in turn cost 28 registers.  k_bucket_acc, BN254: 700001
// points 1.68 -> 1.56 ms a call; BLS12-381, 2^20 points: 3.57 -> 3.49 ms.
template <class F, class ColA, class ColB>
__device__ __forceinline__ void lz_pair(const ColA ca, const ColB cb, Lz<F>& ra, Lz<F>& rb) {
  constexpr int NL = F::NL;
  constexpr int B = F::B;
  uint32_t m[NL], n[NL];
  uint64_t acc = 0, bcc = 0;
  constexpr Words<NL> qc = F::P;
  constexpr Digits<NL> sd = F::SD;
  uint32_t q[NL], qinv = F::QINV;
  int32_t dq[NL];
  if constexpr (F::SPARSE) {
    sparse_digits<F>(dq);
  } else {
#pragma unroll
    for (int j = 0; j < NL; j++) {
      q[j] = qc.w[j];
      asm("" : "+s"(q[j]));
    }
    asm("" : "+s"(qinv));
  }
#pragma unroll
  for (int k = 0; k < 2 * NL - 1; k++) {
#pragma unroll
    for (int s = 0; s < (ColA::len(k) > ColB::len(k) ? ColA::len(k) : ColB::len(k)); s++) {
      if (s < ColA::len(k)) ca.term(acc, k, s);
      if (s < ColB::len(k)) cb.term(bcc, k, s);
    }
#pragma unroll
    for (int i = k < NL ? 0 : k - NL + 1; i < (k < NL ? k : NL); i++) {
      if constexpr (F::SPARSE) {
        const int32_t d = sd.d[k - i];
        if (d > 0) {
          acc += uint64_t(m[i]) * uint32_t(dq[k - i]);
          bcc += uint64_t(n[i]) * uint32_t(dq[k - i]);
        }
        if (d < 0) {
          acc += uint64_t(int64_t(int32_t(m[i])) * int64_t(dq[k - i]));
          bcc += uint64_t(int64_t(int32_t(n[i])) * int64_t(dq[k - i]));
        }
      } else {
        acc += uint64_t(m[i]) * q[k - i];
        bcc += uint64_t(n[i]) * q[k - i];
      }
    }
    if (k < NL) {
      m[k] = uint32_t(acc);
      n[k] = uint32_t(bcc);
      if constexpr (!F::SPARSE) {
        m[k] *= qinv;
        n[k] *= qinv;
      }
      m[k] &= F::MASK;
      n[k] &= F::MASK;
      if constexpr (!F::SPARSE) {  // clears the low B bits
        acc += uint64_t(m[k]) * q[0];
        bcc += uint64_t(n[k]) * q[0];
      }
    } else {
      ra.w[k - NL] = int32_t(uint32_t(acc) & F::MASK);
      rb.w[k - NL] = int32_t(uint32_t(bcc) & F::MASK);
    }
    acc = uint64_t(int64_t(acc) >> B);
    bcc = uint64_t(int64_t(bcc) >> B);
    __builtin_amdgcn_sched_barrier(0);
  }
  ra.w[NL - 1] = int32_t(uint32_t(acc));
  rb.w[NL - 1] = int32_t(uint32_t(bcc));
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

// madd-2008-s from P = U2 - X1 and R = S2 - Y1 on (P not 0 mod p)
template <class C>
__device__ __forceinline__ void xz_madd_tail(Xz<C>& A, const Lz<typename C::F>& P, const Lz<typename C::F>& R) {
  using F = typename C::F;
  const Lz<F> P2 = lz_shl<F>(P, 1), R2 = lz_shl<F>(R, 1);
  Lz<F> PP, RR, PPP, Q, ZZ, ZZZ;
  lz_pair<F>(ColSqr<F>{P, P2}, ColSqr<F>{R, R2}, PP, RR);
  lz_pair<F>(ColMul<F>{P, PP}, ColMul<F>{A.X, PP}, PPP, Q);
  A.X = lz_carry<F>(lz_sub<F>(lz_sub<F>(RR, PPP), lz_shl<F>(Q, 1)));
  lz_pair<F>(ColMul<F>{A.ZZ, PP}, ColMul<F>{A.ZZZ, PPP}, ZZ, ZZZ);
  A.ZZ = ZZ;
  A.ZZZ = ZZZ;
  A.Y = lz_mul2<F>(R, lz_sub<F>(Q, A.X), lz_neg<F>(A.Y), PPP);
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
  Lz<F> P, R;
  lz_pair<F>(ColMul<F>{bx, A.ZZ}, ColMul<F>{by, A.ZZZ}, P, R);
  P = lz_sub<F>(P, A.X);  // |P| < 5p
  R = lz_sub<F>(R, A.Y);  // |R| < 2.5p
  if (lz_maybe_zero<F, 8>(P)) {
    if (lz_is_zero<F>(P)) {
      if (lz_is_zero<F>(R)) xz_mdbl<C>(A, bx, by);
      else inf = true;
      return;
    }
  }
  xz_madd_tail<C>(A, P, R);
}

// dbl-2008-s-1, not for O
template <class C>
__device__ __forceinline__ void xz_dbl(Xz<C>& A) {
  using F = typename C::F;
  const Lz<F> U = lz_carry<F>(lz_shl<F>(A.Y, 1));
  const Lz<F> V = lz_sqr<F>(U);
  const Lz<F> W = lz_mul<F>(U, V);
  const Lz<F> S = lz_mul<F>(A.X, V);
  Lz<F> t;
  if constexpr (C::A_IS_MINUS3) t = lz_mul<F>(lz_sub<F>(A.X, A.ZZ), lz_add<F>(A.X, A.ZZ));
  else t = lz_sqr<F>(A.X);
  const Lz<F> M = lz_carry<F>(lz_add<F>(lz_add<F>(t, t), t));
  A.X = lz_carry<F>(lz_sub<F>(lz_sqr<F>(M), lz_shl<F>(S, 1)));
  A.Y = lz_mul2<F>(M, lz_sub<F>(S, A.X), lz_neg<F>(W), A.Y);
  A.ZZ = lz_mul<F>(V, A.ZZ);
  A.ZZZ = lz_mul<F>(W, A.ZZZ);
}

// add-2008-s: A += B, every case
template <class C>
__device__ __forceinline__ void xz_add(Xz<C>& A, bool& inf, const Xz<C>& B, bool binf) {
  using F = typename C::F;
  if (binf) return;
  if (inf) {
    A = B;
    inf = false;
    return;
  }
  const Lz<F> U1 = lz_mul<F>(A.X, B.ZZ);
  const Lz<F> P = lz_sub<F>(lz_mul<F>(B.X, A.ZZ), U1);
  if (lz_maybe_zero<F, 4>(P)) {
    if (lz_is_zero<F>(P)) {
      if (lz_is_zero<F>(lz_sub<F>(lz_mul<F>(B.Y, A.ZZZ), lz_mul<F>(A.Y, B.ZZZ)))) xz_dbl<C>(A);
      else inf = true;
      return;
    }
  }
  const Lz<F> S1 = lz_mul<F>(A.Y, B.ZZZ);
  const Lz<F> R = lz_sub<F>(lz_mul<F>(B.Y, A.ZZZ), S1);
  const Lz<F> PP = lz_sqr<F>(P);
  const Lz<F> PPP = lz_mul<F>(P, PP);
  const Lz<F> Q = lz_mul<F>(U1, PP);
  A.ZZ = lz_mul<F>(lz_mul<F>(A.ZZ, B.ZZ), PP);
  A.ZZZ = lz_mul<F>(lz_mul<F>(A.ZZZ, B.ZZZ), PPP);
  A.X = lz_carry<F>(lz_sub<F>(lz_sub<F>(lz_sqr<F>(R), PPP), lz_shl<F>(Q, 1)));
  A.Y = lz_mul2<F>(R, lz_sub<F>(Q, A.X), lz_neg<F>(S1), PPP);
}

template <class F>
__device__ __forceinline__ Lz<F> lz_load(const uint32_t* __restrict__ p) {
  return lz_of<F>(fp_load<F>(p));
}

template <class F>
__device__ __forceinline__ void lz_store(uint32_t* __restrict__ p, const Lz<F>& a) {
  Fp<F> r;
#pragma unroll
  for (int i = 0; i < F::NL; i++) r.w[i] = uint32_t(a.w[i]);
  fp_store<F>(p, r);
}

// a stored point: X, Y, ZZ, ZZZ of CW words each; O has a negative lowest limb
// of X, which no other stored X has (a coordinate of a base, or a carried one)
template <class C>
__device__ __forceinline__ void xz_store(uint32_t* __restrict__ p, const Xz<C>& A, bool inf) {
  using F = typename C::F;
  constexpr int CW = F::CW;
  Lz<F> X = A.X;
  if (inf) X.w[0] = -1;
  lz_store<F>(p, X);
  lz_store<F>(p + CW, A.Y);
  lz_store<F>(p + 2 * CW, A.ZZ);
  lz_store<F>(p + 3 * CW, A.ZZZ);
}

template <class C>
__device__ __forceinline__ void xz_load(const uint32_t* __restrict__ p, Xz<C>& A, bool& inf) {
  using F = typename C::F;
  constexpr int CW = F::CW;
  A.X = lz_load<F>(p);
  A.Y = lz_load<F>(p + CW);
  A.ZZ = lz_load<F>(p + 2 * CW);
  A.ZZZ = lz_load<F>(p + 3 * CW);
  inf = A.X.w[0] < 0;
}

// the point in the semi-reduced form of point.h (O: ZZ = 0)
template <class C>
__device__ __forceinline__ XYZZ<C> xz_to_xyzz(const Xz<C>& A, bool inf) {
  using F = typename C::F;
  if (inf) return xyzz_inf<C>();
  XYZZ<C> r;
  r.X = lz_semi<F>(lz_mul<F>(A.X, lz_one<F>()));  // back into (-p, 2p)
  r.Y = lz_semi<F>(A.Y);
  r.ZZ = lz_semi<F>(A.ZZ);
  r.ZZZ = lz_semi<F>(A.ZZZ);
  return r;
}

template <class C, class Fn>
__device__ __forceinline__ void xz_map(Xz<C>& r, const Xz<C>& A, Fn fn) {
#pragma unroll
  for (int i = 0; i < C::F::NL; i++) {
    r.X.w[i] = fn(A.X.w[i]);
    r.Y.w[i] = fn(A.Y.w[i]);
    r.ZZ.w[i] = fn(A.ZZ.w[i]);
    r.ZZZ.w[i] = fn(A.ZZZ.w[i]);
  }
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

// Batched ECDSA verification and signing on secp256r1 and SM2, and batched
// unknown-point multiplication on every curve.
//
// Per request: valid iff 1 <= r, s < n, Q is a curve point other than O, and
// with w = s^-1, u1 = e w, u2 = r w (mod n), R = u1 G + u2 Q is not O and
// R.x mod n = r.  The paper counts a verification as one fixed-point and one
// unknown-point multiplication (Section 5.2).  Two kernels compute it: the
// per-lane form at the end of this file, and first the paper's batched
// affine form, where both multiplications run in one loop over the scalar
// bits from the least significant end, as in its batch PMUL (Section 3.4,
// Algorithm 3):
//
//   step j:  A1 <- A1 + 2^j G   if bit j of u1     (fixed point, table)
//            A2 <- A2 + P       if bit j of u2     (unknown point)
//            P  <- 2 P                              (P = 2^j Q)
//
// All three are affine operations whose denominators go into one
// Montgomery-trick chain per lane, inverted once per step for the whole
// workgroup (Gather-Apply-Scatter, Section 3.2).  The inverse of s mod n is
// batched the same way in F_n.  Finally R = A1 + A2 is one more batched step.
// One request per lane; lanes past the end run dummy requests so that every
// lane reaches every workgroup barrier.
#pragma once
#include "kernels.h"
#include "lazy.h"
#include "quad.h"

namespace eccmi {

enum : int { OP_NOP = 5 };  // alongside CLS_ADD .. CLS_COPY2

template <class C>
struct AffOp {
  int cls;
  Fp<typename C::F> d;  // denominator put into the chain (1 when none is needed)
};

// affine A + B with A, B canonical (infinity flags ia, ib)
template <class C>
__device__ __forceinline__ AffOp<C> plan_add(const Affine<C>& A, bool ia, const Affine<C>& B, bool ib) {
  using F = typename C::F;
  AffOp<C> op;
  op.d = fp_one<F>();
  if (ia && ib) {
    op.cls = CLS_INF;
  } else if (ia) {
    op.cls = CLS_COPY2;
  } else if (ib) {
    op.cls = CLS_COPY1;
  } else if (fp_eq_canonical<F>(A.x, B.x)) {
    if (fp_eq_canonical<F>(A.y, B.y)) {
      op.cls = CLS_DBL;  // y != 0: these curves have no point of order 2
      op.d = fp_dbl<F>(A.y);
    } else {
      op.cls = CLS_INF;
    }
  } else {
    op.cls = CLS_ADD;
    op.d = fp_sub<F>(B.x, A.x);  // normalised: two denominators are multiplied together
  }
  return op;
}

// result of a planned addition given inv = 1 / op.d; canonical output
template <class C>
__device__ __forceinline__ void apply_add(const AffOp<C>& op, const Affine<C>& A, bool ia, const Affine<C>& B, bool ib,
                                          const Fp<typename C::F>& inv, Affine<C>& R, bool& rinf) {
  using F = typename C::F;
  if (op.cls == OP_NOP) {
    R = A;
    rinf = ia;
    return;
  }
  if (op.cls == CLS_INF) {
    rinf = true;
    R = A;
    return;
  }
  if (op.cls == CLS_COPY1) {
    R = A;
    rinf = false;
    return;
  }
  if (op.cls == CLS_COPY2) {
    R = B;
    rinf = false;
    return;
  }
  Fp<F> num = op.cls == CLS_DBL ? tangent_numerator<C>(A.x, fp_one<F>()) : fp_sub_lazy<F>(B.y, A.y);
  Fp<F> lam = fp_mul<F>(num, inv);
  Fp<F> x3 = fp_canonical<F>(fp_sub<F>(fp_sub<F>(fp_sqr<F>(lam), A.x), B.x));
  Fp<F> y3 = fp_canonical<F>(fp_sub<F>(fp_mul<F>(lam, fp_sub_lazy<F>(A.x, x3)), A.y));
  R.x = x3;
  R.y = y3;
  rinf = false;
}

template <class F>
__device__ __forceinline__ bool words_eq8(const uint32_t (&a)[8], const uint32_t (&b)[8]) {
  uint32_t d = 0;
#pragma unroll
  for (int k = 0; k < 8; k++) d |= a[k] ^ b[k];
  return d == 0;
}

// a < b for 8-word little-endian integers
__device__ __forceinline__ bool words_lt8(const uint32_t (&a)[8], const uint32_t (&b)[8]) {
  bool lt = false, decided = false;
#pragma unroll
  for (int k = 7; k >= 0; k--) {
    if (!decided && a[k] != b[k]) {
      lt = a[k] < b[k];
      decided = true;
    }
  }
  return lt;
}

__device__ __forceinline__ bool words_zero8(const uint32_t (&a)[8]) {
  uint32_t o = 0;
#pragma unroll
  for (int k = 0; k < 8; k++) o |= a[k];
  return o == 0;
}

// Loads request i, checks ranges and the public key, and computes
// w = s^-1 (one GAS inversion in F_n for the workgroup), u1 = e w and
// u2 = r w.  Dead or invalid requests continue with dummy values (r = s = 1,
// Q = G) so that every lane reaches every barrier; ok says which are real.
template <class C, int WG>
__device__ __forceinline__ void verify_prologue(const uint8_t* __restrict__ hashes,
                                                const uint32_t* __restrict__ pubkeys,
                                                const uint32_t* __restrict__ sigs, size_t i, bool live,
                                                Fp<typename OrderField<C>::type>* n_tot,
                                                Fp<typename OrderField<C>::type>* n_inv, uint32_t (&rw)[8],
                                                uint32_t (&u1)[8], uint32_t (&u2)[8], Affine<C>& Q, bool& ok) {
  using F = typename C::F;
  using N = typename OrderField<C>::type;
  uint32_t sw[8], ew[8], qx[8], qy[8];
  constexpr Words<8> n32 = N::P32;
  constexpr Words<8> p32 = F::P32;
  ok = live;
  if (live) {
    words_load<F>(sigs + i * 16, rw);
    words_load<F>(sigs + i * 16 + 8, sw);
    words_load<F>(pubkeys + i * 16, qx);
    words_load<F>(pubkeys + i * 16 + 8, qy);
    const uint8_t* h = hashes + i * 32;
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const uint8_t* b = h + 28 - 4 * k;  // big-endian bytes, least significant word last
      ew[k] = (uint32_t(b[0]) << 24) | (uint32_t(b[1]) << 16) | (uint32_t(b[2]) << 8) | uint32_t(b[3]);
    }
    ok = !words_zero8(rw) && words_lt8(rw, n32.w) && !words_zero8(sw) && words_lt8(sw, n32.w) &&
         words_lt8(qx, p32.w) && words_lt8(qy, p32.w) && !(words_zero8(qx) && words_zero8(qy));
  }
  if (ok) {
    Q.x = fp_canonical<F>(fp_to_mont<F>(fp_from_words<F>(qx)));
    Q.y = fp_canonical<F>(fp_to_mont<F>(fp_from_words<F>(qy)));
    ok = affine_on_curve<C>(Q);
  }
  if (!ok) {
#pragma unroll
    for (int k = 0; k < 8; k++) rw[k] = sw[k] = ew[k] = 0;
    rw[0] = sw[0] = 1;
    constexpr Words<F::NL> gx = C::GX, gy = C::GY;
    Q.x = fp_from<F>(gx);
    Q.y = fp_from<F>(gy);
  }
  Fp<N> wm = wg_batch_inverse<N, WG, 3>(fp_to_mont<N>(fp_from_words<N>(sw)), n_tot, n_inv);
  fp_to_words<N>(fp_from_mont<N>(fp_mul<N>(fp_to_mont<N>(fp_from_words<N>(ew)), wm)), u1);
  fp_to_words<N>(fp_from_mont<N>(fp_mul<N>(fp_to_mont<N>(fp_from_words<N>(rw)), wm)), u2);
}

template <class C, int WG>
__global__ void __launch_bounds__(WG) k_verify(const uint8_t* __restrict__ hashes, const uint32_t* __restrict__ pubkeys,
                                               const uint32_t* __restrict__ sigs, size_t m,
                                               const uint32_t* __restrict__ gtab, uint8_t* __restrict__ valid) {
  using F = typename C::F;
  using N = typename OrderField<C>::type;
  constexpr int PW = affine_words<C>();
  __shared__ Fp<F> s_tot[WG / 64], s_inv[WG / 64];
  __shared__ Fp<N> n_tot[WG / 64], n_inv[WG / 64];
  const size_t i = size_t(blockIdx.x) * WG + threadIdx.x;
  const bool live = i < m;
  constexpr Words<8> n32 = N::P32;
  uint32_t rw[8], u1[8], u2[8];
  Affine<C> Q;
  bool ok;
  verify_prologue<C, WG>(hashes, pubkeys, sigs, i, live, n_tot, n_inv, rw, u1, u2, Q, ok);

  // ---- the bit loop ----
  Affine<C> A1, A2, P = Q;
  bool i1 = true, i2 = true;
  A1.x = A1.y = A2.x = A2.y = fp_zero<F>();
  for (int j = 0; j < 256; j++) {
    const bool b1 = (u1[j >> 5] >> (j & 31)) & 1u;
    const bool b2 = (u2[j >> 5] >> (j & 31)) & 1u;
    const Affine<C> Gj = affine_load<C>(gtab + size_t(j) * PW);
    AffOp<C> oa, ob, oc;
    if (b1) {
      oa = plan_add<C>(A1, i1, Gj, false);
    } else {
      oa.cls = OP_NOP;
      oa.d = fp_one<F>();
    }
    if (b2) {
      ob = plan_add<C>(A2, i2, P, false);
    } else {
      ob.cls = OP_NOP;
      ob.d = fp_one<F>();
    }
    oc.cls = CLS_DBL;
    oc.d = fp_dbl<F>(P.y);
    const Fp<F> dab = fp_mul<F>(oa.d, ob.d);
    Fp<F> inv = wg_batch_inverse<F, WG, 4>(fp_mul<F>(dab, oc.d), s_tot, s_inv);
    const Fp<F> inv_c = fp_mul<F>(inv, dab);
    const Fp<F> inv_ab = fp_mul<F>(inv, oc.d);
    const Fp<F> inv_b = fp_mul<F>(inv_ab, oa.d);
    const Fp<F> inv_a = fp_mul<F>(inv_ab, ob.d);
    Affine<C> t;
    bool tinf;
    apply_add<C>(oa, A1, i1, Gj, false, inv_a, t, tinf);
    A1 = t;
    i1 = tinf;
    apply_add<C>(ob, A2, i2, P, false, inv_b, t, tinf);
    A2 = t;
    i2 = tinf;
    apply_add<C>(oc, P, false, P, false, inv_c, t, tinf);
    P = t;
  }
  // ---- R = A1 + A2 ----
  AffOp<C> of = plan_add<C>(A1, i1, A2, i2);
  Fp<F> inv = wg_batch_inverse<F, WG, 4>(of.d, s_tot, s_inv);
  Affine<C> R;
  bool rinf;
  apply_add<C>(of, A1, i1, A2, i2, inv, R, rinf);

  // ---- R.x mod n == r: R.x is below p < 2n, so R.x = r or R.x = r + n ----
  if (live) {
    bool good = ok && !rinf;
    if (good) {
      uint32_t xw[8];
      fp_to_words<F>(fp_from_mont<F>(R.x), xw);
      uint32_t rn[8];
      uint64_t cy = 0;
#pragma unroll
      for (int k = 0; k < 8; k++) {
        uint64_t v = uint64_t(rw[k]) + n32.w[k] + cy;
        rn[k] = uint32_t(v);
        cy = v >> 32;
      }
      good = words_eq8<F>(xw, rw) || (cy == 0 && words_eq8<F>(xw, rn));
    }
    valid[i] = good ? 1 : 0;
  }
}

// ---- latency form: one request per lane --------------------------------------
//
// The loop above inverts once per scalar bit for the whole workgroup, so a
// launch costs 257 inversion latencies however few requests it holds.  This
// form keeps each request's sum on its own lane in projective coordinates
// and inverts twice per launch (s mod n, and the table below):
//   u2 Q: signed 4-bit windows from the most significant end, four Jacobian
//         doublings and one mixed addition of +-T[|d|] = +-|d| Q per window;
//         T[2..8] are made on the lane and normalised to affine with one
//         Montgomery-trick chain and one Gather-Apply-Scatter inversion;
//   u1 G: one mixed XYZZ addition per signed digit of u1, of +-|d| 2^(w j) G
//         from a comb table made once per context (below);
//   R.x mod n = r without an inversion: x = X / ZZ, so the test is X = r ZZ,
//         or X = (r + n) ZZ when r + n < p.
//
// Bound by the instruction stream (one product of the 256-bit primes takes
// about 190 instructions, and one wave per SIMD already issues at 85% of the
// peak).  Signed lazy limbs (lazy.h) take the carries, comparisons and
// multiples of p out of every modular sum; Jacobian doublings take 4 products
// and 4 squarings in 7 reductions where XYZZ takes 7, 2 and 8 (252 of them
// per product); eight signed table entries cost 7 fewer table points than
// fifteen unsigned ones at the same number of windows.  Five-bit windows
// would save ten additions and cost eight more table points, at 17 products
// each: more than they save.
// Measured (one call, unsigned limbs with fifteen-entry tables before): 2^19
// SM2 products 14.36 -> 9.33 ms, 3001 BN254 products 1.78 -> 1.14 ms, 2^16 SM2
// verifications 1.84 -> 1.52 ms, 2^18 SM2 signatures 0.695 -> 0.614 ms, 2^19
// SM2 fixed-point products 1.20 -> 1.00 ms.  Two waves on each SIMD (at most 256
// registers, 2^17 requests a launch) instead of one: 2^19 SM2 products 9.65 ->
// 8.49 ms; three waves take 9.77 ms (spilled registers), and so would two on
// BLS12-381, which keeps one.

constexpr int VT_N = 8;             // table entries d Q, d = 1..8

// words per table entry: X, Y, Z, the chain prefix and a flag word, rounded up
// to whole 16-byte groups
template <class F>
constexpr int vt_slot() {
  return (4 * F::NL + 1 + 3) / 4 * 4;
}

// every access to a table slot is a 16-byte vector access (one access type
// for the whole scratch area)
template <int K>
__device__ __forceinline__ void vt_store(uint32_t* __restrict__ s, const uint32_t (&w)[K]) {
  static_assert(K % 4 == 0, "whole 16-byte groups");
  uint4* v = reinterpret_cast<uint4*>(s);
#pragma unroll
  for (int k = 0; k < K / 4; k++) v[k] = make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
}

template <int K>
__device__ __forceinline__ void vt_load(const uint32_t* __restrict__ s, uint32_t (&w)[K]) {
  static_assert(K % 4 == 0, "whole 16-byte groups");
  const uint4* v = reinterpret_cast<const uint4*>(s);
#pragma unroll
  for (int k = 0; k < K / 4; k++) {
    const uint4 t = v[k];
    w[4 * k] = t.x;
    w[4 * k + 1] = t.y;
    w[4 * k + 2] = t.z;
    w[4 * k + 3] = t.w;
  }
}

template <class F>
__device__ __forceinline__ void vt_pack(uint32_t* __restrict__ w, const Lz<F>& a) {
#pragma unroll
  for (int k = 0; k < F::NL; k++) w[k] = uint32_t(a.w[k]);
}

template <class F>
__device__ __forceinline__ Lz<F> vt_unpack(const uint32_t* __restrict__ w) {
  Lz<F> a;
#pragma unroll
  for (int k = 0; k < F::NL; k++) a.w[k] = int32_t(w[k]);
  return a;
}

// an affine entry: x and y in the first 2 NL words of its slot, written and
// read as whole 16-byte groups
template <class F>
constexpr int vt_affine_words() {
  return (2 * F::NL + 3) / 4 * 4;
}

template <class C>
__device__ __forceinline__ void vt_put_affine(uint32_t* __restrict__ s, const Lz<typename C::F>& x,
                                              const Lz<typename C::F>& y) {
  constexpr int NL = C::F::NL;
  uint32_t w[vt_affine_words<typename C::F>()] = {};
  vt_pack<typename C::F>(w, x);
  vt_pack<typename C::F>(w + NL, y);
  vt_store(s, w);
}

// an affine point as lazy coordinates; x.w[0] < 0 marks O
template <class C>
struct LzAffine {
  Lz<typename C::F> x, y;
};

template <class C>
__device__ __forceinline__ LzAffine<C> vt_get_affine(const uint32_t* __restrict__ s) {
  using F = typename C::F;
  uint32_t w[vt_affine_words<F>()];
  vt_load(s, w);
  LzAffine<C> a;
  a.x = vt_unpack<F>(w);
  a.y = vt_unpack<F>(w + F::NL);
  return a;
}

// the top S bits of a 256-bit value, which is then shifted left by S (the
// digits are read by shifting, so that no register array is indexed at run
// time: such an array would be placed in scratch or LDS memory)
template <int S>
__device__ __forceinline__ uint32_t take_top(uint32_t (&a)[8]) {
  const uint32_t d = a[7] >> (32 - S);
#pragma unroll
  for (int k = 7; k > 0; k--) a[k] = (a[k] << S) | (a[k - 1] >> (32 - S));
  a[0] <<= S;
  return d;
}

// This lane's table T[d] = d Q (d = 1..VT_N) as affine entries: made in
// Jacobian coordinates, then normalised with one Montgomery-trick chain over
// the Z and one Gather-Apply-Scatter inversion for the workgroup (every lane
// must call it).  An entry that is O (Q of order at most 8, possible only off the
// prime-order subgroup) puts 1 into the chain and is stored as the infinity
// marker, which the mixed addition skips.  Q itself must not be O.
template <class C, int WG>
__device__ __forceinline__ void vt_build(uint32_t* __restrict__ tab, const Affine<C>& Q, Fp<typename C::F>* s_tot,
                                         Fp<typename C::F>* s_inv) {
  using F = typename C::F;
  constexpr int NL = F::NL;
  constexpr int SLOT = vt_slot<F>();
  static_assert(vt_affine_words<F>() <= SLOT, "affine entry inside its slot");
  const Lz<F> qx = lz_of<F>(Q.x), qy = lz_of<F>(Q.y);
  Jz<C> T;
  jz_mdbl<C>(T, qx, qy);  // no curve here has a point of order 2
  bool inf = false;
  Lz<F> pref = lz_one<F>();
#pragma unroll 1
  for (int d = 2; d <= VT_N; d++) {
    const Lz<F> z = lz_select<F>(inf, lz_one<F>(), T.Z);
    uint32_t w[SLOT] = {};
    vt_pack<F>(w, T.X);
    vt_pack<F>(w + NL, T.Y);
    vt_pack<F>(w + 2 * NL, z);
    vt_pack<F>(w + 3 * NL, pref);
    w[4 * NL] = inf ? 1u : 0u;
    vt_store(tab + (d - 1) * SLOT, w);
    pref = lz_mul<F>(pref, z);
    if (d < VT_N) jz_madd<C>(T, inf, qx, qy);
  }
  Lz<F> inv = lz_of<F>(wg_batch_inverse<F, WG, 4>(lz_semi<F>(pref), s_tot, s_inv));
#pragma unroll 1
  for (int d = VT_N; d >= 2; d--) {
    uint32_t* sl = tab + (d - 1) * SLOT;
    uint32_t w[SLOT];
    vt_load(sl, w);
    const Lz<F> iz = lz_mul<F>(inv, vt_unpack<F>(w + 3 * NL));  // 1 / Z_d
    inv = lz_mul<F>(inv, vt_unpack<F>(w + 2 * NL));             // 1 / (Z_2 ... Z_(d-1))
    const Lz<F> iz2 = lz_sqr<F>(iz);
    Lz<F> x = lz_mul<F>(vt_unpack<F>(w), iz2);
    const Lz<F> y = lz_mul<F>(vt_unpack<F>(w + NL), lz_mul<F>(iz, iz2));
    if (w[4 * NL]) x = lz_of<F>(fp_inf_marker<F>());
    vt_put_affine<C>(sl, x, y);
  }
  vt_put_affine<C>(tab, qx, qy);
}

// u + sum over j of 8 16^j (256 bits): nibble j of the result minus 8 is
// signed digit j, in [-8, 7], and the carry out is digit 64 (0 or 1)
__device__ __forceinline__ bool signed_nibbles(uint32_t (&u)[8]) {
  uint64_t cy = 0;
#pragma unroll
  for (int k = 0; k < 8; k++) {
    cy += uint64_t(u[k]) + 0x88888888u;
    u[k] = uint32_t(cy);
    cy >>= 32;
  }
  return cy != 0;
}

// A += d Q (d in [-8, 7]) from this lane's table
template <class C>
__device__ __forceinline__ void vt_add_digit(Jz<C>& A, bool& inf, const uint32_t* __restrict__ tab, int d) {
  using F = typename C::F;
  if (d == 0) return;
  const LzAffine<C> T = vt_get_affine<C>(tab + ((d < 0 ? -d : d) - 1) * vt_slot<F>());
  if (T.x.w[0] >= 0) jz_madd<C>(A, inf, T.x, lz_neg_if<F>(T.y, d < 0));
}

// u Q from this lane's table (Q at tab): four doublings and one mixed
// addition per signed digit from the most significant end; u (256 bits) is
// consumed.  While the sum is O the doublings run on Q, unused.
template <class C>
__device__ __forceinline__ void vt_mul(Jz<C>& A, bool& inf, const uint32_t* __restrict__ tab, uint32_t (&u)[8]) {
  using F = typename C::F;
  inf = !signed_nibbles(u);
  const LzAffine<C> Q = vt_get_affine<C>(tab);
  A.X = Q.x;
  A.Y = Q.y;
  A.Z = lz_one<F>();
#pragma unroll 1
  for (int w = 63; w >= 0; w--) {
#pragma unroll 1
    for (int k = 0; k < 4; k++) jz_dbl<C>(A);
    vt_add_digit<C>(A, inf, tab, int(take_top<4>(u)) - 8);
  }
}

// ---- comb tables of the generator ---------------------------------------------
//
// Entry (j, d), d = 1 .. 2^(W-1), at j 2^(W-1) + d - 1: d 2^(W j) G, affine in
// the working form.  Any 256-bit k is the sum over the windows j of
// (f_j - 2^(W-1)) 2^(W j), f_j the W-bit fields of k + sum_j 2^(W j + W - 1).
//
// Two widths.  W = 13: 20 additions, 81,920 points (7.9 MB for the 256-bit
// primes, which passes through the 4 MB L2s but stays in the 256 MB cache
// behind them).  W = 9: 29 additions, 7,424 points (0.7 MB), where device
// memory is capped or fixed.  Unsigned bytes, the earlier form, took 32
// additions of 8,192 points; W = 8 takes 33 of 4,224, and was slower than they
// were (2^19 BLS12-381 fixed-point products 2.88 -> 3.02 ms; 2.61 with 9).  An entry is loaded while the addition of the
// window before it runs, since a gather costs about as long as half an
// addition.
// Measured against the unsigned bytes: 2^19 SM2 fixed-point products 0.97 ->
// 0.66 ms, 2^18 SM2 signatures 0.60 -> 0.45 ms, 2^16 SM2 verifications 1.51 ->
// 1.46 ms (W = 13).
constexpr int COMB_WIDE = 13;
constexpr int COMB_NARROW = 9;
template <int W>
constexpr int comb_windows() {
  return (257 + W - 1) / W;
}
template <int W>
constexpr size_t comb_entries() {
  return size_t(comb_windows<W>()) << (W - 1);
}

// k + sum_j 2^(W j + W - 1) over the windows, 288 bits
template <int W>
__device__ __forceinline__ void comb_fields(const uint32_t (&k)[8], uint32_t (&f)[9]) {
  constexpr Words<9> bias = [] {
    Words<9> b{};
    for (int j = 0; j < comb_windows<W>(); j++) b.w[(W * j + W - 1) / 32] |= 1u << ((W * j + W - 1) % 32);
    return b;
  }();
  uint64_t cy = 0;
#pragma unroll
  for (int i = 0; i < 9; i++) {
    cy += uint64_t(i < 8 ? k[i] : 0u) + bias.w[i];
    f[i] = uint32_t(cy);
    cy >>= 32;
  }
}

// A += k G: the windows first, first + stride, ... of k (all of them with
// first = 0, stride = 1)
template <class C, int W>
__device__ __forceinline__ void comb_add(Xz<C>& A, bool& inf, const uint32_t* __restrict__ gcomb,
                                         const uint32_t (&k)[8], int first = 0, int stride = 1) {
  using F = typename C::F;
  constexpr int PW = affine_words<C>();
  constexpr int D = 1 << (W - 1);
  uint32_t f[9];
  comb_fields<W>(k, f);
  // the field of the window at hand stays at the bottom of f (read by
  // shifting, so that no register array is indexed at run time)
  auto shift = [&](int windows) __attribute__((always_inline)) {
    for (int w = 0; w < windows; w++) {
#pragma unroll
      for (int i = 0; i < 8; i++) f[i] = (f[i] >> W) | (f[i + 1] << (32 - W));
      f[8] >>= W;
    }
  };
  auto digit = [&]() __attribute__((always_inline)) { return int(f[0] & uint32_t(2 * D - 1)) - D; };
  auto load = [&](int j, int d) __attribute__((always_inline)) {
    const int e = (d < 0 ? -d : d) - (d != 0);  // a zero digit reads entry 1, unused
    return affine_load<C>(gcomb + (size_t(j) * D + e) * PW);
  };
  shift(first);
  int d = digit();
  Affine<C> T = load(first, d);
#pragma unroll 1
  for (int j = first; j < comb_windows<W>(); j += stride) {
    const Lz<F> x = lz_of<F>(T.x), y = lz_neg_if<F>(lz_of<F>(T.y), d < 0);
    const bool add = d != 0;
    if (j + stride < comb_windows<W>()) {
      shift(stride);
      d = digit();
      T = load(j + stride, d);
    }
    if (add) xz_madd<C>(A, inf, x, y);
  }
}

// the table: one entry per lane, the bits of d from the most significant end
// (double-and-add of G), then the W j doublings
template <class C, int W, int WG>
__global__ void __launch_bounds__(WG) k_comb_build(uint32_t* __restrict__ gcomb) {
  using F = typename C::F;
  constexpr size_t NE = comb_entries<W>();
  __shared__ Fp<F> s_tot[WG / 64], s_inv[WG / 64];
  const size_t e = size_t(blockIdx.x) * WG + threadIdx.x;
  const bool live = e < NE;
  const uint32_t d = live ? uint32_t(e & ((size_t(1) << (W - 1)) - 1)) + 1u : 1u;
  const int dbls = live ? int(e >> (W - 1)) * W : 0;
  constexpr Words<F::NL> gx = C::GX, gy = C::GY;
  const Lz<F> x = lz_of<F>(fp_from<F>(gx)), y = lz_of<F>(fp_from<F>(gy));
  Jz<C> A;
  A.X = x;
  A.Y = y;
  A.Z = lz_one<F>();
  bool inf = true;
  int left = W + dbls;  // steps: W of double-and-add, then doublings
  uint32_t bits = d << (32 - W);
#pragma unroll 1
  for (; left > 0; left--) {
    jz_dbl<C>(A);
    if (left > dbls) {
      if (bits >> 31) jz_madd<C>(A, inf, x, y);
      bits <<= 1;
    }
  }
  const Lz<F> iz = lz_of<F>(wg_batch_inverse<F, WG>(lz_semi<F>(A.Z), s_tot, s_inv));
  const Lz<F> iz2 = lz_sqr<F>(iz);
  Affine<C> R;
  R.x = lz_canonical<F>(lz_mul<F>(A.X, iz2));
  R.y = lz_canonical<F>(lz_mul<F>(A.Y, lz_mul<F>(iz, iz2)));
  if (live) affine_store<C>(gcomb + e * affine_words<C>(), R);
}

// The affine form (x, y) of a projective point, given lazily, at out as x then
// y (N32 words each), plain or (out_mont) times R' = 2^(32 N32); O as zeros
template <class C>
__device__ __forceinline__ void store_lz_affine(const Lz<typename C::F>& x, const Lz<typename C::F>& y, bool inf,
                                                bool active, uint32_t* __restrict__ out, int out_mont) {
  using F = typename C::F;
  constexpr int N32 = F::N32;
  constexpr Words<F::NL> rout = F::ROUT;
  Lz<F> k = lz_zero<F>();
  k.w[0] = 1;
  // Montgomery product with 1 leaves x; with R' = 2^(32 N32) leaves x R'
  if (out_mont) k = lz_of<F>(fp_from<F>(rout));
  uint32_t xw[N32], yw[N32];
  fp_to_words<F>(lz_canonical<F>(lz_mul<F>(x, k)), xw);
  fp_to_words<F>(lz_canonical<F>(lz_mul<F>(y, k)), yw);
  if (inf) {
#pragma unroll
    for (int j = 0; j < N32; j++) xw[j] = yw[j] = 0;
  }
  if (active) {
    words_store<F>(out, xw);
    words_store<F>(out + N32, yw);
  }
}

// ---- the endomorphism split of one product ---------------------------------------
// On a curve whose every point is in the order-r subgroup (BN254: cofactor 1)
// k P = k1 P + k2 phi(P) with half-length k1, k2 (the split of the MSMs), which
// halves the doublings: 3001 products 1.14 -> 0.86 ms.  BLS12-381 has points
// outside the subgroup, which this call accepts, so it keeps the full scalar.
template <class C>
constexpr bool vt_glv() {
  return C::ID == BN254::ID;
}

// k mod r for any 256-bit k (2^256 < 6 r on BN254)
template <class C>
__device__ __forceinline__ void reduce_order(uint32_t (&k)[8]) {
  constexpr Words<8> r = C::ORDER;
#pragma unroll 1
  for (int t = 0; t < 5; t++) {
    if (words_lt8(k, r.w)) break;
    int64_t br = 0;
#pragma unroll
    for (int i = 0; i < 8; i++) {
      br += int64_t(k[i]) - int64_t(r.w[i]);
      k[i] = uint32_t(br);
      br >>= 32;
    }
  }
}

// k -> the signed nibbles of |k1| (in k) and |k2|, 32 of them in words 4..7,
// and the halves' signs
template <class C>
__device__ __forceinline__ void vt_split(uint32_t (&k)[8], uint32_t (&m2)[8], bool& n1, bool& n2) {
  static_assert(Glv<C>::BITS <= 126, "the signed nibbles of a half end in 128 bits");
  reduce_order<C>(k);
  uint32_t m1[8];
  glv_split<C>(k, m1, n1, m2, n2);  // |halves| < 2^BITS for every k < r
  uint64_t c1 = 0, c2 = 0;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    c1 += uint64_t(m1[i]) + 0x88888888u;
    c2 += uint64_t(m2[i]) + 0x88888888u;
    k[i + 4] = uint32_t(c1);
    m2[i + 4] = uint32_t(c2);
    c1 >>= 32;
    c2 >>= 32;
  }
#pragma unroll
  for (int i = 0; i < 4; i++) k[i] = m2[i] = 0;
}

// words of a slot before beta x of its entry
template <class F>
constexpr int vt_beta_at() {
  return vt_affine_words<F>();
}

// A = k Q for the Q of this lane's table; k is consumed
template <class C>
__device__ __forceinline__ void vt_mul_glv(Jz<C>& A, bool& inf, uint32_t* __restrict__ tab, uint32_t (&k)[8]) {
  using F = typename C::F;
  constexpr int NL = F::NL;
  constexpr int XW = (NL + 3) / 4 * 4;
  static_assert(vt_beta_at<F>() + XW <= vt_slot<F>(), "beta x inside its slot");
  uint32_t m2[8];
  bool n1, n2;
  vt_split<C>(k, m2, n1, n2);
  constexpr Words<NL> beta = Glv<C>::BETA;
#pragma unroll 1
  for (int d = 0; d < VT_N; d++) {
    uint32_t w[XW] = {};
    vt_pack<F>(w, lz_mul<F>(vt_get_affine<C>(tab + d * vt_slot<F>()).x, lz_of<F>(fp_from<F>(beta))));
    vt_store(tab + d * vt_slot<F>() + vt_beta_at<F>(), w);
  }
  inf = true;
  const LzAffine<C> Q = vt_get_affine<C>(tab);
  A.X = Q.x;
  A.Y = Q.y;
  A.Z = lz_one<F>();
#pragma unroll 1
  for (int w = 31; w >= 0; w--) {
#pragma unroll 1
    for (int i = 0; i < 4; i++) jz_dbl<C>(A);
    // the two additions as one piece of code
#pragma unroll 1
    for (int h = 0; h < 2; h++) {
      const int f = int(h ? take_top<4>(m2) : take_top<4>(k)) - 8;
      const int d = (h ? n2 : n1) ? -f : f;
      if (d == 0) continue;
      const uint32_t* sl = tab + ((d < 0 ? -d : d) - 1) * vt_slot<F>();
      LzAffine<C> T = vt_get_affine<C>(sl);
      if (h) {
        uint32_t bw[XW];
        vt_load(sl + vt_beta_at<F>(), bw);
        T.x = vt_unpack<F>(bw);
      }
      jz_madd<C>(A, inf, T.x, lz_neg_if<F>(T.y, d < 0));
    }
  }
}

// ---- the same on four lanes per request ------------------------------------------
// A call of few requests leaves most SIMDs without a wave, and a request's
// doublings are one chain.  Up to QUAD_MAX requests (four lanes of each then
// make one wave on every SIMD) the point operations take a quad of lanes each
// (quad.h); past it every lane has a request of its own.
// Measured: 256 secp256r1 verifications 1.38 -> 0.90 ms, 3001 BN254 products
// 0.86 -> 0.68 ms.
constexpr size_t QUAD_MAX = size_t(1) << 14;

// words per table entry: X, Y, ZZ, ZZZ, then the chain prefix and a flag word
template <class F>
constexpr int qvt_coord() {
  return (F::NL + 1 + 3) / 4 * 4;
}
template <class F>
constexpr int qvt_slot() {
  return 5 * qvt_coord<F>();
}

template <class F>
__device__ __forceinline__ void qvt_store(uint32_t* __restrict__ s, const Lz<F>& a, uint32_t flag = 0) {
  uint32_t w[qvt_coord<F>()] = {};
  vt_pack<F>(w, a);
  w[F::NL] = flag;
  vt_store(s, w);
}

template <class F>
__device__ __forceinline__ Lz<F> qvt_load(const uint32_t* __restrict__ s) {
  uint32_t w[qvt_coord<F>()];
  vt_load(s, w);
  return vt_unpack<F>(w);
}

// vt_build by a quad: entry d is made across the quad and stored one
// coordinate per lane; the chain runs over the ZZZ
template <class C, int WG>
__device__ __forceinline__ void qvt_build(uint32_t* __restrict__ tab, const Affine<C>& Q, Fp<typename C::F>* s_tot,
                                          Fp<typename C::F>* s_inv) {
  using F = typename C::F;
  constexpr int CWQ = qvt_coord<F>();
  constexpr int SLOT = qvt_slot<F>();
  const int q = quad_lane();
  const Qz<C> B = qz_affine<C>(lz_of<F>(Q.x), lz_of<F>(Q.y));
  Qz<C> T = B;
  qz_dbl<C>(T);  // no curve here has a point of order 2
  bool inf = false;
  Lz<F> pref = lz_one<F>();
#pragma unroll 1
  for (int d = 2; d <= VT_N; d++) {
    uint32_t* sl = tab + (d - 1) * SLOT;
    const Lz<F> z = lz_select<F>(inf, lz_one<F>(), quad_perm<F, QUAD_ALL(3)>(T));
    qvt_store<F>(sl + q * CWQ, q == 3 ? z : T);
    if (q == 0) qvt_store<F>(sl + 4 * CWQ, pref, inf ? 1u : 0u);
    pref = lz_mul<F>(pref, z);
    if (d < VT_N) qz_madd<C>(T, inf, B);
  }
  Lz<F> inv = lz_of<F>(wg_batch_inverse<F, WG, 4>(lz_semi<F>(pref), s_tot, s_inv));
  __threadfence_block();  // the quad's lanes read each other's stores
#pragma unroll 1
  for (int d = VT_N; d >= 2; d--) {
    uint32_t* sl = tab + (d - 1) * SLOT;
    uint32_t pw[CWQ];
    vt_load(sl + 4 * CWQ, pw);
    const Lz<F> mine = qvt_load<F>(sl + q * CWQ);
    // 1 / ZZZ_d in lane 0 and 1 / (ZZZ_2 ... ZZZ_(d-1)) in lane 1
    const Lz<F> t = lz_mul<F>(inv, lz_select<F>(q == 0, vt_unpack<F>(pw), quad_perm<F, QUAD_ALL(3)>(mine)));
    const Lz<F> izzz = quad_perm<F, QUAD_ALL(0)>(t);
    inv = quad_perm<F, QUAD_ALL(1)>(t);
    const Lz<F> iz = lz_mul<F>(quad_perm<F, QUAD_ALL(2)>(mine), izzz);  // 1 / Z
    Lz<F> r = lz_mul<F>(mine, lz_select<F>(q == 0, lz_sqr<F>(iz), izzz));  // x in lane 0, y in lane 1
    if (pw[F::NL]) r = lz_of<F>(fp_inf_marker<F>());
    if (q < 2) qvt_store<F>(sl + q * CWQ, r);
    if constexpr (vt_glv<C>()) {
      constexpr Words<F::NL> beta = Glv<C>::BETA;
      const Lz<F> bx = lz_mul<F>(r, lz_of<F>(fp_from<F>(beta)));
      if (q == 0) qvt_store<F>(sl + 2 * CWQ, bx);
    }
  }
  if (q < 2) qvt_store<F>(tab + q * CWQ, B);
  if constexpr (vt_glv<C>()) {
    constexpr Words<F::NL> beta = Glv<C>::BETA;
    const Lz<F> bx = lz_mul<F>(B, lz_of<F>(fp_from<F>(beta)));
    if (q == 0) qvt_store<F>(tab + 2 * CWQ, bx);
  }
  __threadfence_block();
}

// A += d Q (d in [-8, 7]), or d phi(Q) where phi
template <class C>
__device__ __forceinline__ void qvt_add_digit(Qz<C>& A, bool& inf, const uint32_t* __restrict__ tab, int d, bool phi) {
  using F = typename C::F;
  constexpr int CWQ = qvt_coord<F>();
  if (d == 0) return;
  const int q = quad_lane();
  const uint32_t* sl = tab + ((d < 0 ? -d : d) - 1) * qvt_slot<F>();
  Qz<C> B = q < 2 ? qvt_load<F>(sl + (q == 0 && phi ? 2 : q) * CWQ) : lz_one<F>();
  if (quad32<QUAD_ALL(0)>(B.w[0]) < 0) return;  // O
  B = lz_neg_if<F>(B, q == 1 && d < 0);
  qz_madd<C>(A, inf, B);
}

// vt_mul and vt_mul_glv by a quad
template <class C>
__device__ __forceinline__ void qvt_mul(Qz<C>& A, bool& inf, const uint32_t* __restrict__ tab, uint32_t (&u)[8]) {
  using F = typename C::F;
  constexpr int CWQ = qvt_coord<F>();
  const int q = quad_lane();
  A = q < 2 ? qvt_load<F>(tab + q * CWQ) : lz_one<F>();
  if constexpr (vt_glv<C>()) {
    uint32_t m2[8];
    bool n1, n2;
    vt_split<C>(u, m2, n1, n2);
    inf = true;
#pragma unroll 1
    for (int w = 31; w >= 0; w--) {
#pragma unroll 1
      for (int k = 0; k < 4; k++) qz_dbl<C>(A);
#pragma unroll 1
      for (int h = 0; h < 2; h++) {
        const int f = int(h ? take_top<4>(m2) : take_top<4>(u)) - 8;
        qvt_add_digit<C>(A, inf, tab, (h ? n2 : n1) ? -f : f, h != 0);
      }
    }
  } else {
    inf = !signed_nibbles(u);
#pragma unroll 1
    for (int w = 63; w >= 0; w--) {
#pragma unroll 1
      for (int k = 0; k < 4; k++) qz_dbl<C>(A);
      qvt_add_digit<C>(A, inf, tab, int(take_top<4>(u)) - 8, false);
    }
  }
}

// A += k G: each lane sums every fourth window on its own, then the quad adds
// the four sums
template <class C, int W>
__device__ __forceinline__ void qcomb_add(Qz<C>& A, bool& inf, const uint32_t* __restrict__ gcomb,
                                          const uint32_t (&k)[8]) {
  Xz<C> P;
  bool pinf = true;
  P.X = P.Y = P.ZZ = P.ZZZ = lz_one<typename C::F>();
  comb_add<C, W>(P, pinf, gcomb, k, quad_lane(), 4);
  const int fl = pinf ? 1 : 0;
#pragma unroll 1
  for (int s = 0; s < 4; s++) {
    // lane s's point, by rotating the lanes' points one place at each step
    const Qz<C> B = qz_spread<C, 0>(P);
    qz_add<C>(A, inf, B, ((quad32<QUAD_ALL(0)>(fl) | (quad32<QUAD_ALL(1)>(fl) << 1) | (quad32<QUAD_ALL(2)>(fl) << 2) |
                           (quad32<QUAD_ALL(3)>(fl) << 3)) >> s) & 1);
    xz_map<C>(P, P, [](int32_t v) { return quad32<quad_sel(1, 2, 3, 0)>(v); });
  }
}

// A = k G on one lane or on a quad (the sum then in every lane); true if O
template <class C, int W, int LPR>
__device__ __forceinline__ bool comb_sum(Xz<C>& A, const uint32_t* __restrict__ gcomb, const uint32_t (&k)[8]) {
  bool inf = true;
  if constexpr (LPR == 4) {
    Qz<C> S = lz_one<typename C::F>();
    qcomb_add<C, W>(S, inf, gcomb, k);
    A = qz_gather<C>(S);
  } else {
    comb_add<C, W>(A, inf, gcomb, k);
  }
  return inf;
}

// X / ZZ = v for a canonical 256-bit v < p
template <class C>
__device__ __forceinline__ bool x_is(const Xz<C>& A, const uint32_t (&v)[8]) {
  using F = typename C::F;
  return lz_is_zero<F>(lz_sub<F>(lz_mul<F>(lz_of<F>(fp_to_mont<F>(fp_from_words<F>(v))), A.ZZ), A.X));
}

// LPR lanes per request: 1, or 4 (a quad).  scratch: VT_N * vt_slot<F>() words
// (a quad: qvt_slot) per request of the grid, dead ones included
template <class C, int WG, int W, int LPR = 1>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(2))) k_verify_xyzz(const uint8_t* __restrict__ hashes,
                                                    const uint32_t* __restrict__ pubkeys,
                                                    const uint32_t* __restrict__ sigs, size_t m,
                                                    const uint32_t* __restrict__ gcomb,
                                                    uint32_t* __restrict__ scratch, uint8_t* __restrict__ valid) {
  using F = typename C::F;
  using N = typename OrderField<C>::type;
  __shared__ Fp<F> s_tot[WG / 64], s_inv[WG / 64];
  __shared__ Fp<N> n_tot[WG / 64], n_inv[WG / 64];
  const size_t i = (size_t(blockIdx.x) * WG + threadIdx.x) / LPR;
  const bool live = i < m;
  constexpr Words<8> n32 = N::P32;
  constexpr Words<8> p32 = F::P32;
  uint32_t rw[8], u1[8], u2[8];
  Affine<C> Q;
  bool ok;
  verify_prologue<C, WG>(hashes, pubkeys, sigs, i, live, n_tot, n_inv, rw, u1, u2, Q, ok);

  Xz<C> A;  // u2 Q, then u2 Q + u1 G
  bool inf;
  if constexpr (LPR == 4) {
    uint32_t* tab = scratch + i * size_t(VT_N * qvt_slot<F>());
    qvt_build<C, WG>(tab, Q, s_tot, s_inv);
    Qz<C> S;
    qvt_mul<C>(S, inf, tab, u2);
    qcomb_add<C, W>(S, inf, gcomb, u1);
    A = qz_gather<C>(S);
  } else {
    uint32_t* tab = scratch + i * size_t(VT_N * vt_slot<F>());
    vt_build<C, WG>(tab, Q, s_tot, s_inv);
    Jz<C> J;
    vt_mul<C>(J, inf, tab, u2);
    A.X = J.X;
    A.Y = J.Y;
    A.ZZ = lz_sqr<F>(J.Z);
    A.ZZZ = lz_mul<F>(J.Z, A.ZZ);
    comb_add<C, W>(A, inf, gcomb, u1);
  }

  // ---- R.x mod n == r: R.x is below p < 2n, so R.x = r or R.x = r + n ----
  if (live) {
    bool good = ok && !inf;
    if (good) {
      bool eq = x_is<C>(A, rw);
      uint32_t rn[8];
      uint64_t cy = 0;
#pragma unroll
      for (int k = 0; k < 8; k++) {
        uint64_t v = uint64_t(rw[k]) + n32.w[k] + cy;
        rn[k] = uint32_t(v);
        cy = v >> 32;
      }
      if (!eq && cy == 0 && words_lt8(rn, p32.w)) eq = x_is<C>(A, rn);
      good = eq;
    }
    if (threadIdx.x % LPR == 0) valid[i] = good ? 1 : 0;
  }
}

// ---- ECDSA signature generation ---------------------------------------------
//
// Per request: with 1 <= d, k < n, R = k G, r = R.x mod n and
// s = k^-1 (e + r d) mod n, e the hash read big-endian.  A request whose d or
// k is out of range, or whose r or s comes out zero, gets r = s = 0 (the
// caller draws another nonce).  The paper's signing workload is one
// fixed-point multiplication and one inversion mod n (Section 5.2): here k G
// is summed from the comb table in XYZZ coordinates on the lane,
// and 1 / ZZ (for R.x = X / ZZ) and k^-1 are one GAS inversion each per
// workgroup.
template <class C, int WG, int W, int LPR = 1>
__global__ void __launch_bounds__(WG) k_sign(const uint8_t* __restrict__ hashes, const uint32_t* __restrict__ privkeys,
                                             const uint32_t* __restrict__ nonces, size_t m,
                                             const uint32_t* __restrict__ gcomb, uint32_t* __restrict__ sigs) {
  using F = typename C::F;
  using N = typename OrderField<C>::type;
  __shared__ Fp<F> s_tot[WG / 64], s_inv[WG / 64];
  __shared__ Fp<N> n_tot[WG / 64], n_inv[WG / 64];
  const size_t i = (size_t(blockIdx.x) * WG + threadIdx.x) / LPR;
  const bool live = i < m;
  constexpr Words<8> n32 = N::P32;
  uint32_t dw[8], kw[8], ew[8];
  bool ok = live;
  if (live) {
    words_load<N>(privkeys + i * 8, dw);
    words_load<N>(nonces + i * 8, kw);
    const uint8_t* h = hashes + i * 32;
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const uint8_t* b = h + 28 - 4 * k;  // big-endian bytes, least significant word last
      ew[k] = (uint32_t(b[0]) << 24) | (uint32_t(b[1]) << 16) | (uint32_t(b[2]) << 8) | uint32_t(b[3]);
    }
    ok = !words_zero8(dw) && words_lt8(dw, n32.w) && !words_zero8(kw) && words_lt8(kw, n32.w);
  }
  if (!ok) {  // dead or rejected requests continue with d = k = 1, e = 0
#pragma unroll
    for (int k = 0; k < 8; k++) dw[k] = kw[k] = ew[k] = 0;
    dw[0] = kw[0] = 1;
  }

  // ---- R = k G from the comb ----
  Xz<C> A;
  comb_sum<C, W, LPR>(A, gcomb, kw);
  // 0 < k < n, so R != O and ZZ != 0
  const Fp<F> izz = wg_batch_inverse<F, WG, 4>(lz_semi<F>(A.ZZ), s_tot, s_inv);
  uint32_t rw[8];
  fp_to_words<F>(fp_from_mont<F>(lz_semi<F>(lz_mul<F>(A.X, lz_of<F>(izz)))), rw);
  // r = R.x mod n: R.x < p < 2n
  if (!words_lt8(rw, n32.w)) {
    int64_t br = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const int64_t v = int64_t(rw[k]) - int64_t(n32.w[k]) + br;
      rw[k] = uint32_t(v);
      br = v >> 32;
    }
  }

  // ---- s = k^-1 (e + r d) mod n ----
  const Fp<N> kinv = wg_batch_inverse<N, WG, 3>(fp_to_mont<N>(fp_from_words<N>(kw)), n_tot, n_inv);
  const Fp<N> t = fp_add<N>(fp_to_mont<N>(fp_from_words<N>(ew)),
                            fp_mul<N>(fp_to_mont<N>(fp_from_words<N>(rw)), fp_to_mont<N>(fp_from_words<N>(dw))));
  uint32_t sw[8];
  fp_to_words<N>(fp_from_mont<N>(fp_mul<N>(t, kinv)), sw);
  if (live && threadIdx.x % LPR == 0) {
    const bool good = ok && !words_zero8(rw) && !words_zero8(sw);
#pragma unroll
    for (int k = 0; k < 8; k++) {
      rw[k] = good ? rw[k] : 0u;
      sw[k] = good ? sw[k] : 0u;
    }
    words_store<N>(sigs + i * 16, rw);
    words_store<N>(sigs + i * 16 + 8, sw);
  }
}

// ---- batched unknown-point multiplication -----------------------------------
//
// out_i = k_i P_i for points known only at run time (the paper's UPMUL, the
// unknown-point half of its batch PMUL workload, Section 3.4 and Table 5),
// one request per lane: the table of d P_i and signed 4-bit windows of k_i as
// in the per-lane verification, then the result's 1 / Z by one GAS inversion
// per workgroup.  pts are working-form affine points (the infinity
// marker for O); every k_i is a 256-bit integer, taken as is.
template <class C, int WG, int LPR = 1>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(C::NL > 10 ? 1 : 2))) k_pmul(const uint32_t* __restrict__ pts, const uint32_t* __restrict__ ks,
                                             size_t n, uint32_t* __restrict__ scratch, uint32_t* __restrict__ out,
                                             int out_mont) {
  using F = typename C::F;
  constexpr int PW = affine_words<C>();
  __shared__ Fp<F> s_tot[WG / 64], s_inv[WG / 64];
  const size_t i = (size_t(blockIdx.x) * WG + threadIdx.x) / LPR;
  const bool live = i < n;
  Affine<C> P;
  uint32_t k[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  bool pinf = true;
  if (live) {
    P = affine_load<C>(pts + i * PW);
    pinf = fp_is_inf_marker<F>(P.x);
    load_scalar(ks + 8 * i, k);
  }
  if (pinf) {  // O, or a lane past the end: run on G, give O
    constexpr Words<F::NL> gx = C::GX, gy = C::GY;
    P.x = fp_from<F>(gx);
    P.y = fp_from<F>(gy);
  }
  Lz<F> X, Y, iz2, iz3;  // the result is (X iz2, Y iz3)
  bool inf;
  if constexpr (LPR == 4) {
    uint32_t* tab = scratch + i * size_t(VT_N * qvt_slot<F>());
    qvt_build<C, WG>(tab, P, s_tot, s_inv);
    Qz<C> S;
    qvt_mul<C>(S, inf, tab, k);
    inf = inf || pinf;
    const Xz<C> A = qz_gather<C>(S);
    X = A.X;
    Y = A.Y;
    // 1 / (ZZ ZZZ) gives both inverses
    const Lz<F> z = lz_mul<F>(A.ZZ, A.ZZZ);
    const Lz<F> t = lz_of<F>(wg_batch_inverse<F, WG>(inf ? fp_one<F>() : lz_semi<F>(z), s_tot, s_inv));
    iz2 = lz_mul<F>(t, A.ZZZ);
    iz3 = lz_mul<F>(t, A.ZZ);
  } else {
    uint32_t* tab = scratch + i * size_t(VT_N * vt_slot<F>());
    vt_build<C, WG>(tab, P, s_tot, s_inv);
    Jz<C> A;
    if constexpr (vt_glv<C>()) vt_mul_glv<C>(A, inf, tab, k);
    else vt_mul<C>(A, inf, tab, k);
    inf = inf || pinf;
    X = A.X;
    Y = A.Y;
    const Lz<F> iz = lz_of<F>(wg_batch_inverse<F, WG>(inf ? fp_one<F>() : lz_semi<F>(A.Z), s_tot, s_inv));
    iz2 = lz_sqr<F>(iz);
    iz3 = lz_mul<F>(iz, iz2);
  }
  store_lz_affine<C>(lz_mul<F>(X, iz2), lz_mul<F>(Y, iz3), inf, live && threadIdx.x % LPR == 0,
                     out + i * 2 * F::N32, out_mont);
}

// ---- batched unknown-point multiplication in affine coordinates ------------
//
// out_j = k_j P_j by the paper's batch UPMUL (Section 3.4, Algorithm 3): the
// scalar bits are walked from the least significant end; at bit i every
// request j has one point addition R_j = P_j + Q_j (P_j = 2^i P, Q_j the sum
// of the bits so far) and one doubling P_j <- 2 P_j, both affine.  Their two
// denominators t1 = 2 P_j.y (doubling) and t2 = P_j.x - Q_j.x (addition)
// enter one Montgomery-trick chain per lane, which walks the lane's requests;
// only the product T1 before both is kept per request (find-then-recompute:
// T1 t1 is recomputed from T1 and t1 in the decompress step), and the chain
// is inverted once per bit for the whole workgroup (GAS, Section 3.2).  The
// decompress step then finishes the addition first and the doubling second,
// each with its recovered inverse, and Q_j takes R_j when bit i of k_j is
// set: the addition is computed for every bit (a dummy one while Q_j is O),
// as the paper does for constant time.
//
// Request j of lane g is slot t of that lane, j = t T + g (T lanes in the
// grid), and its state lives in limb-major planes over the padded count
// J = T kper, so that a wave's accesses coalesce: P.x, P.y, Q.x, Q.y and the
// stored T1 (NL planes each), then the scalar (8 planes).  Exceptional
// additions (Q_j = O, Q_j = P_j, Q_j = -P_j) put 1 into the chain and are
// resolved in the decompress step; no curve here has a point of order 2, so
// 2^i P is never O and t1 is never 0.
template <class F>
constexpr int upmul_state_words() {
  return 5 * F::NL + 8;
}

enum : int { UP_ADD = 0, UP_COPY_P = 1, UP_TWICE = 2, UP_INF = 3 };

template <class C, int WG>
__global__ void __launch_bounds__(WG) k_upmul_affine(const uint32_t* __restrict__ pts, const uint32_t* __restrict__ ks,
                                                     size_t n, uint32_t kper, uint32_t* __restrict__ state,
                                                     uint32_t* __restrict__ out, int out_mont) {
  using F = typename C::F;
  constexpr int NL = F::NL;
  constexpr int N32 = F::N32;
  constexpr int PW = affine_words<C>();
  __shared__ Fp<F> s_tot[WG / 64], s_inv[WG / 64];
  const size_t T = size_t(gridDim.x) * WG;
  const size_t J = T * kper;
  const size_t g = size_t(blockIdx.x) * WG + threadIdx.x;
  uint32_t* const px = state;
  uint32_t* const py = px + NL * J;
  uint32_t* const qx = py + NL * J;
  uint32_t* const qy = qx + NL * J;
  uint32_t* const mm = qy + NL * J;
  uint32_t* const sc = mm + NL * J;
  const Fp<F> one = fp_one<F>();
  constexpr Words<F::NL> gx = C::GX, gy = C::GY;

  // ---- state: P_j (G with a zero scalar for O and for padding), Q_j = O ----
  for (uint32_t t = 0; t < kper; t++) {
    const size_t j = size_t(t) * T + g;
    Affine<C> P;
    P.x = fp_from<F>(gx);
    P.y = fp_from<F>(gy);
    uint32_t k[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (j < n) {
      const Affine<C> A = affine_load<C>(pts + j * PW);
      if (!fp_is_inf_marker<F>(A.x)) {
        P = A;
        load_scalar(ks + 8 * j, k);
      }
    }
    fp_store_soa<F>(px + j, J, P.x);
    fp_store_soa<F>(py + j, J, P.y);
    fp_store_soa<F>(qx + j, J, fp_inf_marker<F>());
    fp_store_soa<F>(qy + j, J, fp_zero<F>());
#pragma unroll
    for (int w = 0; w < 8; w++) sc[size_t(w) * J + j] = k[w];
  }

  for (int i = 0; i < 256; i++) {
    // compress: M_j = T1 before request j, T1 <- T1 t1 t2
    Fp<F> acc = one;
    for (uint32_t t = 0; t < kper; t++) {
      const size_t j = size_t(t) * T + g;
      const Fp<F> Py = fp_load_soa<F>(py + j, J);
      const Fp<F> t1 = fp_dbl<F>(Py);
      const Fp<F> Px = fp_load_soa<F>(px + j, J);
      const Fp<F> Qx = fp_load_soa<F>(qx + j, J);
      Fp<F> t2 = one;
      if (!fp_is_inf_marker<F>(Qx) && !fp_eq_canonical<F>(Px, Qx)) t2 = fp_sub_lazy<F>(Px, Qx);
      fp_store_soa<F>(mm + j, J, acc);
      acc = fp_mul<F>(fp_mul<F>(acc, t1), t2);
    }
    Fp<F> inv = wg_batch_inverse<F, WG, 20>(acc, s_tot, s_inv);
    // decompress with the addition, then the doubling, of every request
    for (int t = int(kper) - 1; t >= 0; t--) {
      const size_t j = size_t(t) * T + g;
      const Fp<F> M = fp_load_soa<F>(mm + j, J);
      Affine<C> P, Q;
      P.x = fp_load_soa<F>(px + j, J);
      P.y = fp_load_soa<F>(py + j, J);
      Q.x = fp_load_soa<F>(qx + j, J);
      Q.y = fp_load_soa<F>(qy + j, J);
      const bool bit = (sc[size_t(i >> 5) * J + j] >> (i & 31)) & 1u;
      const Fp<F> t1 = fp_dbl<F>(P.y);
      int cls = UP_ADD;
      Fp<F> t2 = one;
      if (fp_is_inf_marker<F>(Q.x)) cls = UP_COPY_P;
      else if (fp_eq_canonical<F>(P.x, Q.x)) cls = fp_eq_canonical<F>(P.y, Q.y) ? UP_TWICE : UP_INF;
      else t2 = fp_sub_lazy<F>(P.x, Q.x);
      const Fp<F> T1t1 = fp_mul<F>(t1, M);   // the discarded product, recomputed
      const Fp<F> t2inv = fp_mul<F>(inv, T1t1);
      inv = fp_mul<F>(inv, t2);              // 1 / (T1 t1)
      const Fp<F> t1inv = fp_mul<F>(inv, M);
      inv = fp_mul<F>(inv, t1);              // 1 / T1: the previous request's total
      Affine<C> R = P;
      if (cls == UP_ADD) {
        const Fp<F> lam = fp_mul<F>(fp_sub_lazy<F>(P.y, Q.y), t2inv);
        R.x = fp_canonical<F>(fp_sub<F>(fp_sub<F>(fp_sqr<F>(lam), P.x), Q.x));
        R.y = fp_canonical<F>(fp_sub<F>(fp_mul<F>(lam, fp_sub_lazy<F>(P.x, R.x)), P.y));
      }
      // the doubling: lambda = (3 x^2 + a) / (2 y)
      const Fp<F> lamd = fp_mul<F>(tangent_numerator<C>(P.x, one), t1inv);
      Affine<C> D;
      D.x = fp_canonical<F>(fp_sub<F>(fp_sub<F>(fp_sqr<F>(lamd), P.x), P.x));
      D.y = fp_canonical<F>(fp_sub<F>(fp_mul<F>(lamd, fp_sub_lazy<F>(P.x, D.x)), P.y));
      if (cls == UP_TWICE) R = D;
      if (cls == UP_INF) {
        R.x = fp_inf_marker<F>();
        R.y = fp_zero<F>();
      }
      fp_store_soa<F>(px + j, J, D.x);
      fp_store_soa<F>(py + j, J, D.y);
      if (bit) {
        fp_store_soa<F>(qx + j, J, R.x);
        fp_store_soa<F>(qy + j, J, R.y);
      }
    }
  }

  // ---- results: Q_j in the boundary form ----
  constexpr Words<F::NL> rout = F::ROUT;
  Fp<F> k1 = fp_zero<F>();
  k1.w[0] = 1;
  const Fp<F> kf = out_mont ? fp_from<F>(rout) : k1;
  for (uint32_t t = 0; t < kper; t++) {
    const size_t j = size_t(t) * T + g;
    if (j >= n) break;
    const Fp<F> Qx = fp_load_soa<F>(qx + j, J);
    const bool qinf = fp_is_inf_marker<F>(Qx);
    uint32_t xw[N32], yw[N32];
    fp_to_words<F>(fp_canonical<F>(fp_mul<F>(Qx, kf)), xw);
    fp_to_words<F>(fp_canonical<F>(fp_mul<F>(fp_load_soa<F>(qy + j, J), kf)), yw);
#pragma unroll
    for (int w = 0; w < N32; w++) {
      xw[w] = qinf ? 0u : xw[w];
      yw[w] = qinf ? 0u : yw[w];
    }
    words_store<F>(out + j * 2 * N32, xw);
    words_store<F>(out + j * 2 * N32 + N32, yw);
  }
}

// ---- fixed-point multiplication from the comb -------------------------------
//
// out_i = k_i G for any 256-bit k_i: one mixed addition per signed digit of
// k_i from the context's comb table (the paper's FPMUL with a precomputed
// table, Section 2.1), in XYZZ coordinates on the lane, then the affine result
// by one GAS inversion per workgroup.
template <class C, int WG, int W, int LPR = 1>
__global__ void __launch_bounds__(WG) k_fixed_base_comb(const uint32_t* __restrict__ ks, size_t n,
                                                        const uint32_t* __restrict__ gcomb, uint32_t* __restrict__ out,
                                                        int out_mont) {
  using F = typename C::F;
  __shared__ Fp<F> s_tot[WG / 64], s_inv[WG / 64];
  const size_t i = (size_t(blockIdx.x) * WG + threadIdx.x) / LPR;
  const bool active = i < n;
  uint32_t k[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (active) load_scalar(ks + 8 * i, k);
  Xz<C> A;
  const bool inf = comb_sum<C, W, LPR>(A, gcomb, k);
  const Lz<F> one = lz_one<F>();
  if (inf) xz_set<C>(A, one, one);
  const Lz<F> t = lz_of<F>(wg_batch_inverse<F, WG>(lz_semi<F>(lz_mul<F>(A.ZZ, A.ZZZ)), s_tot, s_inv));
  store_lz_affine<C>(lz_mul<F>(A.X, lz_mul<F>(t, A.ZZZ)), lz_mul<F>(A.Y, lz_mul<F>(t, A.ZZ)), inf,
                     active && threadIdx.x % LPR == 0, out + i * 2 * F::N32, out_mont);
}

}  // namespace eccmi

// Bucket accumulation of the MSMs: every bucket's points, gathered from the
// bases, are added on one lane (or several, for long buckets) in XYZZ
// coordinates, and the reduction reads the sums in that form.
//
// What bounds it, and why not batch-affine rounds (Section 3): a batched
// affine addition takes 6 products against the 10 (9 reductions) of a mixed
// XYZZ one, but on this device the rounds spend most of their time elsewhere.
// At BLS12-381 2^20 points (16.5 M additions) their products are 1.3 of
// 3.2 ms at the measured product rate (74 10^9 /s); the rest is 734 B of
// traffic per addition (two gathers of the point, prefix products, partial
// sums), the inversion's latency and scans in each of five launches, and the
// canonical forms that equality tests of stored points need.  Here an
// addition reads 154 B (128 of them its point) and does nothing but its products.
// k_bucket_acc keeps the vector units busy for 0.95 of the time in a batch of 512
// MSMs, 0.90 at BLS12-381 2^20 points (2.9 10^13 lane-instructions/s, at the 2.0 GHz
// the clock settles to) and 0.76 at BN254 700001 points (why a quarter of the issue
// slots stays open there has not been shown).
// Measured, rounds and finishing pass before against accumulation and merge
// now: BLS12-381 2^20 points 3.39 -> 2.60 ms (a call 4.55 -> 3.50 ms), 2^16
// 0.74 -> 0.30 ms, 512 uneven MSMs 5.04 -> 3.75 ms, BN254 700001 points 1.77 ->
// 0.95 ms (a call 2.56 -> 1.56 ms).
//
// Work items.  A bucket of n entries is cut into P = ceil(n / cap) nearly
// equal parts, one lane each.  cap is 1.5 times the entries that each lane
// of a full device (two waves on each SIMD) would get, and at least
// ACC_MIN_CAP: large calls cut only the buckets that would outlast the rest,
// small ones cut every bucket, since a lane's additions form a chain.  The
// entries are the call's own, read on the device: zero digits have none, and
// with scalars of few bits (a witness of small values) they are a fraction of
// what the sizes allow.  With cap from that bound, 2^20 BLS12-381 points with
// 8-bit scalars took 3.06 ms a call, 1.78 ms of it in chains of 192 additions on
// 5,600 lanes; now 1.55 ms (all scalars 1: 5.14 -> 3.42 ms, 64 bits: 4.02 -> 2.80).
// Items are ordered by length, longest first, by a counting
// sort, so that the lanes of a wave end together (buckets of uniform scalars
// hold 64 +- 8 entries at 2^20 points, and the longest of 64 lanes is 83) and
// the last waves are short ones.  The partial sums of a cut bucket are added
// by 1 to 4 lanes, as many as the device has for such buckets; by 16 lanes where
// there are more than four; by workgroups of quads when there are very many.
// acuts holds buckets of few parts from its start, of very many
// from the end of its first half, and the others in its second half.
#pragma once
#include "kernels.h"
#include "lazy.h"
#include "quad.h"

namespace eccmi {

constexpr uint32_t ACC_BINS = 1024;       // item lengths told apart by the sort (longer ones share a bin)
constexpr uint32_t ACC_MIN_CAP = 4;
constexpr int ACC_MERGE_LG_LANES = 4;     // at most 16 lanes add the parts of a cut bucket
constexpr uint32_t ACC_MERGE_TARGET = 65536;  // lanes the merge spreads over (one wave per SIMD)
constexpr uint32_t ACC_QUAD_CUTS = 4096;      // bound on the cut buckets up to which a quad takes the place of a lane
constexpr uint32_t ACC_MERGE_FEW = 4;     // parts up to which the lanes follow the number of such buckets
constexpr uint32_t ACC_MERGE_MAX = 128;   // parts beyond which workgroups of quads add them
constexpr uint32_t ACC_BIG_CHUNK = 256;   // parts of a very long bucket per workgroup, at least
constexpr uint32_t ACC_BIG_CHUNKS = 64;   // workgroups a very long bucket is spread over, at most
constexpr uint32_t ACC_ITEMS_LANE = 4;      // parts of a bucket whose items one lane writes, at most
constexpr uint32_t ACC_ITEMS_GROUP = 1024;  // and a group of lanes
constexpr uint32_t ACC_ITEMS_LANES = 16;    // of this many
constexpr int ACC_PLAN_WG = 1024;
constexpr int ACC_WG = 256;
constexpr int ACC_MERGE_WG = 256;

// counters of one call, zeroed before it
struct AccMeta {
  uint32_t items;       // work items
  uint32_t extra;       // parts beyond the first of their bucket (k_acc_items counts this and the next three together)
  uint32_t cut;         // cut buckets of at most ACC_MERGE_FEW parts
  uint32_t cut_mid;     // of more, up to ACC_MERGE_MAX
  uint32_t cut_big;     // of more than that
  uint32_t big_parts;   // the most parts of one bucket among those
  uint32_t hist[ACC_BINS];  // items by bin
  uint32_t cursor[ACC_BINS];
};

struct AccItem {
  uint32_t first, len, slot, pad;  // entries [first, first + len) of the sorted list, summed into psum[slot]
};

struct AccCut {
  uint32_t bucket, parts, extra;  // part 0 at psum[bucket], part j > 0 at psum[B + extra + j - 1]
  uint32_t done;                  // chunks of a very long bucket summed so far
};

struct AccLong {
  uint32_t at, off, bucket, n, extra, parts;
};

// cap for a call of this many bucket entries on a device of `lanes` (two waves
// on each SIMD); entries / cap is at most min(entries / ACC_MIN_CAP, 2 lanes / 3)
__device__ __forceinline__ uint32_t acc_cap(uint32_t entries, uint32_t lanes) {
  const uint32_t c = uint32_t((uint64_t(entries) * 3 / 2 + lanes - 1) / lanes);
  return c < ACC_MIN_CAP ? ACC_MIN_CAP : c;
}

__device__ __forceinline__ uint32_t acc_parts(uint32_t n, uint32_t cap) { return (n + cap - 1) / cap; }

// bin of a bucket's parts: longest first
__device__ __forceinline__ uint32_t acc_bin(uint32_t n, uint32_t parts) {
  const uint32_t len = (n + parts - 1) / parts;
  return ACC_BINS - 1 - (len < ACC_BINS ? len : ACC_BINS - 1);
}

// items per length
static __global__ void __launch_bounds__(ACC_PLAN_WG) k_acc_count(const uint32_t* __restrict__ counts,
                                                                  const uint32_t* __restrict__ offsets, uint32_t B,
                                                                  uint32_t lanes, AccMeta* __restrict__ meta) {
  __shared__ uint32_t s_hist[ACC_BINS];
  const uint32_t cap = acc_cap(offsets[B], lanes);
  for (uint32_t i = threadIdx.x; i < ACC_BINS; i += ACC_PLAN_WG) s_hist[i] = 0;
  __syncthreads();
  for (uint32_t b = blockIdx.x * ACC_PLAN_WG + threadIdx.x; b < B; b += gridDim.x * ACC_PLAN_WG) {
    const uint32_t n = counts[b];
    if (n == 0) continue;
    const uint32_t parts = acc_parts(n, cap);
    atomicAdd(&s_hist[acc_bin(n, parts)], parts);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < ACC_BINS; i += ACC_PLAN_WG)
    if (s_hist[i]) atomicAdd(&meta->hist[i], s_hist[i]);
}

// The items in order of length, and the lists of cut buckets.  Every counter is
// taken from in LDS first and once per workgroup on the device (2,240 cut buckets
// among 131,072 took 31 us of device atomics).  The items of a bucket of more than
// ACC_ITEMS_LANE parts are written by a group of lanes, side by side, or by the
// whole workgroup (2,048 buckets of 64 parts: 41 us with a lane for each).
static __global__ void __launch_bounds__(ACC_PLAN_WG) k_acc_items(const uint32_t* __restrict__ counts,
                                                                  const uint32_t* __restrict__ offsets, uint32_t B,
                                                                  uint32_t lanes, AccMeta* __restrict__ meta,
                                                                  AccItem* __restrict__ items,
                                                                  AccCut* __restrict__ cuts, uint32_t cut_cap) {
  __shared__ uint32_t s_first[ACC_BINS], s_n[ACC_BINS], s_tmp[ACC_PLAN_WG / 64];
  __shared__ uint32_t s_cut[4], s_cut0[4];  // parts beyond the first; cut buckets of few, more and very many parts
  __shared__ uint32_t s_nlong, s_most;
  __shared__ AccLong s_long[ACC_PLAN_WG];
  static_assert(ACC_BINS == ACC_PLAN_WG, "one bin per thread");
  const uint32_t t = threadIdx.x;
  const uint32_t cap = acc_cap(offsets[B], lanes);
  uint32_t total;
  const uint32_t before = block_exclusive_scan<ACC_PLAN_WG>(meta->hist[t], s_tmp, total);
  if (blockIdx.x == 0 && t == 0) meta->items = total;
  const uint32_t b = blockIdx.x * ACC_PLAN_WG + t;
  const uint32_t n = b < B ? counts[b] : 0u;
  const uint32_t parts = acc_parts(n, cap);
  const uint32_t bin = n ? acc_bin(n, parts) : 0u;
  const int kind = parts <= 1 ? 0 : parts <= ACC_MERGE_FEW ? 1 : parts <= ACC_MERGE_MAX ? 2 : 3;
  s_n[t] = 0;
  if (t < 4) s_cut[t] = 0;
  if (t == 0) s_nlong = s_most = 0;
  __syncthreads();
  const uint32_t mine = n ? atomicAdd(&s_n[bin], parts) : 0u;
  const uint32_t my_extra = kind ? atomicAdd(&s_cut[0], parts - 1) : 0u;
  const uint32_t my_cut = kind ? atomicAdd(&s_cut[kind], 1u) : 0u;
  if (kind == 3) atomicMax(&s_most, parts);
  __syncthreads();
  s_first[t] = before + (s_n[t] ? atomicAdd(&meta->cursor[t], s_n[t]) : 0u);
  if (t < 4 && s_cut[t]) s_cut0[t] = atomicAdd(&meta->extra + t, s_cut[t]);
  if (t == 0 && s_most) atomicMax(&meta->big_parts, s_most);
  __syncthreads();
  // part j of np: q entries, one more in each of the last r
  auto put = [&](uint32_t at, uint32_t off, uint32_t bucket, uint32_t q, uint32_t r, uint32_t np, uint32_t extra,
                 uint32_t j) {
    const uint32_t longer = j + r > np ? j + r - np : 0u;  // longer parts before this one
    items[at + j] = AccItem{off + j * q + longer, q + (j + r >= np ? 1u : 0u), j == 0 ? bucket : B + extra + j - 1, 0u};
  };
  if (n != 0) {
    const uint32_t at = s_first[bin] + mine, off = offsets[b];
    uint32_t extra = 0;
    if (kind) {
      extra = s_cut0[0] + my_extra;
      const uint32_t c = s_cut0[kind] + my_cut;
      cuts[kind == 1 ? c : kind == 2 ? cut_cap + c : cut_cap - 1 - c] = AccCut{b, parts, extra, 0u};
    }
    if (parts <= ACC_ITEMS_LANE) {
      const uint32_t q = n / parts, r = n % parts;
      for (uint32_t j = 0; j < parts; j++) put(at, off, b, q, r, parts, extra, j);
    } else {
      s_long[atomicAdd(&s_nlong, 1u)] = AccLong{at, off, b, n, extra, parts};  // one slot per thread at most
    }
  }
  __syncthreads();
  const uint32_t nlong = s_nlong;
  for (uint32_t i = t / ACC_ITEMS_LANES; i < nlong; i += ACC_PLAN_WG / ACC_ITEMS_LANES) {
    const AccLong g = s_long[i];
    if (g.parts > ACC_ITEMS_GROUP) continue;
    const uint32_t q = g.n / g.parts, r = g.n % g.parts;
    for (uint32_t j = t % ACC_ITEMS_LANES; j < g.parts; j += ACC_ITEMS_LANES)
      put(g.at, g.off, g.bucket, q, r, g.parts, g.extra, j);
  }
  if (s_most > ACC_ITEMS_GROUP) {
    for (uint32_t i = 0; i < nlong; i++) {
      const AccLong g = s_long[i];
      if (g.parts <= ACC_ITEMS_GROUP) continue;
      const uint32_t q = g.n / g.parts, r = g.n % g.parts;
      for (uint32_t j = t; j < g.parts; j += ACC_PLAN_WG) put(g.at, g.off, g.bucket, q, r, g.parts, g.extra, j);
    }
  }
}

// One item per lane: its entries added in XYZZ coordinates (madd-2008-s, see
// xz_madd).  The next point is loaded into the registers of the current one
// as soon as its two products are done, so its latency passes behind the
// other seven; the sorted words run two entries ahead.
template <class C>
__global__ void __launch_bounds__(ACC_WG) __attribute__((amdgpu_waves_per_eu(2))) k_bucket_acc(
    const uint32_t* __restrict__ bases, const uint32_t* __restrict__ sorted, const AccMeta* __restrict__ meta,
    const AccItem* __restrict__ items, uint32_t* __restrict__ psum) {
  using F = typename C::F;
  constexpr int PW = affine_words<C>();
  const uint32_t i = blockIdx.x * ACC_WG + threadIdx.x;
  if (i >= meta->items) return;
  const AccItem it = items[i];
  const uint32_t* src = sorted + it.first;
  uint32_t s1 = src[0], s2 = it.len > 1 ? src[1] : 0u;
  Lz<F> bx = lz_load<F>(bases + size_t(s1 & ~SIGN_BIT) * PW);
  Lz<F> by = lz_neg_if<F>(lz_load<F>(bases + size_t(s1 & ~SIGN_BIT) * PW + F::CW), (s1 & SIGN_BIT) != 0);
  Xz<C> A;
  bool inf = true;
#pragma unroll 1
  for (uint32_t k = 0; k < it.len; k++) {
    bool add = !inf;
    Lz<F> P, R;
    if (inf) {
      xz_set<C>(A, bx, by);
      inf = false;
    } else {
      lz_pair<F>(ColMul<F>{bx, A.ZZ}, ColMul<F>{by, A.ZZZ}, P, R);
      P = lz_sub<F>(P, A.X);
      R = lz_sub<F>(R, A.Y);
      if (lz_maybe_zero<F, 8>(P)) {
        if (lz_is_zero<F>(P)) {
          if (lz_is_zero<F>(R)) xz_mdbl<C>(A, bx, by);
          else inf = true;
          add = false;
        }
      }
    }
    if (k + 1 < it.len) {
      const uint32_t s = s2;
      if (k + 2 < it.len) s2 = src[k + 2];
      const uint32_t* p = bases + size_t(s & ~SIGN_BIT) * PW;
      bx = lz_load<F>(p);
      by = lz_load<F>(p + F::CW);
      s1 = s;
    }
    if (add) xz_madd_tail<C>(A, P, R);
    by = lz_neg_if<F>(by, (s1 & SIGN_BIT) != 0);
  }
  xz_store<C>(psum + size_t(it.slot) * xyzz_words<C>(), A, inf);
}

// the partial sums of a cut bucket: lane l of G adds the parts l, l + G, ...,
// then a tree over the lanes (one addition in the code for both); the sum goes
// back to part 0's place.  All 64 lanes of the wave stay in step.
template <class C>
__device__ __forceinline__ void acc_merge(Xz<C>& A, bool& inf, const AccCut& cut, uint32_t l, uint32_t G, uint32_t B,
                                          const uint32_t* __restrict__ psum, int tree) {
  constexpr int XW = xyzz_words<C>();
  const uint32_t mine = l < cut.parts ? (cut.parts - l + G - 1) / G : 0u;
  uint32_t most = mine;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) most = max(most, uint32_t(__shfl_xor(int(most), d, 64)));
  inf = true;
  const uint32_t steps = most + uint32_t(tree);
#pragma unroll 1
  for (uint32_t st = 0; st < steps; st++) {
    Xz<C> Bp;
    bool binf = true;
    if (st < most) {
      if (st < mine) {
        const uint32_t j = l + st * G;
        xz_load<C>(psum + size_t(j == 0 ? cut.bucket : B + cut.extra + j - 1) * XW, Bp, binf);
      }
    } else {
      const int off = 1 << (tree - 1 - int(st - most));
      xz_map<C>(Bp, A, [&](int32_t v) { return __shfl_down(v, off, 64); });
      binf = __shfl_down(int(inf), off, 64) != 0 || l + uint32_t(off) >= G;
    }
    xz_add<C>(A, inf, Bp, binf);
  }
}

// log2 of the lanes (or quads) that add the parts of each of n cut buckets of
// few parts: as many as `target` allows, since a lane's additions form a chain
__device__ __forceinline__ int acc_merge_lanes(uint32_t n, uint32_t target) {
  int lg = 0;
  while ((2u << lg) <= ACC_MERGE_FEW && (n << (lg + 1)) <= target) lg++;
  return lg;
}

template <class C>
__global__ void __launch_bounds__(ACC_MERGE_WG) __attribute__((amdgpu_waves_per_eu(2, 2))) k_acc_merge(
    const AccMeta* __restrict__ meta, const AccCut* __restrict__ cuts, uint32_t cut_cap, uint32_t B,
    uint32_t* __restrict__ psum) {
  const uint32_t waves = gridDim.x * (ACC_MERGE_WG / 64);
  const uint32_t wave = (blockIdx.x * ACC_MERGE_WG + threadIdx.x) / 64;
  // the buckets of more parts first, from the last wave on, then the others
#pragma unroll 1
  for (int pass = 0; pass < 2; pass++) {
    const uint32_t n = pass == 0 ? meta->cut_mid : meta->cut;
    const AccCut* list = pass == 0 ? cuts + cut_cap : cuts;
    const int lgG = pass == 0 ? ACC_MERGE_LG_LANES : acc_merge_lanes(n, ACC_MERGE_TARGET);
    const uint32_t G = 1u << lgG;
    const uint32_t l = threadIdx.x & (G - 1);
    // the wave's cut buckets; the loop's bounds are wave-uniform
    for (uint32_t w = pass == 0 ? waves - 1 - wave : wave; (w << (6 - lgG)) < n; w += waves) {
      const uint32_t i = (w << (6 - lgG)) + ((threadIdx.x & 63u) >> lgG);
      const AccCut cut = i < n ? list[i] : AccCut{0u, 0u, 0u, 0u};
      int tree = 0;  // levels the widest of the wave's buckets needs
      while (tree < lgG && __ballot((1u << tree) < cut.parts) != 0) tree++;
      Xz<C> A;
      bool inf;
      acc_merge<C>(A, inf, cut, l, G, B, psum, tree);
      if (i < n && l == 0) xz_store<C>(psum + size_t(cut.bucket) * xyzz_words<C>(), A, inf);
    }
  }
}

// The same with a quad of lanes in the place of a lane, for calls of at most
// ACC_QUAD_CUTS cut buckets by the plan's bound.  One MSM of the default width 8 has
// 2,048 buckets, all of them cut (whole calls, lanes against quads: 2^10 BLS12-381
// points 590 and 546 us, 2^15 points 834 and 798 us, 2^12 BN254 points 426 and
// 416 us).  At 4,096 buckets of many parts the two are level (2^14 points without
// the endomorphism 934 and 961 us); past it lanes are the faster where as many
// buckets are really cut (2 MSMs of 2^13 points 931 and 976 us), and within 8%
// where the bound counts many that are not.
template <class C>
__global__ void __launch_bounds__(ACC_MERGE_WG) k_acc_merge_quad(const AccMeta* __restrict__ meta,
                                                                 const AccCut* __restrict__ cuts, uint32_t cut_cap,
                                                                 uint32_t B, uint32_t* __restrict__ psum) {
  constexpr int XW = xyzz_words<C>();
  const uint32_t waves = gridDim.x * (ACC_MERGE_WG / 64);
  const uint32_t wave = (blockIdx.x * ACC_MERGE_WG + threadIdx.x) / 64;
  const uint32_t t = (threadIdx.x & 63u) >> 2;  // quad in its wave
#pragma unroll 1
  for (int pass = 0; pass < 2; pass++) {
    const uint32_t n = pass == 0 ? meta->cut_mid : meta->cut;
    const AccCut* list = pass == 0 ? cuts + cut_cap : cuts;
    const int lgG = pass == 0 ? 4 : acc_merge_lanes(n, ACC_MERGE_TARGET / 4);  // quads per bucket
    const uint32_t G = 1u << lgG;
    const uint32_t l = t & (G - 1);
    for (uint32_t w = pass == 0 ? waves - 1 - wave : wave; (w << (4 - lgG)) < n; w += waves) {
      const uint32_t i = (w << (4 - lgG)) + (t >> lgG);
      const AccCut cut = i < n ? list[i] : AccCut{0u, 0u, 0u, 0u};
      int tree = 0;
      while (tree < lgG && __ballot((1u << tree) < cut.parts) != 0) tree++;
      const uint32_t mine = l < cut.parts ? (cut.parts - l + G - 1) / G : 0u;
      uint32_t most = mine;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) most = max(most, uint32_t(__shfl_xor(int(most), d, 64)));
      Qz<C> A = lz_one<typename C::F>();
      bool inf = true;
#pragma unroll 1
      for (uint32_t st = 0; st < most + uint32_t(tree); st++) {
        Qz<C> Bp;
        bool binf = true;
        if (st < most) {
          if (st < mine) {
            const uint32_t j = l + st * G;
            qz_load<C>(psum + size_t(j == 0 ? cut.bucket : B + cut.extra + j - 1) * XW, Bp, binf);
          }
        } else {
          const int off = 1 << (tree - 1 - int(st - most));
#pragma unroll
          for (int k = 0; k < C::F::NL; k++) Bp.w[k] = __shfl_down(A.w[k], 4 * off, 64);
          binf = __shfl_down(int(inf), 4 * off, 64) != 0 || l + uint32_t(off) >= G;
        }
        qz_add<C>(A, inf, Bp, binf);
      }
      if (i < n && l == 0) qz_store<C>(psum + size_t(cut.bucket) * XW, A, inf);
    }
  }
}

// The parts of very long buckets (small or repeated scalars fill a few buckets
// with most of the entries): a workgroup's 64 quads add a chunk of at least
// ACC_BIG_CHUNK parts, a tree through LDS joins them, and the workgroup that ends
// last at a bucket adds its chunks' sums (no workgroup waits for another).
// Bound by that chain: at most 3 additions, 6 levels and the last workgroup's 6
// levels up to 2^14 parts.  2^18 points with 64-bit scalars: one BLS12-381 bucket
// of 2,731 parts took 267 us on one workgroup of lanes, its 9,362 parts now 113 us.
template <class C>
__global__ void __launch_bounds__(ACC_MERGE_WG) k_acc_merge_big(const AccMeta* __restrict__ meta, AccCut* cuts,
                                                                uint32_t cut_cap, uint32_t B, uint32_t* psum) {
  using F = typename C::F;
  constexpr int XW = xyzz_words<C>();
  constexpr uint32_t QUADS = ACC_MERGE_WG / 4;
  static_assert(ACC_BIG_CHUNKS <= QUADS, "one quad per chunk sum");
  __shared__ int32_t s_pt[F::NL * ACC_MERGE_WG];
  __shared__ int32_t s_inf[QUADS];
  __shared__ uint32_t s_last;
  const uint32_t quad = threadIdx.x >> 2;
  const uint32_t n = meta->cut_big;
  const uint32_t most = min(ACC_BIG_CHUNKS, (meta->big_parts + ACC_BIG_CHUNK - 1) / ACC_BIG_CHUNK);
  // every branch below but those on `quad` and on a point's infinity is uniform in the workgroup
  for (uint32_t u = blockIdx.x; u < n * most; u += gridDim.x) {
    AccCut* const list = cuts + (cut_cap - 1 - u % n);
    const AccCut cut = *list;
    const uint32_t per = max(ACC_BIG_CHUNK, (cut.parts + ACC_BIG_CHUNKS - 1) / ACC_BIG_CHUNKS);
    const uint32_t chunks = (cut.parts + per - 1) / per;
    uint32_t base = u / n * per, stride = 1;
    if (base >= cut.parts) continue;
    uint32_t count = min(per, cut.parts - base);
    // the chunk's parts, then (on the last workgroup) the chunks' sums
#pragma unroll 1
    for (int pass = 0;; pass++) {
      int levels = 0;
      while (levels < 6 && (1u << levels) < count) levels++;
      const uint32_t own = (count + QUADS - 1) / QUADS;
      Qz<C> A = lz_one<F>();
      bool inf = true;
#pragma unroll 1
      for (uint32_t st = 0; st < own + uint32_t(levels); st++) {
        Qz<C> Bp = A;
        bool binf = true;
        if (st < own) {
          const uint32_t i = quad + QUADS * st, j = base + stride * i;
          if (i < count) qz_load<C>(psum + size_t(j == 0 ? cut.bucket : B + cut.extra + j - 1) * XW, Bp, binf);
        } else {
          const uint32_t from = quad + (1u << (levels - 1 - int(st - own)));
          __syncthreads();
#pragma unroll
          for (int k = 0; k < F::NL; k++) s_pt[k * ACC_MERGE_WG + threadIdx.x] = A.w[k];
          if (quad_lane() == 0) s_inf[quad] = inf ? 1 : 0;
          __syncthreads();
          if (from < QUADS) {
#pragma unroll
            for (int k = 0; k < F::NL; k++) Bp.w[k] = s_pt[k * ACC_MERGE_WG + from * 4 + quad_lane()];
            binf = s_inf[from] != 0;
          }
        }
        qz_add<C>(A, inf, Bp, binf);
      }
      if (quad == 0) qz_store<C>(psum + size_t(base == 0 ? cut.bucket : B + cut.extra + base - 1) * XW, A, inf);
      if (pass == 1 || chunks == 1) break;
      __threadfence();  // the sum before the count, at device scope: chunks run on other XCDs too
      if (threadIdx.x == 0) s_last = atomicAdd(&list->done, 1u) == chunks - 1 ? 1u : 0u;
      __syncthreads();
      if (!s_last) break;
      __threadfence();
      base = 0;
      stride = per;
      count = chunks;
    }
    __syncthreads();  // LDS is used again
  }
}

// ---- bucket reduction, level A, over the sums above ---------------------------
// The scheme of k_reduce_a (kernels.h) on lazy limbs.

// seg_weighted_sum for lazy points; t_inf: T_t is O
template <class C, class GetT, class PutU>
__device__ __forceinline__ void xz_seg_weighted_sum(Xz<C>& a, bool& inf, int lgS, int lgM, GetT get_T, PutU put_U) {
  const int lane = threadIdx.x & 63;
  const int seg = 1 << lgS;
  const int t = lane & (seg - 1);
  const int nsteps = lgS + lgM + 1 + lgS;
#pragma unroll 1
  for (int st = 0; st < nsteps; st++) {
    if (st == lgS && t == 0) put_U(a, inf);  // the segment total, after the scan
    if (st >= lgS && st < lgS + lgM) {
      if (!inf) xz_dbl<C>(a);
      continue;
    }
    Xz<C> b;
    bool binf;
    if (st < lgS) {
      const int off = 1 << st;
      xz_map<C>(b, a, [&](int32_t v) { return __shfl_down(v, off, 64); });
      binf = __shfl_down(int(inf), off, 64) != 0 || t + off >= seg;
    } else if (st == lgS + lgM) {
      inf = inf || t < 1;
      get_T(b, binf);
    } else {
      const int m = seg >> (st - lgS - lgM);
      xz_map<C>(b, a, [&](int32_t v) { return __shfl_xor(v, m, 64); });
      binf = __shfl_xor(int(inf), m, 64) != 0;
    }
    xz_add<C>(a, inf, b, binf);
  }
}

template <class C, int WG>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(2, 2))) k_reduce_a_xz(
    const uint32_t* __restrict__ counts, const uint32_t* __restrict__ psum, const RedJob* __restrict__ jobs,
    const RedWave* __restrict__ waves, uint32_t nwaves, uint32_t* __restrict__ segU, uint32_t* __restrict__ segY,
    uint32_t* __restrict__ winsum) {
  constexpr int XW = xyzz_words<C>();
  constexpr int NL = C::F::NL;
  const uint32_t gw = (blockIdx.x * WG + threadIdx.x) >> 6;  // uniform per wave
  if (gw >= nwaves) return;
  const uint32_t lane = threadIdx.x & 63;
  const RedWave wv = waves[gw];
  const int lgS = int(wv.lgS);
  const uint32_t slot = lane >> lgS;             // job slot inside the wave
  const uint32_t t = lane & ((1u << lgS) - 1u);  // lane inside the segment
  const bool active = slot < wv.njobs;
  const RedJob jb = jobs[wv.job + (active ? slot : 0u)];
  const int lgLam = int(jb.lgLam);
  const int lgL = int(jb.lgD) - lgLam;
  const uint32_t L = 1u << lgL;
  const uint32_t first = jb.bucket + ((wv.g << 6) + t) * L;  // L buckets from here
  // T lives in LDS (one word per limb and thread, touched by its own thread
  // only): the registers hold one addition's two operands
  __shared__ int32_t s_T[4 * NL * WG];
  int32_t* const sT = s_T + threadIdx.x;
  auto load_T = [&](Xz<C>& P) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NL; i++) {
      P.X.w[i] = sT[(0 * NL + i) * WG];
      P.Y.w[i] = sT[(1 * NL + i) * WG];
      P.ZZ.w[i] = sT[(2 * NL + i) * WG];
      P.ZZZ.w[i] = sT[(3 * NL + i) * WG];
    }
  };
  Xz<C> S;
  bool sinf = true, tinf = true;
  // S += B_k, then T += S: one addition in the code
#pragma unroll 1
  for (uint32_t st = 0; st < 2 * L; st++) {
    Xz<C> Bz;
    bool binf = true;
    const bool second = st & 1u;
    if (second) {
      Bz = S;
      binf = sinf;
      load_T(S);
      sinf = tinf;
    } else if (active) {
      const uint32_t b = first + L - 1 - st / 2;
      if (counts[b]) xz_load<C>(psum + size_t(b) * XW, Bz, binf);
    }
    xz_add<C>(S, sinf, Bz, binf);
    if (second) {
#pragma unroll
      for (int i = 0; i < NL; i++) {
        sT[(0 * NL + i) * WG] = S.X.w[i];
        sT[(1 * NL + i) * WG] = S.Y.w[i];
        sT[(2 * NL + i) * WG] = S.ZZ.w[i];
        sT[(3 * NL + i) * WG] = S.ZZZ.w[i];
      }
      tinf = sinf;
      S = Bz;
      sinf = binf;
    }
  }
  const bool big = lgLam > 6;
  xz_seg_weighted_sum<C>(
      S, sinf, lgS, lgL,
      [&](Xz<C>& b, bool& binf) {
        load_T(b);
        binf = tinf;
      },
      [&](const Xz<C>& U, bool uinf) {
        if (active && big) xyzz_store<C>(segU + size_t(jb.seg_base + wv.g) * XW, xz_to_xyzz<C>(U, uinf));
      });
  if (active && t == 0) {
    const XYZZ<C> Y = xz_to_xyzz<C>(S, sinf);
    if (!big) xyzz_store<C>(winsum + size_t(wv.job + slot) * XW, Y);
    else xyzz_store<C>(segY + size_t(jb.seg_base + wv.g) * XW, Y);
  }
}

// The same with a quad of lanes in the place of a lane: a workgroup of 256 is
// one level-A wave of the plan, and its 64 quads exchange points through LDS.
// All jobs of a workgroup have the same L (Geometry::same_chain): its threads meet
// at barriers once per step.
// Taken while the quads make at most two waves per SIMD (512 waves of the plan on
// this device), since a chain of about 2 L + 13 + log2 L point operations bounds the
// phase there.  Level A, lanes against quads, by waves: 16 (1021 BLS12-381
// points) 218 and 117 us, (4096 BN254 points) 106 and 64 us; 96 (2^12 points, c = 11)
// 232 and 125; 320 (c = 13) 259 and 185; 416 (8 MSMs of 2^12 points) 231 and 177;
// 640 (2^16 points, c = 14) 243 and 273; 1,024 (c = 16) 352 and 468: past the line
// the quad's extra moves cost more than they save.
constexpr int REDUCE_QUAD_WG = 256;

template <class C>
__global__ void __launch_bounds__(REDUCE_QUAD_WG) k_reduce_a_quad(
    const uint32_t* __restrict__ counts, const uint32_t* __restrict__ psum, const RedJob* __restrict__ jobs,
    const RedWave* __restrict__ waves, uint32_t* __restrict__ segU, uint32_t* __restrict__ segY,
    uint32_t* __restrict__ winsum) {
  using F = typename C::F;
  constexpr int XW = xyzz_words<C>();
  constexpr int NL = F::NL;
  __shared__ int32_t s_pt[NL * REDUCE_QUAD_WG];
  __shared__ int32_t s_inf[REDUCE_QUAD_WG / 4];
  const RedWave wv = waves[blockIdx.x];
  const int lgS = int(wv.lgS);
  const uint32_t quad = threadIdx.x >> 2;
  const int q = quad_lane();
  const uint32_t slot = quad >> lgS;             // job slot
  const uint32_t t = quad & ((1u << lgS) - 1u);  // quad inside the segment
  const bool active = slot < wv.njobs;
  const RedJob jb = jobs[wv.job + (active ? slot : 0u)];
  const int lgL = int(jb.lgD) - int(jb.lgLam);
  const uint32_t L = 1u << lgL;
  const uint32_t first = jb.bucket + ((wv.g << 6) + t) * L;
  // the point of quad `from` of this workgroup (every thread takes part)
  auto exchange = [&](const Qz<C>& a, bool inf, uint32_t from, bool valid, Qz<C>& b, bool& binf)
                      __attribute__((always_inline)) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NL; i++) s_pt[i * REDUCE_QUAD_WG + threadIdx.x] = a.w[i];
    if (q == 0) s_inf[quad] = inf ? 1 : 0;
    __syncthreads();
    const uint32_t f = valid ? from : quad;
#pragma unroll
    for (int i = 0; i < NL; i++) b.w[i] = s_pt[i * REDUCE_QUAD_WG + f * 4 + q];
    binf = !valid || s_inf[f] != 0;
  };
  auto put = [&](uint32_t* p, const Qz<C>& a, bool inf) __attribute__((always_inline)) {
    // the semi-reduced form of point.h, one coordinate per lane
    Fp<F> r = lz_semi<F>(lz_mul<F>(a, lz_one<F>()));
    if (inf) r = q < 2 ? fp_one<F>() : fp_zero<F>();
    fp_store<F>(p + q * F::CW, r);
  };
  const bool big = jb.lgLam > 6;
  Qz<C> S = lz_one<F>(), T = S;
  bool sinf = true, tinf = true;
  // one loop, so that the addition appears once: the running sums (S += B_k,
  // T += S), the suffix scan, the addition of T, the butterfly
  const int n_run = int(2 * L), n_scan = n_run + lgS, n_t = n_scan + 1, n_all = n_t + lgS;
#pragma unroll 1
  for (int st = 0; st < n_all; st++) {
    Qz<C> b = S;
    bool binf = sinf;
    const bool second = st < n_run && (st & 1);
    if (second) {
      S = T;
      sinf = tinf;
    } else if (st < n_run) {
      const uint32_t k = first + L - 1 - uint32_t(st) / 2;
      binf = true;
      if (active && counts[k]) qz_load<C>(psum + size_t(k) * XW, b, binf);
    } else if (st < n_scan) {
      const uint32_t off = 1u << (st - n_run);
      exchange(S, sinf, quad + off, t + off < (1u << lgS), b, binf);
    } else if (st < n_t) {
      if (active && t == 0 && big) put(segU + size_t(jb.seg_base + wv.g) * XW, S, sinf);  // the segment total
#pragma unroll 1
      for (int i = 0; i < lgL; i++) qz_dbl<C>(S);
      sinf = sinf || t < 1;
      b = T;
      binf = tinf;
    } else {
      exchange(S, sinf, quad ^ (1u << (lgS - 1 - (st - n_t))), true, b, binf);
    }
    const Qz<C> keep = b;
    const bool kinf = binf;
    qz_add<C>(S, sinf, b, binf);
    if (second) {
      T = S;
      tinf = sinf;
      S = keep;
      sinf = kinf;
    }
  }
  if (active && t == 0) {
    if (!big) put(winsum + size_t(wv.job + slot) * XW, S, sinf);
    else put(segY + size_t(jb.seg_base + wv.g) * XW, S, sinf);
  }
}

}  // namespace eccmi

// Register-blocked NTT pass stages shared by the plain and fused kernels.
//
// Forward transform of a limb (a polynomial modulo q, psi a primitive 2N-th
// root of unity): slot j of the output holds the value at psi^(2 brv(j) + 1),
// brv the logN-bit reversal (bit-reversed evaluation order).
//
// A limb of N 64-bit words (512 KiB at N = 2^16) exceeds one CU's LDS, so a
// transform is two passes over memory, N = R1 x R2 (a = log2 R1, b = log2 R2):
//   * strided pass: the R2 columns (words R2 apart) are independent R1-point
//     transforms: negacyclic forward, with the twiddle psi^brv(2^s + grp) at
//     stage s and group grp;
//   * contiguous pass: block g of R2 contiguous words holds the polynomial
//     modulo X^R2 - psi^(R2 (2 brv_a(g) + 1)).  Twisted by
//     x_i <- x_i psi^((2 brv_a(g) + 1) i) it is a cyclic R2-point transform
//     with omega = psi^(2 R1), whose twiddle for group grp, of any stage, is
//     omega^brv(grp) = psi^brv(grp): one short table for all blocks, and the
//     first group's products are by 1.  The twist is one coalesced table read
//     and one product a point.
// The inverse passes run the cyclic transform in the other order
// (decimation in time: from bit-reversed to natural order, x + w y and
// x - w y with w = omega^-j, j the position inside the half block), then
// multiply word i by its inverse twist (contiguous pass) or by a per-row
// factor that holds psi^(-R2 i) and the pass's scale (strided pass).  Every
// butterfly multiplies before it adds, in both directions, so values grow by
// a bounded step per stage and need (almost) no reductions in between.
//
// Arithmetic (one class per modulus, uniform over a workgroup):
//   * ArF, 2^26 <= q < 2^50 + 2^44: residues are integers in doubles, of
//     either sign.  a w mod q is six full-rate FP64 operations
//       h = a w, c = rint(a (w/q)), r = fma(-c, q, h) + fma(a, w, -h),
//     exact: fma(a, w, -h) is the product's rounding error, h - c q is an
//     integer below 2^53, and a wrong last bit of c moves r by q, not its
//     residue.  With w centred, |r| <= (1/2 + e) q, e the error of c.  Measured
//     on the chip a butterfly takes 9.5 issue slots, against 21.6 for the
//     64-bit integer one;
//   * ArI<LIM>, q < 2^64 / LIM (LIM = 16 below 2^60, else 8): 64-bit integers
//     with Shoup products in [0, 2q), reduced only where the next stage would
//     pass LIM q (the earlier form reduced x in every butterfly).
// The bounds of every stage are computed at compile time (Bounds).
//
// In a pass a thread owns P points of one R-point sub-transform and T = R/P
// threads share it, in layouts of the point index that are switched through
// LDS (Pass2, Pass3 below).
#pragma once
#include "internal.h"

namespace hck {

constexpr int kNttThreads = 256;

// log2(R1), log2(R2) of the two-pass split
constexpr int split_a(int log_n) { return (log_n + 1) / 2; }
constexpr int split_b(int log_n) { return log_n / 2; }

// ---- arithmetic ------------------------------------------------------------

struct ArF {
  using E = double;
  static constexpr bool kFloat = true;
  double q, qi;  // q and its rounded inverse

  // Bounds are in units of q / 1024.  X s, s = 1 + 2^-6 >= q 2^-50, bounds a
  // value in units of 2^50 / 1024; 2^53 is 8192 of them.
  static constexpr int scaled(int x) { return x + x / 64 + 1; }
  static constexpr int kLimit = 8192;
  static constexpr bool fits(int x) { return scaled(x) <= kLimit; }
  // |a w mod q| for |a| <= X q: 1/2 plus the error of c, which is |a| times
  // half an ulp of w/q (2^-55, |w/q| <= 1/2) plus half an ulp of the product
  static constexpr int product(int x) {
    const int s = scaled(x);
    return 512 + s / 32 + 1 + (s <= 2048 ? 64 : s <= 4096 ? 128 : 256);
  }
  static constexpr int kReduced = 514;
  static constexpr int kCanonical = 1024;
  // |a b mod q| of mul2 for |a| <= q, |b| <= q/2: 1/2 plus the errors of c from
  // rounding a b, 1/q and their product, each 2^-53 of q/2 <= 2^49 s (65 and
  // less in units of q / 1024)
  static constexpr int kProduct2 = 512 + 3 * 66;
  static constexpr int reduced(int) { return kReduced; }
  static constexpr int kTrivial = 1;  // leading stages whose products by 1 are left out

  __device__ __forceinline__ E load(uint64_t v) const {  // canonical word
    return __longlong_as_double((long long)(v | 0x4330000000000000ull)) - 4503599627370496.0;
  }
  __device__ __forceinline__ static E raw(uint64_t v) { return __longlong_as_double((long long)v); }
  __device__ __forceinline__ static uint64_t bits(E x) { return (uint64_t)__double_as_longlong(x); }
  // [-q/2, q/2] (and the rounding of c)
  __device__ __forceinline__ E reduce(E x) const {
    return __builtin_fma(-__builtin_rint(x * qi), q, x);
  }
  // after a transform, before a subtraction or exchange: within 1/2
  __device__ __forceinline__ E settle(E x) const { return reduce(x); }
  __device__ __forceinline__ E sub(E a, E b) const { return a - b; }
  template <int X = kLimit>
  __device__ __forceinline__ uint64_t canon(E x) const {
    const E r = reduce(x);
    const E s = (r < 0.0 ? q : 0.0) + 4503599627370496.0;
    return bits(r + s) & 0x000fffffffffffffull;
  }
  __device__ __forceinline__ E mul(E a, Tw w) const {
    const E wv = raw(w.w);
    const E h = a * wv;
    const E c = __builtin_rint(a * raw(w.wp));
    return __builtin_fma(-c, q, h) + __builtin_fma(a, wv, -h);
  }
  // a b mod q for two variable factors, |a b| <= 2^52 q
  __device__ __forceinline__ E mul2(E a, E b) const {
    const E h = a * b;
    const E c = __builtin_rint(h * qi);
    return __builtin_fma(-c, q, h) + __builtin_fma(a, b, -h);
  }
  template <bool RED>
  __device__ __forceinline__ void bfly(E &x, E &y, Tw w) const {
    const E t = mul(y, w);
    const E a = RED ? reduce(x) : x;
    x = a + t;
    y = a - t;
  }
  // product by 1, |y| <= X q / 1024
  template <bool RED, int X>
  __device__ __forceinline__ void bfly1(E &x, E &y) const {
    const E a = RED ? reduce(x) : x, t = RED ? reduce(y) : y;
    x = a + t;
    y = a - t;
  }
};

template <int LIM>
struct ArI {
  using E = uint64_t;
  static constexpr bool kFloat = false;
  uint64_t q, nq;

  static constexpr bool fits(int x) { return x <= LIM * 1024; }
  static constexpr int product(int) { return 2048; }
  static constexpr int kCanonical = 1024;
  static constexpr int kReduced = LIM * 512;
  static constexpr int reduced(int) { return kReduced; }
  static constexpr int kTrivial = LIM >= 16 ? 3 : 1;

  __device__ __forceinline__ E load(uint64_t v) const { return v; }
  __device__ __forceinline__ static E raw(uint64_t v) { return v; }
  __device__ __forceinline__ static uint64_t bits(E x) { return x; }
  __device__ __forceinline__ E half(E x) const { return csub(x, LIM / 2 * q, LIM / 2 * nq); }
  // [0, X q / 1024) -> [0, q)
  template <int X = LIM * 1024>
  __device__ __forceinline__ uint64_t canon(E x) const {
    if constexpr (X > 8192) x = csub(x, 8 * q, 8 * nq);
    if constexpr (X > 4096) x = csub(x, 4 * q, 4 * nq);
    if constexpr (X > 2048) x = csub(x, 2 * q, 2 * nq);
    return csub(x, q, nq);
  }
  __device__ __forceinline__ E settle(E x) const { return canon(x); }
  __device__ __forceinline__ E sub(E a, E b) const { return a - b + q; }  // a, b in [0, q]
  __device__ __forceinline__ E mul(E a, Tw w) const {
    return shoup_lazy(a, w.w, w.wp, Qn{q, nq});
  }
  template <bool RED>
  __device__ __forceinline__ void bfly(E &x, E &y, Tw w) const {
    const E t = mul(y, w);
    const E a = RED ? half(x) : x;
    x = a + t;
    y = a - t + 2 * q;
  }
  template <bool RED, int X>
  __device__ __forceinline__ void bfly1(E &x, E &y) const {
    constexpr int B = ((RED ? (X < kReduced ? X : kReduced) : X) + 1023) / 1024;
    const E a = RED ? half(x) : x, t = RED ? half(y) : y;
    x = a + t;
    y = a - t + B * q;
  }
};

// Runs f with the arithmetic of a modulus (uniform over the workgroup).
template <class F>
__device__ __forceinline__ void with_arith(const ModConst &m, F &&f) {
  if (m.qd != 0.0)
    f(ArF{m.qd, m.qid});
  else if (m.q < (1ull << 60))
    f(ArI<16>{m.q, m.nq});
  else
    f(ArI<8>{m.q, m.nq});
}

// Value bounds (units of q / 1024) on entry to each of S stages, for values
// within X0 on entry to the first, and whether a stage reduces first.  The
// first TRIV stages hold butterflies whose product by 1 is left out (all of
// the first stage's when CYCLIC).
template <class Ar, int S, bool CYCLIC>
struct Bounds {
  int x[S + 1] = {};
  bool red[S + 1] = {};
  constexpr explicit Bounds(int x0) {
    x[0] = x0;
    for (int s = 0; s < S; s++) {
      const bool all = CYCLIC && s == 0, some = CYCLIC && s < Ar::kTrivial;
      int v = x[s];
      for (int pass = 0; pass < 2; pass++) {
        const int p = v + Ar::product(x[s]);
        const int t = 2 * v;
        const int next = all ? t : some && t > p ? t : p;
        x[s + 1] = next;
        if (Ar::fits(next)) break;
        red[s] = true;
        v = Ar::reduced(v);
      }
    }
  }
};

// ---- pass geometries ---------------------------------------------------------

// log2 of the order of the natural-order inverse root table: entry j is
// omega^-j, omega a primitive 2^kRootLog-th root (j < 2^(kRootLog - 1)); an
// R-point stage of half width 2^beta reads entry j << (kRootLog - 1 - beta)
constexpr int kRootLog = 10;

// Twiddles that differ between the lanes of a wavefront are read from a copy
// in LDS, made once per workgroup while the first data loads are in flight: a
// global load in every stage put its latency (several hundred cycles, more
// than a stage's arithmetic) on the path of each.  Lane-uniform twiddles stay
// scalar loads.  Entry i sits at i + i / 4, so that strided reads of 16-byte
// entries spread over the banks.
__device__ __forceinline__ int twidx(int i) { return i + (i >> 2); }
// forward: entries [0, R) (strided) or [0, R/2); inverse: omega_R^-j, j < R/2
template <int COUNT, int STEP, int THREADS>
__device__ __forceinline__ void fill_tw(Tw *l, const Tw *w) {
#pragma unroll
  for (int i0 = 0; i0 < COUNT; i0 += THREADS) {
    const int i = i0 + threadIdx.x;
    if (COUNT % THREADS == 0 || i < COUNT) l[twidx(i)] = w[i * STEP];
  }
}

// Geometry of one pass: R-point sub-transforms of an N-point limb, two
// layouts of P = 2^ceil(log2(R)/2) points a thread: interleaved (thread r
// holds points r + T i) and blocked (r P + v), one LDS exchange between them.
template <int LOGR, int LOGN, bool STRIDED>
struct Pass2 {
  static constexpr int R = 1 << LOGR;
  static constexpr int LOGP = (LOGR + 1) / 2;
  static constexpr int P = 1 << LOGP;
  static constexpr int LT = LOGR - LOGP;
  static constexpr int T = R / P;                 // threads per sub-transform
  static constexpr int THREADS = kNttThreads;
  static constexpr int TR = THREADS / T;          // sub-transforms per workgroup
  static constexpr int N = 1 << LOGN;
  static constexpr int OTHER = N / R;             // sub-transforms per limb
  static constexpr int S = R + R / P + 1;         // LDS words per sub-transform
  static constexpr int LDS_WORDS = TR * S;
  static constexpr int BLOCKS = OTHER / TR;       // workgroups per limb

  __device__ static int lidx(int c, int p) { return c * S + p + (p >> LOGP); }
  // word offset in the limb of point p of sub-transform g
  __device__ static size_t gaddr(int g, int p) {
    return STRIDED ? (size_t)p * OTHER + g : (size_t)g * R + p;
  }
  __device__ static int sub(int tid) { return STRIDED ? tid % TR : tid / T; }
  __device__ static int lane(int tid) { return STRIDED ? tid / TR : tid % T; }
  // point held in register i (interleaved) / v (blocked)
  __device__ static int ipoint(int r, int i) { return r + T * i; }
  __device__ static int bpoint(int r, int v) { return r * P + v; }

  // LDS copies of the lane-dependent twiddles (a barrier must follow).  A
  // 1024-point pass reads them from memory: its data take 68 KB of LDS, and with
  // the copies (88 KB, 104 KB with the inverse's row factors) a CU holds one
  // workgroup instead of two.  N = 2^17 in both directions, us a row: with the
  // copies 2.92 on doubles and 3.90 on integers, without 2.71 and 3.35.
  static constexpr bool TW_LDS = LOGR <= 9;
  static constexpr int TW_LEN = !TW_LDS ? 1 : STRIDED ? R + R / 4 : R / 2 + R / 8;
  __device__ static void fill_forward(Tw *lw, const Tw *w) {
    if constexpr (TW_LDS) fill_tw<STRIDED ? R : R / 2, 1, THREADS>(lw, w);
  }
  __device__ static void fill_inverse(Tw *lw, const Tw *w) {
    if constexpr (TW_LDS) fill_tw<R / 2, 1 << (kRootLog - LOGR), THREADS>(lw, w);
  }

  // contiguous pass, interleaved layout: x_i <- x_i t[i] (t: the limb's twist
  // or inverse-twist table, indexed like the data)
  template <class Ar>
  __device__ static void twist(typename Ar::E (&x)[P], int g, int r, const Tw *t, Ar ar) {
    static_assert(!STRIDED, "twists belong to the contiguous pass");
#pragma unroll
    for (int i = 0; i < P; i++) x[i] = ar.mul(x[i], t[gaddr(g, ipoint(r, i))]);
  }

  // A layout switch exchanges values among the T threads of one
  // sub-transform through its own LDS rows.  In the contiguous pass those
  // threads are consecutive and T divides 64, so they share one wavefront:
  // a wavefront-scope fence keeps the compiler from moving the LDS reads
  // above the writes (or the next writes above the reads), and a wavefront's
  // LDS operations complete in issue order, so no workgroup barrier is
  // needed.  The strided pass spreads a sub-transform over the workgroup.
  static_assert(STRIDED || (T <= 64 && 64 % T == 0), "sub-transform must fit one wavefront");
  __device__ static void exchange_sync() {
    if constexpr (STRIDED) {
      __syncthreads();
    } else {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  template <class E>
  __device__ static void to_blocked(uint64_t *lds, E (&x)[P], int c, int r) {
    E *l = (E *)lds;
#pragma unroll
    for (int i = 0; i < P; i++) l[lidx(c, ipoint(r, i))] = x[i];
    exchange_sync();
#pragma unroll
    for (int v = 0; v < P; v++) x[v] = l[lidx(c, bpoint(r, v))];
    exchange_sync();
  }
  template <class E>
  __device__ static void to_interleaved(uint64_t *lds, E (&x)[P], int c, int r) {
    E *l = (E *)lds;
#pragma unroll
    for (int v = 0; v < P; v++) l[lidx(c, bpoint(r, v))] = x[v];
    exchange_sync();
#pragma unroll
    for (int i = 0; i < P; i++) x[i] = l[lidx(c, ipoint(r, i))];
    exchange_sync();
  }

  // forward stages on values within X0 (units of q / 1024): interleaved in,
  // blocked out
  template <class Ar, int X0>
  __device__ static void forward(uint64_t *lds, typename Ar::E (&x)[P], int c, int r,
                                 const Tw *w, const Tw *lw, Ar ar) {
    constexpr Bounds<Ar, LOGR, !STRIDED> B(X0);
    stages<Ar, X0, 0, LOGP>(x, r, w, lw, ar);
    to_blocked(lds, x, c, r);
    stages<Ar, X0, LOGP, LOGR>(x, r, w, lw, ar);
    static_assert(Ar::fits(B.x[LOGR]), "forward pass out of range");
  }

  // inverse stages: blocked in, interleaved out (before the twist or row
  // factor); w: the natural-order inverse roots
  template <class Ar, int X0>
  __device__ static void inverse(uint64_t *lds, typename Ar::E (&x)[P], int c, int r,
                                 const Tw *w, const Tw *lw, Ar ar) {
    constexpr Bounds<Ar, LOGR, true> B(X0);
    istages<Ar, X0, 0, LT>(x, r, w, lw, ar);
    to_interleaved(lds, x, c, r);
    istages<Ar, X0, LT, LOGR>(x, r, w, lw, ar);
    static_assert(Ar::fits(B.x[LOGR]), "inverse pass out of range");
  }

 private:
  template <class Ar, int X0, int S0, int S1>
  __device__ static void stages(typename Ar::E (&x)[P], int r, const Tw *w, const Tw *lw, Ar ar) {
    if constexpr (S0 < S1) {
      constexpr Bounds<Ar, LOGR, !STRIDED> B(X0);
      constexpr bool IL = S0 < LOGP;
      constexpr int h = IL ? P >> (S0 + 1) : R >> (S0 + 1);
#pragma unroll
      for (int i = 0; i < P; i++) {
        if (i & h) continue;
        const int grp = (IL ? i >> (LOGP - S0) : bpoint(r, i) >> (LOGR - S0)) +
                        (STRIDED ? 1 << S0 : 0);
        if (!STRIDED && IL && S0 < Ar::kTrivial && i >> (LOGP - S0) == 0)
          ar.template bfly1<B.red[S0], B.x[S0]>(x[i], x[i + h]);
        else
          ar.template bfly<B.red[S0]>(x[i], x[i + h],
                                      IL || !TW_LDS ? w[grp] : lw[twidx(grp)]);
      }
      stages<Ar, X0, S0 + 1, S1>(x, r, w, lw, ar);
    }
  }
  template <class Ar, int X0, int S0, int S1>
  __device__ static void istages(typename Ar::E (&x)[P], int r, const Tw *w, const Tw *lw, Ar ar) {
    if constexpr (S0 < S1) {
      constexpr Bounds<Ar, LOGR, true> B(X0);
      constexpr bool BL = S0 < LT;   // blocked layout
      constexpr int h = BL ? 1 << S0 : 1 << (S0 - LT);
#pragma unroll
      for (int i = 0; i < P; i++) {
        if (i & h) continue;
        const int j = BL ? i & (h - 1) : r + T * (i & (h - 1));
        if (BL && S0 < Ar::kTrivial && (i & (h - 1)) == 0)
          ar.template bfly1<B.red[S0], B.x[S0]>(x[i], x[i + h]);
        else
          ar.template bfly<B.red[S0]>(x[i], x[i + h],
                                      BL || !TW_LDS ? w[j << (kRootLog - 1 - S0)]
                                                    : lw[twidx(j << (LOGR - 1 - S0))]);
      }
      istages<Ar, X0, S0 + 1, S1>(x, r, w, lw, ar);
    }
  }
};

// A pass of R = 2^LOGR points, LOGR = 7..9, with P = 8 points a thread (T =
// R / 8 threads a sub-transform; in the contiguous pass inside one wavefront)
// in three layouts of the point index p (bits LOGR-1 .. 0), LM = LOGR - 6:
//   I (interleaved): thread r holds p = r + T k, so register k is the top 3
//     bits (twiddles of the forward stages uniform across the wavefront);
//   M (middle): register k is bits LOGR-4 .. LOGR-6 and the thread the rest,
//     p = (r >> LM) R/8 + k 2^LM + (r mod 2^LM);
//   B (blocked): thread r holds p = 8 r + k, register k the low 3 bits
//     (twiddles of the inverse stages uniform).
// The pass takes two LDS exchanges each way instead of one, and in return a
// thread holds half the points: the fused contiguous passes keep three such
// arrays live, and a strided workgroup (16 columns or more, whole 128-byte
// lines) spreads its work over twice the wavefronts.
template <int LOGR, int LOGN, bool STRIDED>
struct Pass3 {
  static_assert(LOGR >= 7 && LOGR <= 9, "three-layout pass covers 128..512 points");
  static constexpr int R = 1 << LOGR;
  static constexpr int P = 8;
  static constexpr int T = R / P;                 // threads per sub-transform
  // strided: as many columns as the two-layout pass takes (the same grids)
  static constexpr int THREADS = STRIDED ? Pass2<LOGR, LOGN, true>::TR * T : kNttThreads;
  static constexpr int TR = THREADS / T;          // sub-transforms per workgroup
  static constexpr int N = 1 << LOGN;
  static constexpr int OTHER = N / R;             // sub-transforms per limb
  static constexpr int LM = LOGR - 6;
  static constexpr int S = R + R / 8 + 1;         // LDS words per sub-transform
  static constexpr int LDS_WORDS = TR * S;
  static constexpr int BLOCKS = OTHER / TR;       // workgroups per limb
  static_assert(STRIDED || (T <= 64 && 64 % T == 0), "sub-transform must fit one wavefront");

  __device__ static int lidx(int c, int p) { return c * S + p + (p >> 3); }
  __device__ static size_t gaddr(int g, int p) {
    return STRIDED ? (size_t)p * OTHER + g : (size_t)g * R + p;
  }
  __device__ static int sub(int tid) { return STRIDED ? tid % TR : tid / T; }
  __device__ static int lane(int tid) { return STRIDED ? tid / TR : tid % T; }
  __device__ static int ipoint(int r, int k) { return r + T * k; }
  __device__ static int mpoint(int r, int k) {
    return (r >> LM) * (R / 8) + (k << LM) + (r & ((1 << LM) - 1));
  }
  __device__ static int bpoint(int r, int k) { return r * P + k; }
  template <int LAYOUT>
  __device__ static int point(int r, int k) {
    return LAYOUT == 0 ? ipoint(r, k) : LAYOUT == 1 ? mpoint(r, k) : bpoint(r, k);
  }

  static constexpr int TW_LEN = STRIDED ? R + R / 4 : R / 2 + R / 8;
  __device__ static void fill_forward(Tw *lw, const Tw *w) {
    fill_tw<STRIDED ? R : R / 2, 1, THREADS>(lw, w);
  }
  __device__ static void fill_inverse(Tw *lw, const Tw *w) {
    fill_tw<R / 2, 1 << (kRootLog - LOGR), THREADS>(lw, w);
  }

  template <class Ar>
  __device__ static void twist(typename Ar::E (&x)[P], int g, int r, const Tw *t, Ar ar) {
#pragma unroll
    for (int k = 0; k < P; k++) x[k] = ar.mul(x[k], t[gaddr(g, ipoint(r, k))]);
  }

  // contiguous: a wavefront's LDS operations complete in issue order; the
  // fence keeps the compiler from moving them across each other
  __device__ static void sync() {
    if constexpr (STRIDED) {
      __syncthreads();
    } else {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  template <int FROM, int TO, class E>
  __device__ static void exchange(uint64_t *lds, E (&x)[P], int c, int r) {
    E *l = (E *)lds;
#pragma unroll
    for (int k = 0; k < P; k++) l[lidx(c, point<FROM>(r, k))] = x[k];
    sync();
#pragma unroll
    for (int k = 0; k < P; k++) x[k] = l[lidx(c, point<TO>(r, k))];
    sync();
  }
  template <class E>
  __device__ static void to_blocked(uint64_t *lds, E (&x)[P], int c, int r) {
    exchange<0, 2>(lds, x, c, r);
  }
  template <class E>
  __device__ static void to_interleaved(uint64_t *lds, E (&x)[P], int c, int r) {
    exchange<2, 0>(lds, x, c, r);
  }

  // forward stages: interleaved in, blocked out
  template <class Ar, int X0>
  __device__ static void forward(uint64_t *lds, typename Ar::E (&x)[P], int c, int r,
                                 const Tw *w, const Tw *lw, Ar ar) {
    constexpr Bounds<Ar, LOGR, !STRIDED> B(X0);
    stages<Ar, X0, 0, 3>(x, r, w, lw, ar);
    exchange<0, 1>(lds, x, c, r);
    stages<Ar, X0, 3, LOGR - 3>(x, r, w, lw, ar);
    exchange<1, 2>(lds, x, c, r);
    stages<Ar, X0, LOGR - 3, LOGR>(x, r, w, lw, ar);
    static_assert(Ar::fits(B.x[LOGR]), "forward pass out of range");
  }
  // inverse stages: blocked in, interleaved out
  template <class Ar, int X0>
  __device__ static void inverse(uint64_t *lds, typename Ar::E (&x)[P], int c, int r,
                                 const Tw *w, const Tw *lw, Ar ar) {
    constexpr Bounds<Ar, LOGR, true> B(X0);
    istages<Ar, X0, 0, 3>(x, r, w, lw, ar);
    exchange<2, 1>(lds, x, c, r);
    istages<Ar, X0, 3, LOGR - 3>(x, r, w, lw, ar);
    exchange<1, 0>(lds, x, c, r);
    istages<Ar, X0, LOGR - 3, LOGR>(x, r, w, lw, ar);
    static_assert(Ar::fits(B.x[LOGR]), "inverse pass out of range");
  }

 private:
  template <class Ar, int X0, int S0, int S1>
  __device__ static void stages(typename Ar::E (&x)[P], int r, const Tw *w, const Tw *lw, Ar ar) {
    if constexpr (S0 < S1) {
      constexpr Bounds<Ar, LOGR, !STRIDED> B(X0);
      constexpr int LAYOUT = S0 < 3 ? 0 : S0 < LOGR - 3 ? 1 : 2;
      constexpr int bit = LOGR - 1 - S0;   // of the point index
      constexpr int h = 1 << (LAYOUT == 0 ? 2 - S0 : LAYOUT == 1 ? bit - LM : bit);
#pragma unroll
      for (int k = 0; k < P; k++) {
        if (k & h) continue;
        const int grp = (LAYOUT == 0 ? k >> (3 - S0) : point<LAYOUT>(r, k) >> (LOGR - S0)) +
                        (STRIDED ? 1 << S0 : 0);
        if (!STRIDED && LAYOUT == 0 && S0 < Ar::kTrivial && k >> (3 - S0) == 0)
          ar.template bfly1<B.red[S0], B.x[S0]>(x[k], x[k + h]);
        else
          ar.template bfly<B.red[S0]>(x[k], x[k + h], LAYOUT == 0 ? w[grp] : lw[twidx(grp)]);
      }
      stages<Ar, X0, S0 + 1, S1>(x, r, w, lw, ar);
    }
  }
  template <class Ar, int X0, int S0, int S1>
  __device__ static void istages(typename Ar::E (&x)[P], int r, const Tw *w, const Tw *lw, Ar ar) {
    if constexpr (S0 < S1) {
      constexpr Bounds<Ar, LOGR, true> B(X0);
      constexpr int LAYOUT = S0 < 3 ? 2 : S0 < LOGR - 3 ? 1 : 0;
      constexpr int h = 1 << (LAYOUT == 2 ? S0 : LAYOUT == 1 ? S0 - LM : S0 - (LOGR - 3));
#pragma unroll
      for (int k = 0; k < P; k++) {
        if (k & h) continue;
        const int j = LAYOUT == 2 ? k & (h - 1) : point<LAYOUT>(r, k) & ((1 << S0) - 1);
        if (LAYOUT == 2 && S0 < Ar::kTrivial && (k & (h - 1)) == 0)
          ar.template bfly1<B.red[S0], B.x[S0]>(x[k], x[k + h]);
        else
          ar.template bfly<B.red[S0]>(x[k], x[k + h],
                                      LAYOUT == 2 ? w[j << (kRootLog - 1 - S0)]
                                                  : lw[twidx(j << (LOGR - 1 - S0))]);
      }
      istages<Ar, X0, S0 + 1, S1>(x, r, w, lw, ar);
    }
  }
};

// Contiguous pass of R = 2^LOGR points, LOGR = 7 or 8, with P = 4 points a
// thread (T = R / 4 <= 64 threads a sub-transform, inside one wavefront) in
// four layouts: in layout q the thread holds the points that differ in the two
// bits BIT(q), BIT(q) + 1 of the point index (its other bits are the
// thread's), from the top two bits (q = 0) to the low two (q = 3).  A fourth
// layout costs one more LDS exchange than Pass3; in return the fused key
// switching kernels, which keep three to five such arrays live, take half the
// registers and run twice the wavefronts, which hides the latency of their
// loads and of the stages' chains.
template <int LOGR, int LOGN>
struct Pass4 {
  static_assert(LOGR == 7 || LOGR == 8, "four-layout pass covers 128 and 256 points");
  static constexpr bool STRIDED = false;
  static constexpr int R = 1 << LOGR;
  static constexpr int P = 4;
  static constexpr int T = R / P;
  static constexpr int THREADS = kNttThreads;
  static constexpr int TR = THREADS / T;
  static constexpr int N = 1 << LOGN;
  static constexpr int OTHER = N / R;
  // a pad of PAD words every 32 keeps the outer layouts free of bank conflicts
  // and the inner two at two lanes a bank, with constant address offsets
  static constexpr int PAD = LOGR == 8 ? 3 : 5;
  static constexpr int S = R + PAD * (R / 32);
  static constexpr int LDS_WORDS = TR * S;
  static constexpr int BLOCKS = OTHER / TR;
  static constexpr int TW_LEN = R / 2 + R / 8;

  static constexpr int BIT(int q) {
    return q == 0 ? LOGR - 2 : q == 1 ? LOGR - 4 : q == 2 ? LOGR - 6 : 0;
  }
  // layout of stage bit b, forward (top bits first) and inverse (low first)
  static constexpr int fwd_layout(int b) { return (LOGR - 1 - b) / 2; }
  static constexpr int inv_layout(int b) { return b <= 1 ? 3 : (LOGR - 1 - b) / 2; }

  __device__ static int lidx(int c, int p) { return c * S + p + PAD * (p >> 5); }
  __device__ static size_t gaddr(int g, int p) { return (size_t)g * R + p; }
  __device__ static int sub(int tid) { return tid / T; }
  __device__ static int lane(int tid) { return tid % T; }
  template <int Q>
  __device__ static int point(int r, int k) {
    constexpr int b = BIT(Q);
    return ((r >> b) << (b + 2)) | (k << b) | (r & ((1 << b) - 1));
  }
  __device__ static int ipoint(int r, int k) { return point<0>(r, k); }
  __device__ static int bpoint(int r, int k) { return point<3>(r, k); }

  __device__ static void fill_forward(Tw *lw, const Tw *w) { fill_tw<R / 2, 1, THREADS>(lw, w); }
  __device__ static void fill_inverse(Tw *lw, const Tw *w) {
    fill_tw<R / 2, 1 << (kRootLog - LOGR), THREADS>(lw, w);
  }
  template <class Ar>
  __device__ static void twist(typename Ar::E (&x)[P], int g, int r, const Tw *t, Ar ar) {
#pragma unroll
    for (int k = 0; k < P; k++) x[k] = ar.mul(x[k], t[gaddr(g, ipoint(r, k))]);
  }
  __device__ static void sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  template <int FROM, int TO, class E>
  __device__ static void exchange(uint64_t *lds, E (&x)[P], int c, int r) {
    E *l = (E *)lds;
#pragma unroll
    for (int k = 0; k < P; k++) l[lidx(c, point<FROM>(r, k))] = x[k];
    sync();
#pragma unroll
    for (int k = 0; k < P; k++) x[k] = l[lidx(c, point<TO>(r, k))];
    sync();
  }
  template <class E>
  __device__ static void to_blocked(uint64_t *lds, E (&x)[P], int c, int r) {
    exchange<0, 3>(lds, x, c, r);
  }
  template <class E>
  __device__ static void to_interleaved(uint64_t *lds, E (&x)[P], int c, int r) {
    exchange<3, 0>(lds, x, c, r);
  }
  template <class Ar, int X0>
  __device__ static void forward(uint64_t *lds, typename Ar::E (&x)[P], int c, int r,
                                 const Tw *w, const Tw *lw, Ar ar) {
    constexpr Bounds<Ar, LOGR, true> B(X0);
    static_assert(Ar::fits(B.x[LOGR]), "forward pass out of range");
    stages<Ar, X0, 0>(lds, x, c, r, w, lw, ar);
  }
  template <class Ar, int X0>
  __device__ static void inverse(uint64_t *lds, typename Ar::E (&x)[P], int c, int r,
                                 const Tw *w, const Tw *lw, Ar ar) {
    constexpr Bounds<Ar, LOGR, true> B(X0);
    static_assert(Ar::fits(B.x[LOGR]), "inverse pass out of range");
    istages<Ar, X0, 0>(lds, x, c, r, w, lw, ar);
  }

 private:
  template <class Ar, int X0, int S0>
  __device__ static void stages(uint64_t *lds, typename Ar::E (&x)[P], int c, int r, const Tw *w,
                                const Tw *lw, Ar ar) {
    constexpr Bounds<Ar, LOGR, true> B(X0);
    constexpr int bit = LOGR - 1 - S0, Q = fwd_layout(bit), h = 1 << (bit - BIT(Q));
#pragma unroll
    for (int k = 0; k < P; k++) {
      if (k & h) continue;
      const int grp = Q == 0 ? k >> (2 - S0) : point<Q>(r, k) >> (LOGR - S0);
      if (Q == 0 && S0 < Ar::kTrivial && k >> (2 - S0) == 0)
        ar.template bfly1<B.red[S0], B.x[S0]>(x[k], x[k + h]);
      else
        ar.template bfly<B.red[S0]>(x[k], x[k + h], Q == 0 ? w[grp] : lw[twidx(grp)]);
    }
    if constexpr (S0 + 1 < LOGR) {
      constexpr int QN = fwd_layout(bit - 1);
      if constexpr (QN != Q) exchange<Q, QN>(lds, x, c, r);
      stages<Ar, X0, S0 + 1>(lds, x, c, r, w, lw, ar);
    }
  }
  template <class Ar, int X0, int S0>
  __device__ static void istages(uint64_t *lds, typename Ar::E (&x)[P], int c, int r, const Tw *w,
                                 const Tw *lw, Ar ar) {
    constexpr Bounds<Ar, LOGR, true> B(X0);
    constexpr int Q = inv_layout(S0), h = 1 << (S0 - BIT(Q));
#pragma unroll
    for (int k = 0; k < P; k++) {
      if (k & h) continue;
      const int j = Q == 3 ? k & (h - 1) : point<Q>(r, k) & ((1 << S0) - 1);
      if (Q == 3 && S0 < Ar::kTrivial && (k & (h - 1)) == 0)
        ar.template bfly1<B.red[S0], B.x[S0]>(x[k], x[k + h]);
      else
        ar.template bfly<B.red[S0]>(x[k], x[k + h],
                                    Q == 3 ? w[j << (kRootLog - 1 - S0)]
                                           : lw[twidx(j << (LOGR - 1 - S0))]);
    }
    if constexpr (S0 + 1 < LOGR) {
      constexpr int QN = inv_layout(S0 + 1);
      if constexpr (QN != Q) exchange<Q, QN>(lds, x, c, r);
      istages<Ar, X0, S0 + 1>(lds, x, c, r, w, lw, ar);
    }
  }
};

// The pass geometry of a split: strided passes of 128 to 512 points in three
// layouts, contiguous passes of 128 and 256 points in four and of 512 in three,
// smaller ones in two.  Measured against two layouts (16 points a thread) with
// the same arithmetic, N = 2^16: the scaled inverse strided pass of 16 rows
// 10.4 -> 9.7 us, the single-target conversions 26 -> 21 us; against three
// layouts (8 points) the contiguous key product of 8 slots of 24 limbs
// 374 -> 317 us, of one slot 58 -> 46 us.
constexpr int pass_kind(int logr, bool strided) {
  if (strided) return logr >= 7 && logr <= 9 ? 3 : 2;
  return logr == 7 || logr == 8 ? 4 : logr == 9 ? 3 : 2;
}
template <int KIND, int LOGR, int LOGN, bool STRIDED>
struct PassPick {
  using type = Pass2<LOGR, LOGN, STRIDED>;
};
template <int LOGR, int LOGN, bool STRIDED>
struct PassPick<3, LOGR, LOGN, STRIDED> {
  using type = Pass3<LOGR, LOGN, STRIDED>;
};
template <int LOGR, int LOGN>
struct PassPick<4, LOGR, LOGN, false> {
  using type = Pass4<LOGR, LOGN>;
};
template <int LOGR, int LOGN, bool STRIDED>
using Pass = typename PassPick<pass_kind(LOGR, STRIDED), LOGR, LOGN, STRIDED>::type;

// Bounds between the passes: the contiguous pass's twist (and the row factor
// of the inverse strided pass) brings whatever the other stages left to one
// product's bound, which the next stages start from.
template <class Ar>
constexpr int twisted_bound() { return Ar::product(Ar::kFloat ? 8065 : 0); }

// What a basis conversion leaves: within 1/2 where it ran in doubles (S30 of
// ks_fused.hip), fully reduced words where it ran on integers.
template <class Ar, bool S30>
constexpr int converted_bound() { return Ar::kFloat && S30 ? Ar::kReduced : Ar::kCanonical; }
// The same plus ModDown's rounding term, which is within 1/2 (doubles) or a
// fully reduced word (integers).
template <class Ar, bool S30>
constexpr int moddown_bound() {
  return converted_bound<Ar, S30>() + (Ar::kFloat ? Ar::kReduced : Ar::kCanonical);
}

// Slot of the input that lands in slot j under X -> X^g (bit-reversed
// evaluation order: slot j holds the value at psi^(2 brv(j) + 1)).
__device__ __forceinline__ uint32_t galois_src(uint32_t j, uint32_t g, int log_n) {
  const uint32_t shift = 32 - log_n;
  const uint32_t e = 2 * (__brev(j) >> shift) + 1;
  const uint32_t se = (uint32_t)(((uint64_t)e * g) & ((2u << log_n) - 1));
  return __brev((se - 1) >> 1) >> shift;
}

}  // namespace hck

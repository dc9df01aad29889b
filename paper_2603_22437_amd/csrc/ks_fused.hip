// Hybrid key switching with the basis conversions, the key inner product and
// the ModDown tail fused into the NTT passes (ntt_core.h), for a batch of up
// to ks_slots inputs, each with its own switching key.
//
// KeySwitch(d) at level l with a switching key swk(s' -> s); d is read through
// the NTT-domain automorphism X -> X^g (g = 1: no automorphism), so a
// rotation never materializes phi_g(c):
//   K1  inverse contiguous pass of phi_g(d) over Q_l -> y          (gather;
//       also the copies of c0 and phi_g(d) for an output that aliases its
//       input)
//   K2  inverse strided pass, row factors with (Q_j / q_i)^-1      (digit scale)
//   K3  ModUp: per digit j and target limb t not in D_j, the fast basis
//       conversion of y's digit limbs computed at load time, then the
//       forward strided pass -> ext[j][t]
//   K4  special limbs t: forward contiguous pass of every digit's ext, then
//       acc_{0,1}[t] = sum_j d~_j[t] swk_j[t], then the inverse contiguous
//       pass of K5
//   K5  inverse strided pass of acc's P limbs, row factors with (P/p_k)^-1,
//       plus ((P-1)/2) (P/p_k)^-1 (the rounding term of ModDown)
//   K6  ModDown conversion P -> q_i (minus (P-1)/2) at load time, then the
//       forward strided pass -> conv
//   K7  Q limbs: the forward passes and key products of K4 (phi_g(d) itself on
//       the digit's own limbs), kept in registers, then the forward contiguous
//       pass of conv and out_i = (acc_i - conv_i) P^-1 (+ phi_g(addend)_i)
// Switching the special limbs first keeps the Q limbs' accumulators out of
// memory (2 (l + 1) rows a switch, written once and read once).
// Small switches take K4 over all limbs at once, and K7 is the tail alone
// (kTogetherMaxLog).
//
// Workspace: batch slot b occupies rows [b R, (b+1) R) of ws_ks (R rows of N
// words): y [L] | ext [dnum][L+K] | acc [2][L+K] | conv [2][L].  Rows between
// two passes hold words in their modulus' own arithmetic; y, the special rows
// after K5 and the accumulators of the paths that store them are fully
// reduced integers.
// Compiled once per ring, with HCK_LOGN its log2 N (build.py).
#include <algorithm>

#include "ntt_core.h"

namespace hck {

namespace {

// the largest kernel argument list (batch table, geometry, pointers) stays
// within the 4 KiB a kernel can take
static_assert(sizeof(KsBatch) + 256 <= 4096, "kernel arguments beyond 4 KiB");

struct KsGeom {
  uint32_t level, nq, ne, L, K, dnum, alpha, nm;
  uint32_t slot_rows;                       // rows per batch slot
  uint32_t off_ext, off_acc, off_conv;      // row offsets inside a slot
};

// workgroups (at one target each) from which the basis conversions pair
// targets: halved, they still fill the chip twice over at the paired kernel's
// occupancy (about 3 workgroups of 256 threads per CU)
constexpr size_t kPairMinBlocks = 3072;
// Rings whose conversions pair targets: strided passes of up to 256 points.  At
// N = 2^17 the paired workgroup takes 88 KB of LDS and 251 VGPRs, one workgroup
// of four wavefronts a CU, where the single-target one has sixteen: 16 rotations
// of 6 limbs and 2 special primes 1565 us paired, 924 single (moduli of 55 bits),
// 1169 and 796 (50 bits); with one twiddle table for both targets, which leaves
// room for a second workgroup, 1544 and 1087.
template <int LOGN>
constexpr bool kPairs = split_a(LOGN) <= 8;
// tiles up to which the inner products take two sets of wavefronts each: two
// a CU.  One special basis of 8 limbs at N = 2^16 (512 tiles) 22.6 -> 18.9 us;
// 24 limbs (1536 tiles) 45.9 -> 49.1 us, so larger launches do not.
constexpr size_t kSplitMaxBlocks = 512;
// Largest ring at which a switch of at most kSplitMaxBlocks tiles, over all its
// extended limbs, takes every key product in one launch and its accumulators
// through memory.  All its tiles run at once, so its time is the chain of its
// launches, and the Q limbs' products beside the special limbs' take one pass
// a digit off that chain; larger switches are bound by what they move.  One
// switch in its turn, special limbs first / all at once: N = 2^11, one limb and
// one special prime 51.4 / 46.3 us; N = 2^12, 12 limbs and 4 66.7 / 56.6 us;
// N = 2^15, 12 and 4 (512 tiles) 75.4 / 73.4 us, two of them (1024 tiles)
// 92.8 / 93.3 us, four 130 / 140 us; N = 2^17, 2 limbs and 2 (512 tiles)
// 79.0 / 79.6 us.
constexpr int kTogetherMaxLog = 15;

template <int LOGN>
__global__ __launch_bounds__(kNttThreads) void k_ks_intt_gather(
    uint64_t *__restrict__ ws, KsBatch kb, KsGeom kg, const ModConst *__restrict__ mc,
    const Tw *__restrict__ itn, const Tw *__restrict__ itt) {
  using G = Pass<split_b(LOGN), LOGN, false>;
  constexpr int P = G::P;
  __shared__ uint64_t lds[G::LDS_WORDS];
  __shared__ Tw lw[G::TW_LEN];
  const int li = blockIdx.z;  // limb i (modulus i)
  G::fill_inverse(lw, itn + (size_t)li * kRootLen);
  const uint32_t b = blockIdx.y;
  const size_t roff = (size_t)li * G::N;
  const uint64_t *d = kb.d[b];
  const uint32_t galois = kb.galois[b];
  uint64_t *y = ws + (size_t)b * kg.slot_rows * G::N;
  const int c = G::sub(threadIdx.x), r = G::lane(threadIdx.x);
  const int g = blockIdx.x * G::TR + c;
  if (const uint64_t *c0 = kb.add0_src[b]) {
    // an output aliasing its input: copy this tile of c0 and of phi_g(d) for
    // the last launch, which writes the output while other workgroups read
    // both (phi_g(d) into its digit's own ext row, which the ModUp leaves out)
    uint64_t *cp = const_cast<uint64_t *>(kb.add0[b]);
    uint64_t *dp = y + ((size_t)kg.off_ext + li / kg.alpha * kg.ne + li) * G::N;
#pragma unroll
    for (int i = 0; i < P; i++) {
      const size_t pos = G::gaddr(g, G::ipoint(r, i));
      cp[roff + pos] = c0[roff + pos];
      dp[pos] = d[roff + galois_src((uint32_t)pos, galois, LOGN)];
    }
  }
  with_arith(mc[li], [&](auto ar) {
    using Ar = decltype(ar);
    typename Ar::E x[P];
#pragma unroll
    for (int i = 0; i < P; i++)
      x[i] = ar.load(d[roff + galois_src((uint32_t)G::gaddr(g, G::ipoint(r, i)), galois, LOGN)]);
    __syncthreads();
    G::to_blocked(lds, x, c, r);
    G::template inverse<Ar, Ar::kCanonical>(lds, x, c, r, itn + (size_t)li * kRootLen, lw, ar);
    G::twist(x, g, r, itt + roff, ar);
#pragma unroll
    for (int i = 0; i < P; i++) y[roff + G::gaddr(g, G::ipoint(r, i))] = Ar::bits(x[i]);
  });
}

// Fast basis conversion of a thread's P points (interleaved layout of the
// strided pass) at load time, into NT target moduli at once:
//   x[t][i] = sum_{a < na} src[a N + pos_i] c_a  mod q_t
// in [0, q_t), from cv[t][a cstride].w (Montgomery form; the sum stays below
// q_t 2^64).  Points are taken CH at a time, with the CH loads of one source
// limb issued together so that their latencies overlap (one load, then a
// wait, per product leaves the conversion latency-bound); each loaded word
// serves every target.  This form takes any moduli.
template <class G, int NT>
__device__ __forceinline__ void bconv_words(uint64_t (&x)[NT][G::P],
                                            const uint64_t *__restrict__ src,
                                            const ConvC *const (&cv)[NT], uint32_t cstride,
                                            uint32_t na, int g, int r,
                                            const ModConst (&m)[NT]) {
  constexpr int P = G::P;
  constexpr int CH = P / NT;
#pragma unroll
  for (int c0 = 0; c0 < P; c0 += CH) {
    u128 acc[NT][CH];
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int k = 0; k < CH; k++) acc[t][k].lo = acc[t][k].hi = 0;
    for (uint32_t a = 0; a < na; a++) {
      uint64_t v[CH];
#pragma unroll
      for (int k = 0; k < CH; k++) v[k] = src[(size_t)a * G::N + G::gaddr(g, G::ipoint(r, c0 + k))];
#pragma unroll
      for (int t = 0; t < NT; t++) {
        const uint64_t c = cv[t][(size_t)a * cstride].w;
#pragma unroll
        for (int k = 0; k < CH; k++) mac_wide(acc[t][k], v[k], c);
      }
    }
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int k = 0; k < CH; k++) x[t][c0 + k] = redc(acc[t][k], m[t].q, m[t].qinv);
  }
}

// The same sums for moduli below 2^60 (sources v and constants c below
// 2^60), with both factors split into 30-bit halves, v = v1 2^30 + v0 and
// c = c1 2^30 + c0:
//   sum_a v c = L + 2^30 M + 2^60 H,
//   L = sum v0 c0, H = sum v1 c1, M = sum (v0 + v1)(c0 + c1) - L - H.
// L and H stay below na 2^60 <= 2^64 (a digit or the special basis holds at
// most 16 primes); for na <= 8 the true M does too, so its column may wrap on
// the way and three multiply-adds a product do.  Above 8 sources the cross
// products keep two columns (four multiply-adds).  The columns are combined
// into the 128-bit sum (the same integer as above, so the same REDC result)
// once per point.
template <class G, int NT>
__device__ __forceinline__ void bconv_halves(uint64_t (&x)[NT][G::P],
                                             const uint64_t *__restrict__ src,
                                             const ConvC *const (&cv)[NT], uint32_t cstride,
                                             uint32_t na, int g, int r,
                                             const ModConst (&m)[NT]) {
  constexpr int P = G::P;
  constexpr int CH = (P < 8 ? P : 8) / NT;
  constexpr uint32_t kLow30 = (1u << 30) - 1;
#pragma unroll
  for (int c0 = 0; c0 < P; c0 += CH) {
    uint64_t lo[NT][CH], m1[NT][CH], m2[NT][CH], hi[NT][CH];
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int k = 0; k < CH; k++) lo[t][k] = m1[t][k] = m2[t][k] = hi[t][k] = 0;
    uint64_t v[CH], nx[CH];
#pragma unroll
    for (int k = 0; k < CH; k++) nx[k] = src[G::gaddr(g, G::ipoint(r, c0 + k))];
    auto next = [&](uint32_t a) {  // takes limb a's words and loads limb a + 1's
      const size_t n = (size_t)(a + 1 < na ? a + 1 : a) * G::N;
#pragma unroll
      for (int k = 0; k < CH; k++) {
        v[k] = nx[k];
        nx[k] = src[n + G::gaddr(g, G::ipoint(r, c0 + k))];
      }
    };
    if (na <= 8) {
      for (uint32_t a = 0; a < na; a++) {
        next(a);
#pragma unroll
        for (int t = 0; t < NT; t++) {
          const uint64_t c = cv[t][(size_t)a * cstride].w;
          const uint32_t cl = (uint32_t)c & kLow30, ch = (uint32_t)(c >> 30), cs = cl + ch;
#pragma unroll
          for (int k = 0; k < CH; k++) {
            const uint32_t v0 = (uint32_t)v[k] & kLow30, v1 = (uint32_t)(v[k] >> 30);
            lo[t][k] += (uint64_t)v0 * cl;
            hi[t][k] += (uint64_t)v1 * ch;
            m1[t][k] += (uint64_t)(v0 + v1) * cs;
          }
        }
      }
#pragma unroll
      for (int t = 0; t < NT; t++)
#pragma unroll
        for (int k = 0; k < CH; k++) m1[t][k] -= lo[t][k] + hi[t][k];
    } else {
      for (uint32_t a = 0; a < na; a++) {
        next(a);
#pragma unroll
        for (int t = 0; t < NT; t++) {
          const uint64_t c = cv[t][(size_t)a * cstride].w;
          const uint32_t cl = (uint32_t)c & kLow30, ch = (uint32_t)(c >> 30);
#pragma unroll
          for (int k = 0; k < CH; k++) {
            const uint32_t v0 = (uint32_t)v[k] & kLow30, v1 = (uint32_t)(v[k] >> 30);
            lo[t][k] += (uint64_t)v0 * cl;
            m1[t][k] += (uint64_t)v0 * ch;
            m2[t][k] += (uint64_t)v1 * cl;
            hi[t][k] += (uint64_t)v1 * ch;
          }
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int k = 0; k < CH; k++) {
        const wide_t mid = (wide_t)m1[t][k] + m2[t][k];
        const wide_t y = (wide_t)lo[t][k] + (mid << 30) + ((wide_t)hi[t][k] << 60);
        u128 s;
        s.lo = (uint64_t)y;
        s.hi = (uint64_t)(y >> 64);
        x[t][c0 + k] = redc(s, m[t].q, m[t].qinv);
        // reduce this chunk before the next chunk's loads (the empty asm
        // takes the result and orders memory accesses, and emits nothing), so
        // that one chunk's columns are live at a time, not every chunk's
        asm volatile("" ::"v"(x[t][c0 + k]) : "memory");
      }
  }
}

// The sums for targets on doubles, within 1/2 q.  A source word less 2^49 is a
// double v, |v| <= 2^49 + 2^44, and the constant a centred double c.  The sum
// runs in T, which starts at 1.5 2^102 and stays in that binade, so that each
// multiply-add rounds to a multiple of 2^50, and the part rounded off is exact
// in a second multiply-add:
//   T' = T + v c (rounded),  E += v c - (T' - T),  |v c - (T' - T)| <= 2^49,
// four operations a product and no splitting of the source word.  (Splitting
// both factors into 25-bit halves took three multiply-adds a product and about
// seven operations a source: one rotation at N = 2^16 166.5 us against 163.6,
// 21 at level 3 559.6 against 550.6, on one card in turn.)  A source whose prime is not in the floating-point
// range has its bits from 50 on as one more factor v2 < 2^10 with the constant
// c 2^50 = f 2^50 + g mod t, f and g short: v2 f 2^50 is exact in T, v2 g in E.
// T and E are reduced every 8 sources; the host has checked that they stay
// exact over this context's constants (hck_context::conv_f).  The row after the
// last source undoes the 2^49.
template <class G, int NT>
__device__ __forceinline__ void bconv_float(double (&x)[NT][G::P],
                                            const uint64_t *__restrict__ src,
                                            const ConvC *const (&cv)[NT], uint32_t cstride,
                                            uint32_t na, const ModConst *__restrict__ ms, int g,
                                            int r, const ModConst (&m)[NT]) {
  constexpr int P = G::P;
  constexpr int CH = (P < 8 ? P : 8) / NT;
  constexpr uint64_t kExp = 0x4330000000000000ull;               // 2^52 + (low bits)
  constexpr double kOff = 4503599627370496.0 + 562949953421312.0;  // 2^52 + 2^49
  constexpr double kBase = 0x1.8p102;
#pragma unroll
  for (int c0 = 0; c0 < P; c0 += CH) {
    double sum[NT][CH], err[NT][CH];
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int k = 0; k < CH; k++) {
        sum[t][k] = kBase;
        err[t][k] = 0.0;
      }
    // what the columns stand for, an integer below 2^51: a reduction leaves
    // 2^-52 of its argument and q / 2
    auto value = [&](int t, int k) {
      const ArF ar{m[t].qd, m[t].qid};
      return ar.reduce(sum[t][k] - kBase) + ar.reduce(err[t][k]);
    };
    uint64_t v[CH], nx[CH];
#pragma unroll
    for (int k = 0; k < CH; k++) nx[k] = src[G::gaddr(g, G::ipoint(r, c0 + k))];
    for (uint32_t a = 0; a < na; a++) {
      const size_t n = (size_t)(a + 1 < na ? a + 1 : a) * G::N;
#pragma unroll
      for (int k = 0; k < CH; k++) {
        v[k] = nx[k];
        nx[k] = src[n + G::gaddr(g, G::ipoint(r, c0 + k))];
      }
      if (a == 8) {
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
          for (int k = 0; k < CH; k++) {
            err[t][k] = value(t, k);
            sum[t][k] = kBase;
          }
      }
      const bool wide = ms[a].qd == 0.0;  // uniform
      const uint64_t mask = wide ? (1ull << 50) - 1 : ~0ull;
#pragma unroll
      for (int k = 0; k < CH; k++) {
        const double d = __longlong_as_double((long long)((v[k] & mask) | kExp)) - kOff;
#pragma unroll
        for (int t = 0; t < NT; t++) {
          const double c = cv[t][(size_t)a * cstride].c;
          const double next = __builtin_fma(d, c, sum[t][k]);
          err[t][k] += __builtin_fma(d, c, sum[t][k] - next);
          sum[t][k] = next;
        }
        if (wide) {
          const double v2 = (double)(uint32_t)(v[k] >> 50);
#pragma unroll
          for (int t = 0; t < NT; t++) {
            const ConvC &c = cv[t][(size_t)a * cstride];
            sum[t][k] = __builtin_fma(v2, c.f, sum[t][k]);
            err[t][k] = __builtin_fma(v2, c.g, err[t][k]);
          }
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NT; t++) {
      const ArF ar{m[t].qd, m[t].qid};
      const double kt = cv[t][(size_t)na * cstride].c;
#pragma unroll
      for (int k = 0; k < CH; k++) {
        x[t][c0 + k] = ar.reduce(value(t, k) + kt);
        asm volatile("" ::"v"(x[t][c0 + k]) : "memory");  // one chunk at a time
      }
    }
  }
}

// The conversion in a target's arithmetic, within converted_bound.  S30: every
// modulus is below 2^60 and the columns of this context's constants stay exact
// in doubles; other contexts convert on whole words.
template <class G, int NT, bool S30, class Ar>
__device__ __forceinline__ void bconv(typename Ar::E (&x)[NT][G::P],
                                      const uint64_t *__restrict__ src,
                                      const ConvC *const (&cv)[NT], uint32_t cstride, uint32_t na,
                                      const ModConst *__restrict__ ms, int g, int r,
                                      const ModConst (&m)[NT], Ar ar) {
  if constexpr (Ar::kFloat && S30) {
    bconv_float<G, NT>(x, src, cv, cstride, na, ms, g, r, m);
  } else {
    uint64_t u[NT][G::P];
    if constexpr (S30)
      bconv_halves<G, NT>(u, src, cv, cstride, na, g, r, m);
    else
      bconv_words<G, NT>(u, src, cv, cstride, na, g, r, m);
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int i = 0; i < G::P; i++) x[t][i] = ar.load(u[t][i]);
  }
}

// The arithmetic of modulus m in a key-switching kernel: contexts whose
// moduli all lie below 2^60 (S30) need no narrower integer class.
template <bool S30, class F>
__device__ __forceinline__ void with_ks_arith(const ModConst &m, F &&f) {
  if (m.qd != 0.0)
    f(ArF{m.qd, m.qid});
  else if (S30 || m.q < (1ull << 60))
    f(ArI<16>{m.q, m.nq});
  else
    f(ArI<8>{m.q, m.nq});
}

// The conversions' pass: three layouts, except where two targets share a
// workgroup (two arrays of 16 points in two layouts keep more loads of a
// source in flight per register: 224 us against 254 us for 8 slots of 72 rows)
// and for conversions on whole words.
template <int LOGN, bool PAIR, bool S30>
using ConvPass = typename PassPick<PAIR || !S30 ? 2 : pass_kind(split_a(LOGN), true),
                                   split_a(LOGN), LOGN, true>::type;

// K3: workgroup y converts the targets of group y (one, or two of one
// arithmetic) of slot z.  Two targets share the reads of the sources.
template <int LOGN, bool PAIR, bool S30>
__global__ __launch_bounds__((ConvPass<LOGN, PAIR, S30>::THREADS))
__attribute__((amdgpu_waves_per_eu(!PAIR && S30 ? 4 : 3))) void k_modup_strided(
    uint64_t *__restrict__ ws, const ConvGroup *__restrict__ groups,
    const ConvC *__restrict__ conv, KsGeom kg, const ModConst *__restrict__ mc,
    const Tw *__restrict__ tw) {
  using G = ConvPass<LOGN, PAIR, S30>;
  constexpr int P = G::P, NT = PAIR ? 2 : 1;
  __shared__ uint64_t lds[G::LDS_WORDS];
  __shared__ Tw lw[NT][G::TW_LEN];
  const ConvGroup gr = groups[blockIdx.y];
  const uint32_t lo = gr.digit * kg.alpha;
  const uint32_t na = min(kg.alpha, kg.nq - lo);
  uint64_t *slot = ws + (size_t)blockIdx.z * kg.slot_rows * G::N;
  const ConvC *cd = conv + (size_t)gr.digit * (kg.alpha + 1) * kg.nm;
  const uint64_t *src = slot + (size_t)lo * G::N;
  const int c = G::sub(threadIdx.x), r = G::lane(threadIdx.x);
  const int g = blockIdx.x * G::TR + c;
  const int mi[2] = {gr.mod[0], gr.mod[1]};
  const ConvC *cvs[NT];
  ModConst ms[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) {
    cvs[t] = cd + mi[t];
    ms[t] = mc[mi[t]];
    G::fill_forward(lw[t], tw + (size_t)mi[t] * kTwLen);
  }
  with_ks_arith<S30>(ms[0], [&](auto ar) {
    using Ar = decltype(ar);
    typename Ar::E x[NT][P];
    bconv<G, NT, S30>(x, src, cvs, kg.nm, na, mc + lo, g, r, ms, ar);
#pragma unroll
    for (int t = 0; t < NT; t++) {
      if (t == 1 && gr.n < 2) break;
      Ar at = ar;
      if (t == 1) {
        if constexpr (Ar::kFloat) at = Ar{ms[NT - 1].qd, ms[NT - 1].qid};
        else at = Ar{ms[NT - 1].q, ms[NT - 1].nq};
      }
      if (t == 0) __syncthreads();
      G::template forward<Ar, Ar::kCanonical>(lds, x[t], c, r, tw + (size_t)mi[t] * kTwLen, lw[t],
                                              at);
      uint64_t *out = slot + (size_t)gr.row[t] * G::N;
#pragma unroll
      for (int v = 0; v < P; v++) out[G::gaddr(g, G::bpoint(r, v))] = Ar::bits(x[t][v]);
    }
  });
}

// K4 and K7: per extended limb t, the forward contiguous pass of each digit
// and the inner product with the slot's key; then for a special limb the
// inverse contiguous pass of both accumulators, and for a Q limb with TAIL
// ModDown's tail on them in registers (without, they are stored).  The launch
// covers limbs first, first + 1, ... of the list special limbs, then Q limbs.
//
// A workgroup's time is a chain of passes (one a digit, one a polynomial),
// each waiting for its own loads.  In launches that leave the chip room
// (SPLIT) a tile takes two sets of wavefronts: set h takes the digits h,
// h + 2, ..., the sets exchange partial sums through LDS, and set h finishes
// polynomial h, so the chain is half as long.
template <int LOGN, bool TAIL, bool SPLIT>
__global__ __launch_bounds__(kNttThreads * (SPLIT ? 2 : 1))
__attribute__((amdgpu_waves_per_eu(4))) void k_ks_contig_inner(
    uint64_t *__restrict__ ws, KsBatch kb, KsGeom kg, uint32_t first, int canonical,
    const ModConst *__restrict__ mc, const Tw *__restrict__ tw, const Tw *__restrict__ tt,
    const Tw *__restrict__ itn, const Tw *__restrict__ itt, const Tw *__restrict__ pinv) {
  using G = Pass<split_b(LOGN), LOGN, false>;
  constexpr int P = G::P;
  __shared__ uint64_t lds_[SPLIT ? 2 : 1][G::LDS_WORDS];
  // A workgroup of whole wavefronts' sub-transforms covers TILE consecutive
  // words of a row, a wavefront WTILE of them.  Each digit's two
  // key rows over those words are copied into LDS by direct global-to-LDS
  // loads issued before the digit's forward pass, so the copy runs under the
  // transform without holding registers; each wavefront reads only the words
  // it copied (no workgroup barrier).
  constexpr bool KEY_LDS = !SPLIT && split_b(LOGN) >= 7;
  constexpr int TILE = kNttThreads * P, WTILE = 64 * P;
  __shared__ uint64_t ktile[KEY_LDS ? 2 * TILE : 1];
  __shared__ Tw lw[G::TW_LEN];
  const uint32_t z = first + blockIdx.z;
  const uint32_t t = z < kg.K ? kg.nq + z : z - kg.K;
  const uint32_t b = blockIdx.y;
  const uint32_t mi = t < kg.nq ? t : kg.L + (t - kg.nq);
  const ModConst m = mc[mi];
  const int tid = threadIdx.x % kNttThreads;
  const uint32_t set =
      SPLIT ? __builtin_amdgcn_readfirstlane(threadIdx.x / kNttThreads) : 0;
  uint64_t *lds = lds_[set];
  const int c = G::sub(tid), r = G::lane(tid);
  const int g = blockIdx.x * G::TR + c;
  const size_t krow = (size_t)kg.nm * G::N;
  uint64_t *slot = ws + (size_t)b * kg.slot_rows * G::N;
  const uint64_t *d = kb.d[b];
  const uint64_t *key = kb.key[b];
  const uint32_t galois = kb.galois[b];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const size_t tile0 = (size_t)blockIdx.x * TILE;  // first word of the tile in a row
  tw += (size_t)mi * kTwLen;
  tt += (size_t)mi * G::N;
  itn += (size_t)mi * kRootLen;
  if (set == 0) G::fill_forward(lw, tw);
  __syncthreads();
  with_arith(m, [&](auto ar) {
    using Ar = decltype(ar);
    using E = typename Ar::E;
    E a0[P], a1[P], x[P];
#pragma unroll
    for (int i = 0; i < P; i++) a0[i] = a1[i] = 0;
    for (uint32_t j = set; j < kg.dnum; j += SPLIT ? 2 : 1) {
      const uint32_t lo = j * kg.alpha;
      if (lo >= kg.nq) break;
      const uint32_t hi = min(lo + kg.alpha, kg.nq);
      const uint64_t *kbp = key + 2 * j * krow + (size_t)mi * G::N;
      const uint64_t *kap = kbp + krow;
      uint64_t k0[P], k1[P];
      // this wavefront's words of each key row in loads of 16 bytes a lane
      // (1 KiB a load), lane l's bytes landing at 16 l.  Loads complete in
      // issue order, so the copy is issued after the digit's own loads (a wait
      // for those does not wait for it) and before the transform it hides under.
      auto copy_keys = [&]() {
        if constexpr (KEY_LDS) {
#pragma unroll
          for (int rr = 0; rr < 2; rr++) {
            const uint64_t *src = (rr ? kap : kbp) + tile0 + wave * WTILE + 2 * (threadIdx.x % 64);
#pragma unroll
            for (int i = 0; i < P / 2; i++)
              __builtin_amdgcn_global_load_lds(
                  (const void *)(src + 128 * i),
                  (__attribute__((address_space(3))) void *)&ktile[rr * TILE + wave * WTILE + 128 * i],
                  16, 0, 0);
          }
        } else {
#pragma unroll
          for (int i = 0; i < P; i++) {
            const size_t pos = G::gaddr(g, G::ipoint(r, i));
            k0[i] = kbp[pos];
            k1[i] = kap[pos];
          }
        }
      };
      if (t >= lo && t < hi) {
        copy_keys();
        // phi_g(d), or the first launch's copy of it where the output aliases d
        const uint64_t *own = d + (size_t)t * G::N;
        uint32_t gs = galois;
        if (kb.add0_src[b]) {
          own = slot + ((size_t)kg.off_ext + j * kg.ne + t) * G::N;
          gs = 1;
        }
#pragma unroll
        for (int i = 0; i < P; i++)
          x[i] = ar.load(own[galois_src((uint32_t)G::gaddr(g, G::ipoint(r, i)), gs, LOGN)]);
      } else {
        const uint64_t *e = slot + ((size_t)kg.off_ext + j * kg.ne + t) * G::N;
#pragma unroll
        for (int i = 0; i < P; i++) x[i] = Ar::raw(e[G::gaddr(g, G::ipoint(r, i))]);
        G::twist(x, g, r, tt, ar);
        copy_keys();
        G::template forward<Ar, twisted_bound<Ar>()>(lds, x, c, r, tw, lw, ar);
#pragma unroll
        for (int v = 0; v < P; v++) x[v] = ar.settle(x[v]);
        G::to_interleaved(lds, x, c, r);
      }
      // the compiler does not order reads of ktile after the copies into it:
      // wait for this wavefront's copies (all its earlier loads are in use by
      // now) before the first read
      if constexpr (KEY_LDS) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
      for (int i = 0; i < P; i++) {
        if constexpr (KEY_LDS) {
          const size_t pos = G::gaddr(g, G::ipoint(r, i));
          k0[i] = ktile[pos - tile0];
          k1[i] = ktile[TILE + pos - tile0];
        }
        if constexpr (Ar::kFloat) {
          // |x| <= q and a centred key: products within kProduct2
          a0[i] += ar.mul2(x[i], Ar::raw(k0[i]));
          a1[i] += ar.mul2(x[i], Ar::raw(k1[i]));
        } else {
          a0[i] = add_mod(a0[i], redc(mul_wide(x[i], k0[i]), m.q, m.qinv), m.q);
          a1[i] = add_mod(a1[i], redc(mul_wide(x[i], k1[i]), m.q, m.qinv), m.q);
        }
      }
      if constexpr (Ar::kFloat) {
        // reduced after 8 products (a set's: after 4), so that the sum before a
        // reduction, and what the tail takes conv from, stay in range
        static_assert(ArF::fits(ArF::kReduced + 8 * ArF::kProduct2));
        static_assert(ArF::fits(ArF::kReduced + 7 * ArF::kProduct2 + ArF::kReduced));
        static_assert(ArF::fits(2 * (ArF::kReduced + 3 * ArF::kProduct2) + ArF::kReduced));
        if ((j & 7) >= (SPLIT ? 6 : 7)) {
#pragma unroll
          for (int i = 0; i < P; i++) {
            a0[i] = ar.reduce(a0[i]);
            a1[i] = ar.reduce(a1[i]);
          }
        }
      }
    }
    if constexpr (SPLIT) {
      // set 0 gives its sum of polynomial 1 for set 1's of polynomial 0 (the
      // words go to every wavefront's rows: after all of them are done)
      __syncthreads();
#pragma unroll
      for (int i = 0; i < P; i++)
        lds_[set][i * kNttThreads + tid] = Ar::bits(set ? a0[i] : a1[i]);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < P; i++) {
        const E o = Ar::raw(lds_[set ^ 1][i * kNttThreads + tid]);
        const E own = set ? a1[i] : a0[i];
        if constexpr (Ar::kFloat) a0[i] = own + o;
        else a0[i] = add_mod(own, o, m.q);
      }
      __syncthreads();
    }
    // polynomial p's sums in a
    auto tail = [&](const E(&a)[P], uint32_t p) {
      const Tw f = pinv[mi];
      const uint64_t *cin = slot + ((size_t)kg.off_conv + p * kg.L + t) * G::N;
#pragma unroll
      for (int i = 0; i < P; i++) x[i] = Ar::raw(cin[G::gaddr(g, G::ipoint(r, i))]);
      G::twist(x, g, r, tt, ar);
      G::template forward<Ar, twisted_bound<Ar>()>(lds, x, c, r, tw, lw, ar);
#pragma unroll
      for (int v = 0; v < P; v++) x[v] = ar.settle(x[v]);
      G::to_interleaved(lds, x, c, r);
      const uint64_t *add = p == 0 ? kb.add0[b] : kb.add1[b];
      const uint64_t *sum = p == 0 ? kb.sum0[b] : kb.sum1[b];
      uint64_t *out = (p == 0 ? kb.out0[b] : kb.out1[b]) + (size_t)t * G::N;
#pragma unroll
      for (int i = 0; i < P; i++) {
        const size_t pos = G::gaddr(g, G::ipoint(r, i));
        E v = ar.mul(ar.sub(a[i], x[i]), f);
        if (add) v += ar.load(add[(size_t)t * G::N + galois_src((uint32_t)pos, galois, LOGN)]);
        if (sum) v += ar.load(sum[(size_t)t * G::N + pos]);
        out[pos] = ar.template canon<4096>(v);
      }
    };
    // special limbs: ModDown's inverse contiguous pass, while the limb's
    // blocks are at hand
    auto finish = [&](E(&a)[P], uint32_t p) {
      if (t >= kg.nq) {
        if constexpr (Ar::kFloat) {
#pragma unroll
          for (int i = 0; i < P; i++) a[i] = ar.reduce(a[i]);
        }
        G::to_blocked(lds, a, c, r);
        G::template inverse<Ar, Ar::kCanonical>(lds, a, c, r, itn, lw, ar);
        G::twist(a, g, r, itt + (size_t)mi * G::N, ar);
      }
      uint64_t *o = slot + ((size_t)kg.off_acc + p * kg.ne + t) * G::N;
#pragma unroll
      for (int i = 0; i < P; i++)
        o[G::gaddr(g, G::ipoint(r, i))] =
            canonical ? ar.template canon<Ar::kFloat ? 8065 : 2048>(a[i]) : Ar::bits(a[i]);
    };
    if constexpr (!TAIL) {
      __syncthreads();
      if (set == 0) G::fill_inverse(lw, itn);
      __syncthreads();
    }
    if constexpr (SPLIT) {
      if constexpr (TAIL) tail(a0, set);
      else finish(a0, set);
    } else if constexpr (TAIL) {
      tail(a0, 0);
      tail(a1, 1);
    } else {
      finish(a0, 0);
      finish(a1, 1);
    }
  });
}

// K6: workgroup y converts the target limbs of group y (of one poly's groups:
// one limb, or two consecutive ones of one arithmetic) from one read of the K
// special limbs.
template <int LOGN, bool PAIR, bool S30>
__global__ __launch_bounds__((ConvPass<LOGN, PAIR, S30>::THREADS))
__attribute__((amdgpu_waves_per_eu(!PAIR && S30 ? 4 : 3))) void k_moddown_strided(
    uint64_t *__restrict__ ws, const ConvC *__restrict__ down_conv,
    const uint64_t *__restrict__ hneg, const ConvGroup *__restrict__ groups, KsGeom kg,
    const ModConst *__restrict__ mc, const Tw *__restrict__ tw) {
  using G = ConvPass<LOGN, PAIR, S30>;
  constexpr int P = G::P, NT = PAIR ? 2 : 1;
  __shared__ uint64_t lds[G::LDS_WORDS];
  __shared__ Tw lw[NT][G::TW_LEN];
  const uint32_t per = gridDim.y / 2;
  const uint32_t p = blockIdx.y / per;
  const ConvGroup gr = groups[blockIdx.y % per];
  uint64_t *slot = ws + (size_t)blockIdx.z * kg.slot_rows * G::N;
  const uint64_t *src = slot + ((size_t)kg.off_acc + p * kg.ne + kg.nq) * G::N;
  const int c = G::sub(threadIdx.x), r = G::lane(threadIdx.x);
  const int g = blockIdx.x * G::TR + c;
  const int mi[2] = {gr.mod[0], gr.mod[1]};
  const ConvC *cvs[NT];
  ModConst ms[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) {
    cvs[t] = down_conv + mi[t];
    ms[t] = mc[mi[t]];
    G::fill_forward(lw[t], tw + (size_t)mi[t] * kTwLen);
  }
  with_ks_arith<S30>(ms[0], [&](auto ar) {
    using Ar = decltype(ar);
    typename Ar::E x[NT][P];
    bconv<G, NT, S30>(x, src, cvs, kg.nm, kg.K, mc + kg.L, g, r, ms, ar);
#pragma unroll
    for (int t = 0; t < NT; t++) {
      if (t == 1 && gr.n < 2) break;
      Ar at = ar;
      if (t == 1) {
        if constexpr (Ar::kFloat) at = Ar{ms[NT - 1].qd, ms[NT - 1].qid};
        else at = Ar{ms[NT - 1].q, ms[NT - 1].nq};
      }
      // minus (P-1)/2, within 1/2 (doubles) or in [0, q) (integers)
      typename Ar::E h = at.load(hneg[mi[t]]);
      if constexpr (Ar::kFloat) h = at.reduce(h);
#pragma unroll
      for (int i = 0; i < P; i++) x[t][i] += h;
      if (t == 0) __syncthreads();
      G::template forward<Ar, moddown_bound<Ar, S30>()>(lds, x[t], c, r,
                                                        tw + (size_t)mi[t] * kTwLen, lw[t], at);
      uint64_t *out = slot + ((size_t)kg.off_conv + p * kg.L + mi[t]) * G::N;
#pragma unroll
      for (int v = 0; v < P; v++) out[G::gaddr(g, G::bpoint(r, v))] = Ar::bits(x[t][v]);
    }
  });
}

// K7 where the accumulators come from memory (small switches, hoisted
// rotations and shared ModDowns): per Q limb, the forward contiguous pass of
// conv and the tail.  SUM: some slots have further addends (the test for them
// by itself cost 13 hoisted rotations of 13 limbs at N = 2^16 0.4-1 %).
template <int LOGN, bool SUM>
__global__ __launch_bounds__(kNttThreads) void k_moddown_contig_tail(
    uint64_t *__restrict__ ws, KsBatch kb, const Tw *__restrict__ pinv, KsGeom kg,
    const ModConst *__restrict__ mc, const Tw *__restrict__ tw, const Tw *__restrict__ tt) {
  using G = Pass<split_b(LOGN), LOGN, false>;
  constexpr int P = G::P;
  __shared__ uint64_t lds[G::LDS_WORDS];
  __shared__ Tw lw[G::TW_LEN];
  const uint32_t p = blockIdx.z & 1, li = blockIdx.z >> 1;
  G::fill_forward(lw, tw + (size_t)li * kTwLen);
  const uint32_t b = blockIdx.y;
  const uint64_t *slot = ws + (size_t)b * kg.slot_rows * G::N;
  const int c = G::sub(threadIdx.x), r = G::lane(threadIdx.x);
  const int g = blockIdx.x * G::TR + c;
  const uint64_t *cin = slot + ((size_t)kg.off_conv + p * kg.L + li) * G::N;
  const uint64_t *u = slot + ((size_t)kg.off_acc + p * kg.ne + li) * G::N;
  const uint64_t *add = p == 0 ? kb.add0[b] : kb.add1[b];
  const uint64_t *sum = !SUM ? nullptr : p == 0 ? kb.sum0[b] : kb.sum1[b];
  const uint32_t galois = kb.galois[b];
  uint64_t *out = (p == 0 ? kb.out0[b] : kb.out1[b]) + (size_t)li * G::N;
  with_arith(mc[li], [&](auto ar) {
    using Ar = decltype(ar);
    using E = typename Ar::E;
    E x[P];
#pragma unroll
    for (int i = 0; i < P; i++) x[i] = Ar::raw(cin[G::gaddr(g, G::ipoint(r, i))]);
    G::twist(x, g, r, tt + (size_t)li * G::N, ar);
    __syncthreads();
    G::template forward<Ar, twisted_bound<Ar>()>(lds, x, c, r, tw + (size_t)li * kTwLen, lw, ar);
#pragma unroll
    for (int v = 0; v < P; v++) x[v] = ar.settle(x[v]);
    G::to_interleaved(lds, x, c, r);
    const Tw f = pinv[li];
#pragma unroll
    for (int i = 0; i < P; i++) {
      const size_t pos = G::gaddr(g, G::ipoint(r, i));
      E v = ar.mul(ar.sub(ar.load(u[pos]), x[i]), f);
      if (add) v += ar.load(add[(size_t)li * G::N + galois_src((uint32_t)pos, galois, LOGN)]);
      if (sum) v += ar.load(sum[(size_t)li * G::N + pos]);
      out[pos] = ar.template canon<SUM ? 4096 : 3072>(v);
    }
  });
}

// inner product of hoisted rotations: for extended limb t of slot b,
// acc_{0,1}[t] = sum_j phi_g(d~_j)[t] swk_j[t], with d~_j fully transformed in
// slot 0's ext rows (own limbs: phi_g(c1)) and the result, fully reduced, in
// slot b's acc rows
template <int LOGN>
__global__ __launch_bounds__(256) void k_ks_inner_gather(uint64_t *__restrict__ ws,
                                                         const uint64_t *__restrict__ c1,
                                                         KsBatch kb, KsGeom kg,
                                                         const ModConst *__restrict__ mc) {
  constexpr int N = 1 << LOGN;
  const uint32_t pos = blockIdx.x * 256 + threadIdx.x;
  const uint32_t b = blockIdx.y, t = blockIdx.z;
  const uint32_t mi = t < kg.nq ? t : kg.L + (t - kg.nq);
  const ModConst m = mc[mi];
  const uint32_t src = galois_src(pos, kb.galois[b], LOGN);
  const uint64_t *key = kb.key[b];
  const size_t krow = (size_t)kg.nm * N;
  uint64_t *slot = ws + (size_t)b * kg.slot_rows * N;
  auto digits = [&](auto &&f) {
    for (uint32_t j = 0; j < kg.dnum; j++) {
      const uint32_t lo = j * kg.alpha;
      if (lo >= kg.nq) break;
      const uint32_t hi = min(lo + kg.alpha, kg.nq);
      const uint64_t x = (t >= lo && t < hi)
                             ? c1[(size_t)t * N + src]
                             : ws[((size_t)kg.off_ext + j * kg.ne + t) * N + src];
      const uint64_t *kbp = key + 2 * j * krow + (size_t)mi * N;
      f(j, x, kbp[pos], kbp[krow + pos]);
    }
  };
  uint64_t r0, r1;
  if (m.qd != 0.0) {
    const ArF ar{m.qd, m.qid};
    double s0 = 0.0, s1 = 0.0;
    digits([&](uint32_t j, uint64_t x, uint64_t k0, uint64_t k1) {
      const double xd = ar.load(x);  // bounds as in k_ks_contig_inner
      s0 += ar.mul2(xd, ArF::raw(k0));
      s1 += ar.mul2(xd, ArF::raw(k1));
      if ((j & 7) == 7) {
        s0 = ar.reduce(s0);
        s1 = ar.reduce(s1);
      }
    });
    r0 = ar.canon(s0);
    r1 = ar.canon(s1);
  } else {
    u128 s0, s1;
    s0.lo = s0.hi = s1.lo = s1.hi = 0;
    digits([&](uint32_t, uint64_t x, uint64_t k0, uint64_t k1) {
      mac_wide(s0, x, k0);
      mac_wide(s1, x, k1);
    });
    r0 = redc(s0, m.q, m.qinv);
    r1 = redc(s1, m.q, m.qinv);
  }
  slot[((size_t)kg.off_acc + t) * N + pos] = r0;
  slot[((size_t)kg.off_acc + kg.ne + t) * N + pos] = r1;
}

KsGeom make_geom(const hck_context *ctx, uint32_t level) {
  KsGeom kg;
  kg.level = level;
  kg.nq = level + 1;
  kg.ne = level + 1 + ctx->K;
  kg.L = ctx->L;
  kg.K = ctx->K;
  kg.dnum = ctx->dnum;
  kg.alpha = ctx->alpha;
  kg.nm = ctx->L + ctx->K;
  kg.slot_rows = (uint32_t)ws_ks_rows(ctx);
  kg.off_ext = ctx->L;
  kg.off_acc = ctx->L + ctx->dnum * kg.nm;
  kg.off_conv = kg.off_acc + 2 * kg.nm;
  return kg;
}

// K1-K3 for batch slots 0..nb-1 (ModUp into each slot's ext rows)
template <int LOGN>
int ks_modup(hck_context *ctx, const KsBatch &kb, const KsGeom &kg, uint64_t *ws) {
  constexpr int A = split_a(LOGN), B = split_b(LOGN);
  constexpr double N = (double)(1 << LOGN);
  using GA = Pass<A, LOGN, true>;
  using GB = Pass<B, LOGN, false>;
  const uint32_t nq = kg.nq, nb = kb.n, level = kg.level;
  int rc;
  double copies = 0;   // c0 and phi_g(d) tiles copied for outputs that alias their input
  for (uint32_t b = 0; b < nb; b++) copies += kb.add0_src[b] ? 2 * nq : 0;
  timing_begin(ctx, "ks_intt_gather", dim3(GB::BLOCKS, nb, nq), 16.0 * N * (nq * nb + copies),
               0.5 * N * B * nq * nb);
  k_ks_intt_gather<LOGN><<<dim3(GB::BLOCKS, nb, nq), kNttThreads, 0, ctx->stream>>>(
      ws, kb, kg, ctx->d_mod, ctx->d_itn, ctx->split[0].itwist);
  timing_end(ctx);
  {
    LimbMap m;
    m.n = nq * nb;
    for (uint32_t b = 0; b < nb; b++)
      for (uint32_t i = 0; i < nq; i++) {
        m.row[b * nq + i] = (uint16_t)(b * kg.slot_rows + i);
        m.mod[b * nq + i] = (uint8_t)i;
      }
    const RowFactors sc{ctx->d_up_rows + ((size_t)level * kg.L << A), nullptr, nq, false};
    if ((rc = ntt_pass(ctx, ws, m, true, true, &sc))) return rc;
  }
  // in a launch large enough to fill the chip at half the workgroups,
  // consecutive targets of one digit and arithmetic share a workgroup (one
  // read of the digit's limbs for both); small launches keep one target per
  // workgroup and the kernel's lower register count
  const uint32_t targets = ctx->groups[0][level].second;
  const bool paired = kPairs<LOGN> && (size_t)targets * nb * GA::BLOCKS >= kPairMinBlocks;
  const auto gr = ctx->groups[paired][level];
  const ConvC *up_conv = ctx->d_up_conv + (size_t)level * kg.dnum * (kg.alpha + 1) * kg.nm;
  // algorithmic bytes: every digit limb is read once (the targets sharing it
  // re-read it from cache), every output written
  double macs = 0;
  for (uint32_t lo = 0; lo < nq; lo += kg.alpha) {
    const double na = std::min(kg.alpha, nq - lo);
    macs += na * (kg.ne - na);
  }
  const dim3 grid(GA::BLOCKS, gr.second, nb);
  timing_begin(ctx, "ks_modup_strided", grid, 8.0 * N * nb * (nq + targets),
               N * nb * (macs + 0.5 * A * targets));
  const ConvGroup *groups = ctx->d_groups + gr.first;
  const bool s30 = ctx->bconv30 && ctx->conv_f;
  auto launch = [&](auto kernel, int threads) {
    kernel<<<grid, threads, 0, ctx->stream>>>(ws, groups, up_conv, kg, ctx->d_mod, ctx->d_tw);
  };
  if (!s30)
    launch(paired ? k_modup_strided<LOGN, kPairs<LOGN>, false> : k_modup_strided<LOGN, false, false>,
           kNttThreads);
  else if (paired)
    launch(k_modup_strided<LOGN, kPairs<LOGN>, true>, kNttThreads);
  else
    launch(k_modup_strided<LOGN, false, true>, ConvPass<LOGN, false, true>::THREADS);
  timing_end(ctx);
  HCK_HIP(ctx, hipGetLastError());
  return HCK_OK;
}

// K5 and K6 for batch slots 0..nb-1: each slot's special accumulators
// (canonical: fully reduced words, else as k_ks_contig_inner leaves them)
// converted to the Q limbs (conv rows, strided pass done)
template <int LOGN>
int ks_down_conv(hck_context *ctx, uint32_t nb, const KsGeom &kg, uint64_t *ws, bool canonical) {
  constexpr int A = split_a(LOGN);
  constexpr double N = (double)(1 << LOGN);
  using GA = Pass<A, LOGN, true>;
  const uint32_t L = kg.L, K = kg.K, nq = kg.nq, ne = kg.ne;
  int rc;
  {
    LimbMap mp;
    mp.n = 2 * K * nb;
    for (uint32_t b = 0; b < nb; b++)
      for (uint32_t p = 0; p < 2; p++)
        for (uint32_t k = 0; k < K; k++) {
          const uint32_t r = (b * 2 + p) * K + k;
          mp.row[r] = (uint16_t)(b * kg.slot_rows + kg.off_acc + p * ne + nq + k);
          mp.mod[r] = (uint8_t)(L + k);
        }
    const RowFactors sc{ctx->d_down_rows, ctx->d_down_add, K, canonical};
    if ((rc = ntt_pass(ctx, ws, mp, true, true, &sc))) return rc;
  }
  // in a launch large enough to fill the chip at half the workgroups, the K
  // special limbs are read once per pair of target limbs
  const bool paired = kPairs<LOGN> && (size_t)2 * nq * nb * GA::BLOCKS >= kPairMinBlocks;
  const auto gr = ctx->down_groups[paired][kg.level];
  const ConvGroup *groups = ctx->d_groups + gr.first;
  const dim3 grid(GA::BLOCKS, 2 * gr.second, nb);
  // algorithmic bytes: each output's K special limbs read once, its target
  // limbs written
  timing_begin(ctx, "ks_moddown_strided", grid, 8.0 * N * (K + nq) * 2 * nb,
               N * (K + 0.5 * A) * 2 * nq * nb);
  const bool s30 = ctx->bconv30 && ctx->conv_f;
  auto launch = [&](auto kernel, int threads) {
    kernel<<<grid, threads, 0, ctx->stream>>>(ws, ctx->d_down_conv, ctx->d_down_hneg, groups, kg,
                                              ctx->d_mod, ctx->d_tw);
  };
  if (!s30)
    launch(paired ? k_moddown_strided<LOGN, kPairs<LOGN>, false> : k_moddown_strided<LOGN, false, false>,
           kNttThreads);
  else if (paired)
    launch(k_moddown_strided<LOGN, kPairs<LOGN>, true>, kNttThreads);
  else
    launch(k_moddown_strided<LOGN, false, true>, ConvPass<LOGN, false, true>::THREADS);
  timing_end(ctx);
  HCK_HIP(ctx, hipGetLastError());
  return HCK_OK;
}

// K4 over limbs [first, first + limbs) of the list special limbs, Q limbs
template <int LOGN, bool TAIL>
void launch_contig_inner(hck_context *ctx, const KsBatch &kb, const KsGeom &kg, uint64_t *ws,
                         uint32_t first, uint32_t limbs, bool canonical) {
  constexpr int B = split_b(LOGN);
  constexpr double N = (double)(1 << LOGN);
  using GB = Pass<B, LOGN, false>;
  const uint32_t nq = kg.nq, nb = kb.n, alpha = kg.alpha;
  const double digits = (double)((nq + alpha - 1) / alpha);
  const double q_limbs = first + limbs > kg.K ? first + limbs - std::max(first, kg.K) : 0;
  const double p_limbs = limbs - q_limbs;
  double keys = 0;  // distinct keys in the batch
  double adds = 0;
  for (uint32_t b = 0; b < nb; b++) {
    bool seen = false;
    for (uint32_t k = 0; k < b; k++) seen = seen || kb.key[k] == kb.key[b];
    keys += seen ? 0 : 1;
    if (TAIL)
      for (const uint64_t *a : {kb.add0[b], kb.add1[b], kb.sum0[b], kb.sum1[b]}) adds += a ? nq : 0;
  }
  const double ext = nb * (digits * limbs - q_limbs);  // transformed digit limbs
  // accumulators written, or (tail) conv read and outputs written
  const double io = nb * (TAIL ? 4.0 : 2.0) * limbs;
  timing_begin(ctx, TAIL ? "ks_inner_tail" : "ks_contig_inner", dim3(GB::BLOCKS, nb, limbs),
               8.0 * N * (ext + nb * q_limbs + io + adds + 2 * digits * limbs * keys),
               N * (0.5 * B * (ext + 2.0 * nb * (TAIL ? q_limbs : p_limbs)) +
                    2 * digits * limbs * nb + (TAIL ? 2.0 * nb * q_limbs : 0.0)));
  const dim3 grid(GB::BLOCKS, nb, limbs);
  auto launch = [&](auto kernel, int threads) {
    kernel<<<grid, threads, 0, ctx->stream>>>(ws, kb, kg, first, canonical ? 1 : 0, ctx->d_mod,
                                              ctx->d_tw, ctx->split[0].twist, ctx->d_itn,
                                              ctx->split[0].itwist, ctx->d_pinv);
  };
  if ((size_t)grid.x * grid.y * grid.z <= kSplitMaxBlocks)
    launch(k_ks_contig_inner<LOGN, TAIL, true>, 2 * kNttThreads);
  else
    launch(k_ks_contig_inner<LOGN, TAIL, false>, kNttThreads);
  timing_end(ctx);
}

// K5-K7 for batch slots 0..nb-1 with every accumulator (fully reduced) in
// the slots' acc rows; special_contig_done: the special rows have been
// through the inverse contiguous pass
template <int LOGN>
int ks_moddown(hck_context *ctx, const KsBatch &kb, const KsGeom &kg, uint64_t *ws,
               bool special_contig_done) {
  constexpr int B = split_b(LOGN);
  constexpr double N = (double)(1 << LOGN);
  using GB = Pass<B, LOGN, false>;
  const uint32_t nq = kg.nq, nb = kb.n;
  int rc;
  if (!special_contig_done) {
    LimbMap mp;
    mp.n = 2 * kg.K * nb;
    for (uint32_t r = 0; r < mp.n; r++) {
      const uint32_t b = r / (2 * kg.K), p = r / kg.K % 2, k = r % kg.K;
      mp.row[r] = (uint16_t)(b * kg.slot_rows + kg.off_acc + p * kg.ne + nq + k);
      mp.mod[r] = (uint8_t)(kg.L + k);
    }
    if ((rc = ntt_pass(ctx, ws, mp, true, false, nullptr))) return rc;
  }
  if ((rc = ks_down_conv<LOGN>(ctx, nb, kg, ws, special_contig_done))) return rc;
  double adds = 0;
  bool sums = false;
  for (uint32_t b = 0; b < nb; b++) {
    sums = sums || kb.sum0[b] || kb.sum1[b];
    for (const uint64_t *a : {kb.add0[b], kb.add1[b], kb.sum0[b], kb.sum1[b]}) adds += a ? nq : 0;
  }
  timing_begin(ctx, "ks_moddown_tail", dim3(GB::BLOCKS, nb, 2 * nq),
               8.0 * N * (3.0 * 2 * nq * nb + adds), N * (0.5 * B + 1) * 2 * nq * nb);
  auto launch = [&](auto kernel) {
    kernel<<<dim3(GB::BLOCKS, nb, 2 * nq), kNttThreads, 0, ctx->stream>>>(
        ws, kb, ctx->d_pinv, kg, ctx->d_mod, ctx->d_tw, ctx->split[0].twist);
  };
  constexpr bool kSums = LOGN <= kTogetherMaxLog;  // no other caller has any
  launch(kSums && sums ? k_moddown_contig_tail<LOGN, kSums> : k_moddown_contig_tail<LOGN, false>);
  timing_end(ctx);
  HCK_HIP(ctx, hipGetLastError());
  return HCK_OK;
}

template <int LOGN>
int ks_run(hck_context *ctx, const KsBatch &kb, uint32_t level, uint64_t *ws) {
  const KsGeom kg = make_geom(ctx, level);
  int rc;
  if ((rc = ks_modup<LOGN>(ctx, kb, kg, ws))) return rc;
  using GB = Pass<split_b(LOGN), LOGN, false>;
  if (LOGN <= kTogetherMaxLog && (size_t)GB::BLOCKS * kb.n * kg.ne <= kSplitMaxBlocks) {
    launch_contig_inner<LOGN, false>(ctx, kb, kg, ws, 0, kg.ne, true);
    return ks_moddown<LOGN>(ctx, kb, kg, ws, true);
  }
  launch_contig_inner<LOGN, false>(ctx, kb, kg, ws, 0, kg.K, false);
  if ((rc = ks_down_conv<LOGN>(ctx, kb.n, kg, ws, false))) return rc;
  launch_contig_inner<LOGN, true>(ctx, kb, kg, ws, kg.K, kg.nq, false);
  HCK_HIP(ctx, hipGetLastError());
  return HCK_OK;
}

template <int LOGN>
int ks_hoisted(hck_context *ctx, const uint64_t *c0, const uint64_t *c1, uint32_t level,
               const uint32_t *galois, const hck_switch_key *const *keys, uint32_t n,
               uint64_t *const *out0, uint64_t *const *out1) {
  constexpr double N = (double)(1 << LOGN);
  const KsGeom kg = make_geom(ctx, level);
  const uint32_t nq = kg.nq, ne = kg.ne, alpha = kg.alpha;
  int rc;
  KsBatch up;
  up.n = 1;
  up.galois[0] = 1;
  up.d[0] = c1;
  if ((rc = ks_modup<LOGN>(ctx, up, kg, ws_ks(ctx)))) return rc;
  // finish the forward transform of slot 0's extended digits in place
  std::vector<std::pair<uint16_t, uint8_t>> rows;
  for (uint32_t j = 0; j < kg.dnum; j++) {
    const uint32_t lo = j * alpha;
    if (lo >= nq) break;
    const uint32_t hi = std::min(lo + alpha, nq);
    for (uint32_t t = 0; t < ne; t++)
      if (t < lo || t >= hi)
        rows.push_back({(uint16_t)(kg.off_ext + j * ne + t),
                        (uint8_t)(t < nq ? t : kg.L + (t - nq))});
  }
  for (size_t s = 0; s < rows.size(); s += kMaxRows) {
    LimbMap m;
    m.n = (uint32_t)std::min(rows.size() - s, (size_t)kMaxRows);
    for (uint32_t r = 0; r < m.n; r++) {
      m.row[r] = rows[s + r].first;
      m.mod[r] = rows[s + r].second;
    }
    if ((rc = ntt_pass(ctx, ws_ks(ctx), m, false, false, nullptr))) return rc;
  }
  const double digits = (double)((nq + alpha - 1) / alpha);
  const uint32_t limit = ks_batch_limit(ctx, level);
  for (uint32_t s = 0; s < n; s += even_batch(n - s, limit)) {
    KsBatch kb;
    kb.n = even_batch(n - s, limit);
    for (uint32_t b = 0; b < kb.n; b++) {
      kb.key[b] = keys[s + b]->data;
      kb.galois[b] = galois[s + b];
      kb.d[b] = c1;
      kb.out0[b] = out0[s + b];
      kb.out1[b] = out1[s + b];
      kb.add0[b] = c0;
      kb.add1[b] = nullptr;
    }
    timing_begin(ctx, "ks_inner_gather", dim3((1 << LOGN) / 256, kb.n, ne),
                 8.0 * N * ne * (digits + (2 * digits + 2) * kb.n), 2 * digits * N * ne * kb.n);
    k_ks_inner_gather<LOGN><<<dim3((1 << LOGN) / 256, kb.n, ne), 256, 0, ctx->stream>>>(
        ws_ks(ctx), c1, kb, kg, ctx->d_mod);
    timing_end(ctx);
    if ((rc = ks_moddown<LOGN>(ctx, kb, kg, ws_ks(ctx), false))) return rc;
  }
  HCK_HIP(ctx, hipGetLastError());
  return HCK_OK;
}

// K1-K4, then each slot's accumulators added into its extended-basis sum
template <int LOGN>
int ks_pq(hck_context *ctx, const KsBatch &kb, uint32_t level, uint64_t *const *pq,
          const bool *first) {
  constexpr size_t N = 1 << LOGN;
  const KsGeom kg = make_geom(ctx, level);
  const uint32_t nq = kg.nq, ne = kg.ne, nb = kb.n;
  int rc;
  if ((rc = ks_modup<LOGN>(ctx, kb, kg, ws_ks(ctx)))) return rc;
  launch_contig_inner<LOGN, false>(ctx, kb, kg, ws_ks(ctx), 0, ne, true);
  HCK_HIP(ctx, hipGetLastError());
  LimbMap rows;
  rows.n = 2 * ne;
  for (uint32_t r = 0; r < 2 * ne; r++) {
    const uint32_t t = r % ne;
    rows.row[r] = (uint16_t)r;
    rows.mod[r] = (uint8_t)(t < nq ? t : kg.L + (t - nq));
  }
  std::vector<bool> done(nb, false);
  for (uint32_t b = 0; b < nb; b++) {
    if (done[b]) continue;
    std::vector<const uint64_t *> in;
    if (!first[b]) in.push_back(pq[b]);
    for (uint32_t k = b; k < nb; k++)
      if (pq[k] == pq[b]) {
        done[k] = true;
        in.push_back(ws_ks(ctx) + ((size_t)k * kg.slot_rows + kg.off_acc) * N);
      }
    if ((rc = launch_sum_many(ctx, pq[b], in.data(), (uint32_t)in.size(), rows))) return rc;
  }
  return HCK_OK;
}

template <int LOGN>
int md_pq(hck_context *ctx, const KsBatch &kb, uint32_t level, const uint64_t *const *pq) {
  const KsGeom kg = make_geom(ctx, level);
  int rc;
  for (uint32_t b = 0; b < kb.n; b++)
    if ((rc = launch_copy(ctx, ws_ks(ctx) + ((size_t)b * kg.slot_rows + kg.off_acc) * ctx->n,
                          pq[b], (size_t)2 * kg.ne * ctx->n)))
      return rc;
  return ks_moddown<LOGN>(ctx, kb, kg, ws_ks(ctx), true);
}

}  // namespace

template <int LOGN>
int KsRing<LOGN>::run(hck_context *ctx, const KsBatch &kb, uint32_t level, uint64_t *ws) {
  return ks_run<LOGN>(ctx, kb, level, ws);
}

template <int LOGN>
int KsRing<LOGN>::hoisted(hck_context *ctx, const uint64_t *c0, const uint64_t *c1,
                          uint32_t level, const uint32_t *galois,
                          const hck_switch_key *const *keys, uint32_t n, uint64_t *const *out0,
                          uint64_t *const *out1) {
  return ks_hoisted<LOGN>(ctx, c0, c1, level, galois, keys, n, out0, out1);
}

template <int LOGN>
int KsRing<LOGN>::pq(hck_context *ctx, const KsBatch &kb, uint32_t level, uint64_t *const *pq,
                     const bool *first) {
  return ks_pq<LOGN>(ctx, kb, level, pq, first);
}

template <int LOGN>
int KsRing<LOGN>::md(hck_context *ctx, const KsBatch &kb, uint32_t level,
                     const uint64_t *const *pq) {
  return md_pq<LOGN>(ctx, kb, level, pq);
}

template struct KsRing<HCK_LOGN>;

}  // namespace hck

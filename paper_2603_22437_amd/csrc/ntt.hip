// Negacyclic NTT / inverse NTT over many limbs in one launch: the two
// passes of ntt_core.h, each a kernel over every listed limb.
//
// Compiled once per ring, with HCK_LOGN its log2 N (build.py).
#include "ntt_core.h"

namespace hck {

namespace {

// One pass over the rows of `map`, in place.  Words between the two passes
// are in the modulus' own arithmetic (ntt_core.h), words outside a transform
// fully reduced integers.  w: the forward twiddles or inverse roots; tt: the
// contiguous pass's twists; rf: the inverse strided pass's row factors, by
// modulus (rf.period 0) or by (row list index) mod rf.period.
template <class G, bool STRIDED, bool INVERSE, class Ar>
__device__ __forceinline__ void ntt_pass_body(uint64_t *buf, const LimbMap &map,
                                              const Tw *__restrict__ w, const Tw *__restrict__ tt,
                                              const RowFactors &rf, uint64_t *lds, Tw *lw, Tw *lf,
                                              const uint64_t (&u)[G::P], Ar ar) {
  using E = typename Ar::E;
  constexpr int P = G::P;
  const int mi = map.mod[blockIdx.y];
  uint64_t *x_ = buf + (size_t)map.row[blockIdx.y] * G::N;
  const int c = G::sub(threadIdx.x), r = G::lane(threadIdx.x);
  const int g = blockIdx.x * G::TR + c;
  E x[P];
  if constexpr (!INVERSE) {
    w += (size_t)mi * kTwLen;
    G::fill_forward(lw, w);
    if constexpr (STRIDED) {
#pragma unroll
      for (int i = 0; i < P; i++) x[i] = ar.load(u[i]);
      __syncthreads();
      G::template forward<Ar, Ar::kCanonical>(lds, x, c, r, w, lw, ar);
#pragma unroll
      for (int v = 0; v < P; v++) x_[G::gaddr(g, G::bpoint(r, v))] = Ar::bits(x[v]);
    } else {
#pragma unroll
      for (int i = 0; i < P; i++) x[i] = Ar::raw(u[i]);
      G::twist(x, g, r, tt + (size_t)mi * G::N, ar);
      __syncthreads();
      G::template forward<Ar, twisted_bound<Ar>()>(lds, x, c, r, w, lw, ar);
      G::to_interleaved(lds, x, c, r);
#pragma unroll
      for (int i = 0; i < P; i++) x_[G::gaddr(g, G::ipoint(r, i))] = ar.canon(x[i]);
    }
  } else {
    w += (size_t)mi * kRootLen;
    G::fill_inverse(lw, w);
    if constexpr (STRIDED) {
      const int k = rf.period ? (int)(blockIdx.y % rf.period) : mi;
#pragma unroll
      for (int v = 0; v < P; v++) x[v] = rf.canonical ? ar.load(u[v]) : Ar::raw(u[v]);
      const Tw *f = rf.rows + (size_t)k * G::R;
      constexpr bool ROWS_LDS = G::R <= 512;  // as the twiddles (TW_LDS)
      if constexpr (ROWS_LDS)
        for (int i = threadIdx.x; i < G::R; i += G::THREADS) lf[i] = f[i];
      __syncthreads();
      G::template inverse<Ar, twisted_bound<Ar>()>(lds, x, c, r, w, lw, ar);
      const uint64_t add = rf.add ? rf.add[k] : 0;
#pragma unroll
      for (int i = 0; i < P; i++) {
        const int p = G::ipoint(r, i);
        E y = ar.mul(x[i], ROWS_LDS ? lf[p] : f[p]);
        if (rf.add) y += ar.load(add);
        x_[G::gaddr(g, p)] = ar.template canon<3072>(y);
      }
    } else {
#pragma unroll
      for (int i = 0; i < P; i++) x[i] = ar.load(u[i]);
      __syncthreads();
      G::to_blocked(lds, x, c, r);
      G::template inverse<Ar, Ar::kCanonical>(lds, x, c, r, w, lw, ar);
      G::twist(x, g, r, tt + (size_t)mi * G::N, ar);
#pragma unroll
      for (int i = 0; i < P; i++) x_[G::gaddr(g, G::ipoint(r, i))] = Ar::bits(x[i]);
    }
  }
}

// A 1024-point pass is held to the registers of two workgroups a CU, like its
// LDS (TW_LDS).
template <int LOGR, int LOGN, bool STRIDED, bool INVERSE>
__global__ __launch_bounds__((Pass<LOGR, LOGN, STRIDED>::THREADS), LOGR > 9 ? 2 : 1) void k_ntt_pass(
    uint64_t *buf, LimbMap map, const ModConst *__restrict__ mc, const Tw *__restrict__ w,
    const Tw *__restrict__ tt, RowFactors rf) {
  using G = Pass<LOGR, LOGN, STRIDED>;
  __shared__ uint64_t lds[G::LDS_WORDS];
  __shared__ Tw lw[G::TW_LEN];
  __shared__ Tw lf[STRIDED && INVERSE && G::R <= 512 ? G::R : 1];
  // the data loads are issued before the modulus is known, so that their
  // latency and that of its constants overlap
  const uint64_t *in = buf + (size_t)map.row[blockIdx.y] * G::N;
  const int r = G::lane(threadIdx.x);
  const int g = blockIdx.x * G::TR + G::sub(threadIdx.x);
  uint64_t u[G::P];
#pragma unroll
  for (int i = 0; i < G::P; i++)
    u[i] = in[G::gaddr(g, STRIDED && INVERSE ? G::bpoint(r, i) : G::ipoint(r, i))];
  with_arith(mc[map.mod[blockIdx.y]], [&](auto ar) {
    ntt_pass_body<G, STRIDED, INVERSE>(buf, map, w, tt, rf, lds, lw, lf, u, ar);
  });
}

// The centred value of v in [0, ql) (v - ql above half) modulo ar's modulus.
// Doubles: exact below 2^52, and in two 31-bit parts of the signed value
// above (each part's quotient by q stays below 2^36).
__device__ __forceinline__ double lift(uint64_t v, const ModConst &ml, uint64_t, const ModConst &,
                                       ArF ar) {
  if (ml.q < (1ull << 52)) {
    const double d = ar.load(v), qd = (double)ml.q;
    return ar.reduce(d > 0.5 * qd ? d - qd : d);
  }
  const int64_t s = v > (ml.q - 1) / 2 ? (int64_t)v - (int64_t)ml.q : (int64_t)v;
  const double hi = (double)(int32_t)(s >> 31) * 2147483648.0;
  return ar.reduce(ar.reduce(hi) + (double)(uint32_t)(s & 0x7fffffff));
}
template <int LIM>
__device__ __forceinline__ uint64_t lift(uint64_t v, const ModConst &ml, uint64_t ql,
                                         const ModConst &m, ArI<LIM>) {
  const uint64_t t = shoup(v, 1, m.one_shoup, m.q);
  return v > (ml.q - 1) / 2 ? sub_mod(t, ql, m.q) : t;
}

// Rescale, first launch: inverse contiguous pass of polynomial blockIdx.y's
// dropped limb (limb `level` of in) -> limb blockIdx.y of last.
template <int LOGN>
__global__ __launch_bounds__(kNttThreads) void k_rescale_contig_inv(
    uint64_t *__restrict__ last, const uint64_t *__restrict__ in, size_t ps, uint32_t level,
    const ModConst *__restrict__ mc, const Tw *__restrict__ itn, const Tw *__restrict__ itt) {
  using G = Pass<split_b(LOGN), LOGN, false>;
  constexpr int P = G::P;
  __shared__ uint64_t lds[G::LDS_WORDS];
  __shared__ Tw lw[G::TW_LEN];
  const int c = G::sub(threadIdx.x), r = G::lane(threadIdx.x);
  const int g = blockIdx.x * G::TR + c;
  const uint64_t *src = in + blockIdx.y * ps + (size_t)level * G::N;
  uint64_t u[P];
#pragma unroll
  for (int i = 0; i < P; i++) u[i] = src[G::gaddr(g, G::ipoint(r, i))];
  itn += (size_t)level * kRootLen;
  G::fill_inverse(lw, itn);
  with_arith(mc[level], [&](auto ar) {
    using Ar = decltype(ar);
    typename Ar::E x[P];
#pragma unroll
    for (int i = 0; i < P; i++) x[i] = ar.load(u[i]);
    __syncthreads();
    G::to_blocked(lds, x, c, r);
    G::template inverse<Ar, Ar::kCanonical>(lds, x, c, r, itn, lw, ar);
    G::twist(x, g, r, itt + (size_t)level * G::N, ar);
    uint64_t *out = last + (size_t)blockIdx.y * G::N;
#pragma unroll
    for (int i = 0; i < P; i++) out[G::gaddr(g, G::ipoint(r, i))] = Ar::bits(x[i]);
  });
}

// Rescale, second launch (strided passes): the dropped limb's inverse is
// finished (again for every target limb i = blockIdx.y: the pass is short and
// saves a launch and a round trip to memory), each value lifted to its centred
// representative (v - q_l when v > (q_l - 1) / 2) modulo q_i, and the forward
// strided pass of limb i run on it.  tmp gets rows z level + i.  Three launches
// instead of six (two of them copies) a rescale: two polynomials at N = 2^15,
// levels below 12, 29 -> 21 us of kernels, at N = 2^16, 13 limbs, 41 -> 24 us.
template <int LOGN>
__global__ __launch_bounds__((Pass<split_a(LOGN), LOGN, true>::THREADS)) void k_rescale_strided(
    uint64_t *__restrict__ tmp, const uint64_t *__restrict__ last, uint32_t level,
    const ModConst *__restrict__ mc, const Tw *__restrict__ w, const Tw *__restrict__ itn,
    const Tw *__restrict__ rows) {
  using G = Pass<split_a(LOGN), LOGN, true>;
  constexpr int P = G::P;
  __shared__ uint64_t lds[G::LDS_WORDS];
  __shared__ Tw lw[G::TW_LEN], li[G::TW_LEN], lf[G::R];
  const uint32_t i = blockIdx.y, z = blockIdx.z;
  const int c = G::sub(threadIdx.x), r = G::lane(threadIdx.x);
  const int g = blockIdx.x * G::TR + c;
  const uint64_t *src = last + (size_t)z * G::N;
  uint64_t v[P];
#pragma unroll
  for (int k = 0; k < P; k++) v[k] = src[G::gaddr(g, G::bpoint(r, k))];
  w += (size_t)i * kTwLen;
  itn += (size_t)level * kRootLen;
  G::fill_forward(lw, w);
  G::fill_inverse(li, itn);
  for (int k = threadIdx.x; k < G::R; k += G::THREADS) lf[k] = rows[(size_t)level * G::R + k];
  __syncthreads();
  const ModConst m = mc[i], ml = mc[level];
  with_arith(ml, [&](auto ar) {
    using Ar = decltype(ar);
    typename Ar::E x[P];
#pragma unroll
    for (int k = 0; k < P; k++) x[k] = Ar::raw(v[k]);
    G::template inverse<Ar, twisted_bound<Ar>()>(lds, x, c, r, itn, li, ar);
#pragma unroll
    for (int k = 0; k < P; k++) v[k] = ar.template canon<2048>(ar.mul(x[k], lf[G::ipoint(r, k)]));
  });
  with_arith(m, [&](auto ar) {
    using Ar = decltype(ar);
    const uint64_t ql = Ar::kFloat ? 0 : shoup(ml.q, 1, m.one_shoup, m.q);
    typename Ar::E x[P];
#pragma unroll
    for (int k = 0; k < P; k++) x[k] = lift(v[k], ml, ql, m, ar);
    G::template forward<Ar, Ar::kCanonical>(lds, x, c, r, w, lw, ar);
    uint64_t *out = tmp + ((size_t)z * level + i) * G::N;
#pragma unroll
    for (int k = 0; k < P; k++) out[G::gaddr(g, G::bpoint(r, k))] = Ar::bits(x[k]);
  });
}

// Rescale, tail (contiguous pass): finishes the forward transform of the
// lifted limb t and writes out_i = (c_i - t) q_l^-1 mod q_i for i < level
// (inv: q_l^-1 mod q_i).  out may be c.
template <int LOGN>
__global__ __launch_bounds__(kNttThreads) void k_rescale_contig_tail(
    uint64_t *out, const uint64_t *c_in, const uint64_t *__restrict__ tmp, size_t ps,
    uint32_t level, const Tw *__restrict__ inv, const ModConst *__restrict__ mc,
    const Tw *__restrict__ w, const Tw *__restrict__ tt) {
  using G = Pass<split_b(LOGN), LOGN, false>;
  constexpr int P = G::P;
  __shared__ uint64_t lds[G::LDS_WORDS];
  __shared__ Tw lw[G::TW_LEN];
  const uint32_t i = blockIdx.y, z = blockIdx.z;
  G::fill_forward(lw, w + (size_t)i * kTwLen);
  with_arith(mc[i], [&](auto ar) {
    using Ar = decltype(ar);
    const int c = G::sub(threadIdx.x), r = G::lane(threadIdx.x);
    const int g = blockIdx.x * G::TR + c;
    const uint64_t *tin = tmp + ((size_t)z * level + i) * G::N;
    typename Ar::E x[P];
#pragma unroll
    for (int k = 0; k < P; k++) x[k] = Ar::raw(tin[G::gaddr(g, G::ipoint(r, k))]);
    G::twist(x, g, r, tt + (size_t)i * G::N, ar);
    __syncthreads();
    G::template forward<Ar, twisted_bound<Ar>()>(lds, x, c, r, w + (size_t)i * kTwLen, lw, ar);
#pragma unroll
    for (int v = 0; v < P; v++) x[v] = ar.settle(x[v]);
    G::to_interleaved(lds, x, c, r);
    const size_t off = (size_t)z * ps + (size_t)i * G::N;
    const Tw f = inv[i];
#pragma unroll
    for (int k = 0; k < P; k++) {
      const size_t pos = off + G::gaddr(g, G::ipoint(r, k));
      out[pos] = ar.template canon<2048>(ar.mul(ar.sub(ar.load(c_in[pos]), x[k]), f));
    }
  });
}

template <int LOGN>
int run_rescale(hck_context *ctx, uint64_t *out, const uint64_t *in, uint64_t *tmp, uint32_t level,
                uint32_t polys) {
  constexpr int A = split_a(LOGN), B = split_b(LOGN);
  constexpr double N = (double)(1 << LOGN);
  using GA = Pass<A, LOGN, true>;
  using GB = Pass<B, LOGN, false>;
  const size_t ps = (size_t)ctx->L * ctx->n;
  uint64_t *last = tmp, *lift = tmp + (size_t)polys * ctx->n;
  const hck_context::Split &sp = ctx->split[0];
  timing_begin(ctx, "rescale_inv", dim3(GB::BLOCKS, polys), 16.0 * N * polys, 0.5 * N * B * polys);
  k_rescale_contig_inv<LOGN><<<dim3(GB::BLOCKS, polys), kNttThreads, 0, ctx->stream>>>(
      last, in, ps, level, ctx->d_mod, ctx->d_itn, sp.itwist);
  timing_end(ctx);
  timing_begin(ctx, "rescale_strided", dim3(GA::BLOCKS, level, polys),
               8.0 * N * polys * (1 + level), N * (1 + 0.5 * A) * polys * (level + 1));
  k_rescale_strided<LOGN><<<dim3(GA::BLOCKS, level, polys), GA::THREADS, 0, ctx->stream>>>(
      lift, last, level, ctx->d_mod, ctx->d_tw, ctx->d_itn, sp.rows);
  timing_end(ctx);
  timing_begin(ctx, "rescale_tail", dim3(GB::BLOCKS, level, polys), 24.0 * N * polys * level,
               N * (1 + 0.5 * B) * polys * level);
  k_rescale_contig_tail<LOGN><<<dim3(GB::BLOCKS, level, polys), kNttThreads, 0, ctx->stream>>>(
      out, in, lift, ps, level, ctx->d_rescale + (size_t)level * ctx->L, ctx->d_mod, ctx->d_tw,
      sp.twist);
  timing_end(ctx);
  HCK_HIP(ctx, hipGetLastError());
  return HCK_OK;
}

// One pass of the split N = 2^A x 2^(LOGN - A): the strided pass runs the
// first A stages (R1 = 2^A points per sub-transform), the contiguous pass the
// rest, with the tables of that split.
template <int LOGN, int A, bool STRIDED, bool INVERSE>
void launch_split(hck_context *ctx, uint64_t *buf, const LimbMap &map, const RowFactors *sc,
                  const hck_context::Split &sp) {
  constexpr int LOGR = STRIDED ? A : LOGN - A;
  constexpr int N = 1 << LOGN;
  using G = Pass<LOGR, LOGN, STRIDED>;
  static const char *names[2][2] = {{"ntt_fwd_contig", "ntt_fwd_strided"},
                                    {"ntt_inv_contig", "ntt_inv_strided"}};
  const double mm = (0.5 * LOGR + (INVERSE && STRIDED ? 1 : 0)) * N * map.n;
  timing_begin(ctx, names[INVERSE][STRIDED], dim3(G::BLOCKS, map.n), 16.0 * N * map.n, mm);
  const RowFactors rf = sc ? *sc : RowFactors{sp.rows, nullptr, 0, false};
  const Tw *w = INVERSE ? ctx->d_itn : ctx->d_tw, *tt = INVERSE ? sp.itwist : sp.twist;
  const dim3 grid(G::BLOCKS, map.n);
  k_ntt_pass<LOGR, LOGN, STRIDED, INVERSE>
      <<<grid, G::THREADS, 0, ctx->stream>>>(buf, map, ctx->d_mod, w, tt, rf);
  timing_end(ctx);
}

// whether the split 2^A x 2^(LOGN - A) has both passes: at least one
// workgroup per limb, a contiguous sub-transform inside one wavefront, and
// each pass's LDS within a workgroup's share of gfx950's 160 KiB
template <int LOGN, int A>
constexpr bool split_ok() {
  if (A < 2 || LOGN - A < 2) return false;
  using S = Pass<A, LOGN, true>;
  using C = Pass<LOGN - A, LOGN, false>;
  return S::BLOCKS >= 1 && C::BLOCKS >= 1 && C::T <= 64 && 64 % C::T == 0 &&
         S::LDS_WORDS * 8 <= 80 * 1024 && C::LDS_WORDS * 8 <= 80 * 1024;
}

// full transforms on the split the context's NTT tuner chose (ctx->ntt_a;
// the default split_a(LOGN) when 0), one step either side of the default
template <int LOGN, int A, bool INVERSE>
int full_split(hck_context *ctx, uint64_t *buf, const LimbMap &map) {
  if constexpr (split_ok<LOGN, A>()) {
    const hck_context::Split *sp = split_tables(ctx, A);
    if (!sp) return set_error(HCK_EINVAL, "NTT split tables not built");
    launch_split<LOGN, A, !INVERSE, INVERSE>(ctx, buf, map, nullptr, *sp);
    launch_split<LOGN, A, INVERSE, INVERSE>(ctx, buf, map, nullptr, *sp);
    HCK_HIP(ctx, hipGetLastError());
    return HCK_OK;
  } else {
    return set_error(HCK_EINVAL, "NTT split not available for this ring");
  }
}

template <int LOGN, bool INVERSE>
int run_full(hck_context *ctx, uint64_t *buf, const LimbMap &map) {
  constexpr int A = split_a(LOGN);
  const int a = ctx->ntt_a ? ctx->ntt_a : A;
  if (a == A - 1) return full_split<LOGN, A - 1, INVERSE>(ctx, buf, map);
  if (a == A + 1) return full_split<LOGN, A + 1, INVERSE>(ctx, buf, map);
  return full_split<LOGN, A, INVERSE>(ctx, buf, map);
}

template <int LOGN>
int run_one(hck_context *ctx, uint64_t *buf, const LimbMap &map, bool inverse, bool strided,
            const RowFactors *sc) {
  constexpr int A = split_a(LOGN);
  const hck_context::Split &sp = ctx->split[0];
  if (!inverse && strided) launch_split<LOGN, A, true, false>(ctx, buf, map, nullptr, sp);
  if (!inverse && !strided) launch_split<LOGN, A, false, false>(ctx, buf, map, nullptr, sp);
  if (inverse && !strided) launch_split<LOGN, A, false, true>(ctx, buf, map, nullptr, sp);
  if (inverse && strided) launch_split<LOGN, A, true, true>(ctx, buf, map, sc, sp);
  HCK_HIP(ctx, hipGetLastError());
  return HCK_OK;
}

}  // namespace

template <int LOGN>
bool NttRing<LOGN>::split_available(int a) {
  constexpr int A = split_a(LOGN);
  return a == A || (a == A - 1 && split_ok<LOGN, A - 1>()) ||
         (a == A + 1 && split_ok<LOGN, A + 1>());
}

template <int LOGN>
int NttRing<LOGN>::ntt_full(hck_context *ctx, uint64_t *buf, const LimbMap &map, bool inverse) {
  return inverse ? run_full<LOGN, true>(ctx, buf, map) : run_full<LOGN, false>(ctx, buf, map);
}

template <int LOGN>
int NttRing<LOGN>::ntt_pass(hck_context *ctx, uint64_t *buf, const LimbMap &map, bool inverse,
                         bool strided, const RowFactors *sc) {
  return run_one<LOGN>(ctx, buf, map, inverse, strided, sc);
}

template <int LOGN>
int NttRing<LOGN>::rescale(hck_context *ctx, uint64_t *out, const uint64_t *in, uint64_t *tmp,
                           uint32_t level, uint32_t polys) {
  return run_rescale<LOGN>(ctx, out, in, tmp, level, polys);
}

template struct NttRing<HCK_LOGN>;

}  // namespace hck

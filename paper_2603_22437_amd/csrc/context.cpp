// Context: parameter validation, device tables, memory, errors, timing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <string>

#include "internal.h"

namespace hck {

namespace {
thread_local std::string g_last_error;

uint32_t bit_reverse(uint32_t x, uint32_t bits) {
  uint32_t r = 0;
  for (uint32_t i = 0; i < bits; i++) r |= ((x >> i) & 1u) << (bits - 1 - i);
  return r;
}

bool is_prime_u64(uint64_t n) {
  if (n < 2) return false;
  static const uint64_t small[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
  for (uint64_t p : small)
    if (n % p == 0) return n == p;
  uint64_t d = n - 1;
  int r = 0;
  while ((d & 1) == 0) {
    d >>= 1;
    r++;
  }
  for (uint64_t a : small) {
    uint64_t x = h_powmod(a, d, n);
    if (x == 1 || x == n - 1) continue;
    bool comp = true;
    for (int i = 1; i < r; i++) {
      x = h_mulmod(x, x, n);
      if (x == n - 1) {
        comp = false;
        break;
      }
    }
    if (comp) return false;
  }
  return true;
}

// A primitive 2N-th root of unity: psi = x^((q-1)/2N) for the first x >= 3
// with psi^N = -1 (q prime, q = 1 mod 2N).
uint64_t primitive_2n_root(uint64_t q, uint64_t n) {
  for (uint64_t x = 3;; x++) {
    uint64_t psi = h_powmod(x, (q - 1) / (2 * n), q);
    if (h_powmod(psi, n, q) == q - 1) return psi;
  }
}

// psi^k, k < N, and the same of psi^-1
struct Powers {
  std::vector<uint64_t> pw, ipw;
  uint64_t q, n;
  Powers(uint64_t q_, uint64_t n_) : pw(n_), ipw(n_), q(q_), n(n_) {
    const uint64_t psi = primitive_2n_root(q, n), ipsi = h_invmod(psi, q);
    pw[0] = ipw[0] = 1;
    for (uint64_t i = 1; i < n; i++) {
      pw[i] = h_mulmod(pw[i - 1], psi, q);
      ipw[i] = h_mulmod(ipw[i - 1], ipsi, q);
    }
  }
  // psi^e, psi^-e for any e (psi^N = -1)
  uint64_t pos(uint64_t e) const { return at(pw, e); }
  uint64_t neg(uint64_t e) const { return at(ipw, e); }

 private:
  uint64_t at(const std::vector<uint64_t> &v, uint64_t e) const {
    e &= 2 * n - 1;
    return e < n ? v[e] : q - v[e - n];
  }
};

int upload_table(hck_context *ctx, void **dst, const void *src, size_t bytes) {
  if (hipMalloc(dst, bytes) != hipSuccess) {
    *dst = nullptr;
    (void)hipGetLastError();
    return set_error(HCK_ENOMEM, "table allocation failed");
  }
  if (hipMemcpy(*dst, src, bytes, hipMemcpyHostToDevice) != hipSuccess)
    return check_hip(ctx, hipGetLastError(), "table upload");
  return HCK_OK;
}

// The tables of the split 2^log_a x 2^(log_n - log_a) (ntt_core.h): word
// g R2 + i of a limb's twist is psi^((2 brv_a(g) + 1) i); row i's factor of
// the inverse is N^-1 psi^(-R2 i).
int make_split(hck_context *ctx, const std::vector<Powers> &pws, int log_a,
               hck_context::Split *out) {
  const int log_b = (int)ctx->log_n - log_a;
  const size_t n = ctx->n, r1 = (size_t)1 << log_a, r2 = (size_t)1 << log_b, nm = pws.size();
  std::vector<Tw> t(nm * n), it(nm * n), rows(nm * r1);
  for (size_t m = 0; m < nm; m++) {
    const Powers &p = pws[m];
    for (size_t g = 0; g < r1; g++) {
      const uint64_t step = 2ull * bit_reverse((uint32_t)g, (uint32_t)log_a) + 1;
      for (size_t i = 0; i < r2; i++) {
        t[m * n + g * r2 + i] = h_tw(p.pos(step * i), p.q);
        it[m * n + g * r2 + i] = h_tw(p.neg(step * i), p.q);
      }
    }
    const uint64_t ninv = h_invmod(n % p.q, p.q);
    for (size_t i = 0; i < r1; i++)
      rows[m * r1 + i] = h_tw(h_mulmod(ninv, p.neg(r2 * i), p.q), p.q);
  }
  hck_context::Split sp;
  int rc = upload_table(ctx, (void **)&sp.twist, t.data(), t.size() * sizeof(Tw));
  if (!rc) rc = upload_table(ctx, (void **)&sp.itwist, it.data(), it.size() * sizeof(Tw));
  if (!rc) rc = upload_table(ctx, (void **)&sp.rows, rows.data(), rows.size() * sizeof(Tw));
  if (rc) {
    for (void *p : {(void *)sp.twist, (void *)sp.itwist, (void *)sp.rows})
      if (p) (void)hipFree(p);
    return rc;
  }
  *out = sp;
  return HCK_OK;
}

// f and g with f 2^50 + g = e modulo t, both of about sqrt(t): the point
// nearest to (0, e) in the lattice of (f, g) with f 2^50 + g = 0 mod t, over
// its Gauss-reduced basis.  (All values stay below 2^51, products below 2^102.)
void short_pair(int64_t e, uint64_t t, int64_t *f, int64_t *g) {
  using wide = __int128;
  auto nearest = [](wide a, wide b) {
    if (b < 0) a = -a, b = -b;
    return a >= 0 ? (a + b / 2) / b : -((b / 2 - a) / b);
  };
  wide uf = 1, ug = -(wide)h_centred((1ull << 50) % t, t), wf = 0, wg = t;
  for (;;) {
    if (uf * uf + ug * ug > wf * wf + wg * wg) {
      std::swap(uf, wf);
      std::swap(ug, wg);
    }
    const wide m = nearest(uf * wf + ug * wg, uf * uf + ug * ug);
    const wide nf = wf - m * uf, ng = wg - m * ug;
    if (nf * nf + ng * ng >= wf * wf + wg * wg) break;  // each turn shortens w
    wf = nf;
    wg = ng;
  }
  const wide det = uf * wg - ug * wf;
  const wide x = nearest(-(wide)e * wf, det), y = nearest(uf * e, det);
  *f = (int64_t)-(x * uf + y * wf);
  *g = (int64_t)(e - (x * ug + y * wg));
}

// The constants of one conversion's sources src[0..na) (moduli) to modulus t,
// hat(a) = the constant of source a, in rows out[a * stride] and the centring
// row out[na * stride].  Returns whether the conversion in doubles keeps every
// sum exact (bconv_float): over each 8 sources, with |v| <= 2^49 + 2^44 (a
// source in the floating-point range is below 2^50 + 2^44), v2 < 2^10 and what
// each product rounds off within 2^49,
//   sum |c| (2^49 + 2^44) + |f| 2^10 + 2^49 < 2^101,
//   sum 2^49 + |g| 2^10 < 2^53
// (with a margin for the rounding of these sums themselves).
template <class Hat>
bool conv_constants(const std::vector<uint64_t> &src, uint64_t t, Hat &&hat, ConvC *out,
                    size_t stride) {
  const uint64_t r64 = h_r64(t), off = (1ull << 49) % t;
  const double u49 = 562949953421312.0, u50 = 2 * u49;
  uint64_t k = 0;
  bool ok = true;
  double sum = 0, err = 0;
  for (size_t a = 0; a < src.size(); a++) {
    const uint64_t c = hat(a);
    ConvC &o = out[a * stride];
    o.w = h_mulmod(c, r64, t);
    o.c = o.f = o.g = 0;
    if (!h_float_modulus(t)) continue;
    if (a % 8 == 0) {  // later blocks start from the value of those before
      sum = 0;
      err = a ? 2 * u50 : 0;
    }
    o.c = (double)h_centred(c, t);
    k = (uint64_t)(((unsigned __int128)off * c + k) % t);
    if (!h_float_modulus(src[a])) {
      int64_t f, g;
      short_pair(h_centred(h_mulmod(c, (1ull << 50) % t, t), t), t, &f, &g);
      o.f = (double)f * u50;
      o.g = (double)g;
    }
    const auto abs = [](double d) { return d < 0 ? -d : d; };
    sum += abs(o.c) * (u49 + 17592186044416.0) + abs(o.f) * 1024 + u49;
    err += u49 + abs(o.g) * 1024;
    ok = ok && sum < 0.999999 * 0x1p101 && err < 0.999999 * 0x1p53;
  }
  ConvC &o = out[src.size() * stride];
  o.w = 0;
  o.f = o.g = 0;
  o.c = h_float_modulus(t) ? (double)h_centred(k, t) : 0;
  return ok;
}

}  // namespace

int set_error(int code, const std::string &msg) {
  g_last_error = msg;
  return code;
}

int check_hip(hck_context *ctx, hipError_t e, const char *what) {
  if (ctx) ctx->broken = true;
  return set_error(HCK_EDEVICE, std::string("HIP error in ") + what + ": " + hipGetErrorString(e));
}

// one record of the launch trace (hck_trace_enable)
static void trace_note(hck_context *ctx, const char *name, dim3 grid, double bytes,
                       double mulmods) {
  hck_trace_record r{};
  std::strncpy(r.name, name, sizeof(r.name) - 1);
  r.grid[0] = grid.x;
  r.grid[1] = grid.y;
  r.grid[2] = grid.z;
  r.bytes = bytes;
  r.mulmods = mulmods;
  ctx->trace_log.push_back(r);
}

int dev_alloc(hck_context *ctx, uint64_t **p, size_t words) {
  *p = nullptr;
  if (words == 0) return HCK_OK;
  const size_t bytes = words * sizeof(uint64_t);
  if (ctx->capturing)
    return set_error(HCK_EINVAL, "device allocation of " + std::to_string(bytes) +
                                     " bytes during graph capture (run the calls once "
                                     "before capturing them)");
  if (ctx->alloc_fn) {
    *p = (uint64_t *)ctx->alloc_fn(bytes, (void *)ctx->stream, ctx->alloc_user);
    if (!*p)
      return set_error(HCK_ENOMEM, "the allocator hook returned no memory for " +
                                       std::to_string(bytes) + " bytes");
  } else {
    hipError_t e = hipMallocAsync((void **)p, bytes, ctx->stream);
    if (e != hipSuccess) {
      *p = nullptr;
      (void)hipGetLastError();
      return set_error(HCK_ENOMEM, "device allocation of " + std::to_string(bytes) + " bytes failed");
    }
  }
  ctx->live_allocs++;
  ctx->alloc_seq[*p] = ++ctx->alloc_counter;
  if (ctx->trace) trace_note(ctx, "alloc", dim3(0, 0, 0), (double)bytes, 0);
  return HCK_OK;
}

void dev_free(hck_context *ctx, void *p) {
  if (!p) return;
  if (ctx->trace) trace_note(ctx, "free", dim3(0, 0, 0), 0, 0);
  if (ctx->free_fn) ctx->free_fn(p, (void *)ctx->stream, ctx->alloc_user);
  else (void)hipFreeAsync(p, ctx->stream);
  ctx->live_allocs--;
  auto it = ctx->alloc_seq.find(p);
  if (it != ctx->alloc_seq.end()) {
    if (it->second < ctx->graph_mark) ctx->freed_old.push_back(it->second);
    ctx->alloc_seq.erase(it);
  }
}

int ensure_ct(hck_context *ctx, hck_ciphertext *ct, uint32_t polys) {
  if (ct->cap_polys >= polys && ct->data) return HCK_OK;
  if (ct->pooled) polys = std::max(polys, 3u);
  uint64_t *p = nullptr;
  int rc = dev_alloc(ctx, &p, (size_t)polys * ctx->L * ctx->n);
  if (rc) return rc;
  if (ct->data && ct->size) {
    HCK_HIP(ctx, hipMemcpyAsync(p, ct->data, (size_t)ct->size * ctx->L * ctx->n * 8,
                                hipMemcpyDeviceToDevice, ctx->stream));
  }
  dev_free(ctx, ct->data);
  ct->data = p;
  ct->cap_polys = polys;
  return HCK_OK;
}

int ensure_workspace(hck_context *ctx, size_t words) {
  if (ctx->ws_words >= words) return HCK_OK;
  dev_free(ctx, ctx->ws);
  ctx->ws = nullptr;
  ctx->ws_words = 0;
  int rc = dev_alloc(ctx, &ctx->ws, words);
  if (rc) return rc;
  ctx->ws_words = words;
  return HCK_OK;
}

int ensure_lt_scratch(hck_context *ctx, size_t words) {
  if (ctx->lt_scratch_words >= words) return HCK_OK;
  dev_free(ctx, ctx->lt_scratch);
  ctx->lt_scratch = nullptr;
  ctx->lt_scratch_words = 0;
  int rc = dev_alloc(ctx, &ctx->lt_scratch, words);
  if (rc) return rc;
  ctx->lt_scratch_words = words;
  return HCK_OK;
}

int ensure_zero_rows(hck_context *ctx) {
  if (ctx->zero_rows) return HCK_OK;
  const size_t words = (size_t)ctx->L * ctx->n;
  int rc = dev_alloc(ctx, &ctx->zero_rows, words);
  if (rc) return rc;
  HCK_HIP(ctx, hipMemsetAsync(ctx->zero_rows, 0, words * sizeof(uint64_t), ctx->stream));
  return HCK_OK;
}

LimbMap qmap(const hck_context *ctx, uint32_t level) {
  LimbMap m;
  m.n = level + 1;
  for (uint32_t i = 0; i <= level; i++) {
    m.row[i] = (uint16_t)i;
    m.mod[i] = (uint8_t)i;
  }
  return m;
}

LimbMap fullmap(const hck_context *ctx) {
  LimbMap m;
  m.n = ctx->L + ctx->K;
  for (uint32_t i = 0; i < m.n; i++) {
    m.row[i] = (uint16_t)i;
    m.mod[i] = (uint8_t)i;
  }
  return m;
}

uint32_t galois_of_step(const hck_context *ctx, int32_t step) {
  const int64_t slots = ctx->n / 2;
  int64_t k = ((int64_t)step % slots + slots) % slots;
  return (uint32_t)h_powmod(5, (uint64_t)k, 2ull * ctx->n);
}

// ---- timing ----------------------------------------------------------------

void timing_begin(hck_context *ctx, const char *name, dim3 grid, double bytes, double mulmods) {
  if (ctx->trace) trace_note(ctx, name, grid, bytes, mulmods);
  if (!ctx->timing) return;
  hck_context::Timed t;
  t.name = name;
  t.bytes = bytes;
  t.mulmods = mulmods;
  for (hipEvent_t *ev : {&t.start, &t.stop}) {
    if (!ctx->event_pool.empty()) {
      *ev = ctx->event_pool.back();
      ctx->event_pool.pop_back();
    } else if (hipEventCreate(ev) != hipSuccess) {
      return;
    }
  }
  (void)hipEventRecord(t.start, ctx->stream);
  ctx->pending.push_back(t);
}

void timing_end(hck_context *ctx) {
  if (!ctx->timing || ctx->pending.empty()) return;
  (void)hipEventRecord(ctx->pending.back().stop, ctx->stream);
}

int timing_collect(hck_context *ctx) {
  if (ctx->pending.empty()) return HCK_OK;
  HCK_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (auto &t : ctx->pending) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, t.start, t.stop) == hipSuccess) {
      auto &slot = ctx->timing_total[t.name];
      slot.ms += ms;
      slot.launches += 1;
      slot.bytes += t.bytes;
      slot.mulmods += t.mulmods;
    }
    ctx->event_pool.push_back(t.start);
    ctx->event_pool.push_back(t.stop);
  }
  ctx->pending.clear();
  return HCK_OK;
}

// ---- context construction ------------------------------------------------------

static int validate(const hck_params *p) {
  if (!p || !p->q || (p->num_p && !p->p)) return set_error(HCK_EINVAL, "null parameters");
  if (p->log_n < 11 || p->log_n > 17) return set_error(HCK_EPARAMS, "log_n must be in [11, 17]");
  if (p->num_q < 1 || p->num_p < 1) return set_error(HCK_EPARAMS, "need at least one q and one p");
  if (p->num_q + p->num_p > (uint32_t)kMaxLimbs)
    return set_error(HCK_EPARAMS, "L + K exceeds HCK_MAX_LIMBS");
  if (p->dnum < 1 || p->dnum > p->num_q) return set_error(HCK_EPARAMS, "dnum must be in [1, L]");
  const uint64_t two_n = 2ull << p->log_n;
  std::vector<uint64_t> all(p->q, p->q + p->num_q);
  all.insert(all.end(), p->p, p->p + p->num_p);
  uint64_t maxm = 0;
  for (size_t i = 0; i < all.size(); i++) {
    uint64_t m = all[i];
    if (m >= (1ull << 61)) return set_error(HCK_EPARAMS, "modulus not below 2^61");
    if (m % two_n != 1) return set_error(HCK_EPARAMS, "modulus is not 1 mod 2N");
    if (!is_prime_u64(m)) return set_error(HCK_EPARAMS, "modulus is not prime");
    for (size_t j = 0; j < i; j++)
      if (all[j] == m) return set_error(HCK_EPARAMS, "moduli must be distinct");
    maxm = std::max(maxm, m);
  }
  const uint32_t alpha = (p->num_q + p->dnum - 1) / p->dnum;
  if (alpha > 16 || p->num_p > 16)
    return set_error(HCK_EPARAMS, "a digit or the special basis has more than 16 primes");
  for (uint32_t j = 0; j * alpha < p->num_q; j++) {
    unsigned __int128 s = 0;
    for (uint32_t i = j * alpha; i < std::min(p->num_q, (j + 1) * alpha); i++) s += p->q[i];
    if (s >> 64) return set_error(HCK_EPARAMS, "a digit's primes sum to 2^64 or more");
  }
  unsigned __int128 sp = 0;
  for (uint32_t k = 0; k < p->num_p; k++) sp += p->p[k];
  if (sp >> 64) return set_error(HCK_EPARAMS, "the special primes sum to 2^64 or more");
  if ((unsigned __int128)p->dnum * maxm >> 64)
    return set_error(HCK_EPARAMS, "dnum times the largest modulus reaches 2^64");
  return HCK_OK;
}

int build_context(const hck_params *prm, int device, void *stream, hck_context **out) {
  int rc = validate(prm);
  if (rc) return rc;
  HCK_HIP(nullptr, hipSetDevice(device));
  hck_context *ctx = new hck_context();
  ctx->device = device;
  ctx->stream = (hipStream_t)stream;
  ctx->log_n = prm->log_n;
  ctx->n = 1u << prm->log_n;
  ctx->L = prm->num_q;
  ctx->K = prm->num_p;
  ctx->dnum = prm->dnum;
  ctx->alpha = (ctx->L + ctx->dnum - 1) / ctx->dnum;
  ctx->mods.assign(prm->q, prm->q + prm->num_q);
  ctx->mods.insert(ctx->mods.end(), prm->p, prm->p + prm->num_p);
  ctx->bconv30 = std::all_of(ctx->mods.begin(), ctx->mods.end(),
                             [](uint64_t m) { return m < (1ull << 60); });
  const uint32_t nm = ctx->L + ctx->K, n = ctx->n, L = ctx->L, K = ctx->K;

  // per-modulus constants and twiddles
  std::vector<ModConst> mc(nm);
  std::vector<Tw> tw((size_t)nm * kTwLen), itn((size_t)nm * kRootLen);
  std::vector<Powers> pws;
  for (uint32_t m = 0; m < nm; m++) {
    const uint64_t q = ctx->mods[m];
    ModConst &c = mc[m];
    c.q = q;
    c.qinv = h_inv64(q);
    c.r64 = h_r64(q);
    c.r64_shoup = h_shoup(c.r64, q);
    c.ninv = h_invmod(n % q, q);
    c.r2 = h_mulmod(c.r64, c.r64, q);
    c.one_shoup = h_shoup(1, q);
    c.nq = 0 - q;
    c.qd = h_float_modulus(q) ? (double)q : 0.0;
    c.qid = h_float_modulus(q) ? 1.0 / (double)q : 0.0;
    pws.emplace_back(q, n);
    for (uint32_t k = 0; k < (uint32_t)kTwLen; k++)
      tw[(size_t)m * kTwLen + k] = h_tw(pws[m].pos(bit_reverse(k, ctx->log_n)), q);
    for (uint32_t k = 0; k < (uint32_t)kRootLen; k++)
      itn[(size_t)m * kRootLen + k] = h_tw(pws[m].neg((uint64_t)k * (n / kRootLen)), q);
  }

  // ModUp tables: for each level l and digit j with limbs D = [lo, hi),
  // row factors N^-1 (Q_D / q_i)^-1 psi^(-R2 r) mod q_i and the constants
  // Q_D / q_(lo+a) mod m.
  const uint32_t A = ctx->alpha;
  const uint32_t r1 = 1u << ((ctx->log_n + 1) / 2), r2 = n / r1;
  auto row_factors = [&](uint32_t m, uint64_t scale, Tw *out) {
    for (uint32_t r = 0; r < r1; r++)
      out[r] = h_tw(h_mulmod(scale, pws[m].neg((uint64_t)r2 * r), ctx->mods[m]), ctx->mods[m]);
  };
  std::vector<ConvC> up_conv((size_t)L * ctx->dnum * (A + 1) * nm, ConvC{});
  std::vector<Tw> up_rows((size_t)L * L * r1, Tw{0, 0});
  ctx->conv_f = true;
  for (uint32_t l = 0; l < L; l++) {
    for (uint32_t j = 0; j < ctx->dnum; j++) {
      const uint32_t lo = j * A;
      if (lo > l) break;
      const uint32_t hi = std::min(lo + A, l + 1);
      const std::vector<uint64_t> src(ctx->mods.begin() + lo, ctx->mods.begin() + hi);
      auto hat = [&](uint32_t i, uint64_t t) {  // Q_D / q_i mod t
        uint64_t h = 1;
        for (uint32_t k = lo; k < hi; k++)
          if (k != i) h = h_mulmod(h, ctx->mods[k] % t, t);
        return h % t;
      };
      for (uint32_t i = lo; i < hi; i++) {
        const uint64_t q = ctx->mods[i];
        row_factors(i, h_mulmod(h_invmod(hat(i, q), q), mc[i].ninv, q),
                    &up_rows[((size_t)l * L + i) * r1]);
      }
      for (uint32_t m = 0; m < nm; m++) {
        const uint64_t t = ctx->mods[m];
        const bool ok = conv_constants(
            src, t, [&](size_t a) { return hat(lo + (uint32_t)a, t); },
            &up_conv[((size_t)l * ctx->dnum + j) * (A + 1) * nm + m], nm);
        // (a digit is not converted to its own limbs)
        if (m < lo || m >= hi) ctx->conv_f = ctx->conv_f && ok;
      }
    }
  }

  // ModDown tables over P = prod p_k, with the rounding addend h = (P-1)/2.
  std::vector<ConvC> down_conv((size_t)(K + 1) * nm, ConvC{});
  std::vector<Tw> down_rows((size_t)K * r1);
  std::vector<uint64_t> down_add(K);
  const std::vector<uint64_t> specials(ctx->mods.begin() + L, ctx->mods.end());
  auto down_hat = [&](uint32_t k, uint64_t t) {  // P / p_k mod t
    uint64_t h = 1;
    for (uint32_t r = 0; r < K; r++)
      if (r != k) h = h_mulmod(h, specials[r] % t, t);
    return h % t;
  };
  for (uint32_t k = 0; k < K; k++) {
    const uint64_t pk = specials[k];
    const uint64_t hat_inv = h_invmod(down_hat(k, pk), pk);
    row_factors(L + k, h_mulmod(hat_inv, mc[L + k].ninv, pk), &down_rows[(size_t)k * r1]);
    // (P-1)/2 mod p_k = -2^-1 mod p_k
    down_add[k] = h_mulmod(pk - h_invmod(2, pk), hat_inv, pk);
  }
  for (uint32_t m = 0; m < L; m++) {
    const uint64_t t = ctx->mods[m];
    const bool ok = conv_constants(
        specials, t, [&](size_t k) { return down_hat((uint32_t)k, t); }, &down_conv[m], nm);
    ctx->conv_f = ctx->conv_f && ok;
  }

  // targets per workgroup of the basis conversions: single, and pairs of
  // consecutive targets of one arithmetic (the kernel picks the first target's
  // for both; a modulus of 2^60 or more overflows in the class below it)
  std::vector<ConvGroup> groups;
  auto group_targets = [&](const std::vector<ConvGroup> &one, bool pairs) {
    const std::pair<uint32_t, uint32_t> none((uint32_t)groups.size(), 0);
    auto range = none;
    for (size_t i = 0; i < one.size(); i++) {
      ConvGroup g = one[i];
      if (pairs && i + 1 < one.size() && one[i + 1].digit == g.digit &&
          h_arith_class(ctx->mods[g.mod[0]]) == h_arith_class(ctx->mods[one[i + 1].mod[0]])) {
        g.row[1] = one[i + 1].row[0];
        g.mod[1] = one[i + 1].mod[0];
        g.n = 2;
        i++;
      }
      groups.push_back(g);
      range.second++;
    }
    return range;
  };
  for (uint32_t l = 0; l < L; l++) {
    std::vector<ConvGroup> up, down;
    const uint32_t nq = l + 1, ne = nq + K;
    for (uint32_t j = 0; j * A < nq; j++)
      for (uint32_t t = 0; t < ne; t++) {
        if (t >= j * A && t < std::min((j + 1) * A, nq)) continue;
        const uint8_t m = (uint8_t)(t < nq ? t : L + (t - nq));
        const uint16_t row = (uint16_t)(L + j * ne + t);
        up.push_back(ConvGroup{{row, row}, {m, m}, (uint8_t)j, 1});
      }
    for (uint32_t t = 0; t < nq; t++)
      down.push_back(ConvGroup{{0, 0}, {(uint8_t)t, (uint8_t)t}, 0, 1});
    for (int pairs = 0; pairs < 2; pairs++) {
      ctx->groups[pairs].push_back(group_targets(up, pairs));
      ctx->down_groups[pairs].push_back(group_targets(down, pairs));
    }
  }
  std::vector<uint64_t> down_hneg(L);
  std::vector<Tw> pinv(L), rescale((size_t)L * L, Tw{0, 0});
  for (uint32_t i = 0; i < L; i++) {
    const uint64_t q = ctx->mods[i];
    uint64_t pm = 1;
    for (uint32_t k = 0; k < K; k++) pm = h_mulmod(pm, ctx->mods[L + k] % q, q);
    pinv[i] = h_tw(h_invmod(pm, q), q);
    // (P-1)/2 mod q = (P mod q - 1) 2^-1 mod q; stored negated
    const uint64_t h = h_mulmod((pm + q - 1) % q, h_invmod(2, q), q);
    down_hneg[i] = h == 0 ? 0 : q - h;
  }
  for (uint32_t l = 1; l < L; l++)
    for (uint32_t i = 0; i < l; i++)
      rescale[(size_t)l * L + i] =
          h_tw(h_invmod(ctx->mods[l] % ctx->mods[i], ctx->mods[i]), ctx->mods[i]);

  // upload
  auto up = [&](auto **dst, const auto &v) {
    return upload_table(ctx, (void **)dst, v.data(), v.size() * sizeof(v[0]));
  };
  if ((rc = up(&ctx->d_mod, mc)) || (rc = up(&ctx->d_tw, tw)) || (rc = up(&ctx->d_itn, itn)) ||
      (rc = make_split(ctx, pws, (int)(ctx->log_n + 1) / 2, &ctx->split[0])) ||
      (rc = up(&ctx->d_up_conv, up_conv)) || (rc = up(&ctx->d_up_rows, up_rows)) ||
      (rc = up(&ctx->d_down_conv, down_conv)) || (rc = up(&ctx->d_down_rows, down_rows)) ||
      (rc = up(&ctx->d_down_add, down_add)) || (rc = up(&ctx->d_down_hneg, down_hneg)) ||
      (rc = up(&ctx->d_pinv, pinv)) || (rc = up(&ctx->d_rescale, rescale)) ||
      (rc = up(&ctx->d_groups, groups))) {
    hck_context_destroy(ctx);
    return rc;
  }
  *out = ctx;
  return HCK_OK;
}

const hck_context::Split *split_tables(const hck_context *ctx, int a) {
  const int a0 = (ctx->log_n + 1) / 2;
  if (a < a0 - 1 || a > a0 + 1) return nullptr;
  const hck_context::Split &sp = ctx->split[a == a0 ? 0 : a < a0 ? 1 : 2];
  return sp.twist ? &sp : nullptr;
}

int set_ntt_split(hck_context *ctx, int a) {
  const int a0 = (ctx->log_n + 1) / 2;
  if (a == 0 || a == a0) {
    ctx->ntt_a = 0;
    return HCK_OK;
  }
  if (!ntt_split_available(ctx->log_n, a))
    return set_error(HCK_EINVAL, "NTT split " + std::to_string(a) + " not available at log N " +
                                     std::to_string(ctx->log_n));
  if (ctx->capturing) return set_error(HCK_EINVAL, "NTT split change during graph capture");
  hck_context::Split &sp = ctx->split[a < a0 ? 1 : 2];
  if (!sp.twist) {
    std::vector<Powers> pws;
    for (uint64_t q : ctx->mods) pws.emplace_back(q, ctx->n);
    const int rc = make_split(ctx, pws, a, &sp);
    if (rc) return rc;
  }
  ctx->ntt_a = (uint8_t)a;
  return HCK_OK;
}

void track(hck_context *ctx, void *obj, void (*release)(void *)) { ctx->handles[obj] = release; }

void untrack(hck_context *ctx, void *obj) { ctx->handles.erase(obj); }

void track_server(hck_context *ctx, void *srv, void (*release)(void *)) {
  ctx->servers[srv] = release;
}

void untrack_server(hck_context *ctx, void *srv) { ctx->servers.erase(srv); }

void destroy_context(hck_context *ctx) {
  if (!ctx) return;
  (void)hipSetDevice(ctx->device);
  abort_capture(ctx);
  // servers stop their workers first; then every live handle gives back its
  // device memory and is detached
  auto servers = std::move(ctx->servers);
  ctx->servers.clear();
  for (auto &kv : servers) kv.second(kv.first);
  auto handles = std::move(ctx->handles);
  ctx->handles.clear();
  for (auto &kv : handles) kv.second(kv.first);
  if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
  dev_free(ctx, ctx->ws);
  dev_free(ctx, ctx->lt_scratch);
  dev_free(ctx, ctx->zero_rows);
  for (hck_ciphertext *ct : ctx->ct_pool) {
    dev_free(ctx, ct->data);
    delete ct;
  }
  ctx->ct_pool.clear();
  if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
  else (void)hipDeviceSynchronize();
  for (void *p : {(void *)ctx->d_mod, (void *)ctx->d_tw, (void *)ctx->d_itn,
                  (void *)ctx->d_up_conv, (void *)ctx->d_up_rows, (void *)ctx->d_down_conv,
                  (void *)ctx->d_down_rows, (void *)ctx->d_down_add, (void *)ctx->d_down_hneg,
                  (void *)ctx->d_pinv, (void *)ctx->d_rescale, (void *)ctx->d_groups})
    if (p) (void)hipFree(p);
  for (auto &sp : ctx->split)
    for (void *p : {(void *)sp.twist, (void *)sp.itwist, (void *)sp.rows})
      if (p) (void)hipFree(p);
  for (auto &t : ctx->pending) {
    (void)hipEventDestroy(t.start);
    (void)hipEventDestroy(t.stop);
  }
  for (hipEvent_t e : ctx->event_pool) (void)hipEventDestroy(e);
  // the stream-ordered allocator keeps the freed buffers cached in the
  // device's pool; hand them back, so that a destroyed context's workspace
  // and keys (several GB at N = 2^16) do not crowd later allocations
  if (!ctx->alloc_fn) {
    hipMemPool_t pool = nullptr;
    if (hipDeviceGetDefaultMemPool(&pool, ctx->device) == hipSuccess && pool)
      (void)hipMemPoolTrimTo(pool, 0);
    (void)hipGetLastError();
  }
  delete ctx;
}

}  // namespace hck

extern "C" {

const char *hck_last_error(void) { return hck::g_last_error.c_str(); }

int hck_context_create(const hck_params *params, int device, void *hip_stream,
                       hck_context **out) {
  if (!out) return hck::set_error(HCK_EINVAL, "null output");
  *out = nullptr;
  return hck::build_context(params, device, hip_stream, out);
}

int hck_context_destroy(hck_context *ctx) {
  hck::destroy_context(ctx);
  return HCK_OK;
}

int hck_set_allocator(hck_context *ctx, void *(*alloc)(size_t, void *, void *),
                      void (*free_fn)(void *, void *, void *), void *user) {
  if (!ctx) return hck::set_error(HCK_EINVAL, "null context");
  if (!alloc != !free_fn)
    return hck::set_error(HCK_EINVAL, "give both allocator functions or neither");
  if (ctx->live_allocs)
    return hck::set_error(HCK_EINVAL, "the context still holds device buffers of the current "
                                      "allocator");
  ctx->alloc_fn = alloc;
  ctx->free_fn = free_fn;
  ctx->alloc_user = alloc ? user : nullptr;
  return HCK_OK;
}

int hck_context_set_stream(hck_context *ctx, void *hip_stream) {
  if (!ctx) return hck::set_error(HCK_EINVAL, "null context");
  if (ctx->capturing) return hck::set_error(HCK_EINVAL, "stream change during graph capture");
  ctx->stream = (hipStream_t)hip_stream;
  return HCK_OK;
}

int hck_synchronize(hck_context *ctx) {
  if (!ctx) return hck::set_error(HCK_EINVAL, "null context");
  if (ctx->capturing) return hck::set_error(HCK_EINVAL, "wait during graph capture");
  HCK_HIP(ctx, hipStreamSynchronize(ctx->stream));
  return HCK_OK;
}

uint32_t hck_galois_element(const hck_context *ctx, int32_t step) {
  return ctx ? hck::galois_of_step(ctx, step) : 0;
}

int hck_timing_enable(hck_context *ctx, int on) {
  if (!ctx) return hck::set_error(HCK_EINVAL, "null context");
  if (ctx->capturing) return hck::set_error(HCK_EINVAL, "timing during graph capture");
  int rc = hck::timing_collect(ctx);
  ctx->timing = on != 0;
  return rc;
}

int hck_timing_reset(hck_context *ctx) {
  if (!ctx) return hck::set_error(HCK_EINVAL, "null context");
  int rc = hck::timing_collect(ctx);
  ctx->timing_total.clear();
  return rc;
}

int hck_timing_read(hck_context *ctx, const char *name, double *total_ms, uint64_t *launches,
                    double *bytes, double *mulmods) {
  if (!ctx || !name) return hck::set_error(HCK_EINVAL, "null argument");
  int rc = hck::timing_collect(ctx);
  if (rc) return rc;
  hck_context::TimingTotal t;
  auto it = ctx->timing_total.find(name);
  if (it != ctx->timing_total.end()) t = it->second;
  if (total_ms) *total_ms = t.ms;
  if (launches) *launches = t.launches;
  if (bytes) *bytes = t.bytes;
  if (mulmods) *mulmods = t.mulmods;
  return HCK_OK;
}

int hck_trace_enable(hck_context *ctx, int on) {
  if (!ctx) return hck::set_error(HCK_EINVAL, "null context");
  if (on) ctx->trace_log.clear();
  ctx->trace = on != 0;
  return HCK_OK;
}

int hck_trace_read(hck_context *ctx, hck_trace_record *out, size_t cap, size_t *count) {
  if (!ctx || !count || (cap && !out)) return hck::set_error(HCK_EINVAL, "null argument");
  *count = ctx->trace_log.size();
  const size_t n = std::min(cap, ctx->trace_log.size());
  if (n) std::memcpy(out, ctx->trace_log.data(), n * sizeof(hck_trace_record));
  return HCK_OK;
}

int hck_timing_names(hck_context *ctx, char *buf, size_t cap) {
  if (!ctx || !buf || cap == 0) return hck::set_error(HCK_EINVAL, "null argument");
  int rc = hck::timing_collect(ctx);
  if (rc) return rc;
  std::string s;
  for (auto &kv : ctx->timing_total) {
    if (!s.empty()) s += ",";
    s += kv.first;
  }
  std::strncpy(buf, s.c_str(), cap - 1);
  buf[cap - 1] = 0;
  return s.size() < cap ? HCK_OK : hck::set_error(HCK_EINVAL, "buffer too small");
}

}  // extern "C"

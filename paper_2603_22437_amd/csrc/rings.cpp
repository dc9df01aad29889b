// Dispatch to the ring's transforms and key switching: ntt.hip and
// ks_fused.hip are compiled once per ring degree.
#include <algorithm>

#include "internal.h"

namespace hck {

#define HCK_BY_RING(T, CALL)                                           \
  switch (ctx->log_n) {                                                \
    case 11: return T<11>::CALL;                                       \
    case 12: return T<12>::CALL;                                       \
    case 13: return T<13>::CALL;                                       \
    case 14: return T<14>::CALL;                                       \
    case 15: return T<15>::CALL;                                       \
    case 16: return T<16>::CALL;                                       \
    case 17: return T<17>::CALL;                                       \
    default: return set_error(HCK_EPARAMS, "unsupported ring degree"); \
  }

bool ntt_split_available(uint32_t log_n, int a) {
  switch (log_n) {
    case 11: return NttRing<11>::split_available(a);
    case 12: return NttRing<12>::split_available(a);
    case 13: return NttRing<13>::split_available(a);
    case 14: return NttRing<14>::split_available(a);
    case 15: return NttRing<15>::split_available(a);
    case 16: return NttRing<16>::split_available(a);
    case 17: return NttRing<17>::split_available(a);
    default: return false;
  }
}

int ntt_forward(hck_context *ctx, uint64_t *buf, const LimbMap &map) {
  if (map.n == 0) return HCK_OK;
  HCK_BY_RING(NttRing, ntt_full(ctx, buf, map, false))
}

int ntt_inverse(hck_context *ctx, uint64_t *buf, const LimbMap &map) {
  if (map.n == 0) return HCK_OK;
  HCK_BY_RING(NttRing, ntt_full(ctx, buf, map, true))
}

int ntt_pass(hck_context *ctx, uint64_t *buf, const LimbMap &map, bool inverse, bool strided,
             const RowFactors *sc) {
  if (map.n == 0) return HCK_OK;
  HCK_BY_RING(NttRing, ntt_pass(ctx, buf, map, inverse, strided, sc))
}

int rescale_fused(hck_context *ctx, uint64_t *out, const uint64_t *in, uint64_t *tmp,
                  uint32_t level, uint32_t polys) {
  if (level == 0 || polys == 0) return HCK_OK;
  if (level > (uint32_t)kMaxLimbs) return set_error(HCK_EINVAL, "too many limbs");
  HCK_BY_RING(NttRing, rescale(ctx, out, in, tmp, level, polys))
}

// Batches grow where each slot is small (low levels), so that a launch still
// fills the chip; at high levels 8 slots of 24 limbs already do, and larger
// batches measured slower there (more data between the passes of a batch).
uint32_t ks_batch_fit(const hck_context *ctx, uint32_t level) {
  const uint32_t by_rows = (uint32_t)kMaxRows / std::max<uint32_t>(level + 1, 2 * ctx->K);
  return std::max<uint32_t>(1, std::min(ks_slots(ctx), by_rows));
}

uint32_t ks_batch_limit(const hck_context *ctx, uint32_t level) {
  const uint32_t fit = ks_batch_fit(ctx, level);
  if (level < (uint32_t)HCK_MAX_LIMBS && ctx->ks_cap[level])
    return std::min<uint32_t>(fit, ctx->ks_cap[level]);
  return std::min<uint32_t>(fit, std::max<uint32_t>(1, 192 / (level + 1)));
}

int keyswitch_batch(hck_context *ctx, const KsBatch &kb, uint32_t level) {
  if (kb.n == 0) return HCK_OK;
  if (kb.n > ks_slots(ctx)) return set_error(HCK_EINVAL, "batch too large");
  int rc = ensure_workspace(ctx, ws_words_needed(ctx));
  if (rc) return rc;
  return keyswitch_batch_ws(ctx, kb, level, ws_ks(ctx));
}

int keyswitch_batch_ws(hck_context *ctx, const KsBatch &kb, uint32_t level, uint64_t *ws) {
  if (kb.n == 0) return HCK_OK;
  if (level + 1 > (uint32_t)kMaxLimbs || (level + 1) * kb.n > (uint32_t)kMaxRows ||
      2 * ctx->K * kb.n > (uint32_t)kMaxRows)
    return set_error(HCK_EINVAL, "level too high for one batched launch");
  HCK_BY_RING(KsRing, run(ctx, kb, level, ws))
}

int keyswitch_core(hck_context *ctx, const uint64_t *d, uint32_t galois, uint32_t level,
                   const hck_switch_key *key, uint64_t *out0, uint64_t *out1, const uint64_t *add0,
                   const uint64_t *add1) {
  KsBatch kb;
  kb.n = 1;
  kb.key[0] = key->data;
  kb.galois[0] = galois;
  kb.d[0] = d;
  kb.out0[0] = out0;
  kb.out1[0] = out1;
  kb.add0[0] = add0;
  kb.add1[0] = add1;
  return keyswitch_batch(ctx, kb, level);
}

int keyswitch_hoisted(hck_context *ctx, const uint64_t *c0, const uint64_t *c1, uint32_t level,
                      const uint32_t *galois, const hck_switch_key *const *keys, uint32_t n,
                      uint64_t *const *out0, uint64_t *const *out1) {
  if (n == 0) return HCK_OK;
  int rc = ensure_workspace(ctx, ws_words_needed(ctx));
  if (rc) return rc;
  if (level + 1 > (uint32_t)kMaxLimbs || 2 * ctx->K > (uint32_t)kMaxRows)
    return set_error(HCK_EINVAL, "level too high for one batched launch");
  HCK_BY_RING(KsRing, hoisted(ctx, c0, c1, level, galois, keys, n, out0, out1))
}


int keyswitch_pq(hck_context *ctx, const KsBatch &kb, uint32_t level, uint64_t *const *pq,
                 const bool *first) {
  if (kb.n == 0) return HCK_OK;
  if (kb.n > ks_batch_limit(ctx, level)) return set_error(HCK_EINVAL, "batch too large");
  int rc = ensure_workspace(ctx, ws_words_needed(ctx));
  if (rc) return rc;
  HCK_BY_RING(KsRing, pq(ctx, kb, level, pq, first))
}

int moddown_pq(hck_context *ctx, const KsBatch &kb, uint32_t level, const uint64_t *const *pq) {
  if (kb.n == 0) return HCK_OK;
  if (kb.n > ks_batch_limit(ctx, level)) return set_error(HCK_EINVAL, "batch too large");
  int rc = ensure_workspace(ctx, ws_words_needed(ctx));
  if (rc) return rc;
  HCK_BY_RING(KsRing, md(ctx, kb, level, pq))
}

}  // namespace hck

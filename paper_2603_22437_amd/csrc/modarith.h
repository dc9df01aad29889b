// Modular arithmetic for residues below 2^61 on gfx950.
//
// Wide products use the compiler's native 64x64 -> 128-bit forms
// (unsigned __int128, __umul64hi), which gfx950 builds from v_mad_u64_u32,
// v_mul_hi_u32 and v_mul_lo_u32.  Measured on the chip these beat
// hand-placed v_mad_u64_u32 chains: inline asm forces register-pair copies
// for its 64-bit addends and hazard padding the compiler cannot schedule
// away (about 1.9 vs 1.7 T Shoup products/s and 3.1 vs 2.3 T 128-bit
// multiply-accumulates/s over the whole chip).
//
// Reduction schemes:
//   * Shoup, for a known constant w < q with w' = floor(w 2^64 / q):
//       a w mod q = a w - floor(a w' / 2^64) q   in [0, 2q) for any a < 2^64;
//   * Montgomery REDC for a 128-bit T < q 2^64 with qinv = q^-1 mod 2^64:
//       REDC(T) = T 2^-64 mod q  in [0, q);
//     used where a sum of products is reduced once (basis conversion, key
//     inner product): multiplying one factor by 2^64 mod q beforehand cancels
//     the 2^-64.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hck {

struct u128 {
  uint64_t lo, hi;
};

typedef unsigned __int128 wide_t;

// High 64 bits of a * b.
__host__ __device__ __forceinline__ uint64_t mul_hi(uint64_t a, uint64_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __umul64hi(a, b);
#else
  return (uint64_t)(((wide_t)a * b) >> 64);
#endif
}

// Low 64 bits of a * b.
__host__ __device__ __forceinline__ uint64_t mul_lo(uint64_t a, uint64_t b) { return a * b; }

// Full 128-bit product.
__host__ __device__ __forceinline__ u128 mul_wide(uint64_t a, uint64_t b) {
  const wide_t p = (wide_t)a * b;
  u128 r;
  r.lo = (uint64_t)p;
  r.hi = (uint64_t)(p >> 64);
  return r;
}

// acc += a * b (128-bit accumulate; the caller bounds the sum below 2^128).
__host__ __device__ __forceinline__ void mac_wide(u128 &acc, uint64_t a, uint64_t b) {
  wide_t t = ((wide_t)acc.hi << 64) | acc.lo;
  t += (wide_t)a * b;
  acc.lo = (uint64_t)t;
  acc.hi = (uint64_t)(t >> 64);
}

// a w mod q in [0, 2q), for any a < 2^64 and q < 2^63.
__host__ __device__ __forceinline__ uint64_t shoup_lazy(uint64_t a, uint64_t w, uint64_t wp,
                                                        uint64_t q) {
  return mul_lo(a, w) - mul_lo(mul_hi(a, wp), q);
}

// A constant factor modulo q with its companion, for the products of the
// transforms: moduli in the floating-point range (ModConst::qd) hold the
// centred factor and its quotient by q as doubles, others the factor in
// [0, q) and floor(w 2^64 / q).
struct alignas(16) Tw {
  uint64_t w, wp;
};

// A modulus with its negation nq = 2^64 - q.  nq comes from memory, so the
// compiler cannot see that it is -q and keeps "+ k nq" a multiply-add
// (v_mad_u64_u32 takes the addend) and "+ nq" one 64-bit add, where "- k q"
// would be a subtract-with-borrow pair that waits on its carry.
struct Qn {
  uint64_t q, nq;
};

// a w mod q in [0, 2q), the same word as shoup_lazy: a w + qh (2^64 - q)
// = a w - qh q mod 2^64.
__host__ __device__ __forceinline__ uint64_t shoup_lazy(uint64_t a, uint64_t w, uint64_t wp,
                                                        Qn m) {
  return mul_lo(a, w) + mul_lo(mul_hi(a, wp), m.nq);
}

// x - b if x >= b, else x (nb = 2^64 - b).
__host__ __device__ __forceinline__ uint64_t csub(uint64_t x, uint64_t b, uint64_t nb) {
  return x + (x >= b ? nb : 0);
}

__host__ __device__ __forceinline__ uint64_t reduce2(uint64_t a, uint64_t q) {
  return a >= q ? a - q : a;
}

// a w mod q in [0, q).
__host__ __device__ __forceinline__ uint64_t shoup(uint64_t a, uint64_t w, uint64_t wp,
                                                   uint64_t q) {
  return reduce2(shoup_lazy(a, w, wp, q), q);
}

// T 2^-64 mod q in [0, q) for T < q 2^64.
__host__ __device__ __forceinline__ uint64_t redc(u128 t, uint64_t q, uint64_t qinv) {
  uint64_t m = mul_lo(t.lo, qinv);
  uint64_t mh = mul_hi(m, q);
  // T - m q has a zero low word, so its high word is t.hi - mh (no borrow).
  return t.hi >= mh ? t.hi - mh : t.hi + q - mh;
}

__host__ __device__ __forceinline__ uint64_t add_mod(uint64_t a, uint64_t b, uint64_t q) {
  uint64_t s = a + b;
  return s >= q ? s - q : s;
}

__host__ __device__ __forceinline__ uint64_t sub_mod(uint64_t a, uint64_t b, uint64_t q) {
  return a >= b ? a - b : a + q - b;
}

// ---- host-side constant helpers (exact, via unsigned __int128) -----------

inline uint64_t h_mulmod(uint64_t a, uint64_t b, uint64_t q) {
  return (uint64_t)((unsigned __int128)a * b % q);
}

inline uint64_t h_powmod(uint64_t a, uint64_t e, uint64_t q) {
  uint64_t r = 1 % q;
  a %= q;
  for (; e; e >>= 1) {
    if (e & 1) r = h_mulmod(r, a, q);
    a = h_mulmod(a, a, q);
  }
  return r;
}

// Inverse modulo a prime.
inline uint64_t h_invmod(uint64_t a, uint64_t q) { return h_powmod(a % q, q - 2, q); }

// floor(w 2^64 / q), the Shoup companion of w < q.
inline uint64_t h_shoup(uint64_t w, uint64_t q) {
  return (uint64_t)(((unsigned __int128)w << 64) / q);
}

// q^-1 mod 2^64 for odd q (Newton iteration, 6 doublings of precision).
inline uint64_t h_inv64(uint64_t q) {
  uint64_t x = q;  // correct to 3 bits for odd q
  for (int i = 0; i < 6; i++) x *= 2 - q * x;
  return x;
}

// Moduli whose residues the transforms keep in doubles (ntt_core.h): large
// enough that a quotient by q stays exact, small enough that 53 bits hold
// 7.87 q, which the bounds of the passes (ArF::fits) stay within.
inline bool h_float_modulus(uint64_t q) {
  return q >= (1ull << 26) && q < (1ull << 50) + (1ull << 44);
}

// The arithmetic a modulus runs in (with_arith in ntt_core.h): doubles,
// integers below 2^60, integers from 2^60 on.
inline int h_arith_class(uint64_t q) {
  return h_float_modulus(q) ? 0 : q < (1ull << 60) ? 1 : 2;
}

inline uint64_t h_bits(double d) {
  uint64_t u;
  __builtin_memcpy(&u, &d, 8);
  return u;
}

// w in [0, q) centred about 0.
inline int64_t h_centred(uint64_t w, uint64_t q) {
  return w > q / 2 ? (int64_t)w - (int64_t)q : (int64_t)w;
}

inline Tw h_tw(uint64_t w, uint64_t q) {
  if (!h_float_modulus(q)) return Tw{w, h_shoup(w, q)};
  const double c = (double)h_centred(w, q);
  return Tw{h_bits(c), h_bits(c / (double)q)};
}

// 2^64 mod q.
inline uint64_t h_r64(uint64_t q) { return (uint64_t)(((unsigned __int128)1 << 64) % q); }

}  // namespace hck

// Exact convolutions modulo the reconstruction's prime p < 2^63 by
// number-theoretic transforms modulo five 30-bit primes q_i = 1 mod 2^22.
//
// A coefficient of the product of two polynomials over [0, p) with at most
// 2^21 + 1 overlapping terms is an integer below 2^(126 + 21.1); the product
// of the five primes is above 2^149, so its residues modulo them determine it,
// and the Chinese remainder theorem followed by one reduction gives its value
// modulo p exactly.  Five 30-bit primes rather than three 62-bit ones: a
// product modulo q is three multiply instructions (v_mad_u64_u32, v_mul_lo_u32,
// v_mad_u64_u32) against seven or eight, and sums are one-word adds with a
// v_min_u32 in place of compares and selects.
//
// Residues are plain (not in Montgomery form); constants (twiddles, kernels)
// are stored as w 2^32 mod q, so that Montgomery's reduction of x (w 2^32)
// gives x w.  Lazy ranges (D. Harvey, "Faster arithmetic for number-theoretic
// transforms", J. Symb. Comp. 2014): forward butterflies take and give values
// in [0, 4q), inverse ones in [0, 2q).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zr {

constexpr int kNp = 5;            // primes
constexpr int kNttMaxLog = 22;    // q = 1 mod 2^22: transforms up to 2^22
constexpr uint32_t kQ[kNp] = {998244353u, 985661441u, 943718401u, 935329793u, 918552577u};

// ---- constants (evaluated by the compiler) ---------------------------------------

constexpr uint32_t ntt_pow(uint32_t a, uint64_t e, uint32_t q) {
  uint64_t r = 1, b = a;
  for (; e; e >>= 1) {
    if (e & 1) r = r * b % q;
    b = b * b % q;
  }
  return (uint32_t)r;
}
constexpr uint32_t ntt_mont(uint32_t a, uint32_t q) { return (uint32_t)(((uint64_t)a << 32) % q); }
constexpr uint32_t ntt_neg_inv(uint32_t q) {  // -q^-1 mod 2^32
  uint32_t x = 1;
  for (int i = 0; i < 6; ++i) x *= 2 - q * x;
  return 0u - x;
}
// a root of unity of order 2^22 modulo q: (q-1)/2^22-th power of a quadratic nonresidue
constexpr uint32_t ntt_root(uint32_t q) {
  uint32_t g = 2;
  while (ntt_pow(g, (q - 1) / 2, q) == 1) ++g;
  return ntt_pow(g, (q - 1) >> kNttMaxLog, q);
}

struct NttMods {
  uint32_t q[kNp], ni[kNp];  // the primes and -q^-1 mod 2^32
  uint32_t r1[kNp], r2[kNp];  // 2^32 and 2^64 mod q
};
constexpr NttMods ntt_mods() {
  NttMods m{};
  for (int i = 0; i < kNp; ++i) {
    m.q[i] = kQ[i];
    m.ni[i] = ntt_neg_inv(kQ[i]);
    m.r1[i] = ntt_mont(1, kQ[i]);
    m.r2[i] = ntt_mont(m.r1[i], kQ[i]);
  }
  return m;
}
constexpr NttMods kNtt = ntt_mods();

// Garner's constants q_i^-1 mod q_j (i < j) in Montgomery form
struct Garner {
  uint32_t c[kNp][kNp];
};
constexpr Garner ntt_garner() {
  Garner g{};
  for (int j = 0; j < kNp; ++j)
    for (int i = 0; i < j; ++i) g.c[i][j] = ntt_mont(ntt_pow(kQ[i] % kQ[j], kQ[j] - 2, kQ[j]), kQ[j]);
  return g;
}
constexpr Garner kGarner = ntt_garner();

// ---- arithmetic modulo q ------------------------------------------------------------

// a b 2^-32 mod q in [0, 2q) for a < 2^32, b < q
__device__ __forceinline__ uint32_t mmul(uint32_t a, uint32_t b, uint32_t q, uint32_t ni) {
  const uint64_t t = (uint64_t)a * b;
  return (uint32_t)((t + (uint64_t)((uint32_t)t * ni) * q) >> 32);
}
// x < 2m into [0, m): x - m wraps above x when x < m
__device__ __forceinline__ uint32_t red(uint32_t x, uint32_t m) { return min(x, x - m); }

// x < 2^63 modulo q in [0, 4q): xh 2^32 + xl with the two halves weighted by
// 2^64 and 2^32 mod q under one Montgomery reduction (the sum is below 2^62.6)
__device__ __forceinline__ uint32_t ntt_residue(uint64_t x, uint32_t q, uint32_t ni, uint32_t r1, uint32_t r2) {
  const uint64_t t = (uint64_t)(uint32_t)(x >> 32) * r2 + (uint64_t)(uint32_t)x * r1;
  return (uint32_t)((t + (uint64_t)((uint32_t)t * ni) * q) >> 32);
}

// ---- butterflies on E registers --------------------------------------------------------
//
// The transform of x(z) mod z^n - 1 follows the factorisation
// z^(2s) - c^2 = (z^s - c)(z^s + c): at a layer with m blocks, block i splits by
// c = T[i], the same for every element of the block, where T[i] is the root of
// unity at half the van der Corput fraction of i (T[0] = 1, T[1] = sqrt(-1),
// ...), whatever m.  Outputs come in block order, which every product here uses
// as it is.  The inverse runs the same layers backwards with 1/T[i] and leaves
// a factor n, which the stored kernels take out.
//
// L layers on E registers that hold E >> L consecutive blocks, the first of
// them block b0 (tw(u, i) = T[(b0 << u) + i]); FIRST: b0 = 0, T[0] = 1 untouched.
template <int E, int L, bool FIRST, class TW>
__device__ __forceinline__ void ct_layers(uint32_t (&x)[E], uint32_t q, uint32_t ni, const TW& tw) {
  const uint32_t q2 = 2 * q;
#pragma unroll
  for (int u = 0; u < L; ++u) {
    const int span = 1 << (L - 1 - u), blocks = (E >> L) << u;
#pragma unroll
    for (int b = 0; b < blocks; ++b) {
      const bool one = FIRST && b == 0;
      const uint32_t w = one ? 0 : tw(u, b);
#pragma unroll
      for (int j = 0; j < span; ++j) {
        uint32_t& X = x[b * 2 * span + j];
        uint32_t& Y = x[b * 2 * span + j + span];
        const uint32_t a = red(X, q2), y = one ? red(Y, q2) : mmul(Y, w, q, ni);
        X = a + y;
        Y = a - y + q2;
      }
    }
  }
}
template <int E, int L, bool FIRST, class TW>
__device__ __forceinline__ void gs_layers(uint32_t (&x)[E], uint32_t q, uint32_t ni, const TW& tw) {
  const uint32_t q2 = 2 * q;
#pragma unroll
  for (int u = L - 1; u >= 0; --u) {
    const int span = 1 << (L - 1 - u), blocks = (E >> L) << u;
#pragma unroll
    for (int b = 0; b < blocks; ++b) {
      const bool one = FIRST && b == 0;
      const uint32_t w = one ? 0 : tw(u, b);
#pragma unroll
      for (int j = 0; j < span; ++j) {
        uint32_t& X = x[b * 2 * span + j];
        uint32_t& Y = x[b * 2 * span + j + span];
        const uint32_t s = X + Y, d = X - Y + q2;
        X = red(s, q2);
        Y = one ? red(d, q2) : mmul(d, w, q, ni);
      }
    }
  }
}

// ---- transforms of 2^LOGN points by 2^LOGN / 16 threads, 16 points each ------------------
//
// Thread r holds points r + k 2^(LOGN-4) on the natural side and 16 r + k on
// the block-order side; layers run four at a time in registers, with an
// exchange through LDS between.  LDS maps a point to its word (A::at); A::ldl and
// A::stl move the 16 consecutive points of a thread.
// A table of constants.  Passed through an empty asm where a loop would otherwise
// keep every constant of its transforms in registers from one turn to the next.
typedef const __attribute__((address_space(4))) uint32_t* NttTable;
__device__ __forceinline__ NttTable ntt_reload(NttTable t) {
  asm volatile("" : "+s"(t));
  return t;
}

template <int LOGN>
__device__ __forceinline__ uint32_t ntt_idx2(uint32_t r, int k) {
  return ((r >> (LOGN - 8)) << (LOGN - 4)) + (r & ((1u << (LOGN - 8)) - 1)) + ((uint32_t)k << (LOGN - 8));
}

template <int LOGN, class A>
__device__ __forceinline__ void ntt_forward(uint32_t (&x)[16], uint32_t r, const A& lds, NttTable T, uint32_t q,
                                            uint32_t ni) {
  static_assert(LOGN >= 5 && LOGN <= 12, "");
  constexpr int LL = LOGN > 8 ? LOGN - 8 : LOGN - 4;  // layers of the last step
  ct_layers<16, 4, true>(x, q, ni, [&](int, int i) { return T[i]; });
  __syncthreads();  // earlier readers of the exchange area are done
#pragma unroll
  for (int k = 0; k < 16; ++k) lds.at(r + ((uint32_t)k << (LOGN - 4))) = x[k];
  __syncthreads();
  if constexpr (LOGN > 8) {
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = lds.at(ntt_idx2<LOGN>(r, k));
    const uint32_t b0 = r >> (LOGN - 8);
    ct_layers<16, 4, false>(x, q, ni, [&](int u, int i) { return T[(b0 << u) + i]; });
#pragma unroll
    for (int k = 0; k < 16; ++k) lds.at(ntt_idx2<LOGN>(r, k)) = x[k];
    __syncthreads();
  }
  lds.ldl(x, r);
  const uint32_t b0 = r * (16 >> LL);
  ct_layers<16, LL, false>(x, q, ni, [&](int u, int i) { return T[(b0 << u) + i]; });
}

template <int LOGN, class A>
__device__ __forceinline__ void ntt_inverse(uint32_t (&x)[16], uint32_t r, const A& lds, NttTable Ti, uint32_t q,
                                            uint32_t ni) {
  constexpr int LL = LOGN > 8 ? LOGN - 8 : LOGN - 4;
  const uint32_t b0 = r * (16 >> LL);
  gs_layers<16, LL, false>(x, q, ni, [&](int u, int i) { return Ti[(b0 << u) + i]; });
  __syncthreads();
  lds.stl(x, r);
  __syncthreads();
  if constexpr (LOGN > 8) {
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = lds.at(ntt_idx2<LOGN>(r, k));
    const uint32_t b1 = r >> (LOGN - 8);
    gs_layers<16, 4, false>(x, q, ni, [&](int u, int i) { return Ti[(b1 << u) + i]; });
#pragma unroll
    for (int k = 0; k < 16; ++k) lds.at(ntt_idx2<LOGN>(r, k)) = x[k];
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = lds.at(r + ((uint32_t)k << (LOGN - 4)));
  gs_layers<16, 4, true>(x, q, ni, [&](int, int i) { return Ti[i]; });
}

// ---- Chinese remainder ----------------------------------------------------------------

// u_i in [0, 2 q_i) -> the integer they determine, modulo p.  Garner's digits
// d_j < q_j; the value sum_j d_j Qp_j with Qp_j = q_0 .. q_(j-1) mod p is below
// 2^96 and its part above 2^64 below p.
struct CrtP {
  zr_mod M;
  uint64_t Qp[kNp];
};
__device__ __forceinline__ uint64_t ntt_crt(const CrtP& C, const uint32_t (&u)[kNp]) {
  uint32_t d[kNp];
#pragma unroll
  for (int j = 0; j < kNp; ++j) {
    uint32_t v = u[j];
#pragma unroll
    for (int i = 0; i < j; ++i) v = mmul(v - d[i] + 2 * kQ[j], kGarner.c[i][j], kQ[j], kNtt.ni[j]);
    d[j] = red(v, kQ[j]);
  }
  uint64_t lo = d[0], hi = 0;
#pragma unroll
  for (int j = 1; j < kNp; ++j) {
    lo += (uint64_t)d[j] * (uint32_t)C.Qp[j];
    hi += (uint64_t)d[j] * (uint32_t)(C.Qp[j] >> 32);
  }
  const zr_u128 s = (zr_u128)lo + ((zr_u128)hi << 32);
  return zr_mod128(C.M, (uint64_t)(s >> 64), (uint64_t)s);
}

}  // namespace zr

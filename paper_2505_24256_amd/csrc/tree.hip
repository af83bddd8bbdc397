// Transposed Vandermonde solve of a large system by a subproduct tree.
//
// The solve needs s_l = sum_r q_{l,r} v_{r+1} with q_l = M/(z - m_l) for every
// row l, which is W(m_l) for the polynomial part W of M(z) sum_i v_i z^-i: the
// values of a polynomial of degree below t at t points.  With
//   F_u = frac(W/M_u mod z-powers) = sum_{i>=1} f_i z^-i
// for a node u of the subproduct tree (M_u the product of its z - m_l, n its
// size; n coefficients of F_u determine W mod M_u), the root's coefficients are
// the samples themselves, f_i = v_i, and a child's follow from its parent's by
// one product with the sibling's polynomial,
//   f^L_i = sum_{k <= n_R} (M_R)_k f_{i+k},   i = 1..n_L,
// and likewise for the other side (the scaled remainder tree; D. Bernstein,
// "Scaled remainder trees", 2004, and A. Bostan, G. Lecerf, E. Schost, "Tellegen's
// principle into practice", ISSAC 2003).  At a leaf block of B rows, f_1..f_B
// are the samples of a transposed Vandermonde system of those B rows alone with
// master polynomial M_u, whose dot products the quadratic pass then takes: the
// work per row and right-hand side falls from t products to B products and
// log2(t/B) levels of transforms.
//
// Every number is the same integer modulo p as in the quadratic solve, since
// both evaluate the same polynomial identities exactly.
//
// Whole solve, quadratic against tree, one MI355X: t = 9 997, R = 30: 1.07 ->
// 0.56 ms; t = 100 003, R = 17: 49.7 -> 2.27 ms; t = 300 007, R = 40: 781 -> 14.6 ms
// (transforms 11 ms, bound by integer issue and by the residues' traffic; the
// leaves' dot products 1.9 ms).
//
// A node of 2^k rows uses cyclic products of length N = 2^k: sums over i + k <= n
// do not wrap for the coefficients wanted, the upper half of the product of the
// reversed series with the sibling's polynomial.  Transforms of up to 2^12 points run in one
// workgroup's LDS; a longer one is a matrix of N1 rows by 2^12 columns: the
// first log2(N1) layers on columns (the same constants for every column), then
// each row b, twisted by w_N^(rev(b) j) so that it uses the constants of a
// plain transform.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "driver.hpp"
#include "field.hpp"
#include "kernels.hpp"
#include "kernels_dev.hpp"
#include "ntt.hpp"
#include "tree.hpp"

namespace zr {

namespace {

constexpr int kRowLog = 12;                  // longest transform of one workgroup
constexpr uint32_t kRow = 1u << kRowLog;
constexpr uint32_t kLeafLog = 9;             // leaf blocks of 512 rows
constexpr uint32_t kLeaf = 1u << kLeafLog;
static_assert(kLeafLog + 1 >= 10, "the shortest row transform has 2^10 points");

// T[i], 1/T[i], and the powers w^e of the root of order 2^22 in two digits of
// 11 bits (P0: e = 0..2047, P1: e = 2048 i), in Montgomery form.
struct NttTables {
  uint32_t T[kNp][2048], Ti[kNp][2048], P0[kNp][2048], P1[kNp][2048];
};
constexpr NttTables ntt_tables() {
  NttTables t{};
  for (int c = 0; c < kNp; ++c) {
    const uint32_t q = kQ[c], w = ntt_root(q);
    const uint32_t wi = ntt_pow(w, q - 2, q), w11 = ntt_pow(w, 2048, q);
    const uint32_t one = ntt_mont(1, q);
    t.T[c][0] = t.Ti[c][0] = t.P0[c][0] = t.P1[c][0] = one;
    for (int i = 1; i < 2048; ++i) {
      t.P0[c][i] = (uint32_t)((uint64_t)t.P0[c][i - 1] * w % q);
      t.P1[c][i] = (uint32_t)((uint64_t)t.P1[c][i - 1] * w11 % q);
    }
    // T[2^k + j] = T[j] w^(2^22 / 2^(k+2))
    for (int k = 0; k < 11; ++k) {
      const uint32_t r = ntt_pow(w, (uint64_t)1 << (kNttMaxLog - 2 - k), q);
      const uint32_t ri = ntt_pow(wi, (uint64_t)1 << (kNttMaxLog - 2 - k), q);
      for (int j = 0; j < (1 << k); ++j) {
        t.T[c][(1 << k) + j] = (uint32_t)((uint64_t)t.T[c][j] * r % q);
        t.Ti[c][(1 << k) + j] = (uint32_t)((uint64_t)t.Ti[c][j] * ri % q);
      }
    }
  }
  return t;
}
__device__ const NttTables g_tab = ntt_tables();
__device__ __forceinline__ NttTable tab_T(uint32_t c) { return (NttTable)g_tab.T[c]; }
__device__ __forceinline__ NttTable tab_Ti(uint32_t c) { return (NttTable)g_tab.Ti[c]; }

// LDS words of a row transform: 4 spare words per 16 and 16 more per 256, so that
// 16-byte reads at a stride of 16 points, and the two strided patterns, fall on different banks
__host__ __device__ constexpr uint32_t row_pad(uint32_t i) { return i + ((i >> 4) << 2) + ((i >> 8) << 4); }
template <int LOGN>
constexpr uint32_t kRowWords = row_pad(1u << LOGN);

struct RowLds {
  uint32_t* p;
  __device__ __forceinline__ uint32_t& at(uint32_t i) const { return p[row_pad(i)]; }
  __device__ __forceinline__ void ldl(uint32_t (&x)[16], uint32_t r) const {
    const uint4* s = (const uint4*)(p + row_pad(16 * r));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4 v = s[k];
      x[4 * k] = v.x, x[4 * k + 1] = v.y, x[4 * k + 2] = v.z, x[4 * k + 3] = v.w;
    }
  }
  __device__ __forceinline__ void stl(const uint32_t (&x)[16], uint32_t r) const {
    uint4* s = (uint4*)(p + row_pad(16 * r));
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = make_uint4(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
  }
};

template <int C>  // columns of a tile
struct ColLds {
  uint32_t* p;
  uint32_t col;
  __device__ __forceinline__ uint32_t& at(uint32_t i) const { return p[i * C + col]; }
  __device__ __forceinline__ void ldl(uint32_t (&x)[16], uint32_t r) const {
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = p[(16 * r + k) * C + col];
  }
  __device__ __forceinline__ void stl(const uint32_t (&x)[16], uint32_t r) const {
#pragma unroll
    for (int k = 0; k < 16; ++k) p[(16 * r + k) * C + col] = x[k];
  }
};

// Series or polynomials that a level reads: array j at p + j ld, or px for j = jx.
struct Src {
  const uint64_t* p;
  size_t ld;
  const uint64_t* px;
  uint32_t jx;
  __device__ __forceinline__ const uint64_t* at(uint32_t j) const { return j == jx ? px : p + (size_t)j * ld; }
};

// One level of the tree: nodes of N rows, children of h = N/2; nn nodes have
// two children (a last node of at most h rows passes through unchanged).
struct Level {
  uint32_t t, logN, N, h, nn;
  uint32_t R;          // series of the call
  Src f;               // parents' series
  uint64_t* fout;      // children's series [R][t]
  const uint64_t* poly;  // children's polynomials
  uint64_t* pout;      // parents' polynomials
  uint32_t* X;         // column-transformed residues [prime][series or child][node N + s]
  uint32_t* Y;         // products [prime][series][side][...]
  uint32_t* K;         // children's transforms [prime][child][N] times 2^32 / N
  size_t ldX, ldY, ldK;  // words per prime
  // power series of the power sums (one product at a time, nn = 1)
  const uint64_t* root;  // coefficients of M
  uint64_t* g;           // 1/Q, Q the reversed M
  uint64_t* aux;
  uint32_t len;          // terms of a plain source
};

// What a transform reads at point s:
//   kSeries  series j of a node, reversed: f_i at point N - i, zero beyond its n
//   kChild   a child's polynomial: its coefficients and the leading 1
//   kInverse the first len terms of g; kAux the first len terms of aux
//   kRev     Q = rev(M), Q_0 = 1, Q_s = M_(t-s)
//   kDeriv   -Q', coefficients -(s+1) M_(t-1-s), s < t
enum Source { kSeries, kChild, kInverse, kAux, kRev, kDeriv };
template <int SRC>
__device__ __forceinline__ uint64_t source_point(const Level& a, const zr_mod& M, uint32_t j, uint32_t item, uint32_t s) {
  if constexpr (SRC == kSeries) {
    const size_t i = (size_t)item * a.N + (a.N - 1 - s);
    return i < a.t ? a.f.at(j)[i] : 0;
  } else if constexpr (SRC == kChild) {
    const uint32_t n = std::min(a.h, a.t - item * a.h);
    return s < n ? a.poly[(size_t)item * a.h + s] : (s == n ? 1 : 0);
  } else if constexpr (SRC == kInverse) {
    return s < a.len ? a.g[s] : 0;
  } else if constexpr (SRC == kAux) {
    return s < a.len ? a.aux[s] : 0;
  } else if constexpr (SRC == kRev) {
    return s == 0 ? 1 : (s <= a.t ? a.root[a.t - s] : 0);
  } else {
    return s < a.t ? zr_neg(M, zr_mul(M, (s + 1) % M.p, a.root[a.t - 1 - s])) : 0;
  }
}

// Where the product's point s goes:
//   kChildren the upper half is side `side`'s series, point h + ii holding f'_i with i - 1 = h - 1 - ii
//   kParent   the parent's coefficients (the leading term z^n of a full node wraps onto the constant one)
//   kHigh     the upper half into aux; kGrow the lower half, negated, behind the first h terms of g
//   kSums     the first t terms into aux
enum Dest { kChildren, kParent, kHigh, kGrow, kSums };
template <int DST>
__device__ __forceinline__ void store_point(const Level& a, const zr_mod& M, uint32_t j, uint32_t side, uint32_t node,
                                            uint32_t s, uint64_t v) {
  if constexpr (DST == kChildren) {
    const size_t pos = (size_t)node * a.N + side * a.h + (a.N - 1 - s);
    if (pos < a.t) a.fout[(size_t)j * a.t + pos] = v;
  } else if constexpr (DST == kParent) {
    const size_t pos = (size_t)node * a.N + s;
    if (pos >= a.t) return;
    if (s == 0 && a.t - node * a.N >= a.N) v = zr_sub(M, v, 1 % M.p);
    a.pout[pos] = v;
  } else if constexpr (DST == kHigh) {
    a.aux[s - a.h] = v;
  } else if constexpr (DST == kGrow) {
    if (s < a.h) a.g[a.h + s] = zr_neg(M, v);
  } else {
    if (s < a.t) a.aux[s] = v;
  }
}

struct RowK {
  uint32_t q, ni, r1, r2;
};
__device__ __forceinline__ RowK row_mod(const NttMods& m, uint32_t c) { return RowK{m.q[c], m.ni[c], m.r1[c], m.r2[c]}; }

// Twist factors of row b of N1 = N / 2^12 at the thread's points j = r + 256 k:
// w_N^(+-rev(b) j)
template <bool INV>
__device__ __forceinline__ void row_twist(uint32_t (&w)[16], uint32_t logN, uint32_t b, uint32_t r, uint32_t c, const RowK& m) {
  const uint32_t a = logN - kRowLog;
  const uint32_t rev = a ? __brev(b) >> (32 - a) : 0;
  constexpr uint32_t mask = (1u << kNttMaxLog) - 1;
  auto power = [&](uint32_t e) {  // w_N^e or its inverse, Montgomery form
    uint32_t x = (e << (kNttMaxLog - logN)) & mask;
    if (INV) x = (0u - x) & mask;
    return red(mmul(g_tab.P0[c][x & 2047], g_tab.P1[c][x >> 11], m.q, m.ni), m.q);
  };
  w[0] = power(rev * r);
  const uint32_t s1 = power(rev * 256), s2 = power(rev * 512);
  w[1] = red(mmul(w[0], s1, m.q, m.ni), m.q);
#pragma unroll
  for (int k = 2; k < 16; ++k) w[k] = red(mmul(w[k - 2], s2, m.q, m.ni), m.q);
}

// Where point p of a transform's block-ordered output is kept in K: four
// points of each thread side by side, so that lanes read consecutive 16-byte groups
__device__ __forceinline__ void load_k(uint32_t (&x)[16], const uint32_t* k, uint32_t r, uint32_t nt) {
  const uint4* s = (const uint4*)k;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const uint4 v = s[g * nt + r];
    x[4 * g] = v.x, x[4 * g + 1] = v.y, x[4 * g + 2] = v.z, x[4 * g + 3] = v.w;
  }
}

// Transforms of children's polynomials (or of 1/Q): rows of the
// column-transformed residues in X, or (DIRECT, N = 2^LOGN) the polynomials
// themselves.  blockIdx.y = prime.
template <int LOGN, bool DIRECT, int SRC>
__global__ void __launch_bounds__(256) k_tree_kernels(Level a, NttMods mods, uint32_t items) {
  constexpr uint32_t NT = 1u << (LOGN - 4), PER = 256 / NT;
  __shared__ __align__(16) uint32_t sh[PER * kRowWords<LOGN>];
  const uint32_t sub = threadIdx.x / NT, r = threadIdx.x % NT, c = blockIdx.y;
  const uint32_t it0 = blockIdx.x * PER + sub;
  const bool live = it0 < items;
  const uint32_t it = live ? it0 : items - 1;
  const RowK m = row_mod(mods, c);
  const RowLds lds{sh + sub * kRowWords<LOGN>};
  uint32_t x[16];
  if constexpr (DIRECT) {
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = ntt_residue(source_point<SRC>(a, zr_mod{}, 0, it, r + NT * k), m.q, m.ni, m.r1, m.r2);
  } else {
    uint32_t w[16];
    row_twist<false>(w, a.logN, it & ((1u << (a.logN - kRowLog)) - 1), r, c, m);
    const uint32_t* src = a.X + c * a.ldX + (size_t)it * kRow;
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = mmul(src[r + NT * k], w[k], m.q, m.ni);
  }
  ntt_forward<LOGN>(x, r, lds, tab_T(c), m.q, m.ni);
  // times 2^64 / N under one reduction: 2^32 / N
  uint32_t sc = m.r2;
  for (uint32_t i = 0; i < a.logN; ++i) sc = (sc & 1) ? (sc + m.q) >> 1 : sc >> 1;
  uint4* dst = (uint4*)(a.K + c * a.ldK + (size_t)it * (1u << LOGN));
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = red(mmul(x[k], sc, m.q, m.ni), m.q);
  if (live) {
#pragma unroll
    for (int g = 0; g < 4; ++g) dst[g * NT + r] = make_uint4(x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]);
  }
}

// Parents' polynomials: product of the two children's transforms, back along the rows.
template <int LOGN, bool DIRECT>
__global__ void __launch_bounds__(256) k_tree_product(Level a, NttMods mods, uint32_t items) {
  constexpr uint32_t NT = 1u << (LOGN - 4), PER = 256 / NT;
  __shared__ __align__(16) uint32_t sh[PER * kRowWords<LOGN>];
  const uint32_t sub = threadIdx.x / NT, r = threadIdx.x % NT, c = blockIdx.y;
  const uint32_t it0 = blockIdx.x * PER + sub;
  const bool live = it0 < items;
  const uint32_t it = live ? it0 : items - 1;
  const RowK m = row_mod(mods, c);
  const RowLds lds{sh + sub * kRowWords<LOGN>};
  const uint32_t N1 = DIRECT ? 1 : a.N >> kRowLog;
  const uint32_t node = it / N1, b = it % N1;
  uint32_t x[16], y[16];
  const uint32_t* kl = a.K + c * a.ldK + (size_t)(2 * node) * a.N + (size_t)b * (1u << LOGN);
  load_k(x, kl, r, NT);
  load_k(y, kl + a.N, r, NT);
  // both carry 2^32 / N; the product under one reduction carries 2^32 / N^2,
  // and N under a second one leaves 1 / N
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = mmul(mmul(x[k], y[k], m.q, m.ni), a.N, m.q, m.ni);
  ntt_inverse<LOGN>(x, r, lds, tab_Ti(c), m.q, m.ni);
  if constexpr (!DIRECT) {
    uint32_t w[16];
    row_twist<true>(w, a.logN, b, r, c, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = mmul(x[k], w[k], m.q, m.ni);
  }
  if (live) {
    uint32_t* dst = a.Y + c * a.ldY + (size_t)it * (1u << LOGN);
#pragma unroll
    for (int k = 0; k < 16; ++k) dst[r + NT * k] = x[k];
  }
}

// The two products of each node's series, rows: series transform, times the
// sibling's transform, back, for each child.  blockIdx.y = prime, blockIdx.z =
// group of `per` series, which share the registers that hold the two kernels.
template <int LOGN, bool DIRECT>
__global__ void __launch_bounds__(256, 4) k_tree_descend(Level a, NttMods mods, uint32_t items, uint32_t per) {
  constexpr uint32_t NT = 1u << (LOGN - 4), PER = 256 / NT;
  __shared__ __align__(16) uint32_t sh[PER * kRowWords<LOGN>];
  const uint32_t sub = threadIdx.x / NT, r = threadIdx.x % NT, c = blockIdx.y;
  const uint32_t it0 = blockIdx.x * PER + sub;
  const bool live = it0 < items;
  const uint32_t it = live ? it0 : items - 1;
  const RowK m = row_mod(mods, c);
  const RowLds lds{sh + sub * kRowWords<LOGN>};
  const uint32_t N1 = DIRECT ? 1 : a.N >> kRowLog;
  const uint32_t node = it / N1, b = it % N1;
  uint32_t kl[16], kr[16], fw[16], iw[16];
  const uint32_t* kp = a.K + c * a.ldK + (size_t)(2 * node) * a.N + (size_t)b * (1u << LOGN);
  load_k(kl, kp, r, NT);
  load_k(kr, kp + a.N, r, NT);
  if constexpr (!DIRECT) {
    row_twist<false>(fw, a.logN, b, r, c, m);
    row_twist<true>(iw, a.logN, b, r, c, m);
  }
  const uint32_t j1 = std::min(a.R, (blockIdx.z + 1) * per);
  for (uint32_t j = blockIdx.z * per; j < j1; ++j) {
    uint32_t x[16], y[16];
    if constexpr (DIRECT) {
#pragma unroll
      for (int k = 0; k < 16; ++k)
        y[k] = ntt_residue(source_point<kSeries>(a, zr_mod{}, j, node, r + NT * k), m.q, m.ni, m.r1, m.r2);
    } else {
      const uint32_t* src = a.X + c * a.ldX + (size_t)j * a.nn * a.N + (size_t)it * kRow;
#pragma unroll
      for (int k = 0; k < 16; ++k) y[k] = mmul(src[r + NT * k], fw[k], m.q, m.ni);
    }
    ntt_forward<LOGN>(y, r, lds, ntt_reload(tab_T(c)), m.q, m.ni);
#pragma unroll 1
    for (uint32_t side = 0; side < 2; ++side) {
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = mmul(y[k], side ? kl[k] : kr[k], m.q, m.ni);  // the sibling's
      ntt_inverse<LOGN>(x, r, lds, ntt_reload(tab_Ti(c)), m.q, m.ni);
      if constexpr (DIRECT) {
        // only the upper half is wanted
        uint32_t* dst = a.Y + c * a.ldY + ((size_t)(j * 2 + side) * a.nn + node) * a.h;
        if (live) {
#pragma unroll
          for (int k = 8; k < 16; ++k) dst[r + NT * (k - 8)] = x[k];
        }
      } else {
        uint32_t* dst = a.Y + c * a.ldY + (size_t)(j * 2 + side) * a.nn * a.N + (size_t)it * kRow;
        if (live) {
#pragma unroll
          for (int k = 0; k < 16; ++k) dst[r + NT * k] = mmul(x[k], iw[k], m.q, m.ni);
        }
      }
    }
  }
}

// One product: the source's transform times the kernel's, back along the rows.
template <int LOGN, bool DIRECT, int SRC>
__global__ void __launch_bounds__(256) k_tree_conv(Level a, CrtP C, NttMods mods) {
  constexpr uint32_t NT = 1u << (LOGN - 4);
  __shared__ __align__(16) uint32_t sh[256 / NT * kRowWords<LOGN>];
  const uint32_t r = threadIdx.x % NT, c = blockIdx.y, it = blockIdx.x;
  const bool live = threadIdx.x < NT;  // the other threads repeat the work
  const RowK m = row_mod(mods, c);
  const RowLds lds{sh + threadIdx.x / NT * kRowWords<LOGN>};
  uint32_t x[16], w[16];
  if constexpr (DIRECT) {
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = ntt_residue(source_point<SRC>(a, C.M, 0, 0, r + NT * k), m.q, m.ni, m.r1, m.r2);
  } else {
    row_twist<false>(w, a.logN, it, r, c, m);
    const uint32_t* src = a.X + c * a.ldX + (size_t)it * kRow;
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = mmul(src[r + NT * k], w[k], m.q, m.ni);
  }
  ntt_forward<LOGN>(x, r, lds, tab_T(c), m.q, m.ni);
  load_k(w, a.K + c * a.ldK + (size_t)it * (1u << LOGN), r, NT);
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = mmul(x[k], w[k], m.q, m.ni);
  ntt_inverse<LOGN>(x, r, lds, tab_Ti(c), m.q, m.ni);
  if constexpr (!DIRECT) {
    row_twist<true>(w, a.logN, it, r, c, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = mmul(x[k], w[k], m.q, m.ni);
  }
  if (live) {
    uint32_t* dst = a.Y + c * a.ldY + (size_t)it * (1u << LOGN);
#pragma unroll
    for (int k = 0; k < 16; ++k) dst[r + NT * k] = x[k];
  }
}

// The product's values from the five residues, N <= 2^12.  Children: thread =
// (node, upper point), blockIdx.y = side, blockIdx.z = series; else thread =
// (node, point).
template <int DST>
__global__ void __launch_bounds__(256) k_tree_crt(Level a, CrtP C) {
  const uint32_t e = blockIdx.x * 256 + threadIdx.x, side = blockIdx.y, j = blockIdx.z;
  const uint32_t w = DST == kChildren ? a.h : a.N;
  if (e >= a.nn * w) return;
  const uint32_t s = e % w + (DST == kChildren ? a.h : 0);
  if (DST == kHigh && s < a.h) return;
  const uint32_t* src = a.Y + (DST == kChildren ? (size_t)(j * 2 + side) * a.nn * a.h : 0) + e;
  uint32_t u[kNp];
#pragma unroll
  for (int c = 0; c < kNp; ++c) u[c] = src[c * a.ldY];
  store_point<DST>(a, C.M, j, side, e / w, s, ntt_crt(C, u));
}

// ---- column transforms of N1 = 2^A rows -----------------------------------------------
// A <= 4: one thread per column; else tiles of C columns by N1/16 threads each.
template <int A>
struct ColGeom {
  static constexpr uint32_t N1 = 1u << A;
  static constexpr uint32_t TPB = A <= 4 ? 256 : (N1 > 256 ? N1 : 256);
  static constexpr uint32_t C = A <= 4 ? 256 : 16 * TPB / N1;
  static constexpr int E = A <= 4 ? (1 << A) : 16;  // points per thread
  static constexpr uint32_t tiles = kRow / C;
  static constexpr uint32_t words = A <= 4 ? 4 : N1 * C;
  // row of the thread's point k (natural side)
  static __device__ __forceinline__ uint32_t row(uint32_t r, int k) { return A <= 4 ? k : r + ((uint32_t)k << (A > 4 ? A - 4 : 0)); }
  // row of point k on the block-order side
  static __device__ __forceinline__ uint32_t rowb(uint32_t r, int k) { return A <= 4 ? k : 16 * r + k; }
};

// A source's columns into X: blockIdx.x over items (nodes, children, one series) and tiles,
// blockIdx.y = series.
template <int A, int SRC>
__global__ void __launch_bounds__(ColGeom<A>::TPB) k_tree_col_fwd(Level a, zr_mod M) {
  using G = ColGeom<A>;
  __shared__ uint32_t sh[G::words];
  const uint32_t item = blockIdx.x / G::tiles, tile = blockIdx.x % G::tiles, j = blockIdx.y;
  const uint32_t cl = threadIdx.x % G::C, r = threadIdx.x / G::C, col = tile * G::C + cl;
  uint64_t v[G::E];
#pragma unroll
  for (int k = 0; k < G::E; ++k) v[k] = source_point<SRC>(a, M, j, item, G::row(r, k) * kRow + col);
  uint32_t* dst = a.X + ((size_t)j * a.nn + item) * a.N + col;
#pragma unroll 1
  for (int c = 0; c < kNp; ++c) {
    const uint32_t q = kNtt.q[c], ni = kNtt.ni[c];
    uint32_t x[G::E];
#pragma unroll
    for (int k = 0; k < G::E; ++k) x[k] = ntt_residue(v[k], q, ni, kNtt.r1[c], kNtt.r2[c]);
    const NttTable T = tab_T(c);
    if constexpr (A <= 4)
      ct_layers<G::E, A, true>(x, q, ni, [&](int, int i) { return T[i]; });
    else
      ntt_forward<A>(x, r, ColLds<G::C>{sh, cl}, T, q, ni);
#pragma unroll
    for (int k = 0; k < G::E; ++k) dst[c * a.ldX + (size_t)G::rowb(r, k) * kRow] = x[k];
  }
}

// Back along the columns and through the Chinese remainder: children's series
// (blockIdx.y = series, blockIdx.z = side), parents' polynomials, or a power series.
template <int A, int DST>
__global__ void __launch_bounds__(ColGeom<A>::TPB) k_tree_col_inv(Level a, CrtP C) {
  using G = ColGeom<A>;
  __shared__ uint32_t sh[G::words];
  constexpr int K0 = DST == kChildren || DST == kHigh ? G::E / 2 : 0;  // first point wanted
  constexpr int K1 = DST == kGrow ? G::E / 2 : G::E;                    // and one past the last
  const uint32_t node = blockIdx.x / G::tiles, tile = blockIdx.x % G::tiles, j = blockIdx.y, side = blockIdx.z;
  const uint32_t cl = threadIdx.x % G::C, r = threadIdx.x / G::C, col = tile * G::C + cl;
  const uint32_t* src = a.Y + ((size_t)(DST == kChildren ? j * 2 + side : 0) * a.nn + node) * a.N + col;
  uint32_t u[K1 - K0][kNp];
#pragma unroll
  for (int c = 0; c < kNp; ++c) {
    const uint32_t q = kNtt.q[c], ni = kNtt.ni[c];
    uint32_t x[G::E];
#pragma unroll
    for (int k = 0; k < G::E; ++k) x[k] = src[c * a.ldY + (size_t)G::rowb(r, k) * kRow];
    const NttTable T = ntt_reload(tab_Ti(c));
    if constexpr (A <= 4)
      gs_layers<G::E, A, true>(x, q, ni, [&](int, int i) { return T[i]; });
    else
      ntt_inverse<A>(x, r, ColLds<G::C>{sh, cl}, T, q, ni);
#pragma unroll
    for (int k = K0; k < K1; ++k) u[k - K0][c] = x[k];
  }
#pragma unroll
  for (int k = K0; k < K1; ++k)
    store_point<DST>(a, C.M, j, side, node, G::row(r, k) * kRow + col, ntt_crt(C, u[k - K0]));
}

// Newton's first 2^9 terms of 1/Q in one workgroup: g <- g (2 - Q g), doubling,
// with exact sums.  Each product's n sums are split over 512/n threads.
constexpr uint32_t kBase = 512;
__global__ void __launch_bounds__(kBase) k_tree_inverse_base(Level a, zr_mod M) {
  __shared__ uint64_t Q[kBase], g[kBase], e[kBase], part[kBase];
  const uint32_t tid = threadIdx.x;
  Q[tid] = source_point<kRev>(a, M, 0, 0, tid);
  g[tid] = tid == 0 ? 1 % M.p : 0;
  __syncthreads();
  for (uint32_t n = 1; n < kBase; n *= 2) {
    const uint32_t k = tid % n, P = std::min(kBase / n, n), pt = tid / n, len = n / P;
    for (int turn = 0; turn < 2; ++turn) {
      // turn 0: (Q g)_(n+k); turn 1: (e g)_k, the sum over j <= k
      zr_acc192 acc;
      zr_acc_zero(acc);
      if (pt < P)
        for (uint32_t j = pt * len; j < (pt + 1) * len; ++j) {
          if (turn == 0) zr_acc_mac(acc, Q[n + k - j], g[j]);
          else if (j <= k) zr_acc_mac(acc, e[k - j], g[j]);
        }
      part[tid] = zr_acc_reduce(M, acc);
      __syncthreads();
      if (tid < n) {
        uint64_t v = part[k];
        for (uint32_t i = 1; i < P; ++i) v = zr_add(M, v, part[i * n + k]);
        if (turn == 0) e[k] = v;
        else g[n + k] = zr_neg(M, v);
      }
      __syncthreads();
    }
  }
  a.g[tid] = g[tid];
}

// ---- launches of one level ---------------------------------------------------------------

template <int A, int SRC>
void col_fwd(const Level& a, const zr_mod& M, uint32_t items, uint32_t series, hipStream_t s) {
  using G = ColGeom<A>;
  hipLaunchKernelGGL((k_tree_col_fwd<A, SRC>), dim3(items * G::tiles, series), dim3(G::TPB), 0, s, a, M);
}
template <int A, int DST>
void col_inv(const Level& a, const CrtP& C, hipStream_t s) {
  using G = ColGeom<A>;
  hipLaunchKernelGGL((k_tree_col_inv<A, DST>), dim3(a.nn * G::tiles, DST == kChildren ? a.R : 1, DST == kChildren ? 2 : 1),
                     dim3(G::TPB), 0, s, a, C);
}
#define ZR_COL_CASES(F, W, ...)            \
  switch (a.logN - kRowLog) {              \
    case 1: F<1, W>(__VA_ARGS__); break;   \
    case 2: F<2, W>(__VA_ARGS__); break;   \
    case 3: F<3, W>(__VA_ARGS__); break;   \
    case 4: F<4, W>(__VA_ARGS__); break;   \
    case 5: F<5, W>(__VA_ARGS__); break;   \
    case 6: F<6, W>(__VA_ARGS__); break;   \
    case 7: F<7, W>(__VA_ARGS__); break;   \
    case 8: F<8, W>(__VA_ARGS__); break;   \
    case 9: F<9, W>(__VA_ARGS__); break;   \
    case 10: F<10, W>(__VA_ARGS__); break; \
    default: throw Error(ZR_EINVAL);       \
  }

template <int LOGN>
constexpr uint32_t kPer = 256u >> (LOGN - 4);  // transforms per workgroup

// transforms of `items` polynomials into K
template <int SRC>
void level_kernels(const Level& a, const zr_mod& M, uint32_t nc, hipStream_t s) {
  if (a.logN > kRowLog) {
    ZR_COL_CASES(col_fwd, SRC, a, M, nc, 1, s)
    const uint32_t items = nc << (a.logN - kRowLog);
    hipLaunchKernelGGL((k_tree_kernels<kRowLog, false, SRC>), dim3(items, kNp), dim3(256), 0, s, a, kNtt, items);
  } else if (a.logN == 12) {
    hipLaunchKernelGGL((k_tree_kernels<12, true, SRC>), dim3(nc, kNp), dim3(256), 0, s, a, kNtt, nc);
  } else if (a.logN == 11) {
    hipLaunchKernelGGL((k_tree_kernels<11, true, SRC>), dim3(cdiv(nc, kPer<11>), kNp), dim3(256), 0, s, a, kNtt, nc);
  } else {
    hipLaunchKernelGGL((k_tree_kernels<10, true, SRC>), dim3(cdiv(nc, kPer<10>), kNp), dim3(256), 0, s, a, kNtt, nc);
  }
}

template <int DST>
void level_finish(const Level& a, const CrtP& C, hipStream_t s) {
  if (a.logN > kRowLog) {
    ZR_COL_CASES(col_inv, DST, a, C, s)
  } else if (DST == kChildren) {
    hipLaunchKernelGGL((k_tree_crt<DST>), dim3(cdiv((size_t)a.nn * a.h, 256), 2, a.R), dim3(256), 0, s, a, C);
  } else {
    hipLaunchKernelGGL((k_tree_crt<DST>), dim3(cdiv((size_t)a.nn * a.N, 256)), dim3(256), 0, s, a, C);
  }
}

void level_product(const Level& a, const CrtP& C, hipStream_t s) {
  if (a.logN > kRowLog) {
    const uint32_t items = a.nn << (a.logN - kRowLog);
    hipLaunchKernelGGL((k_tree_product<kRowLog, false>), dim3(items, kNp), dim3(256), 0, s, a, kNtt, items);
  } else if (a.logN == 12) {
    hipLaunchKernelGGL((k_tree_product<12, true>), dim3(a.nn, kNp), dim3(256), 0, s, a, kNtt, a.nn);
  } else if (a.logN == 11) {
    hipLaunchKernelGGL((k_tree_product<11, true>), dim3(cdiv(a.nn, kPer<11>), kNp), dim3(256), 0, s, a, kNtt, a.nn);
  } else {
    hipLaunchKernelGGL((k_tree_product<10, true>), dim3(cdiv(a.nn, kPer<10>), kNp), dim3(256), 0, s, a, kNtt, a.nn);
  }
  level_finish<kParent>(a, C, s);
}

// series per workgroup of the descent: as many as leave about 2048 workgroups
uint32_t descend_per(uint32_t blocks, uint32_t R) {
  uint32_t per = 1;
  while (per < 8 && blocks * kNp * cdiv(R, 2 * per) >= 2048) per *= 2;
  return per;
}

void level_descend(const Level& a, const CrtP& C, hipStream_t s) {
  if (a.logN > kRowLog) {
    ZR_COL_CASES(col_fwd, kSeries, a, C.M, a.nn, a.R, s)
    const uint32_t items = a.nn << (a.logN - kRowLog), per = descend_per(items, a.R);
    hipLaunchKernelGGL((k_tree_descend<kRowLog, false>), dim3(items, kNp, cdiv(a.R, per)), dim3(256), 0, s, a, kNtt, items,
                       per);
  } else {
    const uint32_t g = a.logN == 12 ? a.nn : a.logN == 11 ? cdiv(a.nn, kPer<11>) : cdiv(a.nn, kPer<10>);
    const uint32_t per = descend_per(g, a.R);
    const dim3 grid(g, kNp, cdiv(a.R, per));
    if (a.logN == 12) hipLaunchKernelGGL((k_tree_descend<12, true>), grid, dim3(256), 0, s, a, kNtt, a.nn, per);
    else if (a.logN == 11) hipLaunchKernelGGL((k_tree_descend<11, true>), grid, dim3(256), 0, s, a, kNtt, a.nn, per);
    else hipLaunchKernelGGL((k_tree_descend<10, true>), grid, dim3(256), 0, s, a, kNtt, a.nn, per);
  }
  level_finish<kChildren>(a, C, s);
}

// a.aux/a.g <- (source SRC) times the kernel in K
template <int SRC, int DST>
void series_product(const Level& a, const CrtP& C, hipStream_t s) {
  if (a.logN > kRowLog) {
    ZR_COL_CASES(col_fwd, SRC, a, C.M, 1, 1, s)
    hipLaunchKernelGGL((k_tree_conv<kRowLog, false, SRC>), dim3(1u << (a.logN - kRowLog), kNp), dim3(256), 0, s, a, C, kNtt);
  } else if (a.logN == 12) {
    hipLaunchKernelGGL((k_tree_conv<12, true, SRC>), dim3(1, kNp), dim3(256), 0, s, a, C, kNtt);
  } else if (a.logN == 11) {
    hipLaunchKernelGGL((k_tree_conv<11, true, SRC>), dim3(1, kNp), dim3(256), 0, s, a, C, kNtt);
  } else {
    hipLaunchKernelGGL((k_tree_conv<10, true, SRC>), dim3(1, kNp), dim3(256), 0, s, a, C, kNtt);
  }
  level_finish<DST>(a, C, s);
}

// Power sums p_1..p_t of the rows' monomial values into sums, from M alone:
// sum_i p_i x^(i-1) = -Q'(x)/Q(x), Q the reversed M (Newton's identities), with
// 1/Q by Newton's iteration.  They are the samples of the right-hand side whose
// solution is 1 in every row, so that side's value at row l is m_l M'(m_l), the
// denominator of every other side.
void power_sums(uint32_t t, const uint64_t* root, uint64_t* sums, uint32_t* X, size_t ldX, uint32_t* Y, size_t ldY,
                uint32_t* K, size_t ldK, uint64_t* g, const CrtP& C, hipStream_t s) {
  Level a{};
  a.t = t;
  a.nn = 1;
  a.R = 1;
  a.X = X;
  a.Y = Y;
  a.K = K;
  a.ldX = ldX;
  a.ldY = ldY;
  a.ldK = ldK;
  a.root = root;
  a.g = g;
  a.aux = sums;
  hipLaunchKernelGGL(k_tree_inverse_base, dim3(1), dim3(kBase), 0, s, a, C.M);
  uint32_t lg = 9;
  for (; (1u << lg) < t; ++lg) {
    a.logN = lg + 1;
    a.N = 1u << a.logN;
    a.h = a.len = 1u << lg;
    level_kernels<kInverse>(a, C.M, 1, s);
    series_product<kRev, kHigh>(a, C, s);
    series_product<kAux, kGrow>(a, C, s);
  }
  a.logN = lg + 1;
  a.N = 1u << a.logN;
  a.h = a.N / 2;
  a.len = t;
  level_kernels<kInverse>(a, C.M, 1, s);
  series_product<kDeriv, kSums>(a, C, s);
}

// Unknowns from which the denominators come from the power sums, one more
// right-hand side, instead of t^2 steps of the chain pass.
constexpr uint32_t kSumsMinT = 32768;

}  // namespace

// The tree pays from about 10^4 unknowns whatever R, and below that where the
// right-hand sides are many enough for its launches (about 40 of 4 to 10 us).
// Quadratic against tree, microseconds: t = 4500: R = 30 397/415, R = 40 465/432; t = 5500: R = 10 383/407,
// R = 30 497/430; t = 9000: R = 1 435/459, R = 10 665/476; t = 13 000: R = 1
// 629/510, R = 30 1580/617.  Up to 2^21 unknowns: the power sums' last
// transform then has 2^22 points, the primes' limit.
bool tree_applies(uint32_t t, uint32_t R) {
  if (!vsolve_uses_pc() || R == 0 || t > (1u << (kNttMaxLog - 1))) return false;
  return t >= 10000 || (t > 4096 && (uint64_t)t * (R + 10) >= 210000);
}

void tree_solve(const zr_mod& M, uint32_t t, uint32_t R, const uint64_t* mono, const uint64_t* rhs, size_t ld_rhs,
                uint64_t* out, size_t ld_out, int32_t* status, DevArena& A, hipStream_t s) {
  uint32_t logTop = kLeafLog;
  while ((1u << logTop) < t) ++logTop;
  const uint32_t top = 1u << logTop;
  CrtP C;
  C.M = M;
  uint64_t prod = 1 % M.p;
  for (int j = 0; j < kNp; ++j) {
    C.Qp[j] = prod;
    prod = zr_mul(M, prod, kQ[j] % M.p);
  }
  const bool sums = t >= kSumsMinT;
  const uint32_t R1 = R + (sums ? 1 : 0);  // series; the power sums are series 0
  // leaf polynomials by the quadratic product tree, then level by level up:
  // the children's transforms (kept for the way down) and the parents' polynomials
  uint64_t* leafM = A.alloc<uint64_t>(t);
  uint64_t* tmp = A.alloc<uint64_t>(master_tmp_words(t));
  check(master_levels(M, t, kLeaf, mono, leafM, tmp, s));
  uint64_t* poly = A.alloc<uint64_t>(t);
  check(copy_u64(poly, leafM, t, s));
  std::vector<Level> lv;
  for (uint32_t k = kLeafLog + 1; k <= logTop; ++k) {
    Level a{};
    a.t = t;
    a.logN = k;
    a.N = 1u << k;
    a.h = a.N / 2;
    a.nn = t / a.N + (t % a.N > a.h ? 1 : 0);
    a.ldK = (size_t)2 * a.nn * a.N;
    a.K = A.alloc<uint32_t>(a.ldK * kNp);
    a.poly = poly;
    a.pout = poly;
    lv.push_back(a);
  }
  // residue workspace: groups of series small enough for the last-level cache
  const size_t per_series = (size_t)kNp * 4 * 3 * top;
  uint32_t group = (uint32_t)std::max<size_t>(1, std::min<size_t>(R1, (size_t)(160u << 20) / per_series));
  group = cdiv(R1, cdiv(R1, group));
  const size_t ldX = (size_t)std::max(2u, group) * top, ldY = (size_t)2 * group * top;
  uint32_t* X = A.alloc<uint32_t>(ldX * kNp);
  uint32_t* Y = A.alloc<uint32_t>(ldY * kNp);
  {
    TimedLaunch tl("tree_up", s);
    for (Level& a : lv) {
      a.X = X;
      a.Y = Y;
      a.ldX = ldX;
      a.ldY = ldY;
      level_kernels<kChild>(a, M, 2 * a.nn, s);
      level_product(a, C, s);
    }
  }
  uint64_t* F = A.alloc<uint64_t>((size_t)R1 * t);
  uint64_t* ps = nullptr;
  if (sums) {
    TimedLaunch tl("tree_sums", s);
    ps = A.alloc<uint64_t>(top);
    uint64_t* g = A.alloc<uint64_t>(top);
    uint32_t* K = A.alloc<uint32_t>((size_t)2 * top * kNp);
    power_sums(t, poly, ps, X, ldX, Y, ldY, K, (size_t)2 * top, g, C, s);
  }
  // down: the samples are the root's series
  {
    TimedLaunch tl("tree_down", s);
    const Src in = sums ? Src{rhs - ld_rhs, ld_rhs, ps, 0} : Src{rhs, ld_rhs, nullptr, ~0u};
    for (uint32_t j0 = 0; j0 < R1; j0 += group)
      for (size_t i = lv.size(); i-- > 0;) {
        Level a = lv[i];
        a.R = std::min(group, R1 - j0);
        a.fout = F + (size_t)j0 * t;
        a.f = i + 1 == lv.size() ? Src{in.p + (size_t)j0 * ld_rhs, ld_rhs, in.px, j0 == 0 ? in.jx : ~0u}
                                 : Src{F + (size_t)j0 * t, t, nullptr, ~0u};
        level_descend(a, C, s);
      }
  }
  check(hipGetLastError());
  uint64_t* work = A.alloc<uint64_t>(vsolve_leaf_words(t, R1, sums));
  check(vsolve_leaf(M, t, R1, sums, kLeaf, mono, leafM, poly, F, out, ld_out, work, status, s));
}

}  // namespace zr

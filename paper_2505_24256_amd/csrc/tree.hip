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
// 0.39 ms; t = 100 003, R = 17: 49.6 -> 1.66 ms; t = 300 007, R = 40: 781 -> 8.7 ms
// (rows of nodes above 4096 points 2.5 ms, bound by integer issue; rows of smaller nodes
// 1.3 ms, columns 2.3 and Chinese remainder 0.3 ms, near the copy rate by the residues'
// traffic; the leaves' dot products 1.1 ms).  256 uneven systems of 10 to 20 000
// unknowns, R = 30, the large ones through one tree: 52.0 -> 9.0 ms.
//
// A node of 2^k rows uses cyclic products of length N = 2^k: sums over i + k <= n
// do not wrap for the coefficients wanted, the upper half of the product of the
// reversed series with the sibling's polynomial.  Transforms of up to 2^12 points run in one
// workgroup's LDS; a longer one is a matrix of N1 rows by 2^12 columns: the
// first log2(N1) layers on columns (the same constants for every column), then
// each row b, twisted by w_N^(rev(b) j) at the column pass so that it uses the constants
// of a plain transform.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "batch.hpp"
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
constexpr uint32_t kLeafLog = kTreeLeafLog;
constexpr uint32_t kLeaf = kTreeLeaf;
constexpr int kRowMin = 9;  // shortest transform of the rows: half a wave
static_assert(kLeafLog + 1 >= kRowMin, "");

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

// One level of the tree: nodes of N rows, children of h = N/2.  Rows of all
// systems stand in one index space, each system at a multiple of its own top
// node's size (TreeSys::off), largest tops first, so nodes of N rows are the
// aligned ranges of a prefix of it.  A node of at most h rows passes through
// unchanged; one without rows is skipped.
struct Level {
  uint32_t logN, N, h, nn;
  uint32_t R;          // series of the call
  uint32_t j0;         // the first of them
  TreeSys one;         // the only system (sys null), or
  const TreeSys* sys;  // the systems, and the system of each leaf block
  const uint32_t* sys_of;
  uint64_t* sums;        // power sums, series 0 at every level (null: none)
  const uint64_t* poly;  // children's polynomials
  uint64_t* pout;      // parents' polynomials
  uint32_t* X;         // column-transformed residues [prime][series or child][node N + s]
  uint32_t* Y;         // products [prime][series][side][...]
  uint32_t* K;         // children's transforms [prime][child][N] times 2^32 / N
  size_t ldX, ldY, ldK;  // words per prime
  const uint32_t* tw;  // twist factors, 2^twLog words per direction and prime
  uint32_t twLog;
  // power series of the power sums: one product per system, systems item0..
  uint32_t item0;
  uint64_t* g;    // 1/Q, Q the reversed M
  uint64_t* aux;
  uint32_t full;  // kInverse: all t terms (else the first h)
};

template <uint32_t NT>  // threads of a transform: at least a wave, or half of one
__device__ __forceinline__ uint32_t wave_uniform(uint32_t x) {
  return NT >= 64 ? __builtin_amdgcn_readfirstlane(x) : x;
}
// the row's system is the same for all lanes of a wave (two nodes of 512 rows that
// share one lie in one node of 1024)
__device__ __forceinline__ TreeSys sys_at(const Level& a, uint32_t row) {
  return a.sys ? a.sys[a.sys_of[__builtin_amdgcn_readfirstlane(row) >> kLeafLog]] : a.one;
}
__device__ __forceinline__ TreeSys sys_item(const Level& a, uint32_t item) {
  return a.sys ? a.sys[__builtin_amdgcn_readfirstlane(a.item0 + item)] : a.one;
}
__device__ __forceinline__ bool splits(const Level& a, const TreeSys& y, uint32_t node) {
  return y.end > node * a.N + a.h;
}

// What a transform reads at point s:
//   kSeries  series j of a node, reversed: f_i at point N - i, zero beyond its n;
//            the top node's are the samples (series 0 the power sums, where they are made)
//   kChild   a child's polynomial: its coefficients and the leading 1
//   kInverse the first h (or t) terms of g; kAux the first h terms of aux
//   kRev     Q = rev(M), Q_0 = 1, Q_s = M_(t-s)
//   kDeriv   -Q', coefficients -(s+1) M_(t-1-s), s < t
enum Source { kSeries, kChild, kInverse, kAux, kRev, kDeriv };
template <int SRC>
__device__ __forceinline__ uint64_t source_point(const Level& a, const TreeSys& y, const zr_mod& M, uint32_t j,
                                                 uint32_t item, uint32_t s) {
  const uint32_t t = y.end - y.off;
  if constexpr (SRC == kSeries) {
    const uint32_t row = item * a.N + (a.N - 1 - s);
    const uint32_t jj = a.j0 + j;
    const uint64_t* f = a.logN == y.logTop ? y.rhs + (size_t)jj * y.ld_rhs : y.f + (size_t)jj * y.ld;
    if (a.sums && jj == 0) f = a.sums + y.off;
    return row < y.end ? f[row - y.off] : 0;
  } else if constexpr (SRC == kChild) {
    const uint32_t row = item * a.h, n = row < y.end ? std::min(a.h, y.end - row) : 0;
    return s < n ? a.poly[row + s] : (s == n ? 1 : 0);
  } else if constexpr (SRC == kInverse) {
    return s < (a.full ? t : a.h) ? a.g[y.off + s] : 0;
  } else if constexpr (SRC == kAux) {
    return s < a.h ? a.aux[y.off + s] : 0;
  } else if constexpr (SRC == kRev) {
    return s == 0 ? 1 : (s <= t ? a.poly[y.end - s] : 0);
  } else {
    return s < t ? zr_neg(M, zr_mul(M, (s + 1) % M.p, a.poly[y.end - 1 - s])) : 0;
  }
}
// the system an item of a source belongs to
template <int SRC>
__device__ __forceinline__ TreeSys source_sys(const Level& a, uint32_t item) {
  return SRC == kSeries ? sys_at(a, item * a.N) : SRC == kChild ? sys_at(a, item * a.h) : sys_item(a, item);
}

// Where the product's point s goes:
//   kChildren the upper half is side `side`'s series, point h + ii holding f'_i with i - 1 = h - 1 - ii
//   kParent   the parent's coefficients (the leading term z^n of a full node wraps onto the constant one)
//   kHigh     the upper half into aux; kGrow the lower half, negated, behind the first h terms of g
//   kSums     the first t terms into aux
enum Dest { kChildren, kParent, kHigh, kGrow, kSums };
template <int DST>
__device__ __forceinline__ void store_point(const Level& a, const TreeSys& y, const zr_mod& M, uint32_t j, uint32_t side,
                                            uint32_t node, uint32_t s, uint64_t v) {
  if constexpr (DST == kChildren) {
    const uint32_t row = node * a.N + side * a.h + (a.N - 1 - s);
    const uint32_t jj = a.j0 + j;
    uint64_t* f = a.sums && jj == 0 ? a.sums + y.off : y.f + (size_t)jj * y.ld;
    if (row < y.end) f[row - y.off] = v;
  } else if constexpr (DST == kParent) {
    const uint32_t row = node * a.N + s;
    if (row >= y.end) return;
    if (s == 0 && y.end - node * a.N >= a.N) v = zr_sub(M, v, 1 % M.p);
    a.pout[row] = v;
  } else if constexpr (DST == kHigh) {
    a.aux[y.off + s - a.h] = v;
  } else if constexpr (DST == kGrow) {
    if (s < a.h) a.g[y.off + a.h + s] = zr_neg(M, v);
  } else {
    if (s < y.end - y.off) a.aux[y.off + s] = v;
  }
}
template <int DST>
__device__ __forceinline__ TreeSys dest_sys(const Level& a, uint32_t node, bool& live) {
  const TreeSys y = DST == kChildren || DST == kParent ? sys_at(a, node * a.N) : sys_item(a, node);
  live = DST == kChildren || DST == kParent ? splits(a, y, node) : true;
  return y;
}

struct RowK {
  uint32_t q, ni, r1, r2;
};
__device__ __forceinline__ RowK row_mod(const NttMods& m, uint32_t c) { return RowK{m.q[c], m.ni[c], m.r1[c], m.r2[c]}; }

// Twist factors of the column transforms, w_N^(rev(b) j) at row b, column j, and
// their inverses, as [dir][prime][row 2^12 + column].  rev counts the bits of b
// below N/2^12; one table serves every N, since halving N halves rev(b) and squares w_N.
__global__ void __launch_bounds__(256) k_tree_twist(uint32_t* __restrict__ tw, uint32_t logN, NttMods mods) {
  const uint32_t e = blockIdx.x * 256 + threadIdx.x, c = blockIdx.y, inv = blockIdx.z, a = logN - kRowLog;
  const RowK m = row_mod(mods, c);
  constexpr uint32_t mask = (1u << kNttMaxLog) - 1;
  uint32_t x = ((__brev(e >> kRowLog) >> (32 - a)) * (e & (kRow - 1)) << (kNttMaxLog - logN)) & mask;
  if (inv) x = (0u - x) & mask;
  tw[((size_t)(inv * kNp + c) << logN) + e] = red(mmul(g_tab.P0[c][x & 2047], g_tab.P1[c][x >> 11], m.q, m.ni), m.q);
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
  const uint32_t sub = wave_uniform<NT>(threadIdx.x / NT), r = threadIdx.x % NT, c = blockIdx.y;
  const uint32_t it0 = blockIdx.x * PER + sub;
  const bool live = it0 < items;
  const uint32_t it = live ? it0 : items - 1;
  const RowK m = row_mod(mods, c);
  const RowLds lds{sh + sub * kRowWords<LOGN>};
  uint32_t x[16];
  if constexpr (DIRECT) {
    const TreeSys y = source_sys<SRC>(a, it);
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = ntt_residue(source_point<SRC>(a, y, zr_mod{}, 0, it, r + NT * k), m.q, m.ni, m.r1, m.r2);
  } else {
    const uint32_t* src = a.X + c * a.ldX + (size_t)it * kRow;
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = src[r + NT * k];
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
  const uint32_t sub = wave_uniform<NT>(threadIdx.x / NT), r = threadIdx.x % NT, c = blockIdx.y;
  const uint32_t it0 = blockIdx.x * PER + sub;
  const bool live = it0 < items;
  const uint32_t it = live ? it0 : items - 1;
  const RowK m = row_mod(mods, c);
  const RowLds lds{sh + sub * kRowWords<LOGN>};
  const uint32_t lg1 = DIRECT ? 0 : a.logN - kRowLog;
  const uint32_t node = it >> lg1, b = it & ((1u << lg1) - 1);
  uint32_t x[16], y[16];
  const uint32_t* kl = a.K + c * a.ldK + (size_t)(2 * node) * a.N + (size_t)b * (1u << LOGN);
  load_k(x, kl, r, NT);
  load_k(y, kl + a.N, r, NT);
  // both carry 2^32 / N; the product under one reduction carries 2^32 / N^2,
  // and N under a second one leaves 1 / N
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = mmul(mmul(x[k], y[k], m.q, m.ni), a.N, m.q, m.ni);
  ntt_inverse<LOGN>(x, r, lds, tab_Ti(c), m.q, m.ni);
  if (live) {
    uint32_t* dst = a.Y + c * a.ldY + (size_t)it * (1u << LOGN);
#pragma unroll
    for (int k = 0; k < 16; ++k) dst[r + NT * k] = x[k];
  }
}

// The two products of each node's series, rows: series transform, times the
// sibling's transform, back, for each child.  About 160 vector instructions per point
// (three transforms of 12 layers at 8 a butterfly); with the twist factors taken
// out of this pass and the kernels read where they are used it holds 98 VGPRs without
// spills: 90 -> 42 us for 5 series of 3*10^5 rows, about 35 at full issue.  blockIdx.y =
// prime, blockIdx.z = group of `per` series.
template <int LOGN, bool DIRECT>
__global__ void __launch_bounds__(256, 3) k_tree_descend(Level a, NttMods mods, uint32_t items, uint32_t per) {
  constexpr uint32_t NT = 1u << (LOGN - 4), PER = 256 / NT;
  __shared__ __align__(16) uint32_t sh[PER * kRowWords<LOGN>];
  const uint32_t sub = wave_uniform<NT>(threadIdx.x / NT), r = threadIdx.x % NT, c = blockIdx.y;
  const uint32_t it0 = blockIdx.x * PER + sub;
  const uint32_t it = std::min(it0, items - 1);
  const RowK m = row_mod(mods, c);
  const RowLds lds{sh + sub * kRowWords<LOGN>};
  const uint32_t lg1 = DIRECT ? 0 : a.logN - kRowLog;
  const uint32_t node = it >> lg1, b = it & ((1u << lg1) - 1);
  const TreeSys sy = sys_at(a, node * a.N);
  const bool live = it0 < items && splits(a, sy, node);
  if (PER == 1 && !live) return;
  const uint32_t* kp = a.K + c * a.ldK + (size_t)(2 * node) * a.N + (size_t)b * (1u << LOGN);
  const uint32_t j1 = std::min(a.R, (blockIdx.z + 1) * per);
#pragma unroll 1
  for (uint32_t j = blockIdx.z * per; j < j1; ++j) {
    uint32_t y[16];
    if constexpr (DIRECT) {
#pragma unroll
      for (int k = 0; k < 16; ++k)
        y[k] = ntt_residue(source_point<kSeries>(a, sy, zr_mod{}, j, node, r + NT * k), m.q, m.ni, m.r1, m.r2);
    } else {
      const uint32_t* src = a.X + c * a.ldX + (size_t)j * a.nn * a.N + (size_t)it * kRow;
#pragma unroll
      for (int k = 0; k < 16; ++k) y[k] = src[r + NT * k];
    }
    ntt_forward<LOGN>(y, r, lds, ntt_reload(tab_T(c)), m.q, m.ni);
#pragma unroll 1
    for (uint32_t side = 0; side < 2; ++side) {
      uint32_t x[16];
      load_k(x, kp + (side ? 0 : a.N), r, NT);  // the sibling's
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = mmul(y[k], x[k], m.q, m.ni);
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
          for (int k = 0; k < 16; ++k) dst[r + NT * k] = x[k];
        }
      }
    }
  }
}

// One product per item: the source's transform times the kernel's, back along the rows.
template <int LOGN, bool DIRECT, int SRC>
__global__ void __launch_bounds__(256) k_tree_conv(Level a, CrtP C, NttMods mods, uint32_t items) {
  constexpr uint32_t NT = 1u << (LOGN - 4), PER = 256 / NT;
  __shared__ __align__(16) uint32_t sh[PER * kRowWords<LOGN>];
  const uint32_t sub = wave_uniform<NT>(threadIdx.x / NT), r = threadIdx.x % NT, c = blockIdx.y;
  const uint32_t it0 = blockIdx.x * PER + sub;
  const bool live = it0 < items;
  const uint32_t it = live ? it0 : items - 1;
  const RowK m = row_mod(mods, c);
  const RowLds lds{sh + sub * kRowWords<LOGN>};
  uint32_t x[16], w[16];
  if constexpr (DIRECT) {
    const TreeSys y = sys_item(a, it);
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = ntt_residue(source_point<SRC>(a, y, C.M, 0, it, r + NT * k), m.q, m.ni, m.r1, m.r2);
  } else {
    const uint32_t* src = a.X + c * a.ldX + (size_t)it * kRow;
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = src[r + NT * k];
  }
  ntt_forward<LOGN>(x, r, lds, tab_T(c), m.q, m.ni);
  load_k(w, a.K + c * a.ldK + (size_t)it * (1u << LOGN), r, NT);
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = mmul(x[k], w[k], m.q, m.ni);
  ntt_inverse<LOGN>(x, r, lds, tab_Ti(c), m.q, m.ni);
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
  if ((DST == kHigh && s < a.h) || (DST == kGrow && s >= a.h)) return;
  bool live;
  const TreeSys y = dest_sys<DST>(a, e / w, live);
  if (!live) return;
  const uint32_t* src = a.Y + (DST == kChildren ? (size_t)(j * 2 + side) * a.nn * a.h : 0) + e;
  uint32_t u[kNp];
#pragma unroll
  for (int c = 0; c < kNp; ++c) u[c] = src[c * a.ldY];
  store_point<DST>(a, y, C.M, j, side, e / w, s, ntt_crt(C, u));
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
// blockIdx.y = series, blockIdx.z = prime.
template <int A, int SRC>
__global__ void __launch_bounds__(ColGeom<A>::TPB) k_tree_col_fwd(Level a, zr_mod M, NttMods mods) {
  using G = ColGeom<A>;
  __shared__ uint32_t sh[G::words];
  const uint32_t item = blockIdx.x / G::tiles, tile = blockIdx.x % G::tiles, j = blockIdx.y, c = blockIdx.z;
  const uint32_t cl = threadIdx.x % G::C, r = threadIdx.x / G::C, col = tile * G::C + cl;
  const TreeSys y = source_sys<SRC>(a, item);
  if (SRC == kSeries && !splits(a, y, item)) return;
  const RowK m = row_mod(mods, c);
  uint32_t x[G::E], w[G::E];
#pragma unroll
  for (int k = 0; k < G::E; ++k)
    x[k] = ntt_residue(source_point<SRC>(a, y, M, j, item, G::row(r, k) * kRow + col), m.q, m.ni, m.r1, m.r2);
#pragma unroll
  for (int k = 0; k < G::E; ++k) w[k] = a.tw[((size_t)c << a.twLog) + G::rowb(r, k) * kRow + col];
  const NttTable T = tab_T(c);
  if constexpr (A <= 4)
    ct_layers<G::E, A, true>(x, m.q, m.ni, [&](int, int i) { return T[i]; });
  else
    ntt_forward<A>(x, r, ColLds<G::C>{sh, cl}, T, m.q, m.ni);
  uint32_t* dst = a.X + c * a.ldX + ((size_t)j * a.nn + item) * a.N + col;
#pragma unroll
  for (int k = 0; k < G::E; ++k) dst[(size_t)G::rowb(r, k) * kRow] = mmul(x[k], w[k], m.q, m.ni);
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
  bool live;
  const TreeSys y = dest_sys<DST>(a, node, live);
  if (!live) return;
  const uint32_t* src = a.Y + ((size_t)(DST == kChildren ? j * 2 + side : 0) * a.nn + node) * a.N + col;
  uint32_t u[K1 - K0][kNp];
#pragma unroll
  for (int c = 0; c < kNp; ++c) {
    const uint32_t q = kNtt.q[c], ni = kNtt.ni[c];
    uint32_t x[G::E];
#pragma unroll
    for (int k = 0; k < G::E; ++k) {
      const size_t e = (size_t)G::rowb(r, k) * kRow;
      x[k] = mmul(src[c * a.ldY + e], a.tw[((size_t)(kNp + c) << a.twLog) + e + col], q, ni);
    }
    const NttTable T = ntt_reload(tab_Ti(c));
    if constexpr (A <= 4)
      gs_layers<G::E, A, true>(x, q, ni, [&](int, int i) { return T[i]; });
    else
      ntt_inverse<A>(x, r, ColLds<G::C>{sh, cl}, T, q, ni);
#pragma unroll
    for (int k = K0; k < K1; ++k) u[k - K0][c] = x[k];
    // one prime's points live at a time: without the fence the loads of all five come first
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int k = K0; k < K1; ++k)
    store_point<DST>(a, y, C.M, j, side, node, G::row(r, k) * kRow + col, ntt_crt(C, u[k - K0]));
}

// Newton's first 2^9 terms of 1/Q in one workgroup: g <- g (2 - Q g), doubling,
// with exact sums.  Each product's n sums are split over 512/n threads.
constexpr uint32_t kBase = 512;
__global__ void __launch_bounds__(kBase) k_tree_inverse_base(Level a, zr_mod M) {
  __shared__ uint64_t Q[kBase], g[kBase], e[kBase], part[kBase];
  const uint32_t tid = threadIdx.x;
  const TreeSys y = sys_item(a, blockIdx.x);
  Q[tid] = source_point<kRev>(a, y, M, 0, 0, tid);
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
  a.g[y.off + tid] = g[tid];
}

// ---- launches of one level ---------------------------------------------------------------

template <int A, int SRC>
void col_fwd(const Level& a, const zr_mod& M, uint32_t items, uint32_t series, hipStream_t s) {
  using G = ColGeom<A>;
  hipLaunchKernelGGL((k_tree_col_fwd<A, SRC>), dim3(items * G::tiles, series, kNp), dim3(G::TPB), 0, s, a, M, kNtt);
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

// f(length) with the transform's log2 length as a constant
template <class F>
void for_row_log(uint32_t logN, const F& f) {
  switch (logN) {
    case 9: f(std::integral_constant<int, 9>()); break;
    case 10: f(std::integral_constant<int, 10>()); break;
    case 11: f(std::integral_constant<int, 11>()); break;
    case 12: f(std::integral_constant<int, 12>()); break;
    default: throw Error(ZR_EINVAL);
  }
}

// transforms of `items` polynomials into K
template <int SRC>
void level_kernels(const Level& a, const zr_mod& M, uint32_t nc, hipStream_t s) {
  if (a.logN > kRowLog) {
    ZR_COL_CASES(col_fwd, SRC, a, M, nc, 1, s)
    const uint32_t items = nc << (a.logN - kRowLog);
    hipLaunchKernelGGL((k_tree_kernels<kRowLog, false, SRC>), dim3(items, kNp), dim3(256), 0, s, a, kNtt, items);
  } else {
    for_row_log(a.logN, [&](auto L) {
      hipLaunchKernelGGL((k_tree_kernels<L, true, SRC>), dim3(cdiv(nc, kPer<L>), kNp), dim3(256), 0, s, a, kNtt, nc);
    });
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
  } else {
    for_row_log(a.logN, [&](auto L) {
      hipLaunchKernelGGL((k_tree_product<L, true>), dim3(cdiv(a.nn, kPer<L>), kNp), dim3(256), 0, s, a, kNtt, a.nn);
    });
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
    for_row_log(a.logN, [&](auto L) {
      const uint32_t g = cdiv(a.nn, kPer<L>), per = descend_per(g, a.R);
      hipLaunchKernelGGL((k_tree_descend<L, true>), dim3(g, kNp, cdiv(a.R, per)), dim3(256), 0, s, a, kNtt, a.nn, per);
    });
  }
  level_finish<kChildren>(a, C, s);
}

// a.aux or a.g of each of nn systems from item0 <- (source SRC) times the kernel in K
template <int SRC, int DST>
void series_product(const Level& a, const CrtP& C, hipStream_t s) {
  if (a.logN > kRowLog) {
    ZR_COL_CASES(col_fwd, SRC, a, C.M, a.nn, 1, s)
    const uint32_t items = a.nn << (a.logN - kRowLog);
    hipLaunchKernelGGL((k_tree_conv<kRowLog, false, SRC>), dim3(items, kNp), dim3(256), 0, s, a, C, kNtt, items);
  } else {
    for_row_log(a.logN, [&](auto L) {
      hipLaunchKernelGGL((k_tree_conv<L, true, SRC>), dim3(cdiv(a.nn, kPer<L>), kNp), dim3(256), 0, s, a, C, kNtt, a.nn);
    });
  }
  level_finish<DST>(a, C, s);
}

// Power sums p_1..p_t of each system's monomial values, from its M alone:
// sum_i p_i x^(i-1) = -Q'(x)/Q(x), Q the reversed M (Newton's identities), with
// 1/Q by Newton's iteration, all systems a step at a time.  They are the samples
// of the right-hand side whose solution is 1 in every row, so that side's value
// at row l is m_l M'(m_l), the denominator of every other side.
void power_sums(const TreeRun& T, Level a, hipStream_t s) {
  const uint32_t n = (uint32_t)T.sys.size();
  a.R = 1;
  a.K = T.Ks;
  a.ldK = (size_t)2 * T.V;
  a.poly = T.poly;
  a.g = T.g;
  a.aux = T.sums;
  a.item0 = 0;
  a.full = 0;
  hipLaunchKernelGGL(k_tree_inverse_base, dim3(n), dim3(kBase), 0, s, a, T.C.M);
  auto at = [&](uint32_t logN, uint32_t i0, uint32_t i1) {
    a.logN = logN;
    a.N = 1u << logN;
    a.h = a.N / 2;
    a.item0 = i0;
    a.nn = i1 - i0;
  };
  auto tops = [&](uint32_t lg) {  // systems whose top has at least 2^lg rows
    uint32_t i = 0;
    while (i < n && T.sys[i].logTop >= lg) ++i;
    return i;
  };
  for (uint32_t lg = 10; lg <= T.sys[0].logTop; ++lg) {
    at(lg, 0, tops(lg));
    level_kernels<kInverse>(a, T.C.M, a.nn, s);
    series_product<kRev, kHigh>(a, T.C, s);
    series_product<kAux, kGrow>(a, T.C, s);
  }
  a.full = 1;
  for (uint32_t lg = T.sys[0].logTop; lg > kLeafLog; --lg) {
    at(lg + 1, tops(lg + 1), tops(lg));
    if (!a.nn) continue;
    level_kernels<kInverse>(a, T.C.M, a.nn, s);
    series_product<kDeriv, kSums>(a, T.C, s);
  }
}

// Unknowns from which the denominators of one system come from the power sums, one
// more right-hand side, instead of t^2 steps of the chain pass (t = 33 000: about the
// same; 100 003: 3.96 against 0.6 ms; 300 007: 34 against 1.1 ms).
constexpr uint32_t kSumsMinT = 32768;

}  // namespace

// The tree pays from about 5500 unknowns whatever R, and below that where the
// right-hand sides are many enough for its launches (about 45 of 4 to 10 us).
// Quadratic against tree, whole solve, microseconds, on both sides of each line:
// t = 2177: R = 200 511/522, R = 400 904/868; t = 2250: R = 127 395/407, R = 200 521/520, R = 400
// 928/869; t = 2400: R = 80 294/304, R = 100 338/331, R = 200 576/526; t = 2561: R = 37 211/217, R = 43
// 228/229, R = 50 243/234; t = 2700: R = 28 202/202, R = 32 214/209, R = 40 229/222; t = 2945: R = 20
// 199/200, R = 24 214/205; t = 3072: R = 20 195/202, R = 24 217/205, R = 32 230/216; t = 3073: R = 8
// 215/199, R = 12 195/201, R = 16 205/203; t = 3400: R = 8 218/200, R = 15 214/204; t = 4500: R = 1
// 228/251, R = 10 298/267; t = 5500: R = 1 259/262, R = 10 365/272; t = 13 000: R = 1 610/360, R = 30
// 1568/464.  Up to 2^21 unknowns: the power sums' last transform then has 2^22 points,
// the primes' limit.
bool tree_applies(uint32_t t, uint32_t R) {
  if (!vsolve_uses_pc() || R == 0 || t > (1u << (kNttMaxLog - 1))) return false;
  if (t >= 5500) return true;
  if (t > 3072) return R >= 8;
  if (t > 2944) return R >= 24;
  if (t > 2688) return R >= 32;
  if (t > 2560) return R >= 43;
  if (t > 2304) return R >= 100;
  return t > 2240 && R >= 200;
}

uint32_t tree_log_top(uint32_t t) {
  uint32_t lg = kLeafLog;
  while ((1u << lg) < t) ++lg;
  return lg;
}

// Series of one group of R1, of nearly equal groups within kTreeResidueBytes: one
// series' residues and its two products, five primes.
static uint32_t group_size(size_t V, uint32_t R1) {
  const uint32_t most =
      (uint32_t)std::max<size_t>(1, std::min<size_t>(R1, kTreeResidueBytes / ((size_t)kNp * 4 * 3 * V)));
  return cdiv(R1, cdiv(R1, most));
}

void TreeSpace::add(size_t V, uint32_t logTop, uint32_t R1, bool sums) {
  const uint32_t group = group_size(V, R1);
  poly = std::max(poly, 2 * V);
  X = std::max(X, (size_t)std::max(2u, group) * V * kNp);
  Y = std::max(Y, (size_t)2 * group * V * kNp);
  K = std::max(K, (size_t)(logTop - kLeafLog) * 2 * V * kNp);
  if (sums) {
    g = std::max(g, 2 * V);
    Ks = std::max(Ks, (size_t)2 * V * kNp);
  }
  const uint32_t lg = logTop + (sums ? 1 : 0);
  if (lg > kRowLog) twLog = std::max(twLog, lg);
}

size_t TreeSpace::bound(size_t rows, uint32_t logTop, uint32_t R1) {
  const size_t V = std::min<size_t>(rows, kTreeMaxRows), row = 4 * kNp;
  const size_t residues = std::max(4 * row * V, std::min(3 * row * V * R1, kTreeResidueBytes));
  const size_t transforms = 2 * row * V * (logTop - kLeafLog + 1);  // Ks is one level more
  return residues + transforms + 2 * 8 * V + (2 * row << (logTop + 1));
}

void tree_prepare(std::vector<TreeRun>& trees, const zr_mod& M, bool sums, DevArena& A, hipStream_t s) {
  if (trees.empty()) return;
  TreeSpace S;
  for (TreeRun& T : trees) {
    T.V = 0;
    for (TreeSys& y : T.sys) {  // largest tops first: every offset is a multiple of its system's top
      const uint32_t t = y.end - y.off;
      y.off = T.V;
      y.end = T.V + t;
      y.logTop = tree_log_top(t);
      T.V += 1u << y.logTop;
    }
    T.R1 = T.R + (sums ? 1 : 0);
    T.group = group_size(T.V, T.R1);
    S.add(T.V, T.sys[0].logTop, T.R1, sums);
  }
  uint64_t* poly = A.alloc<uint64_t>(S.poly / 2);
  uint64_t* g = sums ? A.alloc<uint64_t>(S.g / 2) : nullptr;
  uint32_t* Ks = sums ? A.alloc<uint32_t>(S.Ks) : nullptr;
  uint32_t* X = A.alloc<uint32_t>(S.X);
  uint32_t* Y = A.alloc<uint32_t>(S.Y);
  uint32_t* K = A.alloc<uint32_t>(S.K);
  uint32_t* tw = S.twLog ? A.alloc<uint32_t>((size_t)2 * kNp << S.twLog) : nullptr;
  for (TreeRun& T : trees) {
    T.C.M = M;
    uint64_t prod = 1 % M.p;
    for (int j = 0; j < kNp; ++j) {
      T.C.Qp[j] = prod;
      prod = zr_mul(M, prod, kQ[j] % M.p);
    }
    T.leafM = A.alloc<uint64_t>(T.V);
    T.sums = sums ? A.alloc<uint64_t>(T.V) : nullptr;
    T.poly = poly;
    T.g = g;
    T.Ks = Ks;
    T.X = X;
    T.Y = Y;
    T.ldX = (size_t)std::max(2u, T.group) * T.V;
    T.ldY = (size_t)2 * T.group * T.V;
    T.tw = tw;
    T.twLog = S.twLog;
    T.make_tw = tw && &T == &trees[0];
    T.K.clear();
    for (uint32_t i = 0; i < T.sys[0].logTop - kLeafLog; ++i) T.K.push_back(K + (size_t)i * 2 * T.V * kNp);
    T.d_sys = nullptr;
    T.d_of = nullptr;
    if (T.sys.size() > 1) {
      std::vector<uint32_t> of(T.V >> kLeafLog);
      for (uint32_t i = 0; i < T.sys.size(); ++i)
        for (uint32_t b = T.sys[i].off >> kLeafLog; b < (T.sys[i].off + (1u << T.sys[i].logTop)) >> kLeafLog; ++b)
          of[b] = i;
      Blob blob;
      const size_t o_sys = blob.add(T.sys), o_of = blob.add(of);
      char* d = blob.upload(A, s);
      T.d_sys = (const TreeSys*)(d + o_sys);
      T.d_of = (const uint32_t*)(d + o_of);
    }
  }
}

static Level tree_level(const TreeRun& T, uint32_t lg) {
  Level a{};
  a.logN = lg;
  a.N = 1u << lg;
  a.h = a.N / 2;
  a.one = T.sys[0];
  a.sys = T.d_sys;
  a.sys_of = T.d_of;
  a.sums = T.sums;
  if (T.d_sys) {
    uint32_t v = 0;
    for (const TreeSys& y : T.sys)
      if (y.logTop >= lg) v += 1u << y.logTop;
    a.nn = v >> lg;
  } else {
    const uint32_t t = T.sys[0].end;
    a.nn = t / a.N + (t % a.N > a.h ? 1 : 0);
  }
  a.poly = T.poly;
  a.pout = T.poly;
  a.X = T.X;
  a.Y = T.Y;
  a.ldX = T.ldX;
  a.ldY = T.ldY;
  a.K = lg > kLeafLog ? T.K[lg - kLeafLog - 1] : nullptr;
  a.ldK = (size_t)2 * T.V;
  a.tw = T.tw;
  a.twLog = T.twLog;
  return a;
}

void tree_build(const TreeRun& T, hipStream_t s) {
  if (T.make_tw)
    hipLaunchKernelGGL(k_tree_twist, dim3(1u << (T.twLog - 8), kNp, 2), dim3(256), 0, s, T.tw, T.twLog, kNtt);
  check(copy_u64(T.poly, T.leafM, T.V, s));
  {
    TimedLaunch tl("tree_up", s);
    for (uint32_t lg = kLeafLog + 1; lg <= T.sys[0].logTop; ++lg) {
      const Level a = tree_level(T, lg);
      level_kernels<kChild>(a, T.C.M, 2 * a.nn, s);
      level_product(a, T.C, s);
    }
  }
  if (T.sums) {
    TimedLaunch tl("tree_sums", s);
    power_sums(T, tree_level(T, kLeafLog + 1), s);
  }
  check(hipGetLastError());
}

void tree_descend(const TreeRun& T, hipStream_t s) {
  {
    TimedLaunch tl("tree_down", s);
    for (uint32_t j0 = 0; j0 < T.R1; j0 += T.group)
      for (uint32_t lg = T.sys[0].logTop; lg > kLeafLog; --lg) {
        Level a = tree_level(T, lg);
        a.j0 = j0;
        a.R = std::min(T.group, T.R1 - j0);
        level_descend(a, T.C, s);
      }
  }
  check(hipGetLastError());
}

TreeSolver::TreeSolver(const zr_mod& M, uint32_t t, uint32_t Rmax, const uint64_t* mono, DevArena& A, hipStream_t s)
    : t_(t), mono_(mono), s_(s), one_(1) {
  TreeRun& T = one_[0];
  T.R = Rmax;
  TreeSys y{};
  y.end = t;
  T.sys.push_back(y);
  tree_prepare(one_, M, t >= kSumsMinT, A, s);
  cap_ = T.group;
  tmp_ = A.alloc<uint64_t>(master_tmp_words(t, kLeaf));
  fixed_ = A.alloc<uint64_t>(vsolve_leaf_fixed_words(t));
}

void TreeSolver::solve(uint32_t R, const uint64_t* rhs, size_t ld_rhs, uint64_t* out, size_t ld_out, int32_t* status,
                       DevArena& W) {
  TreeRun T = one_[0];
  const bool first = !built_;
  if (!first) T.sums = nullptr;  // the denominators are made
  T.R = R;
  T.R1 = R + (T.sums ? 1 : 0);
  T.group = cdiv(T.R1, cdiv(T.R1, cap_));
  TreeSys& y = T.sys[0];
  y.ld_rhs = ld_rhs;
  y.ld = ld_out;
  y.rhs = rhs - (T.sums ? ld_rhs : 0);
  y.f = out - (T.sums ? ld_out : 0);  // read and packed before the unknowns are written
  // before the first launch: a call that fails for memory has written nothing
  uint64_t* work = W.alloc<uint64_t>(vsolve_leaf_words(t_, T.R1, first && !T.sums));
  if (first) {
    // leaf polynomials by the quadratic product tree
    check(master_levels(T.C.M, t_, kLeaf, mono_, T.leafM, tmp_, s_));
    tree_build(T, s_);
    built_ = true;
  }
  tree_descend(T, s_);
  check(vsolve_leaf(T.C.M, t_, T.R1, T.sums, kLeaf, mono_, T.leafM, T.poly, out, ld_out, fixed_, first, work, status,
                    s_));
}

void tree_solve(const zr_mod& M, uint32_t t, uint32_t R, const uint64_t* mono, const uint64_t* rhs, size_t ld_rhs,
                uint64_t* out, size_t ld_out, int32_t* status, DevArena& A, hipStream_t s) {
  TreeSolver(M, t, R, mono, A, s).solve(R, rhs, ld_rhs, out, ld_out, status, A);
}

}  // namespace zr

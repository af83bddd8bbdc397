// Transposed Vandermonde solves of large systems by a subproduct tree.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "driver.hpp"
#include "field.hpp"
#include "ntt.hpp"

namespace zr {

// true when a system of t unknowns and R right-hand sides is solved by the
// tree (the solve variant that zr_solve_variant selects permitting)
bool tree_applies(uint32_t t, uint32_t R);

// The system of vsolve, from the monomial values alone: workspace from A,
// launches on s.
void tree_solve(const zr_mod& M, uint32_t t, uint32_t R, const uint64_t* mono, const uint64_t* rhs, size_t ld_rhs,
                uint64_t* out, size_t ld_out, int32_t* status, DevArena& A, hipStream_t s);

// ---- many systems through one tree ----------------------------------------------------

constexpr uint32_t kTreeLeafLog = 8;  // leaf blocks of 256 rows
constexpr uint32_t kTreeLeaf = 1u << kTreeLeafLog;

// One system: rows [off, end) of the common index space (off set by
// tree_prepare; give off = 0, end = t), the samples of series j at rhs + j ld_rhs, the
// series at f + j ld from the top's children down to the leaf blocks (f may be rhs).
// With power sums, which are series 0, rhs and f stand one series before the first
// right-hand side.
struct TreeSys {
  uint32_t off, end, logTop, pad;
  const uint64_t* rhs;
  uint64_t* f;
  size_t ld_rhs, ld;
};

// log2 of the rows of the top node of t rows
uint32_t tree_log_top(uint32_t t);

// Rows of one tree, at most (a batch's systems beyond it go into further trees, which
// use the same workspace): two series' residues then stay below kTreeResidueBytes.
constexpr uint32_t kTreeMaxRows = 1u << 22;
// Residues of a group of series, at most (bytes).  t = 300 007, 41 series: 9.8 ms with
// 160 MB, which the last-level cache holds, 8.8 with 640, 9.0 with all at once: the
// launches' fill matters more.
constexpr size_t kTreeResidueBytes = (size_t)640 << 20;

// Workspace that trees run one after the other on a stream share, in 32-bit words: the
// largest of each part over the trees added.
struct TreeSpace {
  size_t poly = 0, g = 0;           // whole polynomials; 1/Q of the power sums
  size_t X = 0, Y = 0, K = 0, Ks = 0;  // residues of a group, their products; transforms of all levels; of g
  uint32_t twLog = 0;               // log2 of the longest transform
  // a tree of V rows (at most kTreeMaxRows) whose largest node has 2^logTop, with R1 series
  void add(size_t V, uint32_t logTop, uint32_t R1, bool sums);
  // its bytes at most, for trees with power sums over `rows` rows in all, whatever their
  // division into trees
  static size_t bound(size_t rows, uint32_t logTop, uint32_t R1);
};

struct TreeRun {
  CrtP C;
  std::vector<TreeSys> sys;  // tops in descending order
  uint32_t R;                // right-hand sides of each
  uint32_t V, R1, group;     // rows of the index space; series (the power sums are series 0, if made)
  uint64_t *leafM, *poly, *sums, *g;
  uint32_t *X, *Y, *Ks, *tw;
  uint32_t twLog;
  bool make_tw;  // the first of the trees that share a table of twist factors
  size_t ldX, ldY;
  std::vector<uint32_t*> K;  // children's transforms of each level
  const TreeSys* d_sys;
  const uint32_t* d_of;
};

// Workspace from A, shared by the trees (launched in this order on one stream), and the
// systems' tables (uploaded on s).
void tree_prepare(std::vector<TreeRun>& trees, const zr_mod& M, bool sums, DevArena& A, hipStream_t s);
// From the leaf blocks' polynomials in T.leafM (block b of a system at off + 256 b): the
// whole polynomials into T.poly, the children's transforms, and the power sums.
void tree_build(const TreeRun& T, hipStream_t s);
// From the right-hand sides: every leaf block's series into f (and, with power sums,
// into T.sums).
void tree_descend(const TreeRun& T, hipStream_t s);

// One system whose right-hand sides come in several sets: the tree and the denominators
// are made with the first set.  Workspace from A (which outlives it) for about Rmax
// right-hand sides at a time, and from W during a call.
class TreeSolver {
 public:
  TreeSolver(const zr_mod& M, uint32_t t, uint32_t Rmax, const uint64_t* mono, DevArena& A, hipStream_t s);
  void solve(uint32_t R, const uint64_t* rhs, size_t ld_rhs, uint64_t* out, size_t ld_out, int32_t* status, DevArena& W);

 private:
  uint32_t t_, cap_;  // cap_: series that the residues hold
  const uint64_t* mono_;
  hipStream_t s_;
  std::vector<TreeRun> one_;
  uint64_t *tmp_, *fixed_;
  bool built_ = false;
};

}  // namespace zr

// Transposed Vandermonde solves of large systems by a subproduct tree.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "driver.hpp"
#include "field.hpp"

namespace zr {

// true when a system of t unknowns and R right-hand sides is solved by the
// tree (the solve variant that zr_solve_variant selects permitting)
bool tree_applies(uint32_t t, uint32_t R);

// The system of vsolve, from the monomial values alone: workspace from A,
// launches on s.
void tree_solve(const zr_mod& M, uint32_t t, uint32_t R, const uint64_t* mono, const uint64_t* rhs, size_t ld_rhs,
                uint64_t* out, size_t ld_out, int32_t* status, DevArena& A, hipStream_t s);

}  // namespace zr

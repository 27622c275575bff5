// Predicates of the input check, free of device code so that a plain host
// compiler takes them too (constexpr functions are callable from kernels).
#pragma once
#include <cstdint>

namespace gsofa {

// Row r of a CSR matrix with nnz entries, row_ptr[r] = a and row_ptr[r + 1] = b,
// may be read: [a, b) lies inside the entries and row 0 starts at 0. (b >= a alone
// does not bound the read: in row_ptr {0, 2^30, 5} row 0 ascends and the fall is
// seen by row 1 only.)
constexpr bool csr_row_readable(int64_t r, int32_t a, int32_t b, int32_t nnz) {
    return a >= 0 && b >= a && b <= nnz && (r != 0 || a == 0);
}

}  // namespace gsofa

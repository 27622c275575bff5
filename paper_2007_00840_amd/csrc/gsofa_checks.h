// Decisions free of device code, so that a plain host compiler takes them too
// (constexpr functions are callable from kernels).
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

// How a launch of the block path's factorisation ended: with everything done, for
// want of tiles, or because a wait gave up.
enum BmAbortCode : uint32_t { kBmNoAbort = 0, kBmOverflow = 1, kBmStall = 2 };

// What follows: the results, the launch again with a larger pool if one fits, or the
// traversal. A wait gives up after a number of polls, which a long chain of blocks
// or a device shared with other work can use up: no error of the call.
enum class BmNext { kResults, kAgain, kTraverse };
constexpr BmNext bm_next(uint32_t abort, bool larger_pool_fits) {
    return abort == kBmNoAbort ? BmNext::kResults
                               : abort == kBmOverflow && larger_pool_fits ? BmNext::kAgain : BmNext::kTraverse;
}

}  // namespace gsofa

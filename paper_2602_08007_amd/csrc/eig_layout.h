// Scratch of the small SVD (JacobiBlock::scratch, in doubles): where its parts lie, for the host code that
// carves it and the kernels that index it.
//   [0, 3 k^2)    the three diagonals of the LU factors (inverse iteration); afterwards the triangular factors
//                 of the reflector blocks
//   behind them   d (k), e (k), the eigenvalues (k, ascending), the radius of the spectrum's bracket (1)
#pragma once
#include <cstddef>

namespace tsr {

constexpr size_t eig_tridiag_at(int k) { return (size_t)3 * k * k; }
constexpr size_t eig_scratch_doubles(int k) { return eig_tridiag_at(k) + 3 * (size_t)k + 8; }

// Reflector j of a k x k matrix exists for j + 2 < k; block b holds reflectors 16 b ..: this many.
constexpr int eig_wy_rank(int k, int b) {
    const int left = k - 2 - 16 * b;
    return left < 0 ? 0 : left < 16 ? left : 16;
}
// Entry (row, col) of the triangular factor of block b.  Only row, col < eig_wy_rank(k, b) are stored: a whole
// 16 x 16 factor (256 doubles) would not fit into 3 k^2 for k <= 9.
constexpr size_t eig_wy_at(int b, int row, int col) { return (size_t)b * 256 + row * 16 + col; }

}  // namespace tsr

// Products of fp64 matrices from 8-bit integer matrix instructions (residue.hip).
#pragma once
#include "common.hpp"
#include "residue_math.hpp"

namespace onecomp {
namespace residue {

constexpr int TILE = 256;     // rows and columns of a product tile
constexpr int K_STEP = 64;    // inner ranges begin and end on multiples of this

inline int64_t pad_rows(int64_t n) { return ceil_div(n, TILE) * TILE; }
inline int64_t pad_k(int64_t k) { return ceil_div(k, K_STEP) * K_STEP; }
// bytes of the residues of `rows` rows of k entries, and of the product of `rows` x `cols`
inline size_t operand_bytes(int64_t rows, int64_t k) { return size_t(MODULI) * pad_rows(rows) * pad_k(k); }
inline size_t product_bytes(int64_t rows, int64_t cols) { return size_t(MODULI) * pad_rows(rows) * pad_rows(cols); }

// Residues of a matrix of up to `rows` rows and k columns, one plane per modulus; rows in blocks of 32, columns in blocks
// of 32, such a block (32 x 32 bytes) in the order of the matrix instruction's operand.  data: 256-byte aligned.
struct Operand {
    char* data;
    int64_t plane;    // bytes of a plane
    int64_t block;    // bytes of a row block
    Operand(void* p, int64_t rows, int64_t k)
        : data(static_cast<char*>(p)), plane(pad_rows(rows) * pad_k(k)), block(pad_k(k) * 32) {}
    // the same rows from `row` (a multiple of 32) on
    Operand from(int64_t row) const {
        Operand o = *this;
        o.data += row / 32 * block;
        return o;
    }
};

// ---- left-looking Cholesky -------------------------------------------------------------------------------------------
// shift[i], left[i]: scale and squared norm of row i of L, from the n diagonal entries of the matrix A that is factored
onecomp_status row_bounds(const double* A, int n, int32_t* shift, double* left, hipStream_t stream);
// columns [c0, c0 + width) of rows [r0, n) of L (n x n, row-major) into the same places of R; c0, width multiples of 64, r0
// of 32.  Takes their squares off left[i]; where these exceed it the row gets NO_SHIFT.
onecomp_status convert_columns(const double* L, int n, int r0, int c0, int width, int32_t* shift, double* left,
                               const Operand& R, hipStream_t stream);
// A[r][c] -= sum over k < c0 of L[r][k] L[c][k], rows r in [c0, n), columns c in [c0, c0 + width) up to the row's tile.
// copy: where rows [c0 + 128, c0 + 256) of columns [c0, c0 + 128) also go, rows of 128.  scratch: product_bytes(n - c0, width)
onecomp_status update_columns(double* A, int n, int c0, int width, const int32_t* shift, const Operand& R, double* copy,
                              void* scratch, hipStream_t stream);

// inner[i]: exponent of 1 / V[i][i]
onecomp_status inner_exponents(const double* V, int n, int32_t* inner, hipStream_t stream);

// ---- C = alpha A B with one triangular operand ---------------------------------------------------------------------------
// A m x k, B k x n, C m x n, row-major; lower_b: B is lower triangular (k == n), else A is (m == k); what lies above
// counts as zero whatever it holds, but is read in part, so it has to be there and at rest.  C may be B.  alpha = +-1.
// inner: nullptr, or powers of two by which the k terms of a sum are balanced between the operands: column k of A counts
// 2^inner[k] times, row k of B 2^-inner[k] times, so that what the channels' own scales do to the rows of one and the columns of
// the other cancels.  operands: operand_len bytes of scratch (an upper bound on the columns taken at a time follows from
// it); product: product_len bytes of scratch; shift_a, shift_b: m and n entries.
onecomp_status triangular_product(const double* A, int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc, int m,
                                  int n, int k, bool lower_b, double alpha, void* operands, size_t operand_len, void* product,
                                  size_t product_len, const int32_t* inner, int32_t* shift_a, int32_t* shift_b, hipStream_t stream);

}  // namespace residue
}  // namespace onecomp

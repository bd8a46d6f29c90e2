// Dense kernels of the host factorisation (x86-64 with AVX2 + FMA; AVX-512
// where the CPU has it, chosen at run time).
#pragma once
#include <cstdint>
#include <vector>

namespace scasm {

// C += sign * A * B^T, column-major: A is M x K (lda), B is N x K (ldb), C is
// M x N (ldc); sign is +1 or -1.  Register-blocked 8 x 4 (AVX2) or 16 x 8
// (AVX-512) micro-kernel over packed panels of 256 columns of K; small
// products take a plain loop.
void gemm_nt(int64_t M, int64_t N, int64_t K, double sign, const double* A, int64_t lda, const double* B,
             int64_t ldb, double* C, int64_t ldc);

// Columns [j0, j1) of a panel with ld rows (at most kFactorColumns, updated
// with the columns before them): Cholesky of the diagonal block, then the rows
// below it in strips of registers.  Returns the first column whose pivot is
// not positive, or -1.
constexpr int32_t kFactorColumns = 32;
int64_t factor_columns(double* A, int64_t ld, int64_t j0, int64_t j1);

// The m x K block A (column-major, ld) packed for subtract_outer: panels of 16
// (AVX-512) or 8 rows, k-major, zero padded.
void pack_rows(const double* A, int64_t ld, int64_t m, int64_t K, std::vector<double>& pa);

// T[rel[i], cols[j]] -= sum_k a[i, k] a[b0 + j, k] for the packed rows i >= b0
// + j, 0 <= j < nb; T column-major (ldt), rel indexed by i (from b0 on).
void subtract_outer(const double* pa, int64_t m, int64_t K, int64_t b0, int64_t nb, const int32_t* rel, double* T,
                    int64_t ldt, const int32_t* cols, std::vector<double>& pb);

}  // namespace scasm

// Dense bf16 products of the token-wise library (tw_gemm.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fpdt_tw {

// Start of a library call: forget the realigned weights of the previous call and reuse its scratch.
void begin_call();

// Device scratch that lives until the next begin_call; null if there is not enough memory.
void* scratch(size_t bytes);

// Does the product C [rows, cols] bf16 = A [rows, k] * .. read A where it is (and not a copy in scratch)?
bool reads_in_place(const void* A, int64_t rows, int64_t k, const void* C, int64_t cols);

// C[M,N] (+)= sum_k Aop[m,k] * Bop[n,k], bf16 operands, fp32 accumulation.
//   a_transposed = 0: A is stored [M,K] (leading dimension lda); 1: A is stored [K,M]
//   b_transposed = 0: B is stored [N,K] (ldb);                   1: B is stored [K,N]
//   C row-major [M,N], leading dimension ldc, bf16 or fp32 (c_f32); accumulate: C += instead of C =
//   ldc wider than N, fp32, not accumulating: what follows a row up to a multiple of 4 may be overwritten
//   lda wider than A's rows: they are followed by zeros up to a multiple of 8
//   cache_b: B is a weight that further products of this library call will use again
//   A or B may be what C overwrites
// Only enqueues on `st`.  Returns 0, 1 (HIP failure) or 2 (sizes beyond the launch limits).
int gemm(int a_transposed, int b_transposed, int M, int N, int K, const void* A, int64_t lda, const void* B,
         int64_t ldb, void* C, int64_t ldc, bool c_f32, bool accumulate, bool cache_b, hipStream_t st);

}  // namespace fpdt_tw

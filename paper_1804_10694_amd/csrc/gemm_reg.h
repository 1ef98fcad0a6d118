// Host interface of the register-operand tiles (gemm_reg.hip).
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>

namespace tg {

// Register tile to run a row-major problem of these sizes on, or -1 where the
// schedules of the table are faster (F32 and split-bf16x3 only).
int reg_choice(int64_t M, int64_t N, int64_t K, int dtype);
// The fastest register tile for a batch, whether or not one pays.
int reg_best_tile(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype);
// Whether register tiles pay for `batch` products at fixed strides, where the
// other way copies `copied` elements into another order first.
bool reg_strided_pays(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int64_t copied);
// Whether the tiles' 32-bit offsets reach operands of these strides.  ak / bk:
// A / B has K contiguous (its stride is between rows; otherwise between k).
bool reg_serves(const void* A, bool ak, int64_t lda, const void* B, bool bk, int64_t ldb);
// C[p] = alpha * A[p] * B[p] + beta * C[p], p < batch, operands sA, sB and C
// sC elements apart.  TGEMM_NOT_SUPPORTED where reg_serves is false or the tiles
// are more than one grid holds.
int run_reg(int tile, int dtype, int64_t M, int64_t N, int64_t K, int64_t batch, float alpha, const float* A,
            bool ak, int64_t lda, int64_t sA, const float* B, bool bk, int64_t ldb, int64_t sB, float beta, float* C,
            int64_t ldc, int64_t sC, int group_m, int xcd_remap, hipStream_t s);

}  // namespace tg

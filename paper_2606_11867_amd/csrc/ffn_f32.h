// Launchers of the fp32 FFN kernels (ffn_f32.hip).
#pragma once

#include "common.h"

namespace foremoe {

enum F32Op { kF32GateUpFwd = 0, kF32DownFwd = 1, kF32DownDgrad = 2, kF32GateUpDgrad = 3 };

struct F32RowsArgs {
  const float* A;   // rows: x, h, dy or d_au
  const float* Wt;  // [W, ...] weights
  const float* AU;  // down dgrad: saved [A | U]
  int d, F, W;
  const int32_t* off;
  const int32_t* widx;
  int S;
  int64_t n_cap;
  float* C;
  float* C2;  // gate/up forward: saved [A | U] or NULL
};

// e0, e1: optional timing events of the launch.
void launch_f32_rows(int op, const F32RowsArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1);

// dW[g][m][n] += sum over the rows of slots with gidx g of A[row][m] B[row][n]
void launch_f32_wgrad(const float* A, int lda, const float* B, int ldb, int M, int N, const int32_t* off,
                      const int32_t* gidx, int S, int G, int64_t n_cap, int part, int parts, float* C,
                      hipStream_t st);

}  // namespace foremoe

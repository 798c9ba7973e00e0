// Product epilogues of the many-row kernels, eight consecutive columns of a row
// at a time (16-byte loads and stores); the expressions are k_gemm's.
#pragma once

#include "common.h"
#include "kernels.h"
#include "mma.h"

namespace pdec {

// The eight sums v of columns col .. col + 7 (col a multiple of 8) of a row,
// finished and stored: bias[8] and, by epilogue, the row's residual[8] or its
// (sentence, position).
template <typename WT, int EPI>
__device__ __forceinline__ void finish8(const GemmArgs& a, int row, int col, float* v, const float* bias,
                                        const float* resid, int sent, int pos) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = v[e] + bias[e];
  if constexpr (EPI == EPI_F32) {
    store8<float>(a.out_f32, static_cast<size_t>(row) * a.ldo + col, v);
  } else if constexpr (EPI == EPI_ACT) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (a.act == 2) ? gelu_erf(v[e]) : relu(v[e]);
    store_row8<WT>(static_cast<WT*>(a.out), row, col, a.out_feed ? a.N : 0, a.ldo, v);
  } else if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] + resid[e];
    if (a.out_f32 != nullptr) store8<float>(a.out_f32, static_cast<size_t>(row) * a.ldo + col, v);
    else store8<WT>(static_cast<WT*>(a.out), static_cast<size_t>(row) * a.ldo + col, v);
  } else if constexpr (EPI == EPI_QKV) {
    if (col < a.q_cols) {
      store8<float>(a.out_f32, static_cast<size_t>(row) * a.ldo + col, v);
    } else {
      const int c = col - a.q_cols;
      const int which = c / a.d;
      const int cc = c - which * a.d;
      const int hh = cc / a.dh;
      const int dd = cc - hh * a.dh;
      const size_t idx = ((static_cast<size_t>(sent) * a.H + hh) * a.T + pos) * a.dh + dd;
      store8<WT>(static_cast<WT*>(which == 0 ? a.kc : a.vc), idx, v);
    }
  }
}

}  // namespace pdec

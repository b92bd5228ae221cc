// The fused epilogues and waits that the weight GEMMs share (kernels_gemm.hip, kernels_prompt.hip).
#pragma once
#include "device_common.h"
#include "ham_internal.h"

namespace ham {

// Epilogue of one accumulator element: row m, column nb + r16 of the tile at nb.
// Every lane must call it (the SwiGLU pairing exchanges values between lanes).
template <typename T, int EPI>
__device__ __forceinline__ void epi_tile(const GemmArgs& a, int m, bool ok, int nb, int r16, float v) {
  const int n = nb + r16;
  if constexpr (EPI == EPI_SWIGLU) {
    // a 16-row tile holds gate rows of 8 features then their up rows
    const float u = __shfl_xor(v, 8, WAVE);
    if (ok && r16 < 8) {
      const float sg = v / (1.0f + expf(-v));
      Act<T>::put(a.out, m, a.ldo, nb / 2 + r16, sg * u);
    }
  } else {
    if (!ok) return;
    if constexpr (EPI == EPI_F32) {
      ((float*)a.out)[(size_t)m * a.ldo + n] = v;
    } else if constexpr (EPI == EPI_OP) {
      Act<T>::put(a.out, m, a.ldo, n, v);
    } else if constexpr (EPI == EPI_RESID) {
      float* o = (float*)a.out + (size_t)m * a.ldo;
      o[n] += v;
    } else if constexpr (EPI == EPI_XMASK) {
      if (a.rowmask[m]) ((float*)a.out)[(size_t)m * a.ldo + n] = v;
    }
  }
}

// s_waitcnt with vmcnt <= n (0..63) and lgkmcnt = 0 (expcnt untouched)
template <int N>
__device__ __forceinline__ void wait_vm_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

}  // namespace ham

// Workgroup body of the shared projection R = X B^T (paper Sec. 3.3, Eq. 8).
// Used by the stand-alone projection kernel and, as the producer role, by the
// single-launch decode kernel.
#pragma once
#include "common.hpp"

namespace glowq {

struct ProjArgs {
  const uint16_t* X;   // act dtype [T][K]
  const uint16_t* B;   // act dtype [r][K]
  int T, K, r;
  int ksplit;          // K slices
  int kslice;          // channels per slice, multiple of 32
  float* Rpart;        // stand-alone projection: fp32 [slice][T][r]; in-launch projection
                       // of the decode kernels: 8-byte slots {fp32 bits, launch tag}
  float* R32;          // optional fp32 [T][r]
  uint16_t* R16;       // optional act dtype [T][r]
  Control* ctl;        // control words of the unit's workspace slice
};

// Projection for a handful of tokens (T <= 4), built for the shortest dependency chain:
// one WAVE computes, for one rank j and one of `ksplit` K parts, the T partial sums
// sum_k X[t][k] B[j][k] -- contiguous reads of B and X, all of a batch in flight
// together, fp32 accumulation, a butterfly reduction -- and publishes each as ONE 8-byte
// device-scope store {fp32 bits, low word of the launch tag}.  A slot therefore
// validates itself: no fence, no flag, no ordering between stores, and the wave never
// waits for anything.  The consumers add the parts (r_fetch_finish).  Slot of
// (t, part, j): slots[(t ksplit + part) r + j].
template <int ACT>
__device__ inline void proj_wave_direct(const ProjArgs& a, int wave_global, int lane) {
  const int rank = wave_global % a.r, part = wave_global / a.r;   // a workgroup shares a part
  if (part >= a.ksplit) return;
  const int k_begin = part * a.kslice;
  const int k_end = min(a.K, k_begin + a.kslice);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  const uint16_t* brow = a.B + (size_t)rank * a.K;
  constexpr int BATCH = 4;   // 512-channel steps whose loads are in flight together
  for (int k0 = k_begin + 8 * lane; k0 < k_end; k0 += 512 * BATCH) {
    u32x4_t bv[BATCH], xv[4][BATCH];
#pragma unroll
    for (int it = 0; it < BATCH; ++it) {
      const int k = k0 + 512 * it;
      const bool in = k < k_end;
      const int kc = in ? k : k0;                     // clamped: loaded again, not used
      bv[it] = *(const u32x4_t*)(brow + kc);
      if (!in) bv[it] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (t < a.T) xv[t][it] = *(const u32x4_t*)(a.X + (size_t)t * a.K + kc);
    }
#pragma unroll
    for (int it = 0; it < BATCH; ++it) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (t < a.T) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t bw = bv[it][i], xw = xv[t][it][i];
            float b0, b1, x0, x1;
            if constexpr (ACT == ACT_F16) {
              b0 = (float)__builtin_bit_cast(_Float16, (uint16_t)(bw & 0xffffu));
              b1 = (float)__builtin_bit_cast(_Float16, (uint16_t)(bw >> 16));
              x0 = (float)__builtin_bit_cast(_Float16, (uint16_t)(xw & 0xffffu));
              x1 = (float)__builtin_bit_cast(_Float16, (uint16_t)(xw >> 16));
            } else {
              b0 = __builtin_bit_cast(float, bw << 16);
              b1 = __builtin_bit_cast(float, bw & 0xffff0000u);
              x0 = __builtin_bit_cast(float, xw << 16);
              x1 = __builtin_bit_cast(float, xw & 0xffff0000u);
            }
            acc[t] = __builtin_fmaf(b0, x0, acc[t]);
            acc[t] = __builtin_fmaf(b1, x1, acc[t]);
          }
        }
      }
    }
  }
  const unsigned long long tag_hi = (launch_tag() & 0xffffffffull) << 32;
  unsigned long long* slots = (unsigned long long*)a.Rpart;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (t < a.T) {
      float s = acc[t];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
      if (lane == 0)
        __hip_atomic_store(&slots[((size_t)t * a.ksplit + part) * a.r + rank],
                           tag_hi | (unsigned long long)__builtin_bit_cast(uint32_t, s),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

}  // namespace glowq

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
  float* R32;          // stand-alone projection: its result, fp32 [T][r]
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

// Four 16-byte loads at device scope (not served from an L2 line that may be older than another
// compute unit's store), waited for in the same place.
__device__ inline void load4_device(u32x4_t (&v)[4], const void* p0, const void* p1, const void* p2, const void* p3) {
  asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
               "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\t"
               "s_waitcnt vmcnt(0)"
               : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(p0), "v"(p1), "v"(p2), "v"(p3) : "memory");
}

// Two neighbouring ranks' sums of one K slice (s) are published as self-validating slots {fp32, launch tag} (q: slice 0's
// first one, slices r apart, at most four), and nobody waits for anybody: a thread whose own slots are out looks at its
// elements' slots of all slices once.  If they are complete, s receives their sum in slice order.  Of two slices at least
// one finds the other's slots: a look is issued when the thread's own stores have completed at device scope, so the later
// of the two looks comes behind both stores.  Several may find them all; they hand out the same bits.
__device__ inline void publish_slice(unsigned long long* q, int slice, int r, uint32_t tag, const float (&s)[2]) {
  const unsigned long long tag_hi = (unsigned long long)tag << 32;
#pragma unroll
  for (int e = 0; e < 2; ++e)
    __hip_atomic_store(q + (size_t)slice * r + e, tag_hi | (unsigned long long)__builtin_bit_cast(uint32_t, s[e]),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool look_at_slices(const unsigned long long* q, int ksplit, int r, uint32_t tag, float (&s)[2]) {
  u32x4_t v[4];
  load4_device(v, q, q + (size_t)min(1, ksplit - 1) * r, q + (size_t)min(2, ksplit - 1) * r, q + (size_t)(ksplit - 1) * r);
  bool all = true;
  s[0] = s[1] = 0.f;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const uint32_t w0 = v[p][0], t0 = v[p][1], w1 = v[p][2], t1 = v[p][3];
    all = all && t0 == tag && t1 == tag;
    if (p < ksplit) {
      s[0] += __builtin_bit_cast(float, w0);
      s[1] += __builtin_bit_cast(float, w1);
    }
  }
  return all;
}

constexpr int PROJ_NB = 2;               // 16-rank blocks per workgroup
struct ProjSliced {
  const uint16_t* X;
  const uint16_t* B;
  float* part;             // slots {fp32, tag}: (t ksplit + slice) r + rank (ksplit > 1 only)
  int T, K, r, ksplit, kslice;
  bool slots_only;         // the slices (two at least) stay apart, for the consumers to add
};

// One workgroup of NW waves: tokens 16 tb .., K slice kz, ranks 32 ng .. + 32.  Whoever finds all slices complete adds
// them (see publish_slice); out(t, rank, pair, tag) receives two ranks rounded to the activation type.  lds: NW *
// PROJ_NB * 256 floats.
template <int ACT, int NW, class OUT>
__device__ inline void proj_sliced(const ProjSliced& u, int local, float* lds, OUT out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kz = local % u.ksplit, rest = local / u.ksplit;
  const int n_groups = (u.r + 31) >> 5;
  const int ng = rest % n_groups, tb = rest / n_groups;
  const int i = lane & 15, kq = lane >> 4;
  const int T = u.T, K = u.K, r = u.r, ksplit = u.ksplit;
  // tokens past T and ranks past r: clamped (valid) rows, computed and not stored
  const uint16_t* xrow = u.X + (size_t)min(tb * 16 + i, T - 1) * K + 8 * kq;
  const uint16_t* brow[PROJ_NB];
#pragma unroll
  for (int nb = 0; nb < PROJ_NB; ++nb) brow[nb] = u.B + (size_t)min(ng * 32 + nb * 16 + i, r - 1) * K + 8 * kq;
  const int k_begin = kz * u.kslice, k_end = min(K, k_begin + u.kslice);
  float4_t acc[PROJ_NB];
#pragma unroll
  for (int nb = 0; nb < PROJ_NB; ++nb) acc[nb] = float4_t{0.f, 0.f, 0.f, 0.f};
  constexpr int PB = 4;                          // steps of 32 channels whose loads are in flight together
  for (int k0 = k_begin + wave * 32; k0 < k_end; k0 += PB * NW * 32) {
    u32x4_t xf[PB], bf[PB][PROJ_NB];
#pragma unroll
    for (int s = 0; s < PB; ++s) {
      const int k = k0 + s * NW * 32;
      const bool in = k < k_end;                 // past the end: the first step again, times zero
      const int kc = in ? k : k0;
      xf[s] = *(const u32x4_t*)(xrow + kc);
      if (!in) xf[s] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
      for (int nb = 0; nb < PROJ_NB; ++nb) {
        bf[s][nb] = *(const u32x4_t*)(brow[nb] + kc);
        if (!in) bf[s][nb] = u32x4_t{0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int s = 0; s < PB; ++s)
#pragma unroll
      for (int nb = 0; nb < PROJ_NB; ++nb) acc[nb] = mfma16<ACT>(xf[s], bf[s][nb], acc[nb]);   // D[token][rank]
  }
#pragma unroll
  for (int nb = 0; nb < PROJ_NB; ++nb)
#pragma unroll
    for (int v = 0; v < 4; ++v) lds[((wave * PROJ_NB + nb) * 4 + v) * 64 + lane] = acc[nb][v];
  __syncthreads();
  // thread -> (token, pair of ranks)
  const int tl = tid >> 4, rp = tid & 15;
  const int t = tb * 16 + tl, rank = ng * 32 + 2 * rp;
  if (tid >= 256 || t >= T || rank >= r) return; // (no barrier follows)
  float s[2] = {0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int rl = 2 * rp + e, ln = (rl & 15) + 16 * (tl >> 2);
#pragma unroll
    for (int w = 0; w < NW; ++w) s[e] += lds[((w * PROJ_NB + (rl >> 4)) * 4 + (tl & 3)) * 64 + ln];
  }
  const uint32_t tag = (uint32_t)(launch_tag() & 0xffffffffull);
  if (ksplit > 1) {
    unsigned long long* q = (unsigned long long*)u.part + (size_t)t * ksplit * r + rank;
    publish_slice(q, kz, r, tag, s);
    if (u.slots_only) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // (counts stores, too)
    if (!look_at_slices(q, ksplit, r, tag, s)) return;
  }
  const uint32_t pk = (uint32_t)to_act16<ACT>(s[0]) | ((uint32_t)to_act16<ACT>(s[1]) << 16);
  out(t, rank, pk, tag);
}

}  // namespace glowq

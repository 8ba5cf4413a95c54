// Weight preparation, the two inspection hooks, and the importance scores of GlowQ-S.
//
// quantize_rtn:  fp32 weights -> canonical W4A16 arrays (round to nearest, asymmetric)
// prepare:       canonical W4A16 arrays -> tiled layout the forward kernels read
// debug_unpack:  tiled layout -> q[d_out][d_in] bytes
// debug_dequant: tiled layout -> round_to_act((q - z) * s) through dequant_word(), the
//                library's reference dequantiser (the forward kernels schedule
//                instruction sequences of their own, checked through forward calls)
// importance:    g_ner = ||E_u||^2 / ||W_u||^2 and g_ec = sum_j sigma_j^2 / ||E_u||^2 of one
//                unit (paper Sec. 3.3, Eqs. 10-11), from the full-precision weights, the
//                prepared layout and the stored factors; all sums in float64
#include "common.hpp"
#include "launch.hpp"

namespace glowq {

// one thread per word of a tile record
__global__ void k_prepare(const uint32_t* __restrict__ wq, const uint16_t* __restrict__ scales,
                          const uint16_t* __restrict__ zeros, uint32_t* __restrict__ out,
                          int d_out, int d_in, int G, long long n_words) {
  long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_words) return;
  const int ktiles = d_in / 128;
  const int rec_words = prepared_rec_words(G);
  const int wi = (int)(idx % rec_words);
  const long long tile = idx / rec_words;
  const int kb = (int)(tile % ktiles);
  const int rb = (int)(tile / ktiles);
  uint32_t w;
  if (wi < 256) {
    const int j = wi & 3, lane = wi >> 2;
    const int row = rb * 16 + (lane & 15);
    const int k0 = kb * 128 + 32 * j + 8 * (lane >> 4);
    uint32_t c = 0;
    if (row < d_out) c = wq[(long long)row * (d_in / 8) + k0 / 8];
    w = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w |= ((c >> (8 * i)) & 0xFu) << (4 * i);            // e = 2i     -> nibble i
      w |= ((c >> (8 * i + 4)) & 0xFu) << (4 * i + 16);   // e = 2i + 1 -> nibble i + 4
    }
  } else {
    const int row = rb * 16 + ((wi - 256) & 15);
    const int g = kb * (128 / G) + ((wi - 256) >> 4);
    const int n_groups = d_in / G;
    w = 0x3C00u;   // s = 1, z = 0 for padding rows
    if (row < d_out)
      w = (uint32_t)scales[(long long)row * n_groups + g] |
          ((uint32_t)zeros[(long long)row * n_groups + g] << 16);
  }
  out[idx] = w;
}

// Round-to-nearest asymmetric INT4 per (row, group of G channels) (Sec. 4.1: INT4 weights,
// group size 128 or 64).  One thread per packed word (8 channels); the G / 8 threads of a
// group are neighbouring lanes.  Range widened to contain 0; s = fp16(max((hi - lo) / 15,
// 2^-14)); z = clamp(rint(-lo / s), 0, 15); q = clamp(rint(w / s) + z, 0, 15); float64
// arithmetic on the fp16-rounded s, rint to even.
__global__ void __launch_bounds__(256) k_quantize_rtn(const float* __restrict__ W, int d_out, int d_in, int G,
                                                      uint32_t* __restrict__ wq, uint16_t* __restrict__ scales,
                                                      uint16_t* __restrict__ zeros) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int words = d_in / 8;
  // (whole waves stay in the loop-free path: the total is a multiple of 16 words per row,
  // and lanes past the end only take part in the shuffles)
  const bool live = idx < (long long)d_out * words;
  const long long row = live ? idx / words : 0;
  const int j = live ? (int)(idx - row * words) : 0;
  const float4_t* src = (const float4_t*)(W + row * d_in + 8 * j);
  const float4_t w0 = src[0], w1 = src[1];
  const float w[8] = {w0[0], w0[1], w0[2], w0[3], w1[0], w1[1], w1[2], w1[3]};
  float lo = 0.f, hi = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    lo = fminf(lo, w[e]);
    hi = fmaxf(hi, w[e]);
  }
  for (int o = 1; o < G / 8; o <<= 1) {
    lo = fminf(lo, __shfl_xor(lo, o, 64));
    hi = fmaxf(hi, __shfl_xor(hi, o, 64));
  }
  const double s = fmax(((double)hi - (double)lo) / 15.0, 0x1p-14);
  const uint32_t s_bits = act16_round<ACT_F16>(s);
  const double s_hat = act16_value<ACT_F16>(s_bits);
  const double z = fmin(fmax(__builtin_rint(-(double)lo / s_hat), 0.0), 15.0) + 0.0;   // (+0, never -0)
  uint32_t word = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double q = fmin(fmax(__builtin_rint((double)w[e] / s_hat) + z, 0.0), 15.0);
    word |= (uint32_t)q << (4 * e);
  }
  if (!live) return;
  wq[idx] = word;
  if ((j & (G / 8 - 1)) == 0) {
    const long long g = row * (d_in / G) + (8 * j) / G;
    scales[g] = (uint16_t)s_bits;
    zeros[g] = (uint16_t)act16_round<ACT_F16>(z);
  }
}

__device__ inline uint32_t load_prepared_word(const PreparedView& v, int row, int k) {
  const int lane = (row & 15) + 16 * ((k >> 3) & 3);
  const int j = (k >> 5) & 3;
  return tile_record(v, row >> 4, k >> 7)[lane * 4 + j];
}

__device__ inline uint32_t load_prepared_sz(const PreparedView& v, int row, int k, int G) {
  return tile_record(v, row >> 4, k >> 7)[256 + 16 * ((k & 127) / G) + (row & 15)];
}

// one thread per (row, 8 channels)
__global__ void k_debug_unpack(const void* prepared, int d_out, int d_in, int G,
                               uint8_t* __restrict__ q_out) {
  long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  int words = d_in / 8;
  if (idx >= (long long)d_out * words) return;
  int row = (int)(idx / words), k = (int)(idx % words) * 8;
  PreparedView v = prepared_view(prepared, d_out, d_in, G);
  uint32_t w = load_prepared_word(v, row, k);
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    lo |= prepared_nibble(w, e) << (8 * e);
    hi |= prepared_nibble(w, e + 4) << (8 * e);
  }
  uint2* dst = (uint2*)(q_out + (long long)row * d_in + k);
  *dst = make_uint2(lo, hi);
}

template <int ACT>
__global__ void k_debug_dequant(const void* prepared, int d_out, int d_in, int G,
                                uint16_t* __restrict__ w_out) {
  long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  int words = d_in / 8;
  if (idx >= (long long)d_out * words) return;
  int row = (int)(idx / words), k = (int)(idx % words) * 8;
  PreparedView v = prepared_view(prepared, d_out, d_in, G);
  uint32_t w = load_prepared_word(v, row, k);
  GroupConst<ACT> g;
  g.set(load_prepared_sz(v, row, k, G));
  u32x4_t d = dequant_word<ACT>(w, g);
  *(u32x4_t*)(w_out + (long long)row * d_in + k) = d;
}

// The sums behind the scores, one launch: the leading workgroups take tile records of all modules (Eq. 11: sum of
// (W - What)^2 and of W^2, What the stored weight widened from the activation type), the next ones 128 rows of an A_i each
// (column energies), the last ones a row of B each.  The workgroup that finds all others counted makes the scores of
// the sums.  One wave per (tile record, word index j): lane l holds row l & 15, channels 32 j + 8 (l >> 4) .. + 8,
// so a wave reads 16 rows x 128 contiguous bytes of the fp32 weights (the bytes that matter: 4 of 4.6 per
// weight); four records are asked for together, since a record by itself leaves a workgroup waiting for memory most of
// the time.  5120 rows of 3072, r = 64: 101 us as eight launches behind one another (a record at a time), now 26 and the fill.
// scratch: pairs {error energy, weight energy} of IM_SLOTS groups of workgroups (so that few atomic adds meet at a sum),
// column energies of A, row energies of B, count of workgroups.
constexpr int IM_SLOTS = 32, IM_COL = 2 * IM_SLOTS, IM_ROW = IM_COL + GLOWQ_MAX_RANK, IM_COUNT = IM_ROW + GLOWQ_MAX_RANK;
static_assert((IM_COUNT + 1) * 8 <= GLOWQ_IMPORTANCE_SCRATCH_BYTES, "the sums fit the scratch");
constexpr int IM_RECS = 4, IM_ROWS = 128;         // records per turn; rows of A per workgroup

struct ImportanceArgs {
  const float* W[GLOWQ_MAX_MODULES];
  const uint32_t* prepared[GLOWQ_MAX_MODULES];
  const uint16_t* A[GLOWQ_MAX_MODULES];
  int d_out[GLOWQ_MAX_MODULES], rec_start[GLOWQ_MAX_MODULES], col_start[GLOWQ_MAX_MODULES], n_modules;
  const uint16_t* B;
  int d_in, G, r, n_recs, n_energy, n_cols;       // workgroups of the first two kinds
  double* scratch;
  double* scores;
};

// sum over the workgroup (256 threads); thread 0 has it
__device__ inline double block_sum256(double v, double* lds4) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = v;
  __syncthreads();
  return (lds4[0] + lds4[1]) + (lds4[2] + lds4[3]);
}

template <int ACT>
__global__ void __launch_bounds__(256) k_importance(ImportanceArgs a) {
  __shared__ double part[256 * 9], four[4];
  __shared__ int last;
  const int t = threadIdx.x, wg = blockIdx.x;
  if (wg < a.n_energy) {
    const int j = t >> 6, lane = t & 63, ktiles = a.d_in >> 7, rec_words = prepared_rec_words(a.G);
    double e = 0.0, ww = 0.0;
    for (int rec0 = wg * IM_RECS; rec0 < a.n_recs; rec0 += a.n_energy * IM_RECS) {
      float4_t w0[IM_RECS], w1[IM_RECS];
      uint32_t word[IM_RECS], sz[IM_RECS];
      bool live[IM_RECS];
#pragma unroll
      for (int q = 0; q < IM_RECS; ++q) {
        const int all = min(rec0 + q, a.n_recs - 1);
        int mi = 0;
#pragma unroll
        for (int m = 1; m < GLOWQ_MAX_MODULES; ++m)
          if (m < a.n_modules && all >= a.rec_start[m]) mi = m;
        const int rec = all - a.rec_start[mi], rb = rec / ktiles, kt = rec - rb * ktiles;
        const int row = rb * 16 + (lane & 15), k = kt * 128 + 32 * j + 8 * (lane >> 4);
        live[q] = rec0 + q < a.n_recs && row < a.d_out[mi];
        const float4_t* src = (const float4_t*)(a.W[mi] + (long long)min(row, a.d_out[mi] - 1) * a.d_in + k);
        w0[q] = __builtin_nontemporal_load(src);
        w1[q] = __builtin_nontemporal_load(src + 1);
        const uint32_t* r = a.prepared[mi] + (long long)rec * rec_words;
        word[q] = r[lane * 4 + j];
        sz[q] = r[256 + 16 * ((k & 127) / a.G) + (row & 15)];
      }
#pragma unroll
      for (int q = 0; q < IM_RECS; ++q) {
        GroupConst<ACT> g;
        g.set(sz[q]);
        const u32x4_t d = dequant_word<ACT>(word[q], g);
        const float w[8] = {w0[q][0], w0[q][1], w0[q][2], w0[q][3], w1[q][0], w1[q][1], w1[q][2], w1[q][3]};
        if (live[q]) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t pair = d[i >> 1];
            const double x = (double)w[i], err = x - act16_value<ACT>((i & 1) ? (pair >> 16) : (pair & 0xffffu));
            e += err * err;
            ww += x * x;
          }
        }
      }
    }
    e = block_sum256(e, four);
    ww = block_sum256(ww, four);
    if (t == 0) {
      atomicAdd(&a.scratch[2 * (wg % IM_SLOTS)], e);
      atomicAdd(&a.scratch[2 * (wg % IM_SLOTS) + 1], ww);
    }
  } else if (wg < a.n_energy + a.n_cols) {
    const int at = wg - a.n_energy;
    int mi = 0;
#pragma unroll
    for (int m = 1; m < GLOWQ_MAX_MODULES; ++m)
      if (m < a.n_modules && at >= a.col_start[m]) mi = m;
    // eight ranks per thread, as many rows at once as that leaves
    const int pieces = a.r >> 3, rows = 256 / pieces, piece = t % pieces, sub = t / pieces;
    const int o0 = (at - a.col_start[mi]) * IM_ROWS, o1 = min(a.d_out[mi], o0 + IM_ROWS);
    double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (sub < rows) {
#pragma unroll 4
      for (int o = o0 + sub; o < o1; o += rows) {
        const u32x4_t v = *(const u32x4_t*)(a.A[mi] + (long long)o * a.r + 8 * piece);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t pair = v[i >> 1];
          const double x = act16_value<ACT>((i & 1) ? (pair >> 16) : (pair & 0xffffu));
          s[i] += x * x;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) part[t * 9 + i] = s[i];
    __syncthreads();
    if (t < a.r) {
      double sum = 0.0;
      for (int q = 0; q < rows; ++q) sum += part[(q * pieces + (t >> 3)) * 9 + (t & 7)];
      atomicAdd(&a.scratch[IM_COL + t], sum);
    }
  } else {
    const int j = wg - a.n_energy - a.n_cols;
    double s = 0.0;
    for (int k = 8 * t; k < a.d_in; k += 2048) {
      const u32x4_t v = *(const u32x4_t*)(a.B + (long long)j * a.d_in + k);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t pair = v[i >> 1];
        const double x = act16_value<ACT>((i & 1) ? (pair >> 16) : (pair & 0xffffu));
        s += x * x;
      }
    }
    s = block_sum256(s, four);
    if (t == 0) atomicAdd(&a.scratch[IM_ROW + j], s);
  }
  // the sums are out, then the workgroup is counted
  vm_wait<0>();
  __syncthreads();
  if (t == 0) last = __hip_atomic_fetch_add((int*)&a.scratch[IM_COUNT], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  // scores[0] = g_ner, scores[1] = g_ec: the balanced factors have orthogonal columns / rows with
  // ||a_j||^2 = ||b_j||^2 = sigma_j (Eqs. A.1.9a-b), so sum_j ||a_j||^2 ||b_j||^2 is the captured energy sum_j sigma_j^2
  auto sum_at = [&](int i) { return __hip_atomic_load(a.scratch + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  part[t] = t < 2 * IM_SLOTS ? sum_at(t) : 0.0;
  part[256 + t] = t < a.r ? sum_at(IM_COL + t) * sum_at(IM_ROW + t) : 0.0;
  __syncthreads();
  if (t != 0) return;
  double e = 0.0, w = 0.0, cap = 0.0;
  for (int i = 0; i < IM_SLOTS; ++i) {
    e += part[2 * i];
    w += part[2 * i + 1];
  }
  for (int j = 0; j < a.r; ++j) cap += part[256 + j];
  a.scores[0] = w > 0.0 ? e / w : 0.0;
  a.scores[1] = e > 0.0 ? cap / e : 0.0;
}

hipError_t launch_importance(const glowq_unit& u, const float* const* W_modules, double* scratch,
                             double* scores, hipStream_t st) {
  hipError_t err = launch_fill_zero(scratch, GLOWQ_IMPORTANCE_SCRATCH_BYTES, st);
  if (err != hipSuccess) return err;
  ImportanceArgs a = {};
  a.n_modules = u.n_modules;
  for (int i = 0; i < u.n_modules; ++i) {
    const glowq_module& m = u.modules[i];
    a.W[i] = W_modules[i];
    a.prepared[i] = (const uint32_t*)m.w_prepared;
    a.A[i] = (const uint16_t*)m.A;
    a.d_out[i] = m.d_out;
    a.rec_start[i] = a.n_recs;
    a.col_start[i] = a.n_cols;
    a.n_recs += (m.d_out + 15) / 16 * (u.d_in / 128);
    if (u.r > 0) a.n_cols += (m.d_out + IM_ROWS - 1) / IM_ROWS;
  }
  a.B = (const uint16_t*)u.B;
  a.d_in = u.d_in;
  a.G = u.group_size;
  a.r = u.r;
  const int turns = (a.n_recs + IM_RECS - 1) / IM_RECS;
  a.n_energy = turns < 1024 ? turns : 1024;
  a.scratch = scratch;
  a.scores = scores;
  const dim3 grid((unsigned)(a.n_energy + a.n_cols + u.r)), block(256);
  if (u.act_dtype == GLOWQ_F16) k_importance<ACT_F16><<<grid, block, 0, st>>>(a);
  else k_importance<ACT_BF16><<<grid, block, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_prepare(const uint32_t* wq, const uint16_t* scales, const uint16_t* zeros,
                          int d_out, int d_in, int G, void* prepared, hipStream_t st) {
  long long n_words = (long long)(prepared_total_bytes(d_out, d_in, G) / 4);
  k_prepare<<<dim3((unsigned)((n_words + 255) / 256)), dim3(256), 0, st>>>(
      wq, scales, zeros, (uint32_t*)prepared, d_out, d_in, G, n_words);
  return hipGetLastError();
}

hipError_t launch_quantize_rtn(const float* W, int d_out, int d_in, int G, uint32_t* wq, uint16_t* scales,
                               uint16_t* zeros, hipStream_t st) {
  const long long n = (long long)d_out * (d_in / 8);
  k_quantize_rtn<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(W, d_out, d_in, G, wq, scales, zeros);
  return hipGetLastError();
}

hipError_t launch_debug_unpack(const void* prepared, int d_out, int d_in, int G, uint8_t* q_out,
                               hipStream_t st) {
  long long n = (long long)d_out * (d_in / 8);
  k_debug_unpack<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(prepared, d_out, d_in,
                                                                          G, q_out);
  return hipGetLastError();
}

hipError_t launch_debug_dequant(const void* prepared, int d_out, int d_in, int G, int act,
                                void* w_out, hipStream_t st) {
  long long n = (long long)d_out * (d_in / 8);
  dim3 grid((unsigned)((n + 255) / 256)), block(256);
  if (act == ACT_F16)
    k_debug_dequant<ACT_F16><<<grid, block, 0, st>>>(prepared, d_out, d_in, G, (uint16_t*)w_out);
  else
    k_debug_dequant<ACT_BF16><<<grid, block, 0, st>>>(prepared, d_out, d_in, G, (uint16_t*)w_out);
  return hipGetLastError();
}

}  // namespace glowq

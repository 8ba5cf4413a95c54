// Batched decode and prompts on few or small tiles (more than four tokens, see BATCH_MAX_T):
// Y_i = X dequant(W_q,i)^T + R A_i^T  (paper Eq. 9), R = X B^T (Eq. 8) in the same launch.
//
// What bounds it: the packed weights come from memory once, but with this many tokens the
// activations travel too (T x 256 bytes per 128 channels against 1088 bytes per 16 rows), and a
// weight costs about as many vector-ALU cycles to dequantise as the memory needs to deliver
// it.  Hence:
//  - a workgroup's row waves share one copy of X: each K tile of X (128 channels) is staged
//    in LDS by direct loads, already in operand order (every lane fetches the 16 bytes that
//    the same lane of the matrix instruction holds), so that LDS is written and read 1 KiB
//    lane after lane;
//  - weights and scales take the same way, so that no register holds data in flight: the
//    kernel fits three to four workgroups per compute unit, and a ring of DEPTH K tiles keeps
//    two or three tiles per wave on their way;
//  - all waits are placed by hand (loads of a wave complete in issue order, every stage
//    issues the same number of them), one barrier per K tile;
//  - units of one call share a launch, longest contraction first.
// Four or eight waves per workgroup: RW of them take RB 16-row blocks each, and NW / RW groups share
// the contraction (their sums meet in LDS at the end).  The tile is chosen per launch from the
// units' sizes (choose_batch_tile).
// Measured against one launch per unit with X in registers (up to 32 tokens: 256 registers, one
// wave per SIMD with two token blocks) and against 128- and 64-token tiles of 256 rows beyond: a
// layer of 4096 / 1024 / 14336 at 24 tokens, r = 128, 102 -> 48 us (2.9 TB/s of weights and
// activations); 2 x 14336 rows x 4096 at 8 tokens, bfloat16, 25.5 -> 18.0 us (3.9 TB/s); four
// layers of 1536 / 384 / 6912 at 17 tokens 191 -> 26 us; 3 x 960 rows x 5888 at 124 tokens
// 82 -> 19 us.
//
// The projection workgroups lead the grid: (16-token block, K slice, 32 ranks).  Slices are
// published as self-validating 8-byte slots {fp32, launch tag}; whoever finds them complete
// adds them in slice order, rounds to the activation type and publishes R as slots {two
// 16-bit values, launch tag}, so that a consumer gathers 4 bytes per element of R instead
// of 8 per element and slice.  (With the slices gathered by every consumer, T = 24 at rank 128
// moved 98 KB of device-scope loads per workgroup; a small R is gathered that way all the same, see
// plan_batch_projection.)
#pragma once
#include "arrivals.hpp"
#include "common.hpp"
#include "decode_device.hpp"
#include "proj_device.hpp"
#include "launch.hpp"
#include <algorithm>
#include <cmath>

namespace glowq {

constexpr int BATCH_MAX_UNITS = 16;
constexpr int BATCH_MAX_SLICES = 4;      // of K, across workgroups
static_assert(BATCH_MAX_SLICES < 1 << ARRIVAL_BITS, "a count of slices");
constexpr int BATCH_QUICK_POLLS = 64;    // looks at R with hardly a pause in between
constexpr int BATCH_WB = 1024 + 256;      // bytes per wave and K tile: one record's words, its (s, z) words

struct BatchUnit {
  ModuleArgs mod[GLOWQ_MAX_MODULES];
  const uint16_t* X;
  const uint16_t* B;
  float* part;                 // slots {fp32, tag}: (t ksplit + slice) r + rank
  uint32_t* rslots;            // slots {two ranks, tag}: t r / 2 + rank pair
  Control* ctl;
  int T, K, r, n_modules;
  int n_blocks;                // 16-row blocks of the unit
  int n_groups, n_ttiles;      // its tiles: groups of row blocks x tiles of 16 MB tokens
  int ks;                      // K slices: as many workgroups per tile (see choose_batch_tile)
  unsigned long long* count;   // ks > 1: per tile, slices that are done (see arrivals.hpp); their partial results
  u32x4_t* slab;               // [slice][tile][row wave][row block][token block][lane]
  int restore, out_f32;        // restore 2: the consumers add the projection's slices (see plan_batch_projection)
  int ksplit, kslice;          // K slices of the projection
  int prod_start, n_prod;      // this unit's projection workgroups
  int wg_start;                // first row-block workgroup
};
template <int NB> struct BatchArgs {
  BatchUnit u[NB];
  int n, n_prod;               // units; projection workgroups of all units (they lead the grid)
};

__device__ inline const ModuleArgs& find_batch_module(const BatchUnit& u, int blk) {
  int mi = 0;
#pragma unroll
  for (int i = 1; i < GLOWQ_MAX_MODULES; ++i)
    if (i < u.n_modules && blk >= u.mod[i].blk_start) mi = i;
  return u.mod[mi];
}

// direct global -> LDS loads with a scalar base and a 32-bit lane offset (see lds_dma16)
__device__ inline void lds_dma16_s(const void* base, uint32_t off, uint32_t lds_base) {
  const uint32_t m = __builtin_amdgcn_readfirstlane(lds_base);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               : : "v"(off), "s"(base), "s"(m) : "memory", "m0");
}
__device__ inline void lds_dma4_s(const void* base, uint32_t off, uint32_t lds_base) {
  const uint32_t m = __builtin_amdgcn_readfirstlane(lds_base);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               : : "v"(off), "s"(base), "s"(m) : "memory", "m0");
}
template <typename T> __device__ inline T* scalar_ptr(T* p) {
  const unsigned long long v = (unsigned long long)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (T*)(((unsigned long long)hi << 32) | lo);
}

// One projection workgroup (see proj_sliced): R as slots {two ranks, tag}.
template <int ACT, int NW>
__device__ inline void batch_projection(const BatchUnit& u, int local, float* lds) {
  const ProjSliced p{u.X, u.B, u.part, u.T, u.K, u.r, u.ksplit, u.kslice, u.restore == 2};
  proj_sliced<ACT, NW>(p, local, lds, [&](int t, int rank, uint32_t pair, uint32_t tag) {
    __hip_atomic_store((unsigned long long*)u.rslots + (size_t)t * (u.r >> 1) + (rank >> 1),
                       ((unsigned long long)tag << 32) | pair, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  });
}

// look(): one look of the whole workgroup at R, true where all that this thread saw was of this
// launch; repeated until that holds for every thread.  False (in every thread) if the bounded wait
// expired: the status word is set and the correction left out.
template <class LOOK> __device__ inline bool batch_poll_r(const BatchUnit& u, uint32_t* flag, LOOK look) {
  const int tid = threadIdx.x;
  if (tid == 0) *flag = 0u;
  __syncthreads();
  for (int spin = 0; spin < R_WAIT_POLLS; ++spin) {
    if (!look()) *flag = 1u;
    __syncthreads();
    const bool failed = *flag != 0u;
    if (!failed) return true;
    __syncthreads();
    if (tid == 0) *flag = 0u;
    // (short pauses at first: in the smallest calls R comes while the consumers already look for it,
    // and a pause of a microsecond between two looks cost half of one: 7.1 -> 6.4 us)
    if (spin < BATCH_QUICK_POLLS) __builtin_amdgcn_s_sleep(1);
    else __builtin_amdgcn_s_sleep(32);
    __syncthreads();
  }
  if (tid == 0) atomicOr(&u.ctl->status, 1u);
  return false;
}

// R of the tokens tok0 .. tok0 + n_tok into LDS (act dtype [n_tok][r]), gathered by the whole
// workgroup.  Two loops, so that the descriptor's words that only one of them needs are not loaded
// on the other's way (0.1 us of every call).
template <int ACT, int NT>
__device__ inline bool batch_fetch_r(const BatchUnit& u, bool gather, int tok0, int n_tok, uint32_t* r_lds, uint32_t* flag) {
  const int tid = threadIdx.x;
  const uint32_t tag = (uint32_t)(launch_tag() & 0xffffffffull);
  if (gather)
    return batch_poll_r(u, flag, [&] {
      // a pair of ranks of every slice per thread, added in slice order
      bool ok = true;
      const int hp = u.r >> 1, n_pairs = n_tok * hp;
      for (int el = tid; el < n_pairs; el += NT) {
        const int tok = el / hp;
        const u32x4_t* q = (const u32x4_t*)u.part + (size_t)(tok0 + tok) * u.ksplit * hp + (el - tok * hp);
        u32x4_t v[4];
        load4_device(v, q, q + min(1, u.ksplit - 1) * hp, q + min(2, u.ksplit - 1) * hp, q + (u.ksplit - 1) * hp);
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const uint32_t w0 = v[p][0], t0 = v[p][1], w1 = v[p][2], t1 = v[p][3];
          ok = ok && t0 == tag && t1 == tag;
          if (p < u.ksplit) {
            s0 += __builtin_bit_cast(float, w0);
            s1 += __builtin_bit_cast(float, w1);
          }
        }
        r_lds[el] = (uint32_t)to_act16<ACT>(s0) | ((uint32_t)to_act16<ACT>(s1) << 16);
      }
      return ok;
    });
  const int n_el = n_tok * (u.r >> 2);           // 16-byte units: two slots, four ranks
  const u32x4_t* src = (const u32x4_t*)u.rslots + (size_t)tok0 * (u.r >> 2);
  return batch_poll_r(u, flag, [&] {
    bool ok = true;
    for (int e0 = 0; e0 < n_el; e0 += 4 * NT) {
      u32x4_t v[4];
      load4_device(v, src + min(e0 + tid, n_el - 1), src + min(e0 + NT + tid, n_el - 1),
                   src + min(e0 + 2 * NT + tid, n_el - 1), src + min(e0 + 3 * NT + tid, n_el - 1));
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int el = e0 + k * NT + tid;
        const uint32_t w0 = v[k][0], t0 = v[k][1], w1 = v[k][2], t1 = v[k][3];
        ok = ok && t0 == tag && t1 == tag;
        if (el < n_el) {
          r_lds[2 * el] = w0;
          r_lds[2 * el + 1] = w1;
        }
      }
    }
    return ok;
  });
}

// bfloat16 weights of one word in 17 instructions (see DequantLockstep<ACT_BF16>)
__device__ inline u32x4_t dequant_word_mix(uint32_t w, float s, float c1024, float c64) {
  using D = DequantLockstep<ACT_BF16, 1>;
  const u32x4_t f = nibble_forms_f16(w);
  u32x4_t out;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t fi = f[i];
    const float c = (i & 1) ? c64 : c1024;
    bf16x2_t v;
    v[0] = (__bf16)D::mix<0>(fi, s, c);
    v[1] = (__bf16)D::mix<1>(fi, s, c);
    out[i] = __builtin_bit_cast(uint32_t, v);
  }
  return out;
}

// RB records against MB blocks of 16 tokens.  EXACT (binary16, calls of up to 32 tokens): the
// exact (q - z) are multiplied and the group's fp32 sum is scaled (see decode_tile); with more
// tokens the scaling of the sums would cost more than the rounding multiply of the weights.
template <int ACT, int MB, int RB, bool EXACT, bool G128, class XF>
__device__ inline void batch_tile(const u32x4_t (&w)[RB], const uint32_t (&sz)[RB][2], XF xfrag, float4_t (&acc)[RB][MB]) {
  if constexpr (EXACT) {
#pragma unroll
    for (int b = 0; b < RB; ++b) decode_tile<ACT, MB, G128>(w[b], sz[b][0], sz[b][1], xfrag, acc[b]);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      u32x4_t wf[RB];
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        GroupConst<ACT> g;
        g.set(sz[b][(G128 || j < 2) ? 0 : 1]);
        const uint32_t wj = w[b][j];
        if constexpr (ACT == ACT_BF16) wf[b] = dequant_word_mix(wj, g.s, g.c1024(), g.c64());
        else wf[b] = dequant_word<ACT>(wj, g);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const u32x4_t xf = xfrag(mb, j);
#pragma unroll
        for (int b = 0; b < RB; ++b) acc[b][mb] = mfma16<ACT>(wf[b], xf, acc[b][mb]);   // D[row][token]
      }
    }
  }
}

template <int MB, int RB, int RW, int NW> struct BatchShape {
  static constexpr int KS = NW / RW;                               // groups that share the contraction
  static constexpr int DEPTH = (KS == 1 && MB <= 2) ? 4 : 3;       // K tiles in the ring
  static constexpr int XB = MB * 4096;                             // bytes of X per group and K tile
  static constexpr int STAGE = KS * XB + NW * RB * BATCH_WB;
  static constexpr int XL = 4 * MB / RW;                           // X loads per wave and K tile
  static constexpr int LOADS = XL + 2 * RB;                        // all loads per wave and K tile
  static constexpr int LDS = DEPTH * STAGE;
  static constexpr int WGS = LDS <= 40960 ? 4 : LDS <= 54613 ? 3 : LDS <= 81920 ? 2 : 1;   // per compute unit
  static constexpr int WAVES_EU = WGS * NW / 4;
  static_assert(MB * 4096 + (KS - 1) * RW * RB * MB * 1024 <= LDS, "R and the fold fit the ring");
};

// CUT: some unit's contraction is cut across workgroups (a launch without one runs the code without any of it: with it
// 2 x 14336 rows x 4096 at 8 tokens, bfloat16, took 17.9 instead of 17.7 us).
template <int ACT, int MB, int RB, int RW, int NW, bool EXACT, bool G128, bool CUT, int NB>
__global__ void __launch_bounds__(NW * 64, (BatchShape<MB, RB, RW, NW>::WAVES_EU)) k_decode_batch(BatchArgs<NB> b) {
  using S = BatchShape<MB, RB, RW, NW>;
  __shared__ __attribute__((aligned(1024))) char ring[S::LDS];
  __shared__ uint32_t flag;
  if ((int)blockIdx.x < b.n_prod) {
    int ui = 0;
#pragma unroll
    for (int i = 1; i < NB; ++i)
      if (i < b.n && b.u[i].n_prod > 0 && (int)blockIdx.x >= b.u[i].prod_start) ui = i;
    batch_projection<ACT, NW>(b.u[ui], (int)blockIdx.x - b.u[ui].prod_start, (float*)ring);
    return;
  }
  int ui = 0;
#pragma unroll
  for (int i = 1; i < NB; ++i)
    if (i < b.n && (int)blockIdx.x >= b.u[i].wg_start) ui = i;
  const BatchUnit& u = b.u[ui];
  int grp = (int)blockIdx.x - u.wg_start, tok0 = 0, sl = 0;
  const int ks = CUT ? u.ks : 1, n_tiles = u.n_groups * u.n_ttiles;
  int sk0 = 0, span = u.K >> 7;                   // the slice's K tiles (the divisions stay off whole contractions' way)
  if (CUT && ks > 1) {
    sl = grp / n_tiles;
    grp -= sl * n_tiles;
    sk0 = (u.K >> 7) * sl / ks;
    span = (u.K >> 7) * (sl + 1) / ks - sk0;
  }
  const int tile = grp;
  if (u.n_ttiles > 1) {
    // workgroups go to the eight XCDs round robin: residue class c takes the c-th eighth of the
    // list (token tile fastest), so that the token tiles of a row group share an L2
    const int c = grp & 7, t = c * (n_tiles >> 3) + min(c, n_tiles & 7) + (grp >> 3);
    grp = t / u.n_ttiles;
    tok0 = (t - grp * u.n_ttiles) * 16 * MB;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, kq = lane >> 4;
  const int rw = wave % RW, kg = wave / RW;
  constexpr int REC = G128 ? 1088 : 1152;        // bytes per tile record
  const int ktiles = u.K >> 7, T = u.T, K = u.K;
  const int kt0 = sk0 + span * kg / S::KS, nkt = sk0 + span * (kg + 1) / S::KS - kt0;
  const int n_st = (span + S::KS - 1) / S::KS;    // every group runs this many stages

  // this wave's 16-row blocks; past the unit's last one: that one again, not stored
  const int blk0 = (grp * RW + rw) * RB;
  const char* wsrc[RB];
#pragma unroll
  for (int b_ = 0; b_ < RB; ++b_) {
    const int blk = min(blk0 + b_, u.n_blocks - 1);
    const ModuleArgs& M = find_batch_module(u, blk);
    wsrc[b_] = scalar_ptr((const char*)M.rec + ((size_t)(blk - M.blk_start) * ktiles + kt0) * REC);
  }
  const char* xsrc = scalar_ptr((const char*)u.X + (size_t)kt0 * 256);
  // X: LDS chunk c = 4 mb + j holds, lane after lane, X[tok0 + 16 mb + n][32 j + 8 kq .. + 8]
  uint32_t xoff[S::XL];
#pragma unroll
  for (int i = 0; i < S::XL; ++i) {
    const int c = rw + RW * i;
    xoff[i] = (uint32_t)min(tok0 + 16 * (c >> 2) + n, T - 1) * (uint32_t)K * 2u + (uint32_t)((c & 3) * 64 + kq * 16);
  }
  const uint32_t szoff = 1024u + 4u * (uint32_t)(lane & (G128 ? 15 : 31));
  const uint32_t ring_lds = lds_address(ring);
  const uint32_t x_lds = ring_lds + (uint32_t)(kg * S::XB), w_lds = ring_lds + (uint32_t)(S::KS * S::XB + wave * RB * BATCH_WB);
  auto issue = [&](int st, int slot) {
    // (past the end: the last tile again, into a slot nobody reads; a group without a tile of its
    // own, possible when K has fewer tiles than groups, reads the next group's first one)
    const int k = max(min(st, nkt - 1), 0);
    const uint32_t so = (uint32_t)(slot * S::STAGE);
    const char* xk = scalar_ptr(xsrc + (ptrdiff_t)k * 256);
#pragma unroll
    for (int b_ = 0; b_ < RB; ++b_) {
      const char* wk = scalar_ptr(wsrc[b_] + (ptrdiff_t)k * REC);
      lds_dma16_s(wk, (uint32_t)lane * 16u, w_lds + so + (uint32_t)(b_ * BATCH_WB));
      lds_dma4_s(wk, szoff, w_lds + so + (uint32_t)(b_ * BATCH_WB + 1024));
    }
#pragma unroll
    for (int i = 0; i < S::XL; ++i) lds_dma16_s(xk, xoff[i], x_lds + so + (uint32_t)(rw + RW * i) * 1024u);
  };

  float4_t acc[RB][MB];
#pragma unroll
  for (int b_ = 0; b_ < RB; ++b_)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[b_][mb] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < S::DEPTH - 1; ++s) issue(s, s);
  int slot = 0, slot_new = S::DEPTH - 1;
  for (int st = 0; st < n_st; ++st) {
    // this stage's loads have landed (the ones of the DEPTH - 2 younger stages may be on their
    // way) and so, behind the barrier, have everybody's; everybody is done with the slot that
    // is loaded next (no LDS read of a wave is pending when it arrives here)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((S::DEPTH - 2) * S::LOADS) : "memory");
    issue(st + S::DEPTH - 1, slot_new);
    if (S::KS == 1 || st < nkt) {
      const char* base = ring + slot * S::STAGE;
      const char* ws = base + S::KS * S::XB + wave * RB * BATCH_WB;
      const char* xs = base + kg * S::XB + lane * 16;
      u32x4_t w[RB];
      uint32_t sz[RB][2];
#pragma unroll
      for (int b_ = 0; b_ < RB; ++b_) {
        w[b_] = *(const u32x4_t*)(ws + b_ * BATCH_WB + lane * 16);
        sz[b_][0] = *(const uint32_t*)(ws + b_ * BATCH_WB + 1024 + n * 4);
        sz[b_][1] = G128 ? sz[b_][0] : *(const uint32_t*)(ws + b_ * BATCH_WB + 1088 + n * 4);
      }
      batch_tile<ACT, MB, RB, EXACT, G128>(w, sz, [&](int mb, int j) { return *(const u32x4_t*)(xs + (mb * 4 + j) * 1024); }, acc);
    }
    slot = slot == S::DEPTH - 1 ? 0 : slot + 1;
    slot_new = slot_new == S::DEPTH - 1 ? 0 : slot_new + 1;
  }
  // nothing may be on its way into LDS any more, and everybody is done reading it
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

  const int restore = sl == 0 ? u.restore : 0;   // (the first slice carries the correction)
  if (restore) {                                 // uniform; r > 0
    const int r = u.r, n_tok = min(T - tok0, 16 * MB);
    u32x4_t af[RB][4];
#pragma unroll
    for (int b_ = 0; b_ < RB; ++b_) {
      const int blk = min(blk0 + b_, u.n_blocks - 1);
      const ModuleArgs& M = find_batch_module(u, blk);
      const int row = min((blk - M.blk_start) * 16 + n, M.d_out - 1);
#pragma unroll
      for (int s = 0; s < 4; ++s) {              // correction steps of 32 ranks, dealt to the groups
        const int j0 = 32 * s + 8 * kq;
        af[b_][s] = u32x4_t{0u, 0u, 0u, 0u};
        if (s % S::KS == kg && j0 < r) af[b_][s] = *(const u32x4_t*)(M.A + (size_t)row * r + j0);
      }
    }
    uint32_t* r_lds = (uint32_t*)ring;
    if (batch_fetch_r<ACT, NW * 64>(u, restore == 2, tok0, n_tok, r_lds, &flag)) {
      const uint16_t* R = (const uint16_t*)r_lds;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (s % S::KS == kg && 32 * s < r) {     // uniform per wave
          const int j0 = 32 * s + 8 * kq;
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            // (ranks past r: zero on both sides; tokens past T: never stored)
            u32x4_t rf = u32x4_t{0u, 0u, 0u, 0u};
            if (j0 < r && 16 * mb + n < n_tok) rf = *(const u32x4_t*)(R + (size_t)(16 * mb + n) * r + j0);
#pragma unroll
            for (int b_ = 0; b_ < RB; ++b_)
              acc[b_][mb] = EXACT ? mfma16<ACT>(rf, af[b_][s], acc[b_][mb]) : mfma16<ACT>(af[b_][s], rf, acc[b_][mb]);
          }
        }
      }
    }
  }
  if constexpr (S::KS > 1) {
    // the groups' sums meet in LDS (behind R), added in group order
    float4_t* fold = (float4_t*)(ring + MB * 4096);
    auto at = [&](int g, int b_, int mb) -> float4_t& { return fold[(((g * RW + rw) * RB + b_) * MB + mb) * 64 + lane]; };
    if (kg > 0) {
#pragma unroll
      for (int b_ = 0; b_ < RB; ++b_)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) at(kg - 1, b_, mb) = acc[b_][mb];
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll
      for (int g = 1; g < S::KS; ++g)
#pragma unroll
        for (int b_ = 0; b_ < RB; ++b_)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            const float4_t o = at(g - 1, b_, mb);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[b_][mb][v] += o[v];
          }
    } else if (ks == 1) {
      return;
    }
  }
  if (CUT && ks > 1) {
    // The slice's sums go past the L2s to the unit's slab and the workgroup is counted (the word carries the
    // launch's tag); whoever finds all others counted adds the slices in their order.
    constexpr int PIECES = RW * RB * MB * 64;
    u32x4_t* mine = u.slab + (size_t)tile * PIECES + rw * (RB * MB * 64) + lane;
    const size_t step = (size_t)n_tiles * PIECES;
    if (kg == 0) {
#pragma unroll
      for (int b_ = 0; b_ < RB; ++b_)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) store16_device(mine + sl * step + (b_ * MB + mb) * 64, __builtin_bit_cast(u32x4_t, acc[b_][mb]));
    }
    unsigned long long* word = u.count + tile;
    unsigned long long seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // (on its way with the stores)
    vm_wait<0>();
    __syncthreads();
    if (threadIdx.x == 0) {
      const unsigned long long key = arrival_key(launch_tag());
      uint32_t done;
      do done = arrivals(seen, key);                         // (at most ks rounds: a failure is another slice's success)
      while (!__hip_atomic_compare_exchange_strong(word, &seen, key | (done + 1u), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT));
      flag = done;
    }
    __syncthreads();
    if (flag + 1u != (uint32_t)ks || kg > 0) return;
    // (all slices' values of a block in flight together)
#pragma unroll
    for (int b_ = 0; b_ < RB; ++b_)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        unsigned long long v[BATCH_MAX_SLICES][2];
#pragma unroll
        for (int p = 0; p < BATCH_MAX_SLICES; ++p) {
          const unsigned long long* q = (const unsigned long long*)(mine + min(p, ks - 1) * step + (b_ * MB + mb) * 64);
          v[p][0] = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          v[p][1] = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        acc[b_][mb] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < BATCH_MAX_SLICES; ++p)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = __builtin_bit_cast(float, (uint32_t)(v[p][e >> 1] >> (32 * (e & 1))));
            acc[b_][mb][e] += p < ks ? x : 0.f;
          }
      }
  }
#pragma unroll
  for (int b_ = 0; b_ < RB; ++b_) {
    const int blk = blk0 + b_;
    if (blk >= u.n_blocks) break;
    const ModuleArgs& M = find_batch_module(u, blk);
    const int row0 = (blk - M.blk_start) * 16;
    if constexpr (EXACT) {
      // lane holds row n and tokens 16 mb + 4 kq + v
      if (row0 + n >= M.d_out) continue;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int t = tok0 + 16 * mb + 4 * kq + v;
          if (t < T) {
            const size_t off = (size_t)t * M.ldy + row0 + n;
            const float s = acc[b_][mb][v];
            if (u.out_f32) ((float*)M.Y)[off] = s;
            else ((uint16_t*)M.Y)[off] = to_act16<ACT>(s);
          }
        }
    } else {
      // lane holds rows 4 kq .. + 4 and token 16 mb + n
      if (row0 + 4 * kq >= M.d_out) continue;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int t = tok0 + 16 * mb + n;
        if (t < T) {
          const size_t off = (size_t)t * M.ldy + row0 + 4 * kq;
          const float4_t v = acc[b_][mb];
          if (u.out_f32) {
            *(float4_t*)((float*)M.Y + off) = v;
          } else {
            uint2 pk;
            pk.x = (uint32_t)to_act16<ACT>(v[0]) | ((uint32_t)to_act16<ACT>(v[1]) << 16);
            pk.y = (uint32_t)to_act16<ACT>(v[2]) | ((uint32_t)to_act16<ACT>(v[3]) << 16);
            *(uint2*)((uint16_t*)M.Y + off) = pk;
          }
        }
      }
    }
  }
}

bool batch_compatible(const glowq_unit& a, const glowq_unit& b) {
  return a.T > DEC_SMALL_T && a.T <= BATCH_MAX_T && b.T > DEC_SMALL_T && b.T <= BATCH_MAX_T && a.act_dtype == b.act_dtype &&
         a.group_size == b.group_size && (a.T <= 16) == (b.T <= 16) && (a.T <= 32) == (b.T <= 32);
}
int batch_max_units() { return BATCH_MAX_UNITS; }
int batch_wait_polls() { return R_WAIT_POLLS; }

// Workgroup tiles: 16 mb tokens x 16 rb rw rows, nw / rw groups of waves sharing the contraction.
// What a tile costs, in us per K tile of a wave group: `chain`, when the compute unit has nothing
// else to do, and `busy`, each workgroup's share of a compute unit that is full (binary16,
// bfloat16).  A launch takes the longer of its longest contraction and its share of the chip; a
// workgroup's start, fold, correction and stores weigh `ends` K tiles, and past what the chip holds
// at once the last round is partly empty.
// Measured as calls in a graph over 1250 calls of 5 to 2048 tokens (one unit to two layers, 256 to
// 14336 channels), each on every tile, beyond 64 tokens also on the tiled kernel, and the constants
// fitted to the choice: it is 1.5 % above the best on average up to 64 tokens and 2.1 % beyond (1.6 %
// and 0.7 % in 380 and 70 other calls); with constants of 70 calls and no `ends` it was 4.6 % and 5.6 %.
// The two tiles of two and three row blocks per wave are for 5 to 16 tokens on some thousand rows and a long contraction, where one
// row block per wave leaves a compute unit with one workgroup and a half, and four waves side by side
// leave most compute units empty: 5 tokens x 6456 rows x 8448 17.8 -> 13.4 us, 5 x 3 x 3320 x 12928
// 36.0 -> 25.9 (three row blocks).  A ring deeper than three stages was slower for both (1.07 and
// 1.29 times the time: one workgroup per compute unit).
struct BatchTile {
  int mb, rb, rw, nw;
  float start, ends;
  float chain[2], busy[2];
};
constexpr BatchTile BATCH_TILES[] = {
    {1, 1, 1, 4, 0.00f, 3.61f, {0.25f, 0.48f}, {0.43f, 0.34f}},
    {1, 1, 4, 4, 0.90f, 2.80f, {0.27f, 0.27f}, {0.17f, 0.17f}},
    {1, 1, 4, 8, 0.09f, 4.71f, {0.41f, 0.43f}, {0.29f, 0.29f}},
    {2, 1, 4, 4, 0.21f, 5.56f, {0.32f, 0.28f}, {0.22f, 0.22f}},
    {2, 1, 4, 8, 1.04f, 4.15f, {0.53f, 1.39f}, {0.41f, 0.60f}},
    {4, 1, 4, 4, 1.33f, 6.54f, {0.38f, 0.36f}, {0.38f, 0.41f}},
    {4, 2, 4, 4, 0.26f, 6.01f, {0.53f, 0.65f}, {0.52f, 0.58f}},
    {1, 2, 1, 4, 0.73f, 3.63f, {0.52f, 0.59f}, {0.54f, 0.40f}},
    {1, 3, 1, 4, 0.25f, 5.00f, {0.68f, 0.68f}, {0.68f, 0.72f}},
    {2, 1, 8, 8, 0.28f, 9.30f, {0.33f, 0.36f}, {0.17f, 0.17f}},
};
constexpr int BATCH_N_TILES = sizeof(BATCH_TILES) / sizeof(BATCH_TILES[0]);
// The last tile, 128 rows on eight waves side by side, is for launches of several units of more than 16 tokens that take longer by
// the other tiles' estimate: up to 32 tokens from 14 us on, 33 to 64 from 38 us on.  Its workgroups read X half as often as tiles
// of 64 rows.  Its constants are those of 1791 and 1070 such launches (one to four layers, two to six equal units) on every
// tile and, up to 32 tokens, in one to four slices: beside the other tiles it takes 9.5 % off the time on average up to 32 tokens in
// binary16 and 7.4 in bfloat16, 2.6 and 1.9 beyond; 4.0, 6.4, 2.7 and 2.9 % of the launches are more than 3 % slower for it.  (An
// estimate of nine constants for every tile, of the kind below, took 8.9, 6.8, 0.4 and 0 % off, 5.4, 7.7, 18 and 17 % of the
// launches were slower, 1.5 times as long at most.)  4096 / 14336 at 24 tokens, binary16, 44.8 -> 41.7 us.
constexpr int BATCH_TALL = BATCH_N_TILES - 1;
constexpr BatchTile BATCH_TALL_33 = {2, 1, 8, 8, 0.23f, 4.89f, {0.36f, 0.47f}, {0.32f, 0.34f}};      // at 33 to 64 tokens
constexpr float BATCH_LONG_US = 14.f, BATCH_LONG_US_33 = 38.f;
constexpr float BATCH_TALL_48 = 1.1f;          // up to 48 tokens the tiles of 64 are smaller than they are priced

template <int I> constexpr int batch_tile_resident() {
  constexpr BatchTile t = BATCH_TILES[I];
  return BatchShape<t.mb, t.rb, t.rw, t.nw>::WGS;
}
constexpr int BATCH_RESIDENT[] = {batch_tile_resident<0>(), batch_tile_resident<1>(), batch_tile_resident<2>(),
                                  batch_tile_resident<3>(), batch_tile_resident<4>(), batch_tile_resident<5>(),
                                  batch_tile_resident<6>(), batch_tile_resident<7>(), batch_tile_resident<8>(),
                                  batch_tile_resident<9>()};
static_assert(sizeof(BATCH_RESIDENT) / sizeof(int) == BATCH_N_TILES, "one entry per tile");

// K slices across workgroups, for a long contraction on few rows: its tiles run on while the rest of the chip
// idles (24 tokens x 4096 rows x 14336: 64 workgroups of 56 stages).  What a unit's own shapes allow: 32 K tiles and
// more, at least eight a slice, at most four slices and no more than about a thousand workgroups on tiles of 64 rows x
// 32 tokens.  Up to 32 tokens: a slice of 64 x 4096 results is a megabyte, out to memory and back.
constexpr int BATCH_SLICED_T = 32;
static int unit_row_blocks(const glowq_unit& u) {
  int blocks = 0;
  for (int i = 0; u.modules && i < u.n_modules; ++i) blocks += (u.modules[i].d_out + 15) / 16;
  return blocks;
}
static int batch_slices_allowed(const glowq_unit& u) {
  if (u.d_in < 4096 || u.T <= DEC_SMALL_T || u.T > BATCH_SLICED_T) return 1;
  const int wgs = (unit_row_blocks(u) + 3) / 4;
  if (wgs == 0 || wgs > 512) return 1;
  return std::min(std::min(BATCH_MAX_SLICES, u.d_in / 1024), 1024 / wgs);
}
// A cut unit's place in the launch's room for partial results: a count per tile, then the slabs.  The room is what the
// launch takes and not what its units might (a launch whose pieces do not fit the chip is not cut), and the launches of
// a call, one behind the other on the stream, use the same: at most 256 pieces of 32 KB.  (As a part of every unit's
// slice, by its own shapes, it was 1.6 GB of a stack of 40 layers of 5120 / 13824 at 8 tokens, where nothing is cut.)
static inline int batch_tiles(const glowq_unit& u, const BatchTile& t) {
  return ((unit_row_blocks(u) + t.rb * t.rw - 1) / (t.rb * t.rw)) * ((u.T + 16 * t.mb - 1) / (16 * t.mb));
}
static inline size_t batch_count_bytes(const glowq_unit& u, const BatchTile& t) { return ((size_t)batch_tiles(u, t) * 8 + 255) / 256 * 256; }
static inline size_t batch_unit_slab_bytes(const glowq_unit& u, const BatchTile& t, int ks) {
  return ks == 1 ? 0 : batch_count_bytes(u, t) + (size_t)ks * batch_tiles(u, t) * (t.rw * t.rb * t.mb * 1024);
}
size_t batch_slab_bytes(const glowq_unit* const* units, int n, int tile, const int* slices) {
  size_t bytes = 0;
  for (int k = 0; k < n; ++k) bytes += batch_unit_slab_bytes(*units[k], BATCH_TILES[tile], slices[k]);
  return bytes;
}

// (Tiles of 64 tokens are priced with four token blocks, as in the fit, also where a launch has three.)
// What the tiles from I on cost for units of `blocks` row blocks, `kt` K tiles and T tokens, of which `allowed` K slices
// (a tile at a time as constants, so that a call pays for shifts instead of divisions: one call of the
// smallest group is a few hundred instructions of host code in all).  A contraction is cut where the launch would take
// its length and not its share of the chip: all units to the stages that the longest one is left with, `cut` slices of
// it, and BATCH_SLICE_US for the sum (out to memory, a count, back).  The pieces have to fit the chip one per compute
// unit: beyond, they share what they were to have alone (26 tokens x 3 x 3112 rows x 5120 16.8 -> 20.5 us, 25 x 2 x 3816 x
// 8448 18.5 -> 23.5).  One unit is cut where the estimate falls by 15 %, several where it falls by 10 % (binary16; with less
// a layer of 4096 / 14336 at 16 tokens went from 31.9 to 34.1 us) or at all (bfloat16, whose uncut launches are estimated too
// low: the same layer at 24 tokens 50.8 -> 39.4).  A unit with a correction that is alone in its launch is cut from
// 4096 rows and nine tokens on: a slice that waits for the projection of a long contraction ends no earlier than the whole
// one, and the sum comes on top (64 single units, cold operands, us uncut and cut: 10 tokens x 3 x 192 rows x 9088 11.1 and
// 13.4, 9 x 3 x 1280 x 13568 16.5 and 20.3, 6 x 2 x 2704 x 9984 14.4 and 15.5; 10 x 4768 x 11264 16.5 and 14.6,
// 29 x 4336 x 8448 19.2 and 15.0, 19 x 2 x 2136 x 10880 24.5 and 19.8); in binary16 up to 5120 rows, where three slices
// fill the chip (17 tokens x 3 x 1712 x 11520 22.0 and 24.4, 14 x 3 x 1768 x 10624 18.9 and 22.0).  Layers of 768 / 13056 at 31 tokens 34.1 -> 24.5,
// of 512 / 7552 at 7 tokens (four) 22.7 -> 15.3.
// Several units wait for their projections as well, unless these are small (16 ranks): a launch of less than 400 row blocks
// is not cut, and the wait, BATCH_WAIT_US per K tile of the longest cut contraction, has to leave a microsecond.  (Uncut and cut: two
// of 10 tokens x 3 x 192 rows x 9088, r = 64, 12.9 and 14.6 us, four of 13 x 480 x 9088 15.7 and 18.7, two of 11 x 1168 x 13568 19.2
// and 21.3.  Of 1800 launches that were cut, 600 of them of one to four whole layers, 400 were more than 3 % slower for it, 40 % at
// most; of the 1114 that this leaves 29 are, 19 % at most, and the mean gain is 15 %; 11 of the whole layers run uncut.)
constexpr float BATCH_SLICE_US = 4.0f, BATCH_CUT_ONE = 0.85f, BATCH_CUT_SEVERAL[2] = {0.9f, 1.0f};
constexpr float BATCH_WAIT_US = 5.0f / 32.0f;
constexpr int BATCH_CUT_ONE_BLOCKS = 256, BATCH_CUT_ONE_MOST_F16 = 320, BATCH_CUT_ONE_T = 9, BATCH_CUT_BLOCKS = 400, BATCH_CUT_RANKS = 16;
struct BatchSize {
  int blocks, kt, T, allowed;
};
struct BatchChoice {
  int tile, cut;
  float cost;
};
static inline int batch_stages(int kt, int groups, int slices) { return (kt + groups * slices - 1) / (groups * slices); }
static inline int batch_cut(const BatchSize& u, int groups, int target) {
  return u.allowed == 1 ? 1 : std::min(u.allowed, (batch_stages(u.kt, groups, 1) + target - 1) / target);
}
// What tile I costs, the units cut so that the longest is left with 1 / cut of its stages; pieces: workgroups of units that are.
struct BatchWork {
  long long work, wgs, pieces;
  int chain;
};
static inline BatchWork batch_work(const BatchTile& t, const BatchSize* u, int n, int cut) {
  const int ks = t.nw / t.rw, rows = t.rb * t.rw, tok = 16 * t.mb;
  BatchWork w = {0, 0, 0, 0};
  int target = 0;
  if (cut > 1) {
    for (int k = 0; k < n; ++k) target = std::max(target, batch_stages(u[k].kt, ks, 1));
    target = (target + cut - 1) / cut;
  }
  for (int k = 0; k < n; ++k) {
    const int S = cut > 1 ? batch_cut(u[k], ks, target) : 1, stages = batch_stages(u[k].kt, ks, S);
    const long long wgs = (long long)((u[k].blocks + rows - 1) / rows) * ((u[k].T + tok - 1) / tok) * S;
    w.wgs += wgs;
    w.work += wgs * stages;
    w.chain = std::max(w.chain, stages);
    if (S > 1) w.pieces += wgs;
  }
  return w;
}
static inline float batch_cost(const BatchTile& t, int resident, const BatchWork& w, bool f16, int cut) {
  const float alone = t.chain[f16 ? 0 : 1], busy = t.busy[f16 ? 0 : 1];
  const float share = w.wgs <= 256 * resident ? (float)((w.wgs + 255) / 256) * busy : (float)w.wgs / 256.f * busy + 0.8f * alone;
  return t.start + std::max(((float)w.chain + t.ends) * alone, ((float)w.work / (float)w.wgs + t.ends) * share) + (cut > 1 ? BATCH_SLICE_US : 0.f);
}
template <int I>
static inline void cheapest_batch_tile(const BatchSize* u, int n, bool f16, int max_mb, BatchChoice* best) {
  constexpr BatchTile t = BATCH_TILES[I];
  if (t.mb <= max_mb) {
    const float c = batch_cost(t, BATCH_RESIDENT[I], batch_work(t, u, n, 1), f16, 1);
    if (best->tile < 0 || c < best->cost) *best = BatchChoice{I, 1, c};
  }
  if constexpr (I + 1 < BATCH_TALL) cheapest_batch_tile<I + 1>(u, n, f16, max_mb, best);
}
// the same with every number of slices from two on, on one tile
static void cheapest_cut(int tile, const BatchTile& t, const BatchSize* u, int n, bool f16, int most_cut, BatchChoice* best) {
  for (int cut = 2; cut <= most_cut; ++cut) {
    const BatchWork w = batch_work(t, u, n, cut);
    if (w.pieces > 256) break;
    const float c = batch_cost(t, BATCH_RESIDENT[tile], w, f16, cut);
    if (best->tile < 0 || c < best->cost) *best = BatchChoice{tile, cut, c};
  }
}

// Several units of up to 16 tokens that take longer: the estimate above takes tiles whose waves share the contraction too often, and cuts
// too seldom.  This one is for the two that are best there, 16 rows and 64, in one to four slices: the length of the longest chain
// and the chip's share (the longer of both counts whole, `both` of the other one), workgroups that do not fill whole rounds
// counted half, the projection's workgroups (`proj`: whole places for several us), the call's tokens (`tok`) and groups of 64 (`g64`);
// `slice`: the sum of a cut.  Us.  It is heard where the estimate above has its choice within 15 % of its own, and in bfloat16 not
// where that takes two or three row blocks per wave.  Of 2909 launches on every tile it makes them 2.7 % faster in binary16 and 2.3 in
// bfloat16; 4.6 and 5.6 % of them are more than 3 % slower, 13 % at most.  (Heard always, and with the other tiles, 2.3 and 2.1 % faster,
// 9 and 10 % slower, up to 1.5 times as long.  With the rule for the wait for R, which has to leave a microsecond where the
// estimate above cuts, both lose: binary16 gains 2.1 instead of 2.6 % at 10 % distance, and more launches are slower, not fewer.)
struct BatchFine {
  int tile;
  float start, ends, alone, busy, proj, tok, both, slice, g64;
};
constexpr BatchFine BATCH_FINE[2][2] = {      // binary16, bfloat16
    {{0, 1.725f, 4.684f, 0.367f, 0.383f, 7.843f, 0.159f, 0.266f, 2.802f, 0.003f},
     {1, 1.138f, 7.195f, 0.238f, 0.176f, 4.603f, -0.054f, 0.225f, 2.191f, 0.018f}},
    {{0, 1.874f, 4.249f, 0.384f, 0.399f, 8.406f, 0.163f, 0.190f, 2.783f, 0.006f},
     {1, 1.295f, 6.049f, 0.281f, 0.193f, 5.445f, -0.057f, 0.222f, 1.612f, 0.024f}}};
constexpr float BATCH_FINE_NEAR = 1.15f;
// proj: projection workgroups of the launch, restored or not
static BatchChoice cheapest_fine_tile(const BatchSize* u, int n, bool f16, bool g64, float proj, int most_cut) {
  int T = 0;
  for (int k = 0; k < n; ++k) T = std::max(T, u[k].T);
  BatchChoice best = {-1, 1, 0.f};
  for (const BatchFine& c : BATCH_FINE[f16 ? 0 : 1]) {
    const float scale = (1.f + c.tok * (float)(T - 16) / 16.f) * (g64 ? 1.f + c.g64 : 1.f);
    for (int cut = 1; cut <= most_cut; ++cut) {
      const BatchWork w = batch_work(BATCH_TILES[c.tile], u, n, cut);
      if (cut > 1 && (w.pieces == 0 || w.pieces > 256)) break;
      const float wgs = (float)w.wgs, per_cu = wgs / 256.f, whole = per_cu <= (float)BATCH_RESIDENT[c.tile] ? std::ceil(per_cu) / per_cu : 1.f;
      const float a = ((float)w.chain + c.ends) * c.alone * scale;
      const float b = (((float)w.work + c.ends * wgs) * c.busy * scale * (0.5f + 0.5f * whole) + proj * c.proj) / 256.f;
      const float cost = c.start + std::max(a, b) + c.both * std::min(a, b) + (cut > 1 ? c.slice : 0.f);
      if (best.tile < 0 || cost < best.cost) best = BatchChoice{c.tile, cut, cost};
    }
  }
  return best;
}

// The cheapest tile for these units in one launch, what it is taken to cost (us beyond the launch itself) and, given
// `slices`, the K slices of every unit.
int choose_batch_tile(const glowq_unit* const* units, int n, float* cost, int* slices) {
  const bool f16 = units[0]->act_dtype == GLOWQ_F16, exact = f16 && units[0]->T <= 32;
  BatchSize sizes[BATCH_MAX_UNITS];
  int most_cut = 1, blocks = 0, waiting_kt = 0;
  for (int k = 0; k < n; ++k) {
    const glowq_unit& u = *units[k];
    sizes[k] = BatchSize{unit_row_blocks(u), u.d_in / 128, u.T, 1};
    blocks += sizes[k].blocks;
    if (slices) {
      sizes[k].allowed = batch_slices_allowed(u);
      most_cut = std::max(most_cut, sizes[k].allowed);
      if (sizes[k].allowed > 1 && u.r > BATCH_CUT_RANKS) waiting_kt = std::max(waiting_kt, sizes[k].kt);
    }
  }
  if (n == 1 && units[0]->r > 0 &&
      (blocks < BATCH_CUT_ONE_BLOCKS || (f16 && blocks > BATCH_CUT_ONE_MOST_F16) || sizes[0].T < BATCH_CUT_ONE_T)) most_cut = 1;
  if (n > 1 && waiting_kt > 0 && blocks < BATCH_CUT_BLOCKS) most_cut = 1;
  const int max_mb = exact ? 2 : 4;
  BatchChoice whole = {-1, 1, 0.f}, cut = {-1, 1, 0.f};
  cheapest_batch_tile<0>(sizes, n, f16, max_mb, &whole);
  if (most_cut > 1 && whole.cost > 2.f * BATCH_SLICE_US)
    for (int i = 0; i < BATCH_TALL; ++i)
      if (BATCH_TILES[i].mb <= max_mb) cheapest_cut(i, BATCH_TILES[i], sizes, n, f16, most_cut, &cut);
  auto of_both = [&]() {
    const float wait = n > 1 && waiting_kt > 0 ? std::max(cut.cost - BATCH_SLICE_US, BATCH_WAIT_US * (float)waiting_kt) + 1.f : 0.f;
    const bool better = cut.tile >= 0 && cut.cost < (n > 1 ? BATCH_CUT_SEVERAL[f16 ? 0 : 1] : BATCH_CUT_ONE) * whole.cost && wait < whole.cost;
    return better ? cut : whole;
  };
  BatchChoice best = of_both();
  const int T = units[0]->T;
  if (n > 1 && T <= 64 && best.cost >= (T > 32 ? BATCH_LONG_US_33 : BATCH_LONG_US)) {
    if (T > 16) {
      const BatchTile& tall = T > 32 ? BATCH_TALL_33 : BATCH_TILES[BATCH_TALL];
      const float c = batch_cost(tall, BATCH_RESIDENT[BATCH_TALL], batch_work(tall, sizes, n, 1), f16, 1) * (T > 32 && T <= 48 ? BATCH_TALL_48 : 1.f);
      cheapest_cut(BATCH_TALL, tall, sizes, n, f16, most_cut, &cut);
      if (c < whole.cost) whole = BatchChoice{BATCH_TALL, 1, c};
      best = of_both();
    } else if (f16 || BATCH_TILES[best.tile].rb == 1) {
      float proj = 0.f;
      for (int k = 0; k < n; ++k)
        proj += (float)((units[k]->T + 15) / 16 * std::min(4, (units[k]->d_in + 1023) / 1024) * ((units[k]->r + 31) / 32));
      const BatchChoice fine = cheapest_fine_tile(sizes, n, f16, units[0]->group_size == 64, proj, most_cut);
      const BatchTile& t = BATCH_TILES[fine.tile];
      const float c = batch_cost(t, BATCH_RESIDENT[fine.tile], batch_work(t, sizes, n, fine.cut), f16, fine.cut);
      if (c <= BATCH_FINE_NEAR * best.cost) best = BatchChoice{fine.tile, fine.cut, c};
    }
  }
  *cost = best.cost;
  if (slices) {
    const int ks = BATCH_TILES[best.tile].nw / BATCH_TILES[best.tile].rw;
    int longest = 0;
    for (int k = 0; k < n; ++k) longest = std::max(longest, batch_stages(sizes[k].kt, ks, 1));
    for (int k = 0; k < n; ++k) slices[k] = best.cut == 1 ? 1 : batch_cut(sizes[k], ks, (longest + best.cut - 1) / best.cut);
  }
  return best.tile;
}

// K slices of the projection inside the launch: about 1024 channels each, at most four, and no
// more workgroups than the chip takes beside the first row blocks.
// A call that starts and ends with R waits for the slices' sum to come back from memory once more.
// Where R has no more rank pairs than four waves have threads, and the slices are not long enough to
// hide that hop, the consumers add the slices themselves, four short ones whatever d_in is: a call in
// a graph, 5 tokens x 512 rows x 2048, r = 64, 7.1 -> 5.9 us, 8 tokens x 672 x 1920, r = 32, 7.3 -> 5.7
// (7.0 on the kernel that this one replaced).  Over 313 calls of 5 to 32 tokens none was more than 1 %
// slower by this rule and the gain 2 % on average; with twice the pairs some lose 10 to 20 %.
constexpr int BATCH_GATHER_RANKS = 512, BATCH_GATHER_K = 8192;
void plan_batch_projection(const glowq_unit& u, UnitWorkspace& w) {
  const int pieces = (u.T + 15) / 16 * std::max(1, (u.r + 31) / 32);
  w.gather = u.T * u.r <= BATCH_GATHER_RANKS && u.d_in <= BATCH_GATHER_K;
  const int ksplit = w.gather ? 4 : std::max(1, std::min(std::min(4, (u.d_in + 1023) / 1024), (512 + pieces - 1) / pieces));
  const int steps = u.d_in / 32, per = (steps + ksplit - 1) / ksplit;
  w.kslice = per * 32;
  w.ksplit = (u.d_in + w.kslice - 1) / w.kslice;
}

// Token blocks of a launch's tiles: those of the tile, or three instead of four where nothing is cut and every unit's tokens,
// dealt evenly to as many tiles, fit them (33 to 48 tokens, 65 to 96, ..): a quarter less of X and of the products, and on tiles of
// 64 rows three workgroups per compute unit instead of two.  (Us on four blocks and on three: 88 tokens x 2 x 3272 rows x
// 4224 21.3 and 17.4, 46 x 3 x 5048 x 11008 46.6 and 41.1, 141 x 3 x 3256 x 9600 65.2 and 56.9, four layers of 4992 / 1920 at
// 47 tokens 68.8 and 62.0.)
int batch_token_blocks(const glowq_unit* const* units, int n, int tile, const int* slices) {
  if (BATCH_TILES[tile].mb != 4) return BATCH_TILES[tile].mb;
  for (int k = 0; k < n; ++k) {
    const int tiles = (units[k]->T + 63) / 64;
    if (slices[k] > 1 || units[k]->T > 48 * tiles) return 4;
  }
  return 3;
}

template <int ACT, bool EXACT, bool G128, bool CUT, int NB, int I>
static void launch_batch_tile(const BatchArgs<NB>& b, int tile, int mb, int n_wgs, hipStream_t st) {
  constexpr BatchTile t = BATCH_TILES[I];
  if constexpr (!EXACT && !CUT && t.mb == 4) {
    if (tile == I && mb == 3) {
      k_decode_batch<ACT, 3, t.rb, t.rw, t.nw, EXACT, G128, CUT, NB><<<dim3((unsigned)n_wgs), dim3(t.nw * 64), 0, st>>>(b);
      return;
    }
  }
  if constexpr (!EXACT || t.mb <= 2) {
    if (tile == I) k_decode_batch<ACT, t.mb, t.rb, t.rw, t.nw, EXACT, G128, CUT, NB><<<dim3((unsigned)n_wgs), dim3(t.nw * 64), 0, st>>>(b);
  }
  if constexpr (I + 1 < (NB > 1 ? BATCH_N_TILES : BATCH_TALL)) launch_batch_tile<ACT, EXACT, G128, CUT, NB, I + 1>(b, tile, mb, n_wgs, st);
}

template <bool CUT, int NB>
static void launch_batch_types(const BatchArgs<NB>& b, int ti, int mb, int wg, bool f16, bool exact, bool g128, hipStream_t st) {
  if (exact && g128) launch_batch_tile<ACT_F16, true, true, CUT, NB, 0>(b, ti, mb, wg, st);
  else if (exact) launch_batch_tile<ACT_F16, true, false, CUT, NB, 0>(b, ti, mb, wg, st);
  else if (!f16 && g128) launch_batch_tile<ACT_BF16, false, true, CUT, NB, 0>(b, ti, mb, wg, st);
  else if (!f16) launch_batch_tile<ACT_BF16, false, false, CUT, NB, 0>(b, ti, mb, wg, st);
  else if constexpr (!CUT) {                     // (no call of binary16 past 32 tokens is cut)
    if (g128) launch_batch_tile<ACT_F16, false, true, CUT, NB, 0>(b, ti, mb, wg, st);
    else launch_batch_tile<ACT_F16, false, false, CUT, NB, 0>(b, ti, mb, wg, st);
  }
}

template <int NB>
static hipError_t launch_batch(const glowq_unit* const* units, const UnitWorkspace* ws, const bool* restore, int n,
                               int ti, const int* slices, char* slabs, hipStream_t st) {
  BatchArgs<NB> b;
  const BatchTile tile = BATCH_TILES[ti];
  // longest contraction first: the hardware starts workgroups in index order
  int order[NB];
  for (int i = 0; i < n; ++i) order[i] = i;
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0 && units[order[j]]->d_in > units[order[j - 1]]->d_in; --j) {
      const int t = order[j]; order[j] = order[j - 1]; order[j - 1] = t;
    }
  int n_prod = 0;
  for (int oi = 0; oi < n; ++oi) {
    const glowq_unit& u = *units[order[oi]];
    const UnitWorkspace& w = ws[order[oi]];
    BatchUnit& bu = b.u[oi];
    int blk = 0;
    for (int i = 0; i < u.n_modules; ++i) {
      const glowq_module& m = u.modules[i];
      PreparedView v = prepared_view(m.w_prepared, m.d_out, u.d_in, u.group_size);
      bu.mod[i] = ModuleArgs{v.base, (const uint16_t*)m.A, m.Y, m.d_out, m.ldy, v.rows16, blk};
      blk += v.rows16;
    }
    for (int i = u.n_modules; i < GLOWQ_MAX_MODULES; ++i) bu.mod[i] = bu.mod[0];
    bu.X = (const uint16_t*)u.X;
    bu.B = (const uint16_t*)u.B;
    bu.T = u.T; bu.K = u.d_in; bu.r = u.r; bu.n_modules = u.n_modules;
    bu.n_blocks = blk;
    bu.out_f32 = u.out_dtype == GLOWQ_F32 ? 1 : 0;
    bu.restore = restore[order[oi]] ? 1 + w.gather : 0;
    bu.part = nullptr; bu.rslots = nullptr; bu.ctl = nullptr;
    bu.ks = slices[order[oi]];
    bu.count = nullptr; bu.slab = nullptr;
    if (bu.ks > 1) {
      bu.count = (unsigned long long*)slabs;
      bu.slab = (u32x4_t*)(slabs + batch_count_bytes(u, tile));
      slabs += batch_unit_slab_bytes(u, tile, bu.ks);
    }
    bu.ksplit = w.ksplit; bu.kslice = w.kslice;
    bu.prod_start = n_prod;
    bu.n_prod = 0;
    if (bu.restore) {
      bu.part = (float*)(w.base + w.off_rpart);
      bu.rslots = (uint32_t*)(w.base + w.off_r16);
      bu.ctl = (Control*)w.base;
      bu.n_prod = (u.T + 15) / 16 * w.ksplit * ((u.r + 31) / 32);
      n_prod += bu.n_prod;
    }
  }
  bool cut = false;
  for (int i = 0; i < n; ++i) cut = cut || slices[i] > 1;
  const int mb = batch_token_blocks(units, n, ti, slices);
  int wg = n_prod;
  for (int oi = 0; oi < n; ++oi) {
    b.u[oi].wg_start = wg;
    b.u[oi].n_ttiles = (b.u[oi].T + 16 * mb - 1) / (16 * mb);
    b.u[oi].n_groups = (b.u[oi].n_blocks + tile.rb * tile.rw - 1) / (tile.rb * tile.rw);
    wg += b.u[oi].n_groups * b.u[oi].n_ttiles * b.u[oi].ks;
  }
  for (int i = n; i < NB; ++i) b.u[i] = b.u[0];
  b.n = n;
  b.n_prod = n_prod;
  const bool f16 = units[0]->act_dtype == GLOWQ_F16, g128 = units[0]->group_size == 128;
  const bool exact = f16 && units[0]->T <= 32;
  if (cut) launch_batch_types<true, NB>(b, ti, mb, wg, f16, exact, g128, st);
  else launch_batch_types<false, NB>(b, ti, mb, wg, f16, exact, g128, st);
  return hipGetLastError();
}

// units[i] uses workspace slice ws[i]; all of them pass batch_compatible with units[0].  slabs: batch_slab_bytes of them
hipError_t launch_decode_batch(const glowq_unit* const* units, const UnitWorkspace* ws, const bool* restore, int n,
                               int tile, const int* slices, char* slabs, hipStream_t st) {
  if (n == 1) return launch_batch<1>(units, ws, restore, n, tile, slices, slabs, st);
  return launch_batch<BATCH_MAX_UNITS>(units, ws, restore, n, tile, slices, slabs, st);
}

}  // namespace glowq

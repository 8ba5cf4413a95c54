// Wide tiles of the microscaling product: 256 tokens x 256 rows, one workgroup of four waves per compute unit, waves of
// 128 x 128 in 256 accumulation registers (included by mx.hip behind the arguments of its tiled kernels).
//
// What bounds the 128 x 128 tiles is LDS: waves of 64 x 64 read 12 KiB for sixteen products of 32 cycles, so four waves
// read 96 of the 128 bytes that LDS delivers a cycle while direct loads write another 48.  Waves of 128 x 128 read half of
// that per product and the tile fetches half as much past LDS.  A wave has its SIMD to itself, so nothing may wait:
//  - the K tiles of all tiles of a workgroup are one stream through a ring of three stages (codes and scales of 256 tokens
//    and 256 rows, 50 KiB), loaded three stages ahead; a tile's end does not interrupt it;
//  - the one barrier of a stage stands in its middle, behind its last reads: there the next stage is known to have landed
//    (loads complete in order, the count is placed by hand) and this one's place is free, so that operand reads run half a
//    stage ahead;
//  - slots of one product, each with at most one operand read or one direct load beside it, the loads spread over the
//    whole stage (over half of it: 5 % slower), no branch (the stream passes from tile to tile by selects).
// 2 x 11008 rows x 4096 at 2048 tokens, bfloat16, r = 64: the kernel 170 -> 145 us within a call of 193 -> 162
// (182 -> 154 under the profiler).  In the loop the matrix pipe is busy
// 0.89 of the cycles at 1.88 GHz; with nothing but the products (no loads, no LDS) 0.97 at 2.03: 1.22 against 1.05 us a
// stage.  The rest are a tile's ends (stores of all workgroups at once 5 us, correction 2.5) and the last round of 0.69.
#pragma once

namespace glowq {

constexpr int MXW_BLOCKS = 16, MXW_TOK = 16 * MXW_BLOCKS;        // 16-token (16-row) blocks of a tile
constexpr int MXW_W = MXW_BLOCKS * 2048, MXW_XS = MXW_W + MXW_BLOCKS * 1024, MXW_WS = MXW_XS + MXW_BLOCKS * 64;
constexpr int MXW_STAGE = MXW_WS + MXW_BLOCKS * 64, MXW_RING = 3;
constexpr int MXW_LOADS = 14, MXW_EARLY = 8;                     // of a wave and stage; those issued in the stage before
constexpr int MXW_PANEL = 4;                                     // token tiles per panel of the tile order

// The sums of a wave are the accumulation registers themselves, named by number: sum q is a[4 q .. 4 q + 3].  (As 64
// variables they fill the register file to the last one, and around the ends of a tile the allocator finds no way to
// move them but through scratch.)  Nothing else may live in those registers: build.py reads the listing for that, and for
// the instruction's wait states, which the compiler does not see either.
__device__ inline void sums_claimed() {
#define GLOWQ_TEN(n) "a" #n "0", "a" #n "1", "a" #n "2", "a" #n "3", "a" #n "4", "a" #n "5", "a" #n "6", "a" #n "7", "a" #n "8", "a" #n "9"
  asm volatile("" : : : "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", GLOWQ_TEN(1), GLOWQ_TEN(2), GLOWQ_TEN(3), GLOWQ_TEN(4), GLOWQ_TEN(5), GLOWQ_TEN(6), GLOWQ_TEN(7),
               GLOWQ_TEN(8), GLOWQ_TEN(9), GLOWQ_TEN(10), GLOWQ_TEN(11), GLOWQ_TEN(12), GLOWQ_TEN(13), GLOWQ_TEN(14), GLOWQ_TEN(15), GLOWQ_TEN(16), GLOWQ_TEN(17), GLOWQ_TEN(18), GLOWQ_TEN(19), GLOWQ_TEN(20), GLOWQ_TEN(21),
               GLOWQ_TEN(22), GLOWQ_TEN(23), GLOWQ_TEN(24), "a250", "a251", "a252", "a253", "a254", "a255");
#undef GLOWQ_TEN
}
template <int Q> __device__ __attribute__((always_inline)) inline void sum_clear() {
  asm volatile("v_accvgpr_write_b32 a[%0], 0\n\tv_accvgpr_write_b32 a[%1], 0\n\tv_accvgpr_write_b32 a[%2], 0\n\tv_accvgpr_write_b32 a[%3], 0"
               : : "n"(4 * Q), "n"(4 * Q + 1), "n"(4 * Q + 2), "n"(4 * Q + 3));
}
template <int Q> __device__ __attribute__((always_inline)) inline float4_t sum_read() {
  float x, y, z, w;
  asm volatile("v_accvgpr_read_b32 %0, a[%4]\n\tv_accvgpr_read_b32 %1, a[%5]\n\tv_accvgpr_read_b32 %2, a[%6]\n\tv_accvgpr_read_b32 %3, a[%7]"
               : "=v"(x), "=v"(y), "=v"(z), "=v"(w) : "n"(4 * Q), "n"(4 * Q + 1), "n"(4 * Q + 2), "n"(4 * Q + 3));
  return float4_t{x, y, z, w};
}
// sum Q += a x b (16 bit)
template <int ACT, int Q> __device__ __attribute__((always_inline)) inline void sum_mfma16(u32x4_t a, u32x4_t b) {
  if constexpr (ACT == ACT_F16) asm volatile("v_mfma_f32_16x16x32_f16 a[%0:%1], %2, %3, a[%0:%1]" : : "n"(4 * Q), "n"(4 * Q + 3), "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, a[%0:%1]" : : "n"(4 * Q), "n"(4 * Q + 3), "v"(a), "v"(b));
}
// sum Q += weights x activations (fp4 x fp8, block scales sw, sx)
template <int Q> __device__ __attribute__((always_inline)) inline void sum_mx(u32x4_t w, v8i_t x, int sw, int sx) {
  asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 a[%0:%1], %2, %3, a[%0:%1], %4, %5 op_sel_hi:[0,0,0] cbsz:4"
               : : "n"(4 * Q), "n"(4 * Q + 3), "v"(w), "v"(x), "v"(sw), "v"(sx));
}
// The same with the product between the write of m0 and the direct load that reads it (AT: bytes added to the source and
// to the place in LDS)
template <int Q, int IMM, int AT>
__device__ __attribute__((always_inline)) inline void sum_mx_dma16(u32x4_t w, v8i_t x, int sw, int sx, const void* base, uint32_t off, uint32_t lds_base) {
  asm volatile("s_add_u32 m0, %8, %9\n\tv_mfma_scale_f32_16x16x128_f8f6f4 a[%0:%1], %2, %3, a[%0:%1], %4, %5 op_sel_hi:[0,0,0] cbsz:4\n\t"
               "global_load_lds_dwordx4 %6, %7 offset:%10"
               : : "n"(4 * Q), "n"(4 * Q + 3), "v"(w), "v"(x), "v"(sw), "v"(sx), "v"(off), "s"(base), "s"(lds_base), "n"(IMM), "n"(AT) : "memory", "m0", "scc");
}
template <int Q> __device__ __attribute__((always_inline)) inline void sum_mx_dma4(u32x4_t w, v8i_t x, int sw, int sx, const void* base, uint32_t off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %8\n\tv_mfma_scale_f32_16x16x128_f8f6f4 a[%0:%1], %2, %3, a[%0:%1], %4, %5 op_sel_hi:[0,0,0] cbsz:4\n\t"
               "global_load_lds_dword %6, %7"
               : : "n"(4 * Q), "n"(4 * Q + 3), "v"(w), "v"(x), "v"(sw), "v"(sx), "v"(off), "s"(base), "s"(lds_base) : "memory", "m0");
}
__device__ inline int lds1(uint32_t addr) { return *(const __attribute__((address_space(3))) uint8_t*)addr; }

// where a tile lies: module, token tile, row tile
struct MxWidePlace {
  int module, mt, nt;
};
__device__ inline MxWidePlace mx_wide_place(const MxGemmArgs& a, int tile) {
  int mi = 0;
#pragma unroll
  for (int i = 1; i < GLOWQ_MAX_MODULES; ++i)
    if (i < a.n_modules && tile >= a.mod[i].first_block) mi = i;
  // residue classes of the index share an XCD's L2: class c takes the c-th eighth of the module's list, which runs
  // through panels of token tiles (four of them and eight row tiles: as many bytes of either operand)
  const int local = tile - a.mod[mi].first_block, n_rows = (a.mod[mi].d_out + MXW_TOK - 1) / MXW_TOK, n = n_rows * a.tok_tiles;
  const int c = local & 7, t = c * (n >> 3) + min(c, n & 7) + (local >> 3);
  const int panel = t / (MXW_PANEL * n_rows), width = min(MXW_PANEL, a.tok_tiles - panel * MXW_PANEL);
  const int tl = t - panel * MXW_PANEL * n_rows;
  return MxWidePlace{__builtin_amdgcn_readfirstlane(mi), __builtin_amdgcn_readfirstlane(panel * MXW_PANEL + tl % width),
                     __builtin_amdgcn_readfirstlane(tl / width)};
}

template <int ACT>
__global__ void __launch_bounds__(256, 1) k_mx_wide(MxGemmArgs a, int n_tiles) {
  __shared__ __attribute__((aligned(1024))) uint8_t ring[MXW_RING * MXW_STAGE];
  const int l = threadIdx.x & 63, i = l & 15, g = l >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w >> 1, wn = w & 1;
  const int ktiles = a.d_in / 128, n_tb = (a.T + 15) / 16;
  const uint32_t lds0 = lds_address(ring);

  // the stream of K tiles: sources of the next one to load, and of the tile behind it.  A wave loads four blocks of tokens
  // and four of rows; blocks past the last one repeat it and are not stored, past the last tile its K tiles come again
  struct Source {
    const uint8_t *x, *w, *xs, *ws;
    uint32_t xoff[4], woff[4];       // blocks' offsets (uniform)
    uint32_t xsoff, wsoff;           // of this lane's piece of the scales
  };
  auto source = [&](int tile) {
    Source S;
    const MxWidePlace p = mx_wide_place(a, min(tile, n_tiles - 1));
    const MxModule& m = a.mod[p.module];
    const int tb0 = p.mt * MXW_BLOCKS, rb0 = p.nt * MXW_BLOCKS, n_rb = (m.d_out + 15) / 16;
    S.x = uniform_ptr(a.xcodes + (size_t)tb0 * ktiles * 2048);
    S.xs = uniform_ptr(a.xscales + (size_t)tb0 * ktiles * 64);
    S.w = uniform_ptr((const uint8_t*)m.codes + (size_t)rb0 * ktiles * 1024);
    S.ws = uniform_ptr(m.scales + (size_t)rb0 * ktiles * 64);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      S.xoff[q] = __builtin_amdgcn_readfirstlane((uint32_t)(min(tb0 + 4 * w + q, n_tb - 1) - tb0) * (uint32_t)(ktiles * 2048));
      S.woff[q] = __builtin_amdgcn_readfirstlane((uint32_t)(min(rb0 + 4 * w + q, n_rb - 1) - rb0) * (uint32_t)(ktiles * 1024));
    }
    S.xsoff = (uint32_t)(min(tb0 + 4 * w + g, n_tb - 1) - tb0) * (uint32_t)(ktiles * 64) + i * 4;
    S.wsoff = (uint32_t)(min(rb0 + 4 * w + g, n_rb - 1) - rb0) * (uint32_t)(ktiles * 64) + i * 4;
    return S;
  };
  Source src = source(blockIdx.x), after = source(blockIdx.x + gridDim.x);
  int src_left = __builtin_amdgcn_readfirstlane(ktiles - 1);
  auto advance = [&]() __attribute__((always_inline)) {
    const bool end = src_left == 0;       // uniform; selects instead of a branch, which would end the schedule
    src.x = end ? after.x : src.x + 2048;
    src.xs = end ? after.xs : src.xs + 64;
    src.w = end ? after.w : src.w + 1024;
    src.ws = end ? after.ws : src.ws + 64;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      src.xoff[q] = end ? after.xoff[q] : src.xoff[q];
      src.woff[q] = end ? after.woff[q] : src.woff[q];
    }
    src.xsoff = end ? after.xsoff : src.xsoff;
    src.wsoff = end ? after.wsoff : src.wsoff;
    src_left = end ? ktiles - 1 : src_left - 1;
  };
  const uint32_t land_x = __builtin_amdgcn_readfirstlane(lds0 + w * 8192), land_w = __builtin_amdgcn_readfirstlane(lds0 + MXW_W + w * 4096),
                 land_s = __builtin_amdgcn_readfirstlane(lds0 + MXW_XS + w * 256);
  // loads 0 .. 3: rows, 4 .. 11: tokens, 12, 13: scales
  auto load = [&](int d, uint32_t slot) __attribute__((always_inline)) {
    if (d < 4) lds_dma16_off(src.w + src.woff[d], l * 16, land_w + slot + d * 1024);
    else if (d < 12) lds_dma16_off(src.x + src.xoff[(d - 4) / 2] + (d & 1) * 1024, l * 16, land_x + slot + (d - 4) * 1024);
    else if (d == 12) lds_dma4_off(src.xs, src.xsoff, land_s + slot);
    else lds_dma4_off(src.ws, src.wsoff, land_s + slot + (MXW_WS - MXW_XS));
  };
#pragma unroll
  for (int s = 0; s < 3; ++s) {
#pragma unroll
    for (int d = 0; d < (s < 2 ? MXW_LOADS : MXW_EARLY); ++d) load(d, s * MXW_STAGE);
    if (s < 2) advance();              // (the third time in the loop)
  }

  // operands: a stage multiplies four token blocks with all row blocks, then the other four; the row blocks are replaced
  // by the next stage's behind their last product, the token blocks half a stage ahead
  const uint32_t rd_x = lds0 + wm * 16384 + l * 16, rd_w = lds0 + MXW_W + wn * 8192 + l * 16;
  const uint32_t rd_xs = lds0 + MXW_XS + wm * 512 + l, rd_ws = lds0 + MXW_WS + wn * 512 + l;
  u32x4_t wv[8], xlo[8], xhi[8];
  int ws[8], xs[8];
  // sums: r + 8 tb for row block r and token block tb
  auto clear = [&]() __attribute__((always_inline)) {
    for_each_index<64>([&](auto Q) __attribute__((always_inline)) { sum_clear<Q.value>(); });
    asm volatile("s_nop 1");
  };
  sums_claimed();
  clear();
  vm_wait<MXW_LOADS + MXW_EARLY>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    wv[r] = lds16(rd_w + r * 1024);
    ws[r] = lds1(rd_ws + r * 64);
  }
#pragma unroll
  for (int tb = 0; tb < 4; ++tb) {
    xlo[tb] = lds16(rd_x + tb * 2048);
    xhi[tb] = lds16(rd_x + tb * 2048 + 1024);
    xs[tb] = lds1(rd_xs + tb * 64);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  uint32_t cur = 0, nxt = MXW_STAGE, prv = 2 * MXW_STAGE;      // byte offsets of the stages at hand, next and before
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    for (int kt = 0; kt < ktiles; ++kt) {
      for_each_index<64>([&](auto S) __attribute__((always_inline)) {
        constexpr int s = S.value, half = s / 32, r = s % 32 / 4, tb = 4 * half + s % 4, q = r + 8 * tb;
        if constexpr (s == 32) {
          // this wave's reads of the stage are done and its part of the next one has landed (the loads of the one
          // after may be on their way); behind the barrier everybody's
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(MXW_LOADS) : "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
        // token blocks of the other half
        constexpr int n = s % 32 / 2, fn = (4 * (1 - half) + n / 3) & 7;
        if constexpr (s % 2 == 0 && n < 12) {
          const uint32_t at = half ? nxt : cur;
          if constexpr (n % 3 == 0) xlo[fn] = lds16(rd_x + at + fn * 2048);
          if constexpr (n % 3 == 1) xhi[fn] = lds16(rd_x + at + fn * 2048 + 1024);
          if constexpr (n % 3 == 2) xs[fn] = lds1(rd_xs + at + fn * 64);
        }
        const v8i_t x = __builtin_shufflevector(__builtin_bit_cast(v4i_t, xlo[tb]), __builtin_bit_cast(v4i_t, xhi[tb]), 0, 1, 2, 3, 4, 5, 6, 7);
        // the product, with a direct load behind it in some slots: this stage's place is free behind the barrier
        constexpr int d = s % 4 != 1 ? -1 : half ? s / 4 - 8 : s / 4 < MXW_LOADS - MXW_EARLY ? MXW_EARLY + s / 4 : -1;
        const uint32_t slot = half ? cur : prv;
        if constexpr (d >= 0 && d < 4) sum_mx_dma16<q, d * 1024, 0>(wv[r], x, ws[r], xs[tb], src.w + src.woff[d & 3], l * 16, land_w + slot);
        else if constexpr (d >= 4 && d < 12)
          sum_mx_dma16<q, (d - 4 - (d & 1)) * 1024, (d & 1) * 1024>(wv[r], x, ws[r], xs[tb], src.x + src.xoff[((d - 4) / 2) & 3], l * 16, land_x + slot);
        else if constexpr (d == 12) sum_mx_dma4<q>(wv[r], x, ws[r], xs[tb], src.xs, src.xsoff, land_s + slot);
        else if constexpr (d == 13) sum_mx_dma4<q>(wv[r], x, ws[r], xs[tb], src.ws, src.wsoff, land_s + slot + (MXW_WS - MXW_XS));
        else sum_mx<q>(wv[r], x, ws[r], xs[tb]);
        if constexpr (half && s % 4 == 3) {
          wv[r] = lds16(rd_w + nxt + r * 1024);
          ws[r] = lds1(rd_ws + nxt + r * 64);
        }
        if constexpr (s == 28) advance();
        __builtin_amdgcn_sched_barrier(0);
      });
      const uint32_t t = prv;
      prv = cur;
      cur = nxt;
      nxt = t;
    }
    after = source(tile + 2 * gridDim.x);        // (the stream is in the next tile)
    const MxWidePlace p = mx_wide_place(a, tile);
    const MxModule& m = a.mod[p.module];
    const int row0 = p.nt * MXW_TOK + wn * 128, tok0 = p.mt * MXW_TOK + wm * 128;
    const int rows = m.d_out - row0, toks = a.T - tok0;        // (none for a wave with nothing to store)
    // correction: + R A_i^T (lane (i, g): ranks 32 s + 8 g .. + 8)
    if (a.R16) {
      const auto abase = (const __attribute__((address_space(1))) char*)uniform_ptr(m.A + (size_t)min(row0, m.d_out - 1) * a.r);
      const auto rbase = (const __attribute__((address_space(1))) char*)uniform_ptr(a.R16 + (size_t)min(tok0, a.T - 1) * a.r);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (32 * s < a.r) {        // uniform
          // ranks past r: zeros on both sides (R may hold infinities); rows and tokens past the last are that one again
          const int j0 = 32 * s + 8 * g;
          const uint32_t at = 2u * (uint32_t)min(j0, a.r - 8);
          u32x4_t av[8], rv[8];
#pragma unroll
          for (int r = 0; r < 8; ++r)
            av[r] = *(const __attribute__((address_space(1))) u32x4_t*)(abase + (2u * (uint32_t)(min(r * 16 + i, max(rows, 1) - 1) * a.r) + at));
#pragma unroll
          for (int r = 0; r < 8; ++r)
            rv[r] = *(const __attribute__((address_space(1))) u32x4_t*)(rbase + (2u * (uint32_t)(min(r * 16 + i, max(toks, 1) - 1) * a.r) + at));
          if (32 * s + 32 > a.r) {         // uniform: whole steps multiply while R's later words are on their way
#pragma unroll
            for (int r = 0; r < 8; ++r)
              if (j0 >= a.r) av[r] = rv[r] = u32x4_t{0, 0, 0, 0};
          }
          __builtin_amdgcn_sched_barrier(0);
          asm volatile("s_nop 1");       // (operands that the vector ALU wrote)
          for_each_index<64>([&](auto Q) __attribute__((always_inline)) { sum_mfma16<ACT, Q.value>(av[Q.value % 8], rv[Q.value / 8]); });
        }
      }
    }
    acc_settle();
    // lane holds rows 4 g .. + 4 of each block and token i; 16-bit outputs: eight rows of a pair of blocks per store
    auto ybase = (__attribute__((address_space(1))) char*)uniform_ptr((char*)m.Y + ((size_t)tok0 * m.ldy + row0) * (a.out_f32 ? 4 : 2));
    for_each_index<32>([&](auto P) __attribute__((always_inline)) {
      constexpr int tb = P.value / 4, r = P.value % 4 * 2;
      const uint32_t line = (uint32_t)(tb * 16 + i) * (uint32_t)m.ldy;
      const float4_t v0 = sum_read<8 * tb + r>(), v1 = sum_read<8 * tb + r + 1>();
      if (a.out_f32) {
        const int row = r * 16 + 4 * g;
        if (tb * 16 + i < toks && row < rows) *(__attribute__((address_space(1))) float4_t*)(ybase + (line + row) * 4u) = v0;
        if (tb * 16 + i < toks && row + 16 < rows) *(__attribute__((address_space(1))) float4_t*)(ybase + (line + row + 16) * 4u) = v1;
      } else {
        const int row = (r + (g & 1)) * 16 + 8 * (g >> 1);
        const u32x4_t v = acc_pack_rows<ACT>(v0, v1);
        if (tb * 16 + i < toks && row < rows) *(__attribute__((address_space(1))) u32x4_t*)(ybase + (line + row) * 2u) = v;
      }
    });
    sums_claimed();
    clear();
  }
  vm_wait<0>();        // nothing may still be on its way into LDS when the workgroup ends
}

}  // namespace glowq

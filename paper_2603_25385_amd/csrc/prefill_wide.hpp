// Wide tiles of the tiled kernel: 256 tokens x 256 rows, one workgroup of four waves per compute unit
// (included by prefill.hip behind the descriptors and proj_tile).
//
// What bounds the 128-token tiles is issue: every weight is dequantised once per 128 tokens, which is two
// vector-ALU instructions for each matrix instruction, and the fp32 results of a tile leave no registers for more.
// A wave that has a SIMD to itself holds 64 rows x 256 tokens (256 accumulation registers), so that a weight is
// dequantised once per 256 tokens and one vector-ALU instruction per matrix instruction is left: it issues in the
// shadow of the matrix instruction, as do the operand reads (one per four) and the direct loads.
// X travels global -> LDS in stages of 64 channels through a ring of four.  The one barrier of a stage stands in
// its middle: there every wave has seen its own part of the next stage land (loads complete in order, the count is
// placed by hand), so that the operand reads run ahead across the end of a stage and nothing waits there; the
// stage before it is free, and the loads of the third stage from here go into its place.
// Rows of X are XOR-swizzled by 16-byte chunks on the global-address side, as in k_prefill.
// Measured against the 128-token tiles: 2 x 11008 rows x 4096 at 2048 tokens, bfloat16, 357 -> 294 us; four layers of
// 5120 / 13824 at 1000 tokens 2167 -> 2027 us; a layer of 4096 / 14336 at 512 tokens 241 -> 217 us.  A tile of 4096
// channels takes 151 (binary16) and 161 (bfloat16) of the 131 thousand cycles that its products need, at 1.7 to
// 1.8 GHz: the chip's power sets the clock, and the same loop without the dequantiser is 12 to 17 % faster.
#pragma once

namespace glowq {

constexpr int WD_WAVES = 4, WD_RB = 4, WD_MB = 16;          // 16-row blocks per wave, 16-token blocks per tile
constexpr int WD_TOK = 16 * WD_MB, WD_BLOCKS = WD_WAVES * WD_RB;
constexpr int WD_RING = 4;
constexpr int WD_STAGE = WD_TOK * 64 * 2;                   // bytes of a stage of X
constexpr int WD_WSTG = WD_RB * 1024 + 512;                 // bytes of a wave's weight stage
constexpr int WD_LDS = WD_RING * WD_STAGE + WD_WAVES * WD_WSTG;

// The same with a product between the write of m0 and the load that reads it
template <int ACT, int IMM> __device__ inline void mfma_dma16(float4_t& acc, u32x4_t a, u32x4_t b, const void* base, uint32_t off, uint32_t lds_base) {
  if constexpr (ACT == ACT_F16)
    asm volatile("s_add_u32 m0, %5, %6\n\tv_mfma_f32_16x16x32_f16 %0, %1, %2, %0\n\tglobal_load_lds_dwordx4 %3, %4"
                 : "+a"(acc) : "v"(a), "v"(b), "v"(off), "s"(base), "s"(lds_base), "n"(IMM) : "memory", "m0", "scc");
  else
    asm volatile("s_add_u32 m0, %5, %6\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tglobal_load_lds_dwordx4 %3, %4"
                 : "+a"(acc) : "v"(a), "v"(b), "v"(off), "s"(base), "s"(lds_base), "n"(IMM) : "memory", "m0", "scc");
}
template <int ACT, int IMM> __device__ inline void mfma_dma4(float4_t& acc, u32x4_t a, u32x4_t b, const void* base, uint32_t off, uint32_t lds_base) {
  if constexpr (ACT == ACT_F16)
    asm volatile("s_add_u32 m0, %5, %6\n\tv_mfma_f32_16x16x32_f16 %0, %1, %2, %0\n\tglobal_load_lds_dword %3, %4"
                 : "+a"(acc) : "v"(a), "v"(b), "v"(off), "s"(base), "s"(lds_base), "n"(IMM) : "memory", "m0", "scc");
  else
    asm volatile("s_add_u32 m0, %5, %6\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tglobal_load_lds_dword %3, %4"
                 : "+a"(acc) : "v"(a), "v"(b), "v"(off), "s"(base), "s"(lds_base), "n"(IMM) : "memory", "m0", "scc");
}
// Instructions that the slots before slot `end` of step j have room for beside their product, operand read, wait
// and direct load
template <int NWL> constexpr int wide_room(int j, int end) {
  int room = 0;
  for (int i = 0; i < end; ++i) {
    const bool load = i % 8 == 4 && ((j & 1) || (j == 0 && i / 8 < NWL));
    room += load ? 0 : (i % 4 == 2 || i % 16 == 0) ? 1 : 2;
  }
  return room;
}

// Projection tile of a launch of wide tiles (128 tokens x all ranks, see proj_tile).  It has a compute unit to
// itself, so nothing covers a wait for memory: X and B travel through the ring of four stages, loaded three stages
// ahead.
template <int ACT>
__device__ inline void proj_tile_wide(const PrefillArgs& a, uint8_t* lds) {
  constexpr int RBP = 8 / WD_WAVES, MB = 8, LI = 4, B_AT = 16 * MB * 128;     // loads a stage of X (of B), bytes of X
  int ui = 0;
#pragma unroll
  for (int i = 0; i < PF_MAX_UNITS; ++i)
    if (i < a.n_units && a.unit[i].proj_start >= 0 && (int)blockIdx.x >= a.unit[i].proj_start) ui = i;
  const PfUnit& U = a.unit[ui];
  const int local = (int)blockIdx.x - U.proj_start;
  const int mt = local / U.parts, part = local - mt * U.parts;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kq = lane >> 4;
  const int s_begin = part * U.part_stages, stages = min(U.K >> 6, s_begin + U.part_stages) - s_begin;
  const int tok0 = mt * 16 * MB;
  const char* xtile = (const char*)uniform_ptr(U.X + (size_t)tok0 * U.K + (size_t)s_begin * 64);
  const char* btile = (const char*)uniform_ptr(U.B + (size_t)s_begin * 64);
  uint32_t xoff[LI], boff[LI];       // rows past T (past r) are the last token's (rank's) again, never stored
#pragma unroll
  for (int i = 0; i < LI; ++i) {
    const int row = 32 * i + (tid >> 3);
    const int chunk = (tid & 7) ^ ((row >> 1) & 7);
    xoff[i] = (uint32_t)(min(tok0 + row, U.T - 1) - tok0) * (uint32_t)U.K * 2u + chunk * 16;
    boff[i] = (uint32_t)min(row, U.r - 1) * (uint32_t)U.K * 2u + chunk * 16;
  }
  const uint32_t lds0 = lds_address(lds), land = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
  auto load = [&](int stage) {
    const size_t at = (size_t)min(stage, stages - 1) * 128;
    const uint32_t to = land + (stage & 3) * WD_STAGE;
#pragma unroll
    for (int i = 0; i < LI; ++i) lds_dma16_off(xtile + at, xoff[i], to + i * 4096);
#pragma unroll
    for (int i = 0; i < LI; ++i) lds_dma16_off(btile + at, boff[i], to + B_AT + i * 4096);
  };
  const int rd_sw = (n >> 1) & 7;
  const uint32_t rd[2] = {lds0 + n * 128 + ((kq ^ rd_sw) << 4), lds0 + n * 128 + (((4 + kq) ^ rd_sw) << 4)};
  float4_t acc[RBP][MB];
#pragma unroll
  for (int b = 0; b < RBP; ++b)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[b][mb] = float4_t{0.f, 0.f, 0.f, 0.f};
  load(0);
  load(1);
  load(2);
  for (int s = 0; s < stages; ++s) {
    vm_wait<4 * LI>();               // stage s: two younger ones may be on their way
    __builtin_amdgcn_s_barrier();    // ... everybody's part of it, and everybody is done with stage s - 1
    load(s + 3);
    if (wave * RBP * 16 < U.r) {     // uniform
      const uint32_t at = (s & 3) * WD_STAGE;
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        u32x4_t bw[RBP];
#pragma unroll
        for (int b = 0; b < RBP; ++b) bw[b] = lds16(rd[jj] + at + B_AT + (wave * RBP + b) * 2048);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const u32x4_t x = lds16(rd[jj] + at + mb * 2048);
#pragma unroll
          for (int b = 0; b < RBP; ++b) acc[b][mb] = mfma16<ACT>(bw[b], x, acc[b][mb]);   // D[rank][token]
        }
      }
    }
  }
  vm_wait<0>();                      // nothing may still be on its way into LDS when the ring is used again
  __syncthreads();
  proj_publish<ACT, MB, RBP>(U, acc, mt, part, (uint32_t*)lds);
}

template <int ACT, bool G128>
__global__ void __launch_bounds__(WD_WAVES * 64, 1) k_wide(PrefillArgs a) {
  constexpr int RB = WD_RB, MB = WD_MB;
  constexpr int XI = WD_TOK / (WD_WAVES * 8);        // 16-byte X loads per thread and stage
  constexpr int RW = G128 ? 272 : 288;               // words per tile record
  __shared__ __attribute__((aligned(1024))) uint8_t lds[WD_LDS];
  __shared__ uint32_t corr_failed;                   // a wave's bounded wait for the projection expired

  if ((int)blockIdx.x < a.n_proj_wgs) {
    proj_tile_wide<ACT>(a, lds);
    return;
  }
  int mi = 0;
#pragma unroll
  for (int i = 1; i < PF_MAX_MODS; ++i)
    if (i < a.n_mods && (int)blockIdx.x >= a.mod[i].wg_start) mi = i;
  const PfModule& M = a.mod[mi];
  const PfUnit& U = a.unit[M.unit];
  // tile order: as in k_prefill
  int mt, nt;
  {
    const int local = (int)blockIdx.x - M.wg_start;
    const int n_tiles = M.n_ntiles * U.n_mtiles;
    const int c = local & 7, q = local >> 3;
    const int t = c * (n_tiles >> 3) + min(c, n_tiles & 7) + q;
    const int per_panel = PF_PANEL * M.n_ntiles;
    const int panel = t / per_panel;
    const int width = min(PF_PANEL, U.n_mtiles - panel * PF_PANEL);
    const int tl = t - panel * per_panel;
    nt = __builtin_amdgcn_readfirstlane(tl / width);
    mt = __builtin_amdgcn_readfirstlane(panel * PF_PANEL + (tl - (tl / width) * width));
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kq = lane >> 4;
  const int ktiles = M.nkt, nstages = 2 * ktiles;

  // weights: a 1 KiB load per 16-row block and K tile, and one (two) for the scale/zero words of all four.  Blocks
  // past the module's last one are computed from that one and never stored.
  const int nb0 = nt * WD_BLOCKS + RB * wave;
  constexpr int SZB = G128 ? 64 : 128, SZI = G128 ? 1 : 2, NWL = RB + SZI;
  const char* wptr = (const char*)uniform_ptr(M.rec + ((size_t)min(nb0, M.rows16 - 1) * (U.K >> 7) + M.kt0) * RW);   // the K tile to load next
  const uint32_t block_bytes = (uint32_t)(U.K >> 7) * (RW * 4u);
  auto block_off = [&](int b) { return (uint32_t)(min(nb0 + b, M.rows16 - 1) - min(nb0, M.rows16 - 1)) * block_bytes; };
  uint32_t woff[NWL];                  // byte offsets of this lane's pieces of a K tile
#pragma unroll
  for (int b = 0; b < RB; ++b) woff[b] = block_off(b) + lane * 16;
#pragma unroll
  for (int j = 0; j < SZI; ++j)
    woff[RB + j] = block_off(G128 ? (lane >> 4) : 2 * j + (lane >> 5)) + 1024u + 4u * (G128 ? (lane & 15) : (lane & 31));
  const uint32_t lds0 = lds_address(lds);
  const uint32_t wstage = __builtin_amdgcn_readfirstlane(lds0 + WD_RING * WD_STAGE + wave * WD_WSTG);
  int w_left = ktiles - 1;             // K tiles behind the one at wptr; the last one is loaded again past the end
  auto advance_w = [&]() { wptr += w_left > 0 ? RW * 4 : 0; --w_left; };

  // X: load i of a wave covers eight rows, 128 bytes each; rows past T are the last token's again
  const int tok0 = mt * WD_TOK;
  const char* xtile = (const char*)uniform_ptr(U.X + (size_t)tok0 * U.K + (size_t)M.kt0 * 128);
  uint32_t xoff[XI];
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    const int row = 32 * i + (tid >> 3);
    const int chunk = (tid & 7) ^ ((row >> 1) & 7);
    xoff[i] = (uint32_t)(min(tok0 + row, U.T - 1) - tok0) * (uint32_t)U.K * 2u + chunk * 16;
  }
  const uint32_t xland = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
  int x_left = nstages - 1;            // likewise for stages of X
  auto advance_x = [&]() { xtile += x_left > 0 ? 128 : 0; --x_left; };
  const int rd_sw = (n >> 1) & 7;
  const uint32_t rd0 = lds0 + n * 128 + ((kq ^ rd_sw) << 4), rd1 = lds0 + n * 128 + (((4 + kq) ^ rd_sw) << 4);

  float4_t acc[RB][MB];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[b][mb] = float4_t{0.f, 0.f, 0.f, 0.f};

  u32x4_t wcur[RB];
  uint32_t szcur[RB][2];
  auto take_w = [&]() {
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      wcur[b] = lds16(wstage + lane * 16 + b * 1024);
      szcur[b][0] = lds4(wstage + RB * 1024 + n * 4 + b * SZB);
      szcur[b][1] = G128 ? szcur[b][0] : lds4(wstage + RB * 1024 + n * 4 + b * SZB + 64);
    }
  };
  u32x4_t wf[2][RB];
  GroupConst<ACT> g[RB];
  using DQ = std::conditional_t<ACT == ACT_F16, DequantLockstepF16Shiftless<RB, RB>, DequantLockstep<ACT, RB, RB>>;
  DQ dq;

  GLOWQ_STAMP(0);
  if (tid == 0) corr_failed = 0;       // ordered before its readers by the loop's barriers
#pragma unroll
  for (int j = 0; j < NWL; ++j) {
    if (j < RB) lds_dma16_off(wptr, woff[j], wstage + j * 1024);
    else lds_dma4_off(wptr, woff[j], wstage + RB * 1024 + (j - RB) * 256);
  }
  advance_w();
#pragma unroll
  for (int s = 0; s < 3; ++s) {
#pragma unroll
    for (int i = 0; i < XI; ++i) lds_dma16_off(xtile, xoff[i], xland + s * WD_STAGE + i * 4096);
    if (s < 2) advance_x();            // (the third time in the loop)
  }
  vm_wait<2 * XI>();                   // the weights and stage 0
  __builtin_amdgcn_s_barrier();
  take_w();
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    g[b].set(szcur[b][0]);
    dq.set_group(b, g[b]);
    wf[0][b] = dequant_word<ACT>(wcur[b][0], g[b]);
  }
  GLOWQ_STAMP(1);

  // One K tile: four steps of 32 channels, each 64 products in fenced slots of one; behind the products of step j
  // the words of step j + 1 are dequantised.  A matrix instruction holds the matrix core for 16 cycles and leaves
  // room for two more instructions of any kind (a third costs its 4 cycles), so every slot gets at most two:
  // operand reads in slots 2 mod 4, direct loads and the write of m0 in slots 4 mod 8, the dequantiser in
  // what is left (wide_room).  Operands are read two groups of four fragments ahead, and a group's last
  // one read is the first one used, so that one wait serves four.
  // (Against one wait a fragment and uneven slots: 19.9 -> 18.5 cycles a product in binary16, 20.6 -> 19.6 in bfloat16.)
  constexpr int XN = 16;
  u32x4_t xq[XN];                      // fragment f (step f / 16, token block f % 16) in xq[f % 16]
  auto xread = [&](int f, uint32_t p0, uint32_t p1) __attribute__((always_inline)) {
    const int st = f >> 5, jj = (f >> 4) & 1, mb = f & 15;
    return lds16((jj ? p1 : p0) + (uint32_t)(st * WD_STAGE + mb * 2048));
  };
#pragma unroll
  for (int f = 0; f < 8; ++f) xq[f] = xread(f, rd0, rd1);
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acc_settled(acc[b][mb]);
  acc_settle();                        // (the zeros of the first products)
  uint32_t cur = 0;                    // byte offset of the K tile's two stages in the ring
  for (int kt = 0; kt < ktiles; ++kt) {
    const uint32_t p0 = rd0 + cur, p1 = rd1 + cur;
    const uint32_t q0 = rd0 + (cur ^ (2 * WD_STAGE));
    // places of the two stages that are loaded during this K tile
    const uint32_t land1 = xland + (cur ^ (2 * WD_STAGE)) + WD_STAGE, land2 = xland + cur;
    for_each_index<4>([&](auto J) __attribute__((always_inline)) {
      constexpr int j = J.value, jn = (j + 1) & 3;       // the step being dequantised: jn
      constexpr bool new_group = G128 ? (j == 3) : ((j & 1) == 1);
      u32x4_t (&wa)[RB] = wf[j & 1];
      u32x4_t (&wn)[RB] = wf[jn & 1];
      if constexpr (j & 1) {
        // the middle of stage 2 kt + (j >> 1): in flight and younger than the next stage's X are one stage of X
        // and, in the first stage, the next tile's weights; in the second stage those have to be there too
        vm_wait<j == 1 ? XI + NWL : XI>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      for_each_index<RB * MB>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = I.value, b = i % RB, q = i / 16, mb = 4 * q + 3 - (i % 16) / RB;   // the group's last fragment first
        constexpr int f = MB * j + mb;
        if constexpr (i % 4 == 2) {
          constexpr int fn = MB * j + 4 * (q + 2) + (i % 16) / 4;       // two groups ahead
          xq[fn % XN] = fn < 4 * MB ? xread(fn, p0, p1) : xread(fn - 4 * MB, q0, q0);
        }
        // the next tile's words
        if constexpr (j == 3 && i % 2 == 1 && i / 2 < RB) {
          wcur[i / 2] = lds16(wstage + lane * 16 + (i / 2) * 1024);
          szcur[i / 2][0] = lds4(wstage + RB * 1024 + n * 4 + (i / 2) * SZB);
          szcur[i / 2][1] = G128 ? szcur[i / 2][0] : lds4(wstage + RB * 1024 + n * 4 + (i / 2) * SZB + 64);
        }
        // the product (D[row][token]), with a direct load behind it in some slots
        constexpr int d = i / 8;
        if constexpr (j == 0 && i % 8 == 4 && d < RB) mfma_dma16<ACT, (d % RB) * 1024>(acc[b][mb], wa[b], xq[f % XN], wptr, woff[d % RB], wstage);
        else if constexpr (j == 0 && i % 8 == 4 && d < NWL) mfma_dma4<ACT, RB * 1024 + (d >= RB && d < NWL ? d - RB : 0) * 256>(acc[b][mb], wa[b], xq[f % XN], wptr, woff[d < NWL ? d : 0], wstage);
        else if constexpr ((j & 1) && i % 8 == 4) mfma_dma16<ACT, d * 4096>(acc[b][mb], wa[b], xq[f % XN], xtile, xoff[d], j == 1 ? land1 : land2);
        else mfma_acc<ACT>(acc[b][mb], wa[b], xq[f % XN]);
        if constexpr (j == 2 && i == 4) advance_w();
        if constexpr (j == 2 && i == 12) advance_x();
        if constexpr (j == 0 && i == 60) advance_x();
        // its vector-ALU shadow, in the last step behind the words' own LDS reads
        constexpr int S0 = j == 3 ? 24 : new_group ? 2 * RB : 0, w = (i - (S0 - 2 * RB)) / 2;
        if constexpr (new_group && i >= S0 - 2 * RB && i < S0 && i % 2 == 1) {
          g[w].set(szcur[w][G128 ? 0 : (jn >> 1)]);
          dq.set_group(w, g[w]);
        }
        constexpr int NO = DQ::N_OPS, all = wide_room<NWL>(j, RB * MB) - wide_room<NWL>(j, S0);
        constexpr int lo = i < S0 ? 0 : (wide_room<NWL>(j, i) - wide_room<NWL>(j, S0)) * NO / all;
        constexpr int hi = i < S0 ? 0 : (wide_room<NWL>(j, i + 1) - wide_room<NWL>(j, S0)) * NO / all;
        for_each_index<hi - lo>([&](auto O) __attribute__((always_inline)) { dq.op(lo + O.value, wcur, jn, g, wn); });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    cur ^= 2 * WD_STAGE;
  }
  vm_wait<0>();        // nothing may still be on its way into LDS when the ring is used again or the workgroup ends
  GLOWQ_STAMP(4);

  // correction: r more channels in stages of 64, [A_i] against [R] (see k_prefill); R comes from the projection
  // tiles of 128 tokens that this tile covers
  if (U.restore && M.corr) {
    const int rstages = (U.r + 63) >> 6;                       // 1 or 2
    bool ready = wait_tile_ready(U.flags + 8 * (2 * mt), U.status);
    if (tok0 + 128 < U.T) ready = wait_tile_ready(U.flags + 8 * (2 * mt + 1), U.status) && ready;
    if (!ready && lane == 0) atomicOr(&corr_failed, 1u);
    __syncthreads();   // (the ring is idle from here on)
    const bool apply = *(volatile uint32_t*)&corr_failed == 0;
    if (apply) {
      const char* rtile = (const char*)uniform_ptr(U.R16 + (size_t)tok0 * U.r);
#pragma unroll
      for (int rs = 0; rs < 2; ++rs)
#pragma unroll
        for (int i = 0; i < XI; ++i) {
          const int row = 32 * i + (tid >> 3);
          const int chunk = (tid & 7) ^ ((row >> 1) & 7);
          const int rank = min(64 * rs + 8 * chunk, U.r - 8);
          const uint32_t off = (uint32_t)((min(tok0 + row, U.T - 1) - tok0) * U.r + rank) * 2u;
          if (rs < rstages) lds_dma16_off_coherent(rtile, off, xland + rs * WD_STAGE + i * 4096);
        }
      u32x4_t af[2][2][RB];
#pragma unroll
      for (int rs = 0; rs < 2; ++rs)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int b = 0; b < RB; ++b) {
            // ranks past r: zeros
            const int j0 = 64 * rs + 32 * jj + 8 * kq;
            const int row = min((nb0 + b) * 16 + n, M.d_out - 1);
            af[rs][jj][b] = u32x4_t{0u, 0u, 0u, 0u};
            if (j0 < U.r) af[rs][jj][b] = *(const u32x4_t*)(M.A + (size_t)row * U.r + j0);
          }
      vm_wait<0>();
      // ... and zeros in LDS over the valid rank's words that were loaded there (R may hold infinities): each thread in
      // the places that its own loads have filled
      if (U.r & 31) {
#pragma unroll
        for (int rs = 0; rs < 2; ++rs)
          if (rs < rstages && 64 * rs + 8 * ((tid & 7) ^ ((tid >> 4) & 7)) >= U.r)
#pragma unroll
            for (int i = 0; i < XI; ++i)
              *(__attribute__((address_space(3))) u32x4_t*)(xland + rs * WD_STAGE + i * 4096 + lane * 16) = u32x4_t{0u, 0u, 0u, 0u};
      }
      __syncthreads();
#pragma unroll
      for (int rs = 0; rs < 2; ++rs)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          if (64 * rs + 32 * jj < U.r) {                       // uniform
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
              const u32x4_t x = lds16((jj ? rd1 : rd0) + (uint32_t)(rs * WD_STAGE + mb * 2048));
#pragma unroll
              for (int b = 0; b < RB; ++b) mfma_acc<ACT>(acc[b][mb], af[rs][jj][b], x);
            }
          }
        }
    }
  }
  GLOWQ_STAMP(5);
  acc_settle();
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc_settled(acc[b][mb]);
  // store: lane holds token (mb, n) and rows 4 kq + {0..3} of each 16-row block; 16-bit outputs exchange two blocks'
  // rows between lane groups, so that every lane stores eight rows (16 bytes)
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int tok = tok0 + mb * 16 + n;
#pragma unroll
    for (int b = 0; b < RB; b += 2) {
      if (M.out_f32) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int row = (nb0 + b + q) * 16 + 4 * kq;
          if (tok < U.T && row < M.d_out) *(float4_t*)((float*)M.Y + (size_t)tok * M.ldy + row) = acc[b + q][mb];
        }
      } else {
        const u32x4_t v = acc_pack_rows<ACT>(acc[b][mb], acc[b + 1][mb]);
        const int row = (nb0 + b + (kq & 1)) * 16 + 8 * (kq >> 1);
        if (tok < U.T && row < M.d_out) *(u32x4_t*)((uint16_t*)M.Y + (size_t)tok * M.ldy + row) = v;
      }
    }
  }
  GLOWQ_STAMP(6);
}

}  // namespace glowq

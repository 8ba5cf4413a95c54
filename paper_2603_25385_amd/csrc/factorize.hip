// Shared factors of one unit's stacked quantisation error, computed on the GPU
// (paper Alg. 1 and App. A.3-A.4: randomised range finder with power steps on the
// covariance-aligned error, small SVD, balanced split, lift back).  Offline work, no part
// of the forward.  Everything is float64.
//
//   Ms     = E_cat Sigma_x^(1/2)            E_cat = [W_i - dequant(W_q,i)]_i stacked by rows
//   Y      = Ms Omega,  q times  Y <- Ms (Ms^T Y)
//   Q      = orth(Y)                        Cholesky QR in passes (wide sketches: Gram-Schmidt)
//   Bs     = Q^T Ms = U~ S V^T              rotations from the rows' Gram matrix (wide: one-sided
//                                           Jacobi on the rows)
//   A      = Q U~_r S_r^(1/2),  B = S_r^(1/2) V_r^T Sigma_x^(-1/2)
//
// The algorithm in the paper first replaces the m x d stack by the d x d triangular factor
// of its thin QR, so that a dense SVD of the core is affordable.  With the operator form of
// the range finder (App. A.3: only products with M and M^T are needed) the products run on
// the stack itself here: Q_e M = E_cat Sigma_x^(1/2), so every quantity below is Q_e times
// (or equal to) its counterpart on the core and A, B come out the same; forming the Gram
// matrix or a Householder QR of the stack would cost m d^2 operations against
// (2q + 2) m d (r + p) for the products.
//
// The matrix products are float64 matrix-core contractions (16x16x4); where K is cut into slices
// their partial results are added in slice order, and the Gram matrices' parts in workgroup order, so
// results do not depend on timing.
#include "common.hpp"
#include "launch.hpp"
#include "ranking.hpp"
#include <algorithm>
#include <utility>

namespace glowq {

typedef double double4_t __attribute__((ext_vector_type(4)));

constexpr int FZ_NT = 5;            // 16-column blocks per pass of a product (80 columns)

// ---------------------------------------------------------------------------------------
// the stack
// ---------------------------------------------------------------------------------------
// Thread idx: root[idx] and inv_root[idx] (no sigma: neither), element idx of Omega in rows of ld (the layout of every
// narrow operand below; zeros behind column l), counter idx.
__global__ void __launch_bounds__(256) k_setup(const double* __restrict__ sigma, int d, double* __restrict__ root,
                                               double* __restrict__ inv_root, const double* __restrict__ Omega, int l,
                                               int ld, double* __restrict__ Z, int* __restrict__ counters, int n_counters) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx < n_counters) counters[idx] = 0;
  if (sigma && idx < d) {
    const double s = sigma[idx];
    const double r = s > 0.0 ? sqrt(s) : 0.0;
    root[idx] = r;
    inv_root[idx] = r > 0.0 ? 1.0 / r : 0.0;    // (pseudo-inverse on a zero variance)
  }
  if (idx >= d * ld) return;
  const int k = idx / ld, c = idx - k * ld;
  Z[idx] = c < l ? Omega[(long long)k * l + c] : 0.0;
}

// Ms[o][k] = (W[o][k] - What[o][k]) * root[k], What the stored 16-bit weight, rows of all modules one after the other.
// A workgroup per tile record, four rows per wave, two channels per lane: a wave reads 512 contiguous bytes of
// W and writes a contiguous KiB of Ms per row (with eight channels per lane, 64 bytes each a row apart, and a
// launch per module: 5120 rows of 3072 in 100 us, now 30; the bytes at a copy's rate: 40).
struct StackArgs {
  const float* W[GLOWQ_MAX_MODULES];
  const uint32_t* prepared[GLOWQ_MAX_MODULES];
  int d_out[GLOWQ_MAX_MODULES], rec_start[GLOWQ_MAX_MODULES], n_modules;      // first record of a module
  long long row_start[GLOWQ_MAX_MODULES];
  int d_in, G;
};

template <int ACT>
__global__ void __launch_bounds__(256) k_error_stack(StackArgs a, const double* __restrict__ root, double* __restrict__ Ms) {
  int mi = 0;
#pragma unroll
  for (int q = 1; q < GLOWQ_MAX_MODULES; ++q)
    if (q < a.n_modules && (int)blockIdx.x >= a.rec_start[q]) mi = q;
  const int rec = (int)blockIdx.x - a.rec_start[mi], ktiles = a.d_in >> 7, d_out = a.d_out[mi];
  const int rb = rec / ktiles, kt = rec - rb * ktiles;
  const int lane = threadIdx.x & 63, row0 = 4 * (threadIdx.x >> 6);      // row within the record
  const uint32_t* r = a.prepared[mi] + (long long)rec * prepared_rec_words(a.G);
  const int k = kt * 128 + 2 * lane;
  const float* W = a.W[mi] + (long long)(rb * 16 + row0) * a.d_in + k;
  double* dst = Ms + (a.row_start[mi] + rb * 16 + row0) * a.d_in + k;
  const int live = min(4, d_out - rb * 16 - row0);
  // lane's pair of channels: nibbles i and i + 4 of word j of record lane row + 16 ((k >> 3) & 3)
  const int word = 64 * ((lane >> 2) & 3) + (lane >> 4), i = lane & 3, sz = 256 + 16 * (2 * lane / a.G);
  double2 rt = make_double2(1.0, 1.0);
  if (root) rt = *(const double2*)(root + k);
  float2 w[4];
  uint32_t c[4], g[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (q < live) w[q] = *(const float2*)(W + (long long)q * a.d_in);
    c[q] = r[4 * (row0 + q) + word];
    g[q] = r[sz + row0 + q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (q >= live) break;
    GroupConst<ACT> gc;
    gc.set(g[q]);
    const uint32_t pair = dequant_pair<ACT>(c[q] >> (4 * i), gc);
    double2 e = make_double2((double)w[q].x - act16_value<ACT>(pair & 0xffffu), (double)w[q].y - act16_value<ACT>(pair >> 16));
    e.x *= rt.x;
    e.y *= rt.y;
    *(double2*)(dst + (long long)q * a.d_in) = e;
  }
}

// ---------------------------------------------------------------------------------------
// float64 products on the matrix cores.  v_mfma_f64_16x16x4: lane l holds A[l & 15][l >> 4],
// B[l >> 4][l & 15] and, in register v, D[(l >> 4) + 4 v][l & 15].  Slice ks of a product goes to
// P[ks][M][ldp]; rows, columns and K past the edge are clamped on the load and dropped (zeroed, for K) afterwards.
// ---------------------------------------------------------------------------------------
struct GemmShape {
  int M, N, K;
  int n0;          // first column of this pass
  int kslice;      // stages per slice
  int n_slices;
  int row_tiles;   // ceil(M / 64)
};

// the four waves' tiles added in wave order, in wave 0's registers (k_lift, whose waves share the contraction)
template <int RB, int NT>
__device__ inline void fold_waves(double4_t (&acc)[RB][NT], double* fold, int wave, int lane) {
  for (int w = 1; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int v = 0; v < 4; ++v) fold[((rb * NT + nt) * 4 + v) * 64 + lane] = acc[rb][nt][v];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[rb][nt][v] += fold[((rb * NT + nt) * 4 + v) * 64 + lane];
    }
    __syncthreads();
  }
}

// The products with the stack (and Gram matrices): C = A B or, TN, C = A^T B, by workgroups of 64
// rows of C x 16 NT columns x a slice of K.  Both operands travel global -> LDS in stages of 32 channels
// through two buffers (the next stage is on its way while one is multiplied), a wave owns 16 rows
// and all columns.  The matrix instruction takes 64 cycles, so eight LDS reads and a barrier per 40 of
// them cost nothing; what counts is that no wave waits for memory in front of its products and that
// the narrow operand crosses the L2s once per 64 rows.  Two workgroups share a compute unit.  (Operands
// straight to registers, 32 rows a workgroup and the channels dealt to its waves: 5120 x 80 over 3072
// 81 us, 3072 x 80 over 5120 66 us; this 54 and 60.  The products alone, 64 cycles each at 2.4 GHz: 32 us.
// Stages of 16 channels in a ring of four: 56 and 63 us, so memory is not what it waits for.)
// A's rows are XOR-swizzled by 16-byte chunks on the global-address side where lanes read down a
// column of them (A B).  lda, ldb even, both operands 16-byte aligned and readable up to a whole 16
// columns; what is read there reaches only rows and columns of C that are not stored.  K is a multiple of 32, or TN:
// channels past it are read from the last one and multiplied by zero.
template <bool TN, int NT>
__global__ void __launch_bounds__(256, 2) k_gemm_ring(const double* __restrict__ A, long long lda,
                                                      const double* __restrict__ B, long long ldb,
                                                      double* __restrict__ P, long long ldp, GemmShape s) {
  constexpr int A_BYTES = 64 * 32 * 8, STAGE = A_BYTES + 32 * NT * 128;
  __shared__ __attribute__((aligned(1024))) uint8_t ring[2 * STAGE];
  const int tile = blockIdx.x % s.row_tiles, ks = blockIdx.x / s.row_tiles;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, i = l & 15, g = l >> 4;
  const int st0 = ks * s.kslice, n_st = min((s.K + 31) / 32 - st0, s.kslice);
  const uint32_t lds0 = lds_address(ring);
  auto issue = [&](int st, int buf) {
    const int k0 = 32 * (st0 + st);
    const uint32_t base = lds0 + (uint32_t)(buf * STAGE);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = 4 * w + j;                       // a KiB: four rows of 32 channels, or two channels of 64 rows
      const double* src;
      if (TN) {
        const long long col = min((long long)tile * 64 + 2 * (l & 31), lda - 2);
        src = A + (long long)min(k0 + 2 * q + (l >> 5), s.K - 1) * lda + col;
      } else {
        const int row = 4 * q + g;
        src = A + (long long)min(tile * 64 + row, s.M - 1) * lda + k0 + 2 * (i ^ (row & 15));
      }
      lds_dma16(src, base + (uint32_t)q * 1024u);
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int q = w * NT + j, piece = q * 64 + l, ch = piece / (8 * NT), at = piece - ch * (8 * NT);
      lds_dma16(B + (long long)min(k0 + ch, s.K - 1) * ldb + s.n0 + 2 * at, base + A_BYTES + (uint32_t)q * 1024u);
    }
  };
  double4_t acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = double4_t{0.0, 0.0, 0.0, 0.0};
  issue(0, 0);
  vm_wait<0>();
  __syncthreads();
  for (int st = 0; st < n_st; ++st) {
    const int buf = st & 1;
    if (st + 1 < n_st) issue(st + 1, buf ^ 1);
    const uint8_t* L = ring + buf * STAGE;
    const double* Bl = (const double*)(L + A_BYTES);
    const int left = s.K - 32 * (st0 + st);          // (TN: channels from here to the end)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      // channels of instruction t: 4 t + g, or 8 (t >> 1) + 2 g + (t & 1) (a 16-byte chunk holds two)
      const int ch = TN ? 4 * t + g : 8 * (t >> 1) + 2 * g + (t & 1);
      double a;
      if (TN) {
        a = ((const double*)L)[ch * 64 + 16 * w + i];
        a = ch < left ? a : 0.0;
      } else {
        a = ((const double*)(L + (16 * w + i) * 256 + (((4 * (t >> 1) + g) ^ i) << 4)))[t & 1];
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        acc[nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Bl[ch * (16 * NT) + 16 * nt + i], acc[nt], 0, 0, 0);
    }
    vm_wait<0>();          // this wave's loads of the next stage have landed ...
    __syncthreads();       // ... and everybody's; everybody is done reading this one
  }
  double* Ps = P + (long long)ks * s.M * ldp;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = tile * 64 + 16 * w + g + 4 * v, col = s.n0 + 16 * nt + i;
      if (row < s.M && col < s.N) Ps[(long long)row * ldp + col] = acc[nt][v];
    }
}

// C[row][col] (or C[col][row] when transposed) = sum over slices, in slice order
__global__ void k_reduce_slices(const double* __restrict__ P, long long ldp, int n_slices, int M, int N,
                                double* __restrict__ C, long long ldc, int transposed) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long long)M * N) return;
  const int row = (int)(idx / N), col = (int)(idx - (long long)row * N);
  double sum = 0.0;
  for (int sl = 0; sl < n_slices; ++sl) sum += P[((long long)sl * M + row) * ldp + col];
  if (transposed) C[(long long)col * ldc + row] = sum;
  else C[(long long)row * ldc + col] = sum;
}

struct GemmPlan {
  int kslice, n_slices, row_tiles;
};

// Products with the stack: the number of slices whose workgroups, dealt to 256 compute units, need the fewest
// stages on the fullest one.  A workgroup's start and end weigh two stages; one that has a compute unit to itself
// takes 8 % longer a stage (nothing covers its barriers); a slice's partial results weigh a twelfth.  (From 3 to 16 slices
// of the two products named at k_gemm_ring; us: 3 / 4 / 5 / 6 / 8 / 10 / 12 / 16 slices of the first 55 / 73 / 63 / 54 / 60 /
// 60 / 56 / 56, of the second 99 / 77 / 64 / 87 / 71 / 60 / 76 / 60.)
static GemmPlan plan_ring(int M, int K) {
  GemmPlan p;
  p.row_tiles = (M + 63) / 64;
  const int stages = (K + 31) / 32;
  double best = 0.0;
  for (int want = 1; want <= 16 && want <= stages; ++want) {
    const int per = (stages + want - 1) / want, n = (stages + per - 1) / per;
    const int rounds = (p.row_tiles * n + 255) / 256;
    const double cost = (rounds == 1 ? 1.08 : rounds) * (per + 2) + 0.08 * n;
    if (want == 1 || cost < best) {
      best = cost;
      p.kslice = per;
      p.n_slices = n;
    }
  }
  return p;
}

static size_t slice_doubles(const GemmPlan& p, int M, int N) {
  return (size_t)p.n_slices * (size_t)M * (size_t)((N + 15) / 16 * 16);
}

template <bool TN, int NT>
static void launch_gemm_pass(const double* A, long long lda, const double* B, long long ldb, double* P,
                             long long ldp, const GemmShape& s, hipStream_t st) {
  k_gemm_ring<TN, NT><<<dim3((unsigned)(s.row_tiles * s.n_slices)), dim3(256), 0, st>>>(A, lda, B, ldb, P, ldp, s);
}

// C [M][N] = A B (K a multiple of 32) or, TN, A^T B through the slice buffer.  `left`: the sum over the slices is left to
// the caller, and *left their number.
template <bool TN>
static hipError_t gemm(const double* A, long long lda, const double* B, long long ldb, double* C,
                       long long ldc, bool c_transposed, int M, int N, int K, double* slices,
                       hipStream_t st, int* left = nullptr) {
  const GemmPlan p = plan_ring(M, K);
  const long long ldp = (N + 15) / 16 * 16;
  GemmShape s;
  s.M = M; s.N = N; s.K = K;
  s.kslice = p.kslice; s.n_slices = p.n_slices; s.row_tiles = p.row_tiles;
  for (int n0 = 0; n0 < N; n0 += 16 * FZ_NT) {
    s.n0 = n0;
    const int nt = (std::min(N - n0, 16 * FZ_NT) + 15) / 16;
    switch (nt) {
      case 1: launch_gemm_pass<TN, 1>(A, lda, B, ldb, slices, ldp, s, st); break;
      case 2: launch_gemm_pass<TN, 2>(A, lda, B, ldb, slices, ldp, s, st); break;
      case 3: launch_gemm_pass<TN, 3>(A, lda, B, ldb, slices, ldp, s, st); break;
      case 4: launch_gemm_pass<TN, 4>(A, lda, B, ldb, slices, ldp, s, st); break;
      default: launch_gemm_pass<TN, 5>(A, lda, B, ldb, slices, ldp, s, st); break;
    }
  }
  if (left) {
    *left = p.n_slices;
    return hipGetLastError();
  }
  const long long n = (long long)M * N;
  k_reduce_slices<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(slices, ldp, p.n_slices, M, N, C,
                                                                          ldc, c_transposed ? 1 : 0);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Q = orth(Y) for sketches of up to FZ_SMALL columns: Cholesky QR, iterated.  A pass forms the
// Gram matrix of Y (matrix cores), factors it in one workgroup's LDS and multiplies Y with the
// inverse factor (k_pass; column by column, three launches each, 80 columns x 5120 rows took 1930 us).  A Cholesky factor of a Gram matrix only resolves columns whose part
// outside the span of the columns before them is well above its rounding.  So a column whose
// share of norm^2 outside that span falls below FZ_ACCEPT is deferred: this pass takes the
// span out of it but does not project anybody on it, and the next pass, where it starts at
// length one again, decides anew.  `kept` follows the product of those shares; a column that
// kept less than FZ_RANK_TOL2 of its norm^2 is dependent and cleared.  The passes end when all
// remaining columns were accepted with pivots above one half, i.e. when the columns were
// orthogonal before the pass up to what the pass itself corrects to rounding.  Two passes for a
// sketch of condition 10^4, five for 10^12.
// ---------------------------------------------------------------------------------------
constexpr int FZ_SMALL = 128;
constexpr int FZ_QR_PASSES = 6;
constexpr double FZ_ACCEPT = 1e-8;
constexpr double FZ_RANK_TOL2 = 1e-24;      // a column whose norm^2 fell by this factor is dependent
constexpr int FZ_PASS_THREADS = 1024;
enum { FZ_PENDING = 0, FZ_KEPT = 1, FZ_DROPPED = 2 };

// 1 / sqrt(x) to working precision: the hardware's estimate and two Newton steps
__device__ inline double inv_sqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  y = y * __builtin_fma(-h * y, y, 1.5);
  return y * __builtin_fma(-h * y, y, 1.5);
}

// D += sum over 16 channels of A B, 16 x 16 blocks of doubles anywhere (element (i, k) of A at
// A[i ai + k ak], and so on): four matrix instructions.
__device__ inline double4_t block_product(const double* A, int ai, int ak, const double* B, int bk, double4_t acc) {
  const int l = (int)threadIdx.x & 63, i = l & 15, g = l >> 4;
#pragma unroll
  for (int t = 0; t < 4; ++t)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[i * ai + (4 * t + g) * ak], B[(4 * t + g) * bk + i], acc, 0, 0, 0);
  return acc;
}
__device__ inline double read_lane(double v, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// lane J's value of every row of 16 lanes, in all its lanes
template <int J> __device__ inline double row_broadcast(double v) {
  const long long u = __builtin_amdgcn_update_dpp(0ll, __builtin_bit_cast(long long, v), 0x150 | J, 0xf, 0xf, true);
  return __builtin_bit_cast(double, u);
}
// lane `from`'s value (any lane of the wave)
__device__ inline double lane_permute(double v, int from) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * from, (int)(uint32_t)u);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * from, (int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Step J of a diagonal block (see block_cholesky): lane (i, g) holds rows 4 q + g of column i in a[q].
// Columns behind J take the multiple of column J out of themselves, column J is scaled where it is the
// inverse's.
template <int J, class PIVOT>
__device__ __attribute__((always_inline)) inline void diagonal_steps(double (&a)[4], int i, int g, bool& used, PIVOT& pivot) {
  if constexpr (J < 16) {
    constexpr int QJ = J >> 2, GJ = J & 3;
    const double mine = lane_permute(a[QJ], i + 16 * GJ);          // row J of this lane's column
    double own = 0.0;
    const double ri = pivot.take(J, read_lane(a[QJ], J + 16 * GJ), own);
    const double w = -mine * ri * ri;
    const bool behind = i > J, at = i == J;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double v = row_broadcast<J>(a[q]);
      const double moved = __builtin_fma(v, w, a[q]), scaled = a[q] * own;
      const bool above = q < QJ || (q == QJ && g < GJ);
      double x = behind ? moved : (at && above ? scaled : a[q]);
      if (q == QJ && g == GJ) x = behind ? w : (at ? own : a[q]);
      a[q] = x;
    }
    if (at) used = ri > 0.0;
    diagonal_steps<J + 1>(a, i, g, used, pivot);
  }
}

// Cholesky factor R (upper, S = R^T R) of a symmetric matrix of nb x nb blocks of 16 in LDS
// (S [16 nb][LD], upper blocks and whole diagonal blocks), by one workgroup; with INVERSE, S
// ends as the upper triangular T = R^-1, without it as R.  Panels of 16 rows: one wave factors
// and inverts the diagonal block, four rows of a column per lane, matrix instructions do the rest.
// The serial chain of the diagonal block's sixteen steps bounds it; what a step needs of a lane's own column
// comes through a row broadcast, what it needs of the pivot row through one permutation under the
// latency of the square root, and the decisions about pivots stay in registers until the panel is done (with a
// column per lane and the pivots' state in LDS 80 columns took 41 us, now 25).
// PIVOT: begin(J) before panel J's steps; take(j, d, own) returns 1 / sqrt(d) if column 16 J + j is to be used and 0 if not,
// `own` then scales what stays of its own column in T; end(J).  E, F, Rb: LDS, 256, 256 and 16 LD
// doubles (Rb only with INVERSE).
template <bool INVERSE, class PIVOT>
__device__ inline void block_cholesky(double* S, int LD, int nb, double* E, double* F, double* Rb, PIVOT pivot) {
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, i = lane & 15, g = lane >> 4, waves = (int)blockDim.x >> 6;
  auto put = [&](double* D, int ld, double4_t v) {
#pragma unroll
    for (int q = 0; q < 4; ++q) D[(g + 4 * q) * ld + i] = v[q];
  };
  auto get = [&](const double* D, int ld) {
    double4_t v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = D[(g + 4 * q) * ld + i];
    return v;
  };
  const double4_t zero = double4_t{0.0, 0.0, 0.0, 0.0};
  for (int J = 0; J < nb; ++J) {
    double* Sj = S + 16 * J * LD;                    // block row J
    __syncthreads();
    if (wave == 0) {
      double a[4];
      bool used = false;
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = Sj[(4 * q + g) * LD + 16 * J + i];
      pivot.begin(J);
      diagonal_steps<0>(a, i, g, used, pivot);
      pivot.end(J);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double f = 4 * q + g <= i ? a[q] : 0.0;
        F[(4 * q + g) * 16 + i] = f;
        E[(4 * q + g) * 16 + i] = used ? f : 0.0;
      }
    }
    __syncthreads();
    // row J of the factor, E^T S_JK, and of the inverse, -E R_JK
    for (int K = J + (INVERSE ? 1 : 0) + wave; K < nb; K += waves) {
      double* R = INVERSE ? Rb + 16 * K : Sj + 16 * K;
      const int LR = LD;
      const double4_t v = block_product(E, 1, 16, Sj + 16 * K, LD, zero);
      put(R, LR, v);
      if (INVERSE) {
        const double4_t u = block_product(E, 16, 1, R, LR, zero);
        put(Sj + 16 * K, LD, -u);
      }
    }
    __syncthreads();
    const double* R = INVERSE ? Rb : Sj;
    const int rest = nb - 1 - J, below = rest * rest, total = below + (INVERSE ? J * rest : 0);
    for (int b = wave; b < total; b += waves) {
      if (b < below) {
        const int I = J + 1 + b / rest, K = J + 1 + b % rest;
        if (K < I) continue;
        double* D = S + 16 * I * LD + 16 * K;
        const double4_t v = block_product(R + 16 * I, 1, LD, R + 16 * K, LD, zero);
        put(D, LD, get(D, LD) - v);
      } else {
        const int I = (b - below) / rest, K = J + 1 + (b - below) % rest;
        double* D = S + 16 * I * LD + 16 * K;
        put(D, LD, block_product(S + 16 * I * LD + 16 * J, LD, 1, Sj + 16 * K, LD, get(D, LD)));
      }
    }
    if (INVERSE) {
      __syncthreads();
      for (int I = wave; I <= J; I += waves) {
        double* D = S + 16 * I * LD + 16 * J;
        if (I < J) put(D, LD, block_product(D, LD, 1, F, 16, zero));
        else put(D, LD, get(F, 16));
      }
    }
  }
  __syncthreads();
}

// The decisions about the columns of a sketch.  Kept: scaled to length one; deferred: as the projections left it; dropped:
// cleared
struct SketchPivot {
  const double* scale;
  int *st, *pending;
  double* least;
  bool last;
  uint32_t dropped, kept, deferred;    // of the panel's columns
  double lowest;
  __device__ inline void begin(int J) {
    dropped = (uint32_t)__builtin_amdgcn_ballot_w64(scale[16 * J + (threadIdx.x & 15)] == 0.0);
    kept = deferred = 0;
  }
  __device__ inline double take(int j, double d, double& own) {
    const bool out = (dropped >> j) & 1u, keep = !out && d > FZ_ACCEPT;
    const double ri = keep ? inv_sqrt(d) : 0.0;
    own = keep ? ri : (out || last ? 0.0 : 1.0);
    lowest = keep ? fmin(lowest, d) : lowest;
    kept |= (keep ? 1u : 0u) << j;
    deferred |= (!keep && !out ? 1u : 0u) << j;
    return ri;
  }
  __device__ inline void end(int J) {
    const int t = threadIdx.x;
    if (t < 16) st[16 * J + t] = (kept >> t) & 1u ? FZ_KEPT : ((deferred >> t) & 1u && !last ? FZ_PENDING : FZ_DROPPED);
    if (t == 0) {
      *least = lowest;
      if (deferred) *pending = 1;
    }
  }
};

// The factor of a pass of the orthonormalisation, by one workgroup.  S: Gram matrix (upper blocks, rows of LD);
// Tinv (upper triangular): Y Tinv is the next Y.
template <int NB, int LD>
__device__ inline void cholesky_step(double* S, int l, double* Tinv, long long ldt, double* kept, int* state, int* done,
                                     int pass) {
  __shared__ double Rb[16 * LD], E[256], F[256], scale[16 * NB];
  __shared__ int st[16 * NB], pending;
  __shared__ double least;
  const int t = threadIdx.x, nb = (l + 15) >> 4, n16 = 16 * nb;
  const bool last = pass == FZ_QR_PASSES - 1;
  if (t < n16) {
    const double gg = t < l ? S[t * LD + t] : 0.0;
    double k2 = pass && t < l ? kept[t] : 1.0;
    int s0 = pass && t < l ? state[t] : FZ_PENDING;
    if (pass && s0 == FZ_PENDING) k2 *= gg;
    if (!(gg > 0.0) || k2 <= FZ_RANK_TOL2) s0 = FZ_DROPPED;
    scale[t] = s0 == FZ_DROPPED ? 0.0 : 1.0 / sqrt(gg);
    st[t] = s0;
    if (t < l) kept[t] = k2;
  }
  if (t == 0) {
    least = 1.0;
    pending = 0;
  }
  __syncthreads();
  for (int idx = t; idx < n16 * n16; idx += FZ_PASS_THREADS) {
    const int i = idx / n16, k = idx - i * n16;
    const double w = scale[i] * scale[k];
    S[i * LD + k] = w > 0.0 && (i >> 4) <= (k >> 4) ? S[i * LD + k] * w : 0.0;
  }
  block_cholesky<true>(S, LD, nb, E, F, Rb, SketchPivot{scale, st, &pending, &least, last, 0, 0, 0, 1.0});
  for (int idx = t; idx < l * l; idx += FZ_PASS_THREADS) {
    const int i = idx / l, k = idx - i * l;
    Tinv[(long long)i * ldt + k] = k >= i ? scale[i] * S[i * LD + k] : 0.0;
  }
  if (t < l) state[t] = st[t];
  if (t == 0) *done = pending == 0 && least > 0.5 ? pass + 1 : 1 << 30;
}

// ---------------------------------------------------------------------------------------
// The same for wider sketches: classical Gram-Schmidt, every column projected twice.  Y is [m][ld], l
// columns, l <= 256.  Workgroup b owns rows [b rpw, (b + 1) rpw), rpw <= 256, in every
// launch; sums over rows go through per-workgroup partials that every workgroup adds in the
// same order.  Three launches per column j:
//   phase 0: finish column j - 1 (scale by 1 / norm, or clear a column that the projections
//            took below the rank threshold); partial c1 = Q^T y_j, partial |y_j|^2
//   phase 1: y_j -= Q c1; partial c2 = Q^T y_j
//   phase 2: y_j -= Q c2; partial |y_j|^2
// and one more phase 0 with j = l that only finishes the last column.
// ---------------------------------------------------------------------------------------
struct CgsBuffers {
  double* c1;       // [n_groups][256]
  double* c2;       // [n_groups][256]
  double* norm;     // [n_groups]      |y_j|^2 after both projections
  double* norm0;    // [2][n_groups]   |y_j|^2 before, by parity of j
};

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

// sum of one value per thread over the block; every thread gets the result
__device__ inline double block_sum(double v, double* lds4) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = v;
  __syncthreads();
  return lds4[0] + lds4[1] + lds4[2] + lds4[3];
}

// dot[t] = sum over the rows [r0, r1) of Y[k][t] * ycol[k - r0] for every column t < j, by all 256
// threads: the rows are dealt to 256 / CW thread groups of CW >= j columns, whose partial sums
// meet in `part` (256 doubles of LDS); thread t < j returns the sum, in group order
__device__ inline double cgs_dots(const double* __restrict__ Y, long long ld, int r0, int r1, int j,
                                  const double* ycol, double* part) {
  const int t = threadIdx.x;
  const int CW = j <= 64 ? 64 : (j <= 128 ? 128 : 256), n_sub = 256 / CW;
  const int col = t & (CW - 1), sub = t / CW;
  double dot = 0.0;
  if (col < j) {
#pragma unroll 8
    for (int k = r0 + sub; k < r1; k += n_sub) dot += Y[(long long)k * ld + col] * ycol[k - r0];
  }
  __syncthreads();
  part[t] = dot;
  __syncthreads();
  double sum = 0.0;
  if (t < j)
    for (int sgrp = 0; sgrp < n_sub; ++sgrp) sum += part[sgrp * CW + t];
  return sum;
}

__global__ void __launch_bounds__(256) k_cgs(double* __restrict__ Y, long long ld, int m, int l, int rpw,
                                             int n_groups, int j, int phase, CgsBuffers cb) {
  __shared__ double c[256];
  __shared__ double ycol[256];
  __shared__ double red[4];
  const int t = threadIdx.x, b = blockIdx.x;
  const int r0 = b * rpw, r1 = min(m, r0 + rpw);
  if (phase == 0) {
    if (j > 0) {
      // finish column j - 1 (every workgroup adds the partial norms in the same order)
      double n2 = 0.0, n0 = 0.0;
      for (int gq = t; gq < n_groups; gq += 256) {
        n2 += cb.norm[gq];
        n0 += cb.norm0[(size_t)((j - 1) & 1) * n_groups + gq];
      }
      n2 = block_sum(n2, red);
      n0 = block_sum(n0, red);
      const double scale = (n2 > FZ_RANK_TOL2 * n0 && n2 > 0.0) ? 1.0 / sqrt(n2) : 0.0;
      for (int k = r0 + t; k < r1; k += 256) Y[(long long)k * ld + (j - 1)] *= scale;
      __syncthreads();       // (the scaled column is read below, by other threads)
    }
    if (j >= l) return;
    for (int k = r0 + t; k < r1; k += 256) ycol[k - r0] = Y[(long long)k * ld + j];
    __syncthreads();
    double nn = 0.0;
    const double dot = cgs_dots(Y, ld, r0, r1, j, ycol, c);
    cb.c1[(size_t)b * 256 + t] = dot;
    for (int k = r0 + t; k < r1; k += 256) nn += ycol[k - r0] * ycol[k - r0];
    nn = block_sum(nn, red);
    if (t == 0) cb.norm0[(size_t)(j & 1) * n_groups + b] = nn;
    return;
  }
  // phases 1 and 2: coefficients, in workgroup order
  const double* part = phase == 1 ? cb.c1 : cb.c2;
  double ct = 0.0;
  if (t < j) {
#pragma unroll 16
    for (int gq = 0; gq < n_groups; ++gq) ct += part[(size_t)gq * 256 + t];
  }
  c[t] = ct;
  __syncthreads();
  // sixteen lanes per row: y_k -= sum_i Q[k][i] c[i]   (every lane runs the same number of
  // rounds, so that the shuffles below see whole waves)
  const int slot = t >> 4, sub = t & 15;
  for (int kb = r0; kb < r1; kb += 16) {
    const int k = kb + slot;
    double sum = 0.0;
    if (k < r1)
      for (int i = sub; i < j; i += 16) sum += Y[(long long)k * ld + i] * c[i];
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (sub == 0 && k < r1) {
      const double y = Y[(long long)k * ld + j] - sum;
      Y[(long long)k * ld + j] = y;
      ycol[k - r0] = y;
    }
  }
  __syncthreads();
  if (phase == 1) {
    const double dot = cgs_dots(Y, ld, r0, r1, j, ycol, c);     // (c is free again: barrier inside)
    cb.c2[(size_t)b * 256 + t] = dot;
  } else {
    double nn = 0.0;
    for (int k = r0 + t; k < r1; k += 256) nn += ycol[k - r0] * ycol[k - r0];
    nn = block_sum(nn, red);
    if (t == 0) cb.norm[b] = nn;
  }
}

// ---------------------------------------------------------------------------------------
// SVD of Bs [l][d] by one-sided Jacobi rotations of its rows (Hestenes): a rotation of rows
// (a, b) makes them orthogonal; at convergence row a is sigma_a v_a^T and the accumulated
// rotations, applied to the columns of Um, leave U~ in Um.  One launch per round of a round-robin schedule over n = l rounded up to even players
// (n / 2 disjoint pairs, a workgroup each); a sweep is n - 1 rounds.  counters[w] counts the
// rotations of sweep w; once a sweep made none, the launches of later sweeps return at once.
// ---------------------------------------------------------------------------------------
constexpr int FZ_MAX_SWEEPS = 16;
constexpr double FZ_JACOBI_TOL2 = 1e-28;     // rotate while (a.b)^2 > tol^2 |a|^2 |b|^2, tol = 1e-14

constexpr int FZ_JT = 1024;       // threads of a Jacobi workgroup
constexpr int FZ_JC = 4;          // elements of each row a thread keeps in registers

__global__ void __launch_bounds__(FZ_JT) k_jacobi_round(double* __restrict__ Bs, long long ldb, int d,
                                                        double* __restrict__ Um, long long ldu, int l, int n,
                                                        int round, int sweep, int* counters) {
  __shared__ double red[3][FZ_JT / 64];
  if (sweep > 0 && counters[sweep - 1] == 0) return;
  const int k = blockIdx.x, t = threadIdx.x;
  int a, b;
  if (k == 0) { a = n - 1; b = round; }
  else { a = (round + k) % (n - 1); b = (round - k + (n - 1)) % (n - 1); }
  if (a >= l || b >= l) return;      // the odd player out
  double* ra = Bs + (long long)a * ldb;
  double* rb = Bs + (long long)b * ldb;
  double xa[FZ_JC], xb[FZ_JC];
  double aa = 0.0, bb = 0.0, ab = 0.0;
#pragma unroll
  for (int c = 0; c < FZ_JC; ++c) {
    const int i = t + c * FZ_JT;
    xa[c] = i < d ? ra[i] : 0.0;
    xb[c] = i < d ? rb[i] : 0.0;
    aa += xa[c] * xa[c]; bb += xb[c] * xb[c]; ab += xa[c] * xb[c];
  }
  for (int i = t + FZ_JC * FZ_JT; i < d; i += FZ_JT) {
    const double x = ra[i], y = rb[i];
    aa += x * x; bb += y * y; ab += x * y;
  }
  aa = wave_sum(aa); bb = wave_sum(bb); ab = wave_sum(ab);
  if ((t & 63) == 0) { red[0][t >> 6] = aa; red[1][t >> 6] = bb; red[2][t >> 6] = ab; }
  __syncthreads();
  aa = bb = ab = 0.0;
#pragma unroll
  for (int w = 0; w < FZ_JT / 64; ++w) { aa += red[0][w]; bb += red[1][w]; ab += red[2][w]; }
  if (!(ab * ab > FZ_JACOBI_TOL2 * aa * bb)) return;
  if (t == 0) atomicAdd(&counters[sweep], 1);
  const double zeta = (bb - aa) / (2.0 * ab);
  const double tt = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
  const double cs = 1.0 / sqrt(1.0 + tt * tt), sn = cs * tt;
#pragma unroll
  for (int c = 0; c < FZ_JC; ++c) {
    const int i = t + c * FZ_JT;
    if (i < d) {
      ra[i] = cs * xa[c] - sn * xb[c];
      rb[i] = sn * xa[c] + cs * xb[c];
    }
  }
  for (int i = t + FZ_JC * FZ_JT; i < d; i += FZ_JT) {
    const double x = ra[i], y = rb[i];
    ra[i] = cs * x - sn * y;
    rb[i] = sn * x + cs * y;
  }
  for (int i = t; i < l; i += FZ_JT) {
    double* u = Um + (long long)i * ldu;
    const double x = u[a], y = u[b];
    u[a] = cs * x - sn * y;
    u[b] = sn * x + cs * y;
  }
}

// The same for up to FZ_SMALL rows, through the l x l Gram matrix G of the rows.  G = L L^T
// (Cholesky), and one-sided rotations V make the columns of Z = L V orthogonal: then G = Z Z^T,
// the columns of Z divided by their lengths are the rotation U itself, and nothing has to be
// collected beside Z.  One workgroup with Z in LDS: 16 lanes per pair of columns, all pairs of a
// round at once, one barrier per round.  U is applied to the long rows by one product, and the
// next pass starts from their new Gram matrix, which knows every small row relative to its own
// length: a second pass removes what the first one's rounding left (relative to the largest
// row), a third only runs when the second still found something to rotate.  Any orthogonal U is
// exact work whatever G was, so a pivot that is only rounding is replaced by FZ_PIVOT and costs
// convergence, not accuracy.  Up to FZ_DIRECT rows the first pass takes the road below instead, where it can.  80 rows of 3072:
// 510 us in seven to eight sweeps of 79 rounds, bound by issue and LDS (1600 cycles a round); two-sided rotations with three barriers a
// round followed by one launch per round on the long rows took 1830 + 1620 us.
constexpr int FZ_SVD_PASSES = 3;
constexpr int FZ_SMALL_SWEEPS = 12;
constexpr double FZ_LAST_SWEEP2 = 1e-15;
constexpr double FZ_QUIET2 = 1e-26;         // rows whose (a.b)^2 is below this share of |a|^2 |b|^2 need no further pass
constexpr double FZ_PIVOT = 1e-13;          // of a unit diagonal: below, the row's remainder is rounding

// sum over the 16 lanes of a DPP row, in every lane
template <int ROR> __device__ inline double row_rotate(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x120 | ROR, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x120 | ROR, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ inline double row_sum16(double v) {
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  v += row_rotate<1>(v);
  return v;
}

struct GramPivot {
  double* tiny;
  uint32_t rounding;                   // the panel's columns whose pivot is only that
  __device__ inline void begin(int) { rounding = 0; }
  __device__ inline double take(int j, double d, double& own) {
    const bool real = d > FZ_PIVOT;
    own = real ? inv_sqrt(d) : 0.0;
    rounding |= (real ? 0u : 1u) << j;
    return own;
  }
  __device__ inline void end(int J) {
    const int t = threadIdx.x;
    if (t < 16 && ((rounding >> t) & 1u)) tiny[16 * J + t] = sqrt(FZ_PIVOT);
  }
};

__device__ inline double load_device(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_device(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// U from its columns in the rows of Zt; Um_new = Um_old U (pass 0: U)
template <int LD>
__device__ inline void store_rotation(const double* Zt, int l, double* __restrict__ U, const double* __restrict__ Um_old,
                                      double* __restrict__ Um_new, long long ldu, int pass) {
  const int t = threadIdx.x;
  for (int idx = t; idx < l * l; idx += FZ_PASS_THREADS) {
    const int i = idx / l, k = idx - i * l;
    double v = Zt[k * LD + i];
    U[(long long)i * ldu + k] = v;
    if (pass > 0) {
      v = 0.0;
      for (int c = 0; c < l; ++c) v += Um_old[(long long)i * ldu + c] * Zt[k * LD + c];
    }
    Um_new[(long long)i * ldu + k] = v;
  }
}

// NQ: 16-element pieces of a column (l <= 16 NQ).  Zt: Gram matrix (upper blocks, rows of LD), then Zt[k] is column k
// of Z.  Returns true, with Zt's diagonal as it was, if the rows are orthogonal already; else U is the rotation, and
// Um_new = Um_old U the rotations so far (pass 0: U).
template <int NQ, int LD>
__device__ inline bool rotation_step(double* Zt, int l, double* __restrict__ U, const double* __restrict__ Um_old,
                                     double* __restrict__ Um_new, long long ldu, int pass) {
  constexpr int LW = 16 * NQ;
  __shared__ double E[256], F[256], len2[16 * NQ], tiny[16 * NQ];
  __shared__ int rotated[2];
  const int t = threadIdx.x;
  if (t < LW) {
    const double gg = t < l ? Zt[t * LD + t] : 0.0;
    len2[t] = gg > 0.0 ? sqrt(gg) : 0.0;            // (row lengths for now)
    tiny[t] = 0.0;
  }
  if (t == 0) rotated[0] = 0;
  __syncthreads();
  for (int idx = t; idx < LW * LW; idx += FZ_PASS_THREADS) {
    const int i = idx / LW, k = idx - i * LW;
    const double w = len2[i] * len2[k];
    const bool upper = (i >> 4) <= (k >> 4);
    const double c = upper && w > 0.0 ? Zt[i * LD + k] / w : 0.0;
    if (i != k && c * c > FZ_QUIET2) rotated[0] = 1;
  }
  __syncthreads();
  if (pass > 0 && rotated[0] == 0) return true;     // already orthogonal: nothing to apply
  for (int idx = t; idx < LW * LW; idx += FZ_PASS_THREADS) {
    const int i = idx / LW, k = idx - i * LW;
    const double w = len2[i] * len2[k];
    Zt[i * LD + k] = (i >> 4) <= (k >> 4) && w > 0.0 ? Zt[i * LD + k] / w : 0.0;
  }
  __syncthreads();
  {
    block_cholesky<false>(Zt, LD, NQ, E, F, nullptr, GramPivot{tiny, 0});
    // column j of Z: row j of the factor, every element scaled back by its row's length
    for (int idx = t; idx < LW * LW; idx += FZ_PASS_THREADS) {
      const int j = idx / LW, k = idx - j * LW;
      Zt[j * LD + k] = k < j ? 0.0 : (k == j && tiny[j] > 0.0 ? tiny[j] : Zt[j * LD + k]) * len2[k];
    }
  }
  const int n = (l + 1) & ~1, pairs = n / 2, p = t >> 4, sub = t & 15;
  for (int sweep = 0; sweep < FZ_SMALL_SWEEPS; ++sweep) {
    __syncthreads();
    if (t == 0) rotated[sweep & 1] = 0;
    for (int i = p; i < l; i += 64) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const double x = Zt[i * LD + sub + 16 * q];
        s += x * x;
      }
      s = row_sum16(s);
      if (sub == 0) len2[i] = s;
    }
    for (int round = 0; round < n - 1; ++round) {
      __syncthreads();
      if (p >= pairs) continue;
      int a, b;
      if (p == 0) { a = n - 1; b = round; }
      else {
        a = round + p;
        if (a >= n - 1) a -= n - 1;
        b = round - p;
        if (b < 0) b += n - 1;
      }
      if (a >= l || b >= l) continue;               // the odd player out
      double* za = Zt + a * LD + sub;
      double* zb = Zt + b * LD + sub;
      double xa[NQ], xb[NQ], ab = 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        xa[q] = za[16 * q];
        xb[q] = zb[16 * q];
        ab += xa[q] * xb[q];
      }
      ab = row_sum16(ab);
      const double aa = len2[a], bb = len2[b];
      if (!(ab * ab > FZ_JACOBI_TOL2 * aa * bb)) continue;
      // the tangent of the angle from the hardware's estimates (the next sweep takes what they
      // leave), cosine and sine to working precision: they must belong to one angle
      const double zeta = (bb - aa) * 0.5 * __builtin_amdgcn_rcp(ab);
      const double az = fmin(fabs(zeta), 1e100), h = __builtin_fma(az, az, 1.0);
      const double tt = copysign(__builtin_amdgcn_rcp(az + h * __builtin_amdgcn_rsq(h)), zeta);
      const double cs = inv_sqrt(__builtin_fma(tt, tt, 1.0)), sn = cs * tt;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        za[16 * q] = cs * xa[q] - sn * xb[q];
        zb[16 * q] = sn * xa[q] + cs * xb[q];
      }
      if (sub == 0) {
        len2[a] = fmax(aa - tt * ab, 0.0);
        len2[b] = bb + tt * ab;
        // (rotations this small leave the square of it: no other sweep has to look)
        if (ab * ab > FZ_LAST_SWEEP2 * aa * bb) rotated[sweep & 1] = 1;
      }
    }
    __syncthreads();
    if (rotated[sweep & 1] == 0) break;
  }
  __syncthreads();
  // U = Z with columns of length one (a zero row of G is a direction of its own)
  for (int i = p; i < l; i += 64) {
    double s = 0.0;
    for (int q = 0; q < NQ; ++q) {
      const double x = Zt[i * LD + sub + 16 * q];
      s += x * x;
    }
    s = row_sum16(s);
    const double is = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
    for (int q = 0; q < NQ; ++q) {
      const int k = sub + 16 * q;
      Zt[i * LD + k] = s > 0.0 ? Zt[i * LD + k] * is : (k == i ? 1.0 : 0.0);
    }
  }
  __syncthreads();
  store_rotation<LD>(Zt, l, U, Um_old, Um_new, ldu, pass);
  return false;
}

// ---------------------------------------------------------------------------------------
// The first rotation of up to FZ_DIRECT rows by another road: the eigenvectors of the Gram matrix, through its
// tridiagonal form (Householder), bisection on sign counts of the leading minors, one twisted factorisation per eigenvalue
// (Parlett and Dhillon: the solve starts at the row where it leaves the least residual), the
// reflections applied backwards, and U <- U (3 - U^T U) / 2, which makes vectors of close eigenvalues
// orthogonal to rounding.  A rotation to the accuracy of the largest row is all that the first pass has to give: any orthogonal U
// is exact work, the next pass measures what is left on the rows themselves and rotates the rest away.  So a
// spectrum that spans more than FZ_DIRECT_RANGE, and vectors that come out far from orthogonal
// (eigenvalues equal to rounding), are left to the rotations below.  One workgroup: a chain of barriers (two a
// column) and of dependent float64 instructions.
// 80 rows of 3072, us: 155 (tridiagonal 64, bisection 37, twisted factorisations 32, reflections 12, orthogonality 10) where
// the rotations take 510; what the rows have left is then 5e-16 of their lengths.
// ---------------------------------------------------------------------------------------
// (both matrices of 96 columns, with the pads that spread their columns over the banks, are past the LDS)
constexpr int FZ_DIRECT = 80;
constexpr double FZ_DIRECT_RANGE = 1e-6;     // smallest over largest eigenvalue
constexpr double FZ_ORTHO_TRIES = 0.25, FZ_ORTHO_ONE = 1e-8;   // |U^T U - 1| that can be mended at all, and by one step

template <int CTRL> __device__ inline double dpp_move(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// sum over eight neighbouring lanes, in all of them: lanes ^ 1, ^ 2, and the mirror image
__device__ inline double sum8(double v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  return v;
}
// 1 / x to working precision: the hardware's estimate and two Newton steps
__device__ inline double inv(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
  return __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
}
__device__ inline double pivot_guard(double q) { return fabs(q) < 0x1p-60 ? copysign(0x1p-60, q) : q; }

// f(0), .. f(N - 1) with compile-time indexes
template <class F, int... I> __device__ __attribute__((always_inline)) inline void static_for(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __attribute__((always_inline)) inline void static_for(F f) {
  static_for(f, std::make_integer_sequence<int, N>{});
}

// How many eigenvalues of the tridiagonal matrix lie below x: sign changes of its leading minors,
// p_i = (d_i - x) p_i-1 - e_i-1^2 p_i-2, their sign bits collected in a word.  de[i] = {d_i, -e_i-1^2}, zeros behind l;
// sixteen elements travel in the lanes of a row and are broadcast from there.  One multiply-add of a step waits for the
// step before (with two more of them in that chain 4100 cycles for 80 steps, now 3100).
__device__ inline int eigenvalues_below(const double2* de, int l, double x) {
  double p = 1.0, pp = 0.0;
  int below = 0;
  auto high = [](double v) { return (uint32_t)(__builtin_bit_cast(unsigned long long, v) >> 32); };
  for (int i0 = 0; i0 < l; i0 += 16) {
    const int n = min(16, l - i0);
    const double2 v = de[i0 + (threadIdx.x & 15)];
    uint32_t signs = high(p) >> 31;                  // of the minor before the chunk, then of its own
    static_for<16>([&](auto J) __attribute__((always_inline)) {      // (behind l too: no branch parts the steps)
      constexpr int j = J.value;
      const double next = __builtin_fma(row_broadcast<j>(v.x) - x, p, row_broadcast<j>(v.y) * pp);
      pp = p;
      p = next;
      signs = __builtin_amdgcn_alignbit(signs, high(p), 31);
      if constexpr (j == 7 || j == 15) {
        const int ex = max(__builtin_amdgcn_frexp_exp(p), __builtin_amdgcn_frexp_exp(pp));
        p = __builtin_amdgcn_ldexp(p, -ex);
        pp = __builtin_amdgcn_ldexp(pp, -ex);
      }
    });
    below += __popc((signs ^ (signs >> 1)) & (((1u << n) - 1u) << (16 - n)));
  }
  return below;
}

// Zt: Gram matrix (upper blocks, rows of LD).  True: eigenvector k is row k of Zt, rows of LV, V undefined; false: Zt
// undefined.  V: LDS,
// 16 NQ rows of LV (lanes that go down a column of either meet other banks).
template <int NQ, int LD, int LV>
__device__ inline bool eigenvectors(double* Zt, double* V, int l) {
  constexpr int LW = 16 * NQ, E = 2 * NQ;
  __shared__ double pb[2 * LW], beta[LW], lam[LW], off[LW], len[LW];
  __shared__ double2 de[LW];
  __shared__ unsigned long long worst;
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, row = t >> 3, sub = t & 7;
  const int i16 = lane & 15, g = lane >> 4;
  // lanes 8 row .. 8 row + 7 hold a row of the matrix: columns sub + 8 q; scaled by a power of two to a largest element of about one
  if (t == 0) {
    double top = 0.0;
    for (int i = 0; i < l; ++i) top = fmax(top, Zt[i * LD + i]);
    pb[0] = top;
  }
  __syncthreads();
  const double top = pb[0];
  __syncthreads();
  if (!(top > 0.0) || !(top < 1e300)) return false;
  const int scale = -__builtin_amdgcn_frexp_exp(top);
  double A[E];
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const int c = sub + 8 * q;
    const bool upper = (row >> 4) <= (c >> 4);
    A[q] = row < l && c < l ? __builtin_amdgcn_ldexp(upper ? Zt[row * LD + c] : Zt[c * LD + row], scale) : 0.0;
  }
  if (t < LW) {
    de[t] = make_double2(0.0, 0.0);
    beta[t] = off[t] = pb[t] = 0.0;
  }
  // H_k = 1 - beta_k v_k v_k^T takes column k's elements behind k + 1 to zero: its vector, by the wave of row k, an element or
  // two per lane (by the row's eight lanes, ten elements each and their selects, a column took 2700 cycles, now 2000)
  auto reflect = [&](int k) {
    if (row == k) {
#pragma unroll
      for (int q = 0; q < E; ++q) pb[LW + sub + 8 * q] = A[q];
    }
    __builtin_amdgcn_wave_barrier();
    constexpr int NE = (LW + 63) / 64;
    const double* x = pb + LW;
    double e[NE], s2 = 0.0;
#pragma unroll
    for (int n = 0; n < NE; ++n) {
      const int c = lane + 64 * n;
      e[n] = x[min(c, LW - 1)];
      const double z = c > k + 1 && c < LW ? e[n] : 0.0;
      s2 = __builtin_fma(z, z, s2);
    }
    const double x0 = k + 1 < l ? x[min(k + 1, LW - 1)] : 0.0, dk = x[k];
    s2 = row_sum16(s2);
    s2 = (read_lane(s2, 0) + read_lane(s2, 16)) + (read_lane(s2, 32) + read_lane(s2, 48));
    double alpha = x0, v0 = 0.0, b = 0.0;
    if (s2 > 0.0) {
      const double n2 = __builtin_fma(x0, x0, s2), rs = inv_sqrt(n2);
      double n = n2 * rs;
      n = __builtin_fma(__builtin_fma(-n, n, n2), 0.5 * rs, n);
      alpha = x0 >= 0.0 ? -n : n;
      v0 = x0 - alpha;
      b = inv(n * (n + fabs(x0)));
    }
#pragma unroll
    for (int n = 0; n < NE; ++n) {
      const int c = lane + 64 * n;
      const double head = c == k + 1 ? v0 : 0.0, tail = b > 0.0 ? e[n] : 0.0;
      if (c < LW) V[k * LV + c] = c > k + 1 ? tail : head;
    }
    if (lane == 0) {
      de[k].x = dk;
      beta[k] = b;
      off[k] = alpha;
      if (k + 1 < l) de[k + 1].y = -alpha * alpha;
    }
  };
  __syncthreads();
  if (wave == 0) reflect(0);
  __syncthreads();
  // A <- H_k A H_k = A - v w^T - w v^T, w = p - (beta / 2) (p.v) v, p = beta A v
  static_for<NQ>([&](auto Q) {
    constexpr int Q0 = 2 * Q.value;                  // columns up to 8 Q0 are done (a copy of the code for every 16: each is fetched once)
    for (int k = 8 * Q0; k < min(8 * Q0 + 16, l - 2); ++k) {
      const bool alive = 8 * wave + 7 > k && 8 * wave < l;       // (uniform) rows behind k are in this wave
      double v[E], vr = 0.0, b = 0.0;
      if (alive) {
        double part[2] = {0.0, 0.0};
#pragma unroll
        for (int q = Q0; q < E; ++q) v[q] = V[k * LV + sub + 8 * q];
        vr = V[k * LV + row];
        b = beta[k];
#pragma unroll
        for (int q = Q0; q < E; ++q) part[q & 1] = __builtin_fma(A[q], v[q], part[q & 1]);
        const double pr = sum8(part[0] + part[1]);
        if (sub == 0) pb[row] = b * pr;
      }
      __syncthreads();
      if (alive) {
        double w[E], part[2] = {0.0, 0.0};
#pragma unroll
        for (int q = Q0; q < E; ++q) w[q] = pb[sub + 8 * q];
        const double pr = pb[row];
#pragma unroll
        for (int q = Q0; q < E; ++q) part[q & 1] = __builtin_fma(v[q], w[q], part[q & 1]);
        const double K = 0.5 * b * sum8(part[0] + part[1]);
        const double wr = __builtin_fma(-K, vr, pr);
#pragma unroll
        for (int q = Q0; q < E; ++q) A[q] = __builtin_fma(-wr, v[q], __builtin_fma(-vr, __builtin_fma(-K, v[q], w[q]), A[q]));
        if (wave == (k + 1) >> 3) reflect(k + 1);
      }
      __syncthreads();
    }
  });
  if (wave == (l - 1) >> 3) reflect(l - 1);
  __syncthreads();
  // eigenvalue k by three points at a time, a lane each: two bits a round
  if (wave < 4) {
    const int k = 21 * wave + lane / 3, pt = lane - lane / 3 * 3, lead = lane / 3 * 3;
    double lo = 1e300, hi = -1e300;
    for (int i = lane; i < l; i += 64) {
      const double r = (i > 0 ? fabs(off[i - 1]) : 0.0) + fabs(off[i]);
      lo = fmin(lo, de[i].x - r);
      hi = fmax(hi, de[i].x + r);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo = fmin(lo, __shfl_xor(lo, o, 64));
      hi = fmax(hi, __shfl_xor(hi, o, 64));
    }
    lo -= 0x1p-48;
    hi += 0x1p-48;
    for (int it = 0; it < 29; ++it) {
      const double step = 0.25 * (hi - lo);
      const int n = eigenvalues_below(de, l, __builtin_fma((double)(pt + 1), step, lo));
      const int n0 = __shfl(n, lead, 64), n1 = __shfl(n, lead + 1, 64), n2 = __shfl(n, lead + 2, 64);
      const int j = n0 > k ? 0 : (n1 > k ? 1 : (n2 > k ? 2 : 3));      // the quarter that eigenvalue k is in
      hi = j == 3 ? hi : __builtin_fma((double)(j + 1), step, lo);
      lo = __builtin_fma((double)j, step, lo);
    }
    if (pt == 0 && lane < 63 && k < l) lam[k] = 0.5 * (lo + hi);
  }
  __syncthreads();
  if (!(lam[0] > FZ_DIRECT_RANGE * lam[l - 1])) return false;
  // T - lambda = L+ D+ L+^T = U- D- U-^T, lane t: eigenvalue t; D+ in column t of Zt, and once the row `at` of the least
  // residual is known, D- behind it; then the vector from that row both ways in their place.  (D- in global memory, and every
  // loop unrolled: 50 us, most of it for code that is fetched and run once.)
  if (t < 128 && t < l) {
    const double x = lam[t];
    double* z = Zt + t;
    double r = 0.0;
    for (int i = 0; i < l; ++i) {
      const double q = pivot_guard(__builtin_fma(de[i].y, r, de[i].x - x));       // (de[0].y is zero)
      r = inv(q);
      z[i * LV] = q;
    }
    double least = 1e300, e2 = 0.0;
    int at = 0;
    r = 0.0;
    for (int i = l - 1; i >= 0; --i) {
      const double d = de[i].x - x, q = pivot_guard(__builtin_fma(e2, r, d));
      const double gm = fabs(z[i * LV] + q - d);
      at = gm < least ? i : at;
      least = fmin(gm, least);
      r = inv(q);
      e2 = de[i].y;
    }
    e2 = r = 0.0;
    for (int i = l - 1; i > 0; --i) {
      const double q = pivot_guard(__builtin_fma(e2, r, de[i].x - x));
      r = inv(q);
      e2 = de[i].y;
      if (i > at) z[i * LV] = q;
    }
    double v = 1.0, n2 = 1.0;
    for (int i = l - 1; i >= 0; --i) {
      const double f = -off[i] * inv(z[i * LV]) * v;
      v = i < at ? f : v;
      n2 = i < at ? __builtin_fma(v, v, n2) : n2;
      if (i <= at) z[i * LV] = v;
    }
    v = 1.0;
    for (int i = 1; i < l; ++i) {
      const double f = -off[i - 1] * inv(z[i * LV]) * v;
      v = i > at ? f : v;
      n2 = i > at ? __builtin_fma(v, v, n2) : n2;
      if (i > at) z[i * LV] = v;
    }
    len[t] = inv_sqrt(n2);
  }
  __syncthreads();
  // back through the reflections: lanes 8 row .. hold vector `row`
  if (row < l) {
#pragma unroll
    for (int q = 0; q < E; ++q) A[q] = sub + 8 * q < l ? Zt[(sub + 8 * q) * LV + row] * len[row] : 0.0;
    static_for<NQ>([&](auto Q) {
      constexpr int Q0 = E - 2 - 2 * Q.value;
      for (int k = min(8 * Q0 + 15, l - 3); k >= 8 * Q0; --k) {
        double v[E], part[2] = {0.0, 0.0};
#pragma unroll
        for (int q = Q0; q < E; ++q) v[q] = V[k * LV + sub + 8 * q];
        const double b = beta[k];
#pragma unroll
        for (int q = Q0; q < E; ++q) part[q & 1] = __builtin_fma(v[q], A[q], part[q & 1]);
        const double dot = -b * sum8(part[0] + part[1]);
#pragma unroll
        for (int q = Q0; q < E; ++q) A[q] = __builtin_fma(dot, v[q], A[q]);
      }
    });
  }
  __syncthreads();
  if (row < LW) {
#pragma unroll
    for (int q = 0; q < E; ++q) Zt[row * LV + sub + 8 * q] = row < l ? A[q] : 0.0;
  }
  // to orthogonal vectors: V = Zt Zt^T, Zt <- (3 - V) / 2 Zt
  constexpr int WAVES = FZ_PASS_THREADS / 64, ALL = NQ * NQ, MY = (ALL + WAVES - 1) / WAVES;
  for (int it = 0; it < 4; ++it) {
    if (t == 0) worst = 0;
    __syncthreads();
    double4_t out[MY];
    double far_off = 0.0;
#pragma unroll
    for (int m = 0; m < MY; ++m) {
      const int b = wave + WAVES * m, I = b / NQ, K = b - I * NQ;
      out[m] = double4_t{0.0, 0.0, 0.0, 0.0};
      if (b < ALL) {
#pragma unroll
        for (int e = 0; e < 4 * NQ; ++e)
          out[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(Zt[(16 * I + i16) * LV + 4 * e + g], Zt[(16 * K + i16) * LV + 4 * e + g], out[m], 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * I + g + 4 * v, c = 16 * K + i16;
          const double o = r < l && c < l ? out[m][v] - (r == c ? 1.0 : 0.0) : 0.0;
          far_off = fabs(o) < 1.0 ? fmax(far_off, fabs(o)) : 1.0;       // (a NaN counts as one)
          V[r * LV + c] = r == c ? 1.0 - 0.5 * o : -0.5 * o;
        }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) far_off = fmax(far_off, __shfl_xor(far_off, o, 64));
    if (lane == 0) atomicMax(&worst, __builtin_bit_cast(unsigned long long, far_off));
    __syncthreads();
    const double dev = __builtin_bit_cast(double, worst);
    if (!(dev < FZ_ORTHO_TRIES)) return false;
#pragma unroll
    for (int m = 0; m < MY; ++m) {
      const int b = wave + WAVES * m, I = b / NQ, K = b - I * NQ;
      out[m] = double4_t{0.0, 0.0, 0.0, 0.0};
      if (b < ALL) {
#pragma unroll
        for (int e = 0; e < 4 * NQ; ++e)
          out[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(V[(16 * I + i16) * LV + 4 * e + g], Zt[(4 * e + g) * LV + 16 * K + i16], out[m], 0, 0, 0);
      }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MY; ++m) {
      const int b = wave + WAVES * m, I = b / NQ, K = b - I * NQ;
      if (b < ALL) {
#pragma unroll
        for (int v = 0; v < 4; ++v) Zt[(16 * I + g + 4 * v) * LV + 16 * K + i16] = out[m][v];
      }
    }
    __syncthreads();
    if (dev < FZ_ORTHO_ONE) return true;
  }
  return false;
}

// ---------------------------------------------------------------------------------------
// A pass of the orthonormalisation (rows of Y) or of the rotations (SVD: rows of Bs^T), one launch: every workgroup
// takes its rows through LDS, 64 at a time, multiplies them with the factor of the pass before, stores them
// and adds their part of the new Gram matrix; the workgroup that finds all others counted
// adds the parts and takes the next factor from the sum.  As the launches gram, sum, factor and product a pass that had nothing
// left to do cost four times 4.4 us (queued launches follow each other no faster), and there are four such passes for an
// ordinary sketch.  Parts are added in two levels of about the square root of the workgroups, in workgroup order, so that no
// workgroup reads all of them (80 parts of 30 KB at 80 columns); they travel past the L2s (device-scope stores,
// a wait for them, a count).  The counts start at zero and whoever was last puts the zero back.  Nothing waits.
// pass 0 adds the slices of the product before it into Y instead of applying a factor.
// 5120 x 80, us: a pass 80 -> 52 (25 of them the factor, 9 the sum of the parts), a pass with nothing to do 18.5 -> 4.5.
// ---------------------------------------------------------------------------------------
struct PassArgs {
  double* Y;               // [rows][ld]
  const double* slices;    // [n_slices][rows][ld], read by pass 0
  double* factor;          // [l][ld]
  double* parts;           // [workgroups + groups][blocks][256]
  int* counters;           // [groups + 1]
  int rows, l, ld, n_slices;
  int rows_per_wg, group, n_groups;     // rows of a workgroup (a multiple of 64), workgroups of a group
  int* done;
  int pass, passes;
  // orthonormalisation
  double* kept;
  int* state;
  // rotations; what the last pass leaves: singular values and their order, l x r matrix that takes Q to A
  double* Um[2];           // pass p writes Um[p & 1]
  int* sel;                // which of them holds the rotations
  double* sigma_sorted;
  int* perm;
  double* sigma_out;       // or NULL
  double* lift;            // [l][r16]
  int r, r16;
};
constexpr int FZ_PASS_ROWS = 64, FZ_PASS_WGS = 128, FZ_PASS_GROUP = 12;
constexpr int FZ_COUNTERS = 16;          // at least FZ_PASS_GROUP + 1, and FZ_MAX_SWEEPS

// the caller's stores are out and it is counted; true for the workgroup that was last of n
__device__ inline bool last_of(int* counter, int n) {
  __shared__ int last;
  vm_wait<0>();
  __syncthreads();
  if (threadIdx.x == 0) {
    last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
    if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  return last != 0;
}

// The singular values from the Gram matrix of orthogonal rows (its diagonal), their order (see
// rank_of), and P[i][jr] = U~[i][perm jr] sqrt(sigma_jr), the l x r matrix that takes Q to A (Alg. 1, lift and balance)
__device__ inline void sort_and_lift(const PassArgs& a, const double* S, int LD) {
  __shared__ double sigma[FZ_SMALL];
  __shared__ int order[FZ_SMALL];
  const int t = threadIdx.x;
  if (t < a.l) {
    const double s = S[t * LD + t];
    const int rank = rank_of([&](int b) { return S[b * LD + b]; }, a.l, t);
    const double sg = sqrt(s);
    sigma[rank] = sg;
    order[rank] = t;
    a.sigma_sorted[rank] = sg;
    a.perm[rank] = t;
    if (a.sigma_out) a.sigma_out[rank] = sg;
  }
  __syncthreads();
  const double* Um = a.Um[*a.sel];
  for (int idx = t; idx < a.l * a.r; idx += FZ_PASS_THREADS) {
    const int i = idx / a.r, jr = idx - i * a.r;
    a.lift[(long long)i * a.r16 + jr] = Um[(long long)i * a.ld + order[jr]] * sqrt(sigma[jr]);
  }
}

template <int NB, bool SVD>
__global__ void __launch_bounds__(FZ_PASS_THREADS) k_pass(PassArgs a) {
  constexpr int LW = 16 * NB, LT = LW + 2, LD = SVD ? LW + (NB > 6 ? 4 : 16) : LW + 2;   // (the pad spreads columns over the banks)
  constexpr int WAVES = FZ_PASS_THREADS / 64, BLOCKS = NB * (NB + 1) / 2, GB = (BLOCKS + WAVES - 1) / WAVES;
  constexpr int RBS = FZ_PASS_ROWS / 16, TASKS = RBS * NB, AT = (TASKS + WAVES - 1) / WAVES;
  constexpr int S_SIZE = LW * LD > FZ_PASS_ROWS * LT ? LW * LD : FZ_PASS_ROWS * LT;
  __shared__ double S[S_SIZE];         // 64 rows of Y, then the Gram matrix
  const bool apply = a.pass > 0;
  const int done = apply ? *a.done : 0;
  if (apply && done < a.pass) return;
  const bool gram = SVD || !apply || (a.pass < a.passes && done != a.pass);
  const int t = threadIdx.x, lane = t & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wg = blockIdx.x;
  auto block_at = [&](int b, int& I, int& K) {
    for (I = 0; b >= NB - I; ++I) b -= NB - I;
    K = I + b;
  };
  double4_t acc[GB];
#pragma unroll
  for (int q = 0; q < GB; ++q) acc[q] = double4_t{0.0, 0.0, 0.0, 0.0};
  const int r_end = min(a.rows, (wg + 1) * a.rows_per_wg);
  for (int r0 = wg * a.rows_per_wg; r0 < r_end; r0 += FZ_PASS_ROWS) {
    for (int idx = t; idx < FZ_PASS_ROWS * LW / 2; idx += FZ_PASS_THREADS) {
      const int row = idx / (LW / 2), c = 2 * (idx - row * (LW / 2));
      double2 v = make_double2(0.0, 0.0);
      if (r0 + row < r_end && c < a.l) {
        const long long at = (long long)(r0 + row) * a.ld + c;
        if (apply) {
          v = *(const double2*)(a.Y + at);
        } else {
#pragma unroll 4
          for (int sl = 0; sl < a.n_slices; ++sl) {
            const double2 p = *(const double2*)(a.slices + (long long)sl * a.rows * a.ld + at);
            v.x += p.x;
            v.y += p.y;
          }
          *(double2*)(a.Y + at) = v;
        }
        if (c + 1 >= a.l) v.y = 0.0;
      }
      S[row * LT + c] = v.x;
      S[row * LT + c + 1] = v.y;
    }
    __syncthreads();
    if (apply) {
      double4_t out[AT];
#pragma unroll
      for (int q = 0; q < AT; ++q) {
        const int task = wave + WAVES * q, rb = task % RBS, cb = task / RBS, col = 16 * cb + i;
        out[q] = double4_t{0.0, 0.0, 0.0, 0.0};
        if (task < TASKS) {
          for (int kb = 0; kb < (SVD ? NB : cb + 1); ++kb) {
            double f[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int ch = 16 * kb + 4 * e + g;
              f[e] = ch < a.l && col < a.l ? a.factor[(long long)ch * a.ld + col] : 0.0;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
              out[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(S[(16 * rb + i) * LT + 16 * kb + 4 * e + g], f[e], out[q], 0, 0, 0);
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < AT; ++q) {
        const int task = wave + WAVES * q, rb = task % RBS, cb = task / RBS, col = 16 * cb + i;
        if (task < TASKS) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = 16 * rb + g + 4 * v;
            S[row * LT + col] = out[q][v];
            if (r0 + row < r_end && col < a.l) a.Y[(long long)(r0 + row) * a.ld + col] = out[q][v];
          }
        }
      }
      __syncthreads();
    }
    if (gram) {
#pragma unroll
      for (int q = 0; q < GB; ++q) {
        const int b = wave + WAVES * q;
        if (b < BLOCKS) {
          int I, K;
          block_at(b, I, K);
#pragma unroll
          for (int e = 0; e < FZ_PASS_ROWS / 4; ++e)
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(S[(4 * e + g) * LT + 16 * I + i], S[(4 * e + g) * LT + 16 * K + i],
                                                          acc[q], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }
  if (!gram) return;
  constexpr int SIZE = BLOCKS * 256;   // a part: block after block, register after register
#pragma unroll
  for (int q = 0; q < GB; ++q) {
    const int b = wave + WAVES * q;
    if (b < BLOCKS) {
#pragma unroll
      for (int v = 0; v < 4; ++v) store_device(a.parts + (long long)wg * SIZE + b * 256 + v * 64 + lane, acc[q][v]);
    }
  }
  const int grp = wg / a.group, first = grp * a.group, members = min(a.group, (int)gridDim.x - first);
  auto sum = [&](const double* p, int n, int e) {
    double v[FZ_PASS_GROUP], s = 0.0;
#pragma unroll
    for (int k = 0; k < FZ_PASS_GROUP; ++k) v[k] = load_device(p + (long long)min(k, n - 1) * SIZE + e);
#pragma unroll
    for (int k = 0; k < FZ_PASS_GROUP; ++k) s += k < n ? v[k] : 0.0;
    return s;
  };
  if (!last_of(a.counters + grp, members)) return;
  double* parts2 = a.parts + (long long)gridDim.x * SIZE;
  for (int e = t; e < SIZE; e += FZ_PASS_THREADS) store_device(parts2 + (long long)grp * SIZE + e, sum(a.parts + (long long)first * SIZE, members, e));
  if (!last_of(a.counters + a.n_groups, a.n_groups)) return;
  auto whole = [&]() {
    for (int e = t; e < SIZE; e += FZ_PASS_THREADS) {
      int I, K;
      block_at(e >> 8, I, K);
      S[(16 * I + ((e >> 4) & 3) + 4 * ((e >> 6) & 3)) * LD + 16 * K + (e & 15)] = sum(parts2, a.n_groups, e);
    }
    __syncthreads();
  };
  whole();
  if constexpr (!SVD) {
    cholesky_step<NB, LD>(S, a.l, a.factor, a.ld, a.kept, a.state, a.done, a.pass);
  } else {
    if constexpr (16 * NB <= FZ_DIRECT) {
      __shared__ double V[LW * LT];
      if (a.pass == 0) {
        if (eigenvectors<NB, LD, LT>(S, V, a.l)) {
          store_rotation<LT>(S, a.l, a.factor, nullptr, a.Um[0], a.ld, 0);
          if (t == 0) {
            *a.sel = 0;
            *a.done = 1 << 30;
          }
          return;
        }
        __syncthreads();
        whole();
      }
    }
    const bool orthogonal = a.pass == a.passes ||
                            rotation_step<NB, LD>(S, a.l, a.factor, a.Um[(a.pass & 1) ^ 1], a.Um[a.pass & 1], a.ld, a.pass);
    if (orthogonal) sort_and_lift(a, S, LD);
    else if (t == 0) *a.sel = a.pass & 1;
    if (t == 0) *a.done = orthogonal ? a.pass : 1 << 30;
  }
}

template <bool SVD>
static hipError_t launch_passes(PassArgs a, hipStream_t st) {
  const int tiles = (a.rows + FZ_PASS_ROWS - 1) / FZ_PASS_ROWS, per = (tiles + FZ_PASS_WGS - 1) / FZ_PASS_WGS;
  a.rows_per_wg = per * FZ_PASS_ROWS;
  const int wgs = (tiles + per - 1) / per;
  for (a.group = 1; a.group * a.group < wgs; ++a.group) {}
  a.n_groups = (wgs + a.group - 1) / a.group;
  const dim3 grid((unsigned)wgs), block(FZ_PASS_THREADS);
  for (a.pass = 0; a.pass <= a.passes; ++a.pass) {
    switch ((a.l + 15) / 16) {
      case 1: case 2: k_pass<2, SVD><<<grid, block, 0, st>>>(a); break;
      case 3: k_pass<3, SVD><<<grid, block, 0, st>>>(a); break;
      case 4: k_pass<4, SVD><<<grid, block, 0, st>>>(a); break;
      case 5: k_pass<5, SVD><<<grid, block, 0, st>>>(a); break;
      case 6: k_pass<6, SVD><<<grid, block, 0, st>>>(a); break;
      default: k_pass<8, SVD><<<grid, block, 0, st>>>(a); break;
    }
  }
  return hipGetLastError();
}

// doubles of the parts of either kind of pass, whatever the rows
static size_t pass_part_doubles(int l) {
  const size_t nb = l > 96 ? 8 : std::max(2, (l + 15) / 16);
  return (FZ_PASS_WGS + FZ_PASS_GROUP) * nb * (nb + 1) / 2 * 256;
}

__global__ void k_identity(double* U, long long ld, int l) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= l * l) return;
  const int a = idx / l, i = idx - a * l;
  U[(long long)a * ld + i] = a == i ? 1.0 : 0.0;
}

// sig2[a] = |row a of Bs|^2; one block per row.  Element (a, i) of Bs is at a rs + i cs.
__global__ void __launch_bounds__(256) k_row_norms(const double* __restrict__ Bs, long long rs, long long cs, int d,
                                                   double* sig2) {
  __shared__ double red[4];
  const double* r = Bs + (long long)blockIdx.x * rs;
  double s = 0.0;
  for (int i = threadIdx.x; i < d; i += 256) s += r[i * cs] * r[i * cs];
  s = block_sum(s, red);
  if (threadIdx.x == 0) sig2[blockIdx.x] = s;
}

// order of the singular values (see rank_of); one block
__global__ void __launch_bounds__(256) k_sort_sigma(const double* sig2, int l, double* sigma_sorted, int* perm) {
  const int a = threadIdx.x;
  if (a >= l) return;
  const double s = sig2[a];
  const int rank = rank_of([&](int b) { return sig2[b]; }, l, a);
  sigma_sorted[rank] = sqrt(s);
  perm[rank] = a;
}

// P[i][jr] = U~[i][perm jr] sqrt(sigma_jr): the l x r matrix that takes Q to A (Alg. 1,
// lift and balance)
__global__ void k_build_lift(const double* __restrict__ Um, long long ldu, const double* sigma_sorted,
                             const int* perm, int l, int r, double* P, long long ldp) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= l * r) return;
  const int i = idx / r, jr = idx - i * r;
  P[(long long)i * ldp + jr] = Um[(long long)i * ldu + perm[jr]] * sqrt(sigma_sorted[jr]);
}

// A_i = rows of Q P, B[jr][k] = row perm jr of Bs / sqrt(sigma_jr) * Sigma_x^(-1/2)[k], both rounded once to the
// activation type.  The leading workgroups take 32 rows of Q x 16 NT columns of P each (the
// channels dealt to the waves), the others 256 elements of B.
struct LiftArgs {
  const double* Q;         // [m][ldq], l columns
  const double* P;         // [l][ldp], r columns
  long long ldq, ldp;
  int m, l, r, n0, row_tiles;
  int n_modules, row_start[GLOWQ_MAX_MODULES];
  uint16_t* A[GLOWQ_MAX_MODULES];
  // element (a, i) of Um^T Bs at rows[a rs + i cs]
  const double* rows;
  long long rs, cs;
  const double* sigma_sorted;
  const int* perm;
  const double* inv_root;  // or NULL
  int d;
  uint16_t* B;
};

template <int ACT, int NT>
__global__ void __launch_bounds__(256) k_lift(LiftArgs a) {
  __shared__ double fold[2 * NT * 256];
  const int t = threadIdx.x;
  if ((int)blockIdx.x >= a.row_tiles) {
    const long long idx = (long long)((int)blockIdx.x - a.row_tiles) * 256 + t;
    if (idx >= (long long)a.r * a.d) return;
    const int jr = (int)(idx / a.d), k = (int)(idx - (long long)jr * a.d);
    const double s = a.sigma_sorted[jr];
    double v = s > 0.0 ? a.rows[(long long)a.perm[jr] * a.rs + k * a.cs] / sqrt(s) : 0.0;
    if (a.inv_root) v *= a.inv_root[k];
    a.B[idx] = (uint16_t)act16_round<ACT>(v);
    return;
  }
  const int wave = t >> 6, l = t & 63, i = l & 15, g = l >> 4, row0 = (int)blockIdx.x * 32;
  const int per = (a.l + 63) / 64 * 16, kbeg = wave * per, kend = min(a.l, kbeg + per);
  double4_t acc[2][NT];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[rb][nt] = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int k0 = kbeg; k0 < kend; k0 += 4) {
    const int k = k0 + g, kc = min(k, a.l - 1);
    double q[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const double v = a.Q[(long long)min(a.m - 1, row0 + 16 * rb + i) * a.ldq + kc];
      q[rb] = k < kend ? v : 0.0;
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const double b = a.P[(long long)kc * a.ldp + min(a.r - 1, a.n0 + 16 * nt + i)];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) acc[rb][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(q[rb], b, acc[rb][nt], 0, 0, 0);
    }
  }
  fold_waves<2, NT>(acc, fold, wave, l);
  if (wave != 0) return;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = row0 + 16 * rb + g + 4 * v;
      if (row >= a.m) continue;
      int mi = 0;
#pragma unroll
      for (int q = 1; q < GLOWQ_MAX_MODULES; ++q)
        if (q < a.n_modules && row >= a.row_start[q]) mi = q;
      uint16_t* dst = a.A[mi] + (long long)(row - a.row_start[mi]) * a.r;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int col = a.n0 + 16 * nt + i;
        if (col < a.r) dst[col] = (uint16_t)act16_round<ACT>(acc[rb][nt][v]);
      }
    }
}

template <int ACT>
static hipError_t launch_lift(LiftArgs a, hipStream_t st) {
  a.row_tiles = (a.m + 31) / 32;
  for (a.n0 = 0; a.n0 < a.r; a.n0 += 16 * FZ_NT) {
    // (B with the first pass of columns)
    const unsigned n_b = a.n0 == 0 ? (unsigned)(((long long)a.r * a.d + 255) / 256) : 0u;
    const dim3 grid((unsigned)a.row_tiles + n_b), block(256);
    switch ((std::min(a.r - a.n0, 16 * FZ_NT) + 15) / 16) {
      case 1: k_lift<ACT, 1><<<grid, block, 0, st>>>(a); break;
      case 2: k_lift<ACT, 2><<<grid, block, 0, st>>>(a); break;
      case 3: k_lift<ACT, 3><<<grid, block, 0, st>>>(a); break;
      case 4: k_lift<ACT, 4><<<grid, block, 0, st>>>(a); break;
      default: k_lift<ACT, 5><<<grid, block, 0, st>>>(a); break;
    }
  }
  return hipGetLastError();
}

__global__ void k_copy_doubles(const double* src, double* dst, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
static size_t up256(size_t b) { return (b + 255) & ~(size_t)255; }

FactorizePlan plan_factorize(const glowq_unit& u, int r, int p) {
  FactorizePlan f;
  long long m = 0;
  for (int i = 0; i < u.n_modules; ++i) m += u.modules[i].d_out;
  f.m = m;
  f.d = u.d_in;
  f.l = r + p;
  f.l16 = (f.l + 15) / 16 * 16;
  f.r16 = (r + 15) / 16 * 16;
  f.n_groups = (int)((m + 255) / 256);                 // at most 256 rows per group ...
  if (f.n_groups < 64) f.n_groups = (int)(m < 64 ? m : 64);   // ... and few groups: their partial sums are added serially
  f.rpw = (int)((m + f.n_groups - 1) / f.n_groups);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += up256(bytes); return o; };
  f.off_ms = take((size_t)m * f.d * 8);
  f.off_y = take((size_t)m * f.l16 * 8);
  f.off_z = take((size_t)f.d * f.l16 * 8);
  f.off_bs = take((size_t)f.l * f.d * 8);
  f.off_ut = take((size_t)f.l * f.l16 * 8);
  f.off_parts = take(f.l <= FZ_SMALL ? pass_part_doubles(f.l) * 8 : 0);
  f.off_lift = take((size_t)f.l * f.r16 * 8);
  const size_t sl = std::max(slice_doubles(plan_ring((int)m, f.d), (int)m, f.l),     // Y = Ms Omega, Y = Ms Z
                             slice_doubles(plan_ring(f.d, (int)m), f.d, f.l));       // Z = Ms^T Y, Bs^T = Ms^T Q
  f.off_slices = take(sl * 8);
  f.off_root = take((size_t)f.d * 8);
  f.off_inv_root = take((size_t)f.d * 8);
  f.off_c1 = take((size_t)f.n_groups * 256 * 8);
  f.off_c2 = take((size_t)f.n_groups * 256 * 8);
  f.off_norm = take((size_t)f.n_groups * 8);
  f.off_norm0 = take((size_t)2 * f.n_groups * 8);
  f.off_sig2 = take(256 * 8);
  f.off_sigma = take(256 * 8);
  f.off_perm = take(256 * 4);
  f.off_counters = take(FZ_COUNTERS * 4);
  f.off_rot = take((size_t)f.l * f.l16 * 8);
  f.off_um2 = take((size_t)f.l * f.l16 * 8);
  f.off_kept = take(256 * 8);
  f.off_state = take(256 * 4);
  f.off_done = take(3 * 4);
  f.bytes = off;
  return f;
}

hipError_t launch_factorize(const glowq_unit& u, const float* const* W_modules, const double* sigma_x,
                            int r, int p, int q, const double* Omega, char* ws, void* const* A_out,
                            void* B_out, double* sigma_out, hipStream_t st) {
  const FactorizePlan f = plan_factorize(u, r, p);
  const bool f16 = u.act_dtype == GLOWQ_F16;
  const int m = (int)f.m, d = f.d, l = f.l;
  double* Ms = (double*)(ws + f.off_ms);
  double* Y = (double*)(ws + f.off_y);
  double* Z = (double*)(ws + f.off_z);
  double* Bs = (double*)(ws + f.off_bs);
  double* Um = (double*)(ws + f.off_ut);
  double* lift = (double*)(ws + f.off_lift);
  double* factor = (double*)(ws + f.off_rot);      // [l][l16]: the matrix a pass multiplies with
  double* slices = (double*)(ws + f.off_slices);
  double* root = sigma_x ? (double*)(ws + f.off_root) : nullptr;
  double* inv_root = sigma_x ? (double*)(ws + f.off_inv_root) : nullptr;
  double* sig2 = (double*)(ws + f.off_sig2);
  double* sigma_sorted = (double*)(ws + f.off_sigma);
  int* perm = (int*)(ws + f.off_perm);
  int* counters = (int*)(ws + f.off_counters);
  CgsBuffers cb;
  cb.c1 = (double*)(ws + f.off_c1);
  cb.c2 = (double*)(ws + f.off_c2);
  cb.norm = (double*)(ws + f.off_norm);
  cb.norm0 = (double*)(ws + f.off_norm0);

  hipError_t err = hipSuccess;
  k_setup<<<dim3((unsigned)((d * f.l16 + 255) / 256)), dim3(256), 0, st>>>(sigma_x, d, root, inv_root, Omega, l, f.l16, Z,
                                                                          counters, FZ_COUNTERS);
  // the stack, scaled by Sigma_x^(1/2) (Alg. 1, core construction)
  StackArgs sa = {};
  sa.n_modules = u.n_modules;
  sa.d_in = d;
  sa.G = u.group_size;
  long long row_off = 0;
  int recs = 0;
  for (int i = 0; i < u.n_modules; ++i) {
    const glowq_module& mod = u.modules[i];
    sa.W[i] = W_modules[i];
    sa.prepared[i] = (const uint32_t*)mod.w_prepared;
    sa.d_out[i] = mod.d_out;
    sa.rec_start[i] = recs;
    sa.row_start[i] = row_off;
    recs += (mod.d_out + 15) / 16 * (d / 128);
    row_off += mod.d_out;
  }
  if (f16) k_error_stack<ACT_F16><<<dim3((unsigned)recs), dim3(256), 0, st>>>(sa, root, Ms);
  else k_error_stack<ACT_BF16><<<dim3((unsigned)recs), dim3(256), 0, st>>>(sa, root, Ms);
  // sketch and power steps (Alg. 1, range finding)
  const bool small = l <= FZ_SMALL;
  int n_slices = 0;                                // (small: the first pass of the orthonormalisation adds the last ones)
  err = gemm<false>(Ms, d, Z, f.l16, Y, f.l16, false, m, l, d, slices, st, small && q == 0 ? &n_slices : nullptr);
  for (int it = 0; it < q && err == hipSuccess; ++it) {
    err = gemm<true>(Ms, d, Y, f.l16, Z, f.l16, false, d, l, m, slices, st);
    if (err == hipSuccess) err = gemm<false>(Ms, d, Z, f.l16, Y, f.l16, false, m, l, d, slices, st, small && it == q - 1 ? &n_slices : nullptr);
  }
  if (err != hipSuccess) return err;
  // orthonormal basis of the range, compressed matrix Bs = Q^T Ms and its SVD
  const double* rows;          // element (a, i) of Um^T Bs at a rows_rs + i rows_cs
  long long rows_rs, rows_cs;
  if (small) {
    int* done = (int*)(ws + f.off_done);
    PassArgs pa = {};
    pa.slices = slices;
    pa.factor = factor;
    pa.parts = (double*)(ws + f.off_parts);
    pa.counters = counters;
    pa.l = l; pa.ld = f.l16;
    pa.Y = Y;
    pa.n_slices = n_slices;
    pa.rows = m;
    pa.done = done;
    pa.passes = FZ_QR_PASSES;
    pa.kept = (double*)(ws + f.off_kept);
    pa.state = (int*)(ws + f.off_state);
    err = launch_passes<false>(pa, st);
    if (err != hipSuccess) return err;
    double* BsT = Z;                                                               // [d][l16]
    err = gemm<true>(Ms, d, Y, f.l16, BsT, f.l16, false, d, l, m, slices, st, &n_slices);     // Ms^T Q
    if (err != hipSuccess) return err;
    pa.Y = BsT;
    pa.n_slices = n_slices;
    pa.rows = d;
    pa.done = done + 1;
    pa.passes = FZ_SVD_PASSES;
    pa.Um[0] = Um;
    pa.Um[1] = (double*)(ws + f.off_um2);
    pa.sel = done + 2;
    pa.sigma_sorted = sigma_sorted;
    pa.perm = perm;
    pa.sigma_out = sigma_out;
    pa.lift = lift;
    pa.r = r; pa.r16 = f.r16;
    err = launch_passes<true>(pa, st);
    if (err != hipSuccess) return err;
    rows = BsT;
    rows_rs = 1;
    rows_cs = f.l16;
  } else {
    for (int j = 0; j <= l; ++j) {
      k_cgs<<<dim3((unsigned)f.n_groups), dim3(256), 0, st>>>(Y, f.l16, m, l, f.rpw, f.n_groups, j, 0, cb);
      if (j == l) break;
      if (j > 0) {
        k_cgs<<<dim3((unsigned)f.n_groups), dim3(256), 0, st>>>(Y, f.l16, m, l, f.rpw, f.n_groups, j, 1, cb);
        k_cgs<<<dim3((unsigned)f.n_groups), dim3(256), 0, st>>>(Y, f.l16, m, l, f.rpw, f.n_groups, j, 2, cb);
      } else {
        // the first column has nothing to be projected against: its norm is the one just taken
        k_cgs<<<dim3((unsigned)f.n_groups), dim3(256), 0, st>>>(Y, f.l16, m, l, f.rpw, f.n_groups, 0, 2, cb);
      }
    }
    err = gemm<true>(Ms, d, Y, f.l16, Bs, d, true, d, l, m, slices, st);           // (Ms^T Q)^T
    if (err != hipSuccess) return err;
    k_identity<<<dim3((unsigned)((l * l + 255) / 256)), dim3(256), 0, st>>>(Um, f.l16, l);
    const int n = (l + 1) & ~1;
    for (int sweep = 0; sweep < FZ_MAX_SWEEPS; ++sweep)
      for (int round = 0; round < n - 1; ++round)
        k_jacobi_round<<<dim3((unsigned)(n / 2)), dim3(FZ_JT), 0, st>>>(Bs, d, d, Um, f.l16, l, n, round, sweep, counters);
    rows = Bs;
    rows_rs = d;
    rows_cs = 1;
    k_row_norms<<<dim3((unsigned)l), dim3(256), 0, st>>>(rows, rows_rs, rows_cs, d, sig2);
    k_sort_sigma<<<dim3(1), dim3(256), 0, st>>>(sig2, l, sigma_sorted, perm);
    // truncate, balance
    k_build_lift<<<dim3((unsigned)((l * r + 255) / 256)), dim3(256), 0, st>>>(Um, f.l16, sigma_sorted, perm, l, r, lift, f.r16);
    if (sigma_out) k_copy_doubles<<<dim3(1), dim3(256), 0, st>>>(sigma_sorted, sigma_out, l);
  }
  // lift
  LiftArgs la = {};
  la.Q = Y; la.P = lift;
  la.ldq = f.l16; la.ldp = f.r16;
  la.m = m; la.l = l; la.r = r;
  la.n_modules = u.n_modules;
  row_off = 0;
  for (int i = 0; i < u.n_modules; ++i) {
    la.row_start[i] = (int)row_off;
    la.A[i] = (uint16_t*)A_out[i];
    row_off += u.modules[i].d_out;
  }
  la.rows = rows; la.rs = rows_rs; la.cs = rows_cs;
  la.sigma_sorted = sigma_sorted;
  la.perm = perm;
  la.inv_root = inv_root;
  la.d = d;
  la.B = (uint16_t*)B_out;
  return f16 ? launch_lift<ACT_F16>(la, st) : launch_lift<ACT_BF16>(la, st);
}

}  // namespace glowq

// Host-side launch entry points implemented by the .hip files (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "../../include/glowq.h"

namespace glowq {

// Layout of one unit's slice of the caller's workspace.
struct UnitWorkspace {
  char* base;         // start of the slice (256-byte aligned)
  size_t bytes;       // size of the slice
  size_t off_counters;  // T > 64: per token tile, a ready flag and an arrival counter of K parts
  // The next two areas hold what the kernel that serves the call puts there (T > 64: either of two).
  size_t off_rpart;   // partial sums of the projection: 8-byte slots {fp32, launch tag},
                      // [T][ksplit][r] (few-token and batched kernels; first launch of a microscaling call,
                      // at most four slices: past 64 tokens these fill the area); fp32 [part][T][r] (tiled kernel,
                      // glowq_shared_proj)
  size_t off_r16;     // R in the activation type: 8-byte slots {two ranks, launch tag}, [T][r / 2]
                      // (batched kernel); [T][r] (tiled kernel)
  size_t off_splitk;  // T > 64: fp32 slabs of a long contraction cut into K slices (0 bytes if not cut)
  size_t splitk_bytes;
  size_t ctl_bytes;   // leading bytes that must be zero between calls
  int ksplit;         // K slices of the projection
  int kslice;         // channels per slice (multiple of 32)
  int gather;         // the consumers of R add the slices themselves (see plan_batch_projection)
  int kstride;        // ksplit rounded up to a multiple of 4 (sizes the partial-sum area)
  int pf_parts;       // T > 64: K parts of a projection tile inside the GEMM launch
  int pf_part_stages; // 64-channel stages per such part
};

// decode path: the few-token kernel (T <= 4) or the batched one, whatever the shapes; beyond it the
// choice between the batched and the tiled kernel is made for each launch
static inline bool is_decode(int T) { return T <= 64; }

UnitWorkspace plan_unit_workspace(const glowq_unit& u, char* base);

hipError_t launch_prepare(const uint32_t* wq, const uint16_t* scales, const uint16_t* zeros,
                          int d_out, int d_in, int G, void* prepared, hipStream_t st);
hipError_t launch_quantize_rtn(const float* W, int d_out, int d_in, int G, uint32_t* wq, uint16_t* scales,
                               uint16_t* zeros, hipStream_t st);
hipError_t launch_debug_unpack(const void* prepared, int d_out, int d_in, int G, uint8_t* q_out,
                               hipStream_t st);
hipError_t launch_debug_dequant(const void* prepared, int d_out, int d_in, int G, int act,
                                void* w_out, hipStream_t st);
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t st);
hipError_t launch_importance(const glowq_unit& u, const float* const* W_modules, double* scratch,
                             double* scores, hipStream_t st);
// Workspace of the factorisation of one unit's stacked error (byte offsets, 256-aligned).
struct FactorizePlan {
  long long m;        // rows of the stack
  int d, l, l16, r16; // channels; sketch width r + p; both widths rounded up to 16
  int n_groups, rpw;  // row groups of the orthonormalisation and rows per group
  size_t off_ms, off_y, off_z, off_bs, off_ut, off_parts, off_lift, off_slices, off_root,
      off_inv_root, off_c1, off_c2, off_norm, off_norm0, off_sig2, off_sigma, off_perm,
      off_counters, off_rot, off_um2, off_kept, off_state, off_done;
  size_t bytes;
};
FactorizePlan plan_factorize(const glowq_unit& u, int r, int p);
hipError_t launch_factorize(const glowq_unit& u, const float* const* W_modules, const double* sigma_x,
                            int r, int p, int q, const double* Omega, char* ws, void* const* A_out,
                            void* B_out, double* sigma_out, hipStream_t st);
// Microscaling variant (MXFP4 weights, MXFP8 activations), up to 16 tokens.
struct MxWorkspace {
  size_t off_rpart;         // fp32 partial sums of the projection, [ks][16][r]
  size_t off_xcodes;        // E4M3 codes of the activations in fragment order, whole 16-token blocks
  size_t off_xscales;       // their E8M0 block scales, likewise
  size_t bytes;
  int ks, kslice;           // K slices of the projection and channels per slice
};
constexpr int MX_MAX_TOKENS = 16;
size_t mx_prepared_bytes(int d_out, int d_in);
MxWorkspace plan_mx_workspace(const glowq_unit& u);
hipError_t launch_mx_prepare(const uint32_t* codes, const uint8_t* scales, int d_out, int d_in, void* prepared,
                             hipStream_t st);
hipError_t launch_mx_quantize_x(const void* X, int T, int d_in, int act, uint8_t* codes, uint8_t* scales,
                                hipStream_t st);
hipError_t launch_mx_forward(const glowq_unit& u, bool restore, char* workspace, hipStream_t st);
void mx_route(const glowq_unit& u, glowq_route* route);
void mx_front_shape(const glowq_unit& u, int32_t* shape);      // of the first launch: token blocks, rank blocks, waves, slices
int mx_tile_tokens(const glowq_unit& u);      // tokens of the call's workgroup tiles (0: not tiled)
// slices' start offsets in units of 256 bytes (every slice is 256-byte aligned)
constexpr int STATUS_BATCH = 256;
struct StatusBatch {
  uint32_t off256[STATUS_BATCH];
  int n;
};
hipError_t launch_status_count(const void* ws, const StatusBatch& b, bool first, uint32_t* out,
                               hipStream_t st);

struct ProjArgs;
ProjArgs make_proj_args(const glowq_unit& u, const UnitWorkspace& ws, float* R32);

// R = X B^T, stand-alone: fp32 partial sums per K slice, then a second launch adds them in
// slice order into R32.
hipError_t launch_proj(const glowq_unit& u, const UnitWorkspace& ws, float* R32, hipStream_t st);
// T <= 4: streaming pass over the prepared weights; when restore, the projection runs
// in the first workgroups of the same launch
bool decode_batch_compatible(const glowq_unit& a, const glowq_unit& b);
int decode_max_batch();
int decode_wait_polls();
hipError_t launch_decode_multi(const glowq_unit* const* units, const UnitWorkspace* ws,
                               const bool* restore, int n, hipStream_t st);
// T > 4: the same with X shared through LDS; compatible units share a launch.  All calls of up to
// 64 tokens go this way, those beyond where that is estimated to be the faster one, up to this
// many tokens (the workspace of a unit holds the slots up to here)
constexpr int BATCH_MAX_T = 2048;
void plan_batch_projection(const glowq_unit& u, UnitWorkspace& w);
// the workgroup tile for these units in one launch, what it is taken to cost and, where contractions may be cut (else
// NULL), the K slices of every unit; then the bytes behind the units' workspace slices that such a launch keeps its
// partial results in
int choose_batch_tile(const glowq_unit* const* units, int n, float* cost, int* slices);
int batch_wait_polls();
bool batch_compatible(const glowq_unit& a, const glowq_unit& b);
int batch_max_units();
size_t batch_slab_bytes(const glowq_unit* const* units, int n, int tile, const int* slices);
int batch_token_blocks(const glowq_unit* const* units, int n, int tile, const int* slices);     // of 16, in the launch's tiles
hipError_t launch_decode_batch(const glowq_unit* const* units, const UnitWorkspace* ws, const bool* restore, int n,
                               int tile, const int* slices, char* slabs, hipStream_t st);
// The other calls of T > 64: tiled matrix-core GEMM, correction folded in as an extra K slab.
// One launch covers several compatible units (same types and group size).
bool prefill_compatible(const glowq_unit& a, const glowq_unit& b);
int prefill_max_units();
int prefill_max_modules();
// K slices of every unit of a launch: where the unit's shapes ask for them, the workspace has the
// slabs (`slabs`) and the module table has room.  Returns the bytes (of `room`) behind the units' workspace slices that the
// launch takes for more slices than that
size_t plan_prefill_slices(const glowq_unit* const* units, int n, bool slabs, size_t room, int* slices);
// ... and fewer of them where a launch of several units on wide tiles is taken to end sooner so
void fewer_wide_slices(const glowq_unit* const* units, int n, int* slices);
// the tiles that the launch, cut into these slices, takes, and what it is taken to cost (dealt false: on tiles that all hold
// 128 tokens)
enum { PF_TILE_LARGE = 0, PF_TILE_HALF = 1, PF_TILE_WIDE = 2 };
int choose_prefill_tile(const glowq_unit* const* units, const int* slices, int n, float* cost, bool dealt = true);
int prefill_token_blocks(const glowq_unit* const* units, int n, int tile);
int prefill_wait_polls();
hipError_t launch_prefill_multi(const glowq_unit* const* units, const UnitWorkspace* ws, const bool* restore,
                                int n_units, int tile, const int* slices, char* behind, hipStream_t st);
int prefill_k_slices(const glowq_unit& u);
size_t prefill_splitk_bytes(const glowq_unit& u);

}  // namespace glowq

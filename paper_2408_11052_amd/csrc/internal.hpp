// Internal launch wrappers shared by the C-ABI layer (not part of the ABI).
#pragma once

#include "common.hpp"
#include "crl.h"
#include "gemm.hpp"

namespace crl {

// timing.hip: opt-in HIP-event timing of single launches (see crl_timing_*).
struct KTimer {
  bool on;
  int slot;
  hipEvent_t a, b;
  hipStream_t s;
  double flops, bytes;
};
KTimer timing_begin(const char* name, double flops, double bytes, hipStream_t s);
void timing_end(KTimer& t);
#define CRL_TIMED(name, flops, bytes, stream, ...)                   \
  do {                                                               \
    ::crl::KTimer _crl_t = ::crl::timing_begin(name, flops, bytes, stream); \
    __VA_ARGS__;                                                     \
    ::crl::timing_end(_crl_t);                                       \
  } while (0)

// gemm.hip: dispatch on storage type / operand layouts / output type.
hipError_t launch_gemm(GemmParams& P, bool bf16, int la, int lb, bool out_bf16,
                       hipStream_t s);
// One layer's weight gradient (Pw: MC x MC, FP32 out or deferred split-K
// partials) and input gradient (Px: KC x KC, storage-type out, unsplit) in one
// launch; gemm_pair_ok tells whether the two can share one (no split-K
// reduction left to run; a BF16 dX whose K is whole stages).
bool gemm_pair_ok(const GemmParams& Pw, const GemmParams& Px, bool bf16);
hipError_t launch_gemm_dw_dx(GemmParams& Pw, GemmParams& Px, bool bf16, hipStream_t s);
// dpsi = G^T phi (Pc: MC x MC) and dphi = G psi (Pr: KC x MC) of the
// materialised critic matrix in one launch, FP32; splits stay unreduced.
hipError_t launch_gemm_obj(GemmParams& Pc, GemmParams& Pr, hipStream_t s);
// Split factor, chunk and tile for a batch of problems (fills P.splits,
// P.k_chunk, P.tile, P.tiles): the largest power of two that keeps the launch
// within target_wgs workgroups and every split at least min_steps K steps deep.
void plan_split_k(GemmParams& P, bool bf16, int target_wgs, int min_steps = 4);
void set_tile(GemmParams& P, int tile);    // tile (kTile*) and tile counts of a planned launch
int64_t gemm_tiles128(const GemmDesc& d);  // 128 x 128 tiles of one problem
// Block width (128, or 64 when no problem is wider) of the fragment order that
// a launch's deferred split-K partials take.
int frag_bn(const GemmParams& P);
// Floats of one split's deferred partial of problem g: whole 128 x bn blocks.
int64_t frag_partial_floats(const GemmParams& P, int g, int bn);

// kernels.hip
hipError_t launch_relabel(const float* obs, const float* act, int E, int T,
                          int d_s, int d_a, int d_g, int goal_lo, uint64_t seed,
                          const int64_t* step, const uint64_t* thr, int B,
                          int32_t* idx, void* x_sa, int ld_sa, void* x_g, int ld_g,
                          void* x_sg, int ld_sg, bool bf16, hipStream_t s);

// replay.hip: the ring buffer
hipError_t launch_replay_insert(float* obs, float* act, int32_t* traj, int E, int C, int d_s,
                                int d_a, const float* nobs, const float* nact,
                                const int32_t* ntraj, int U, int64_t* count, hipStream_t s);
hipError_t launch_ring_relabel(const float* obs, const float* act, const int32_t* traj, int E,
                               int C, const int64_t* count, int d_s, int d_a, int d_g,
                               int goal_lo, uint64_t seed, const int64_t* step,
                               const uint64_t* thr, int n_thr, int B, int32_t* idx, void* x_sa,
                               int ld_sa, void* x_g, int ld_g, void* x_sg, int ld_sg, bool bf16,
                               hipStream_t s);

struct LnArgs {
  const void* Z[2];     // [B][N] pre-LN values
  void* H[2];           // [B][N] Swish(LN(z)) out
  float* mu[2];
  float* rstd[2];
  const float* g[2];    // LN scale
  const float* b[2];    // LN offset
  // backward
  const void* dH[2];
  void* dZ[2];
  float* part[2];       // [ln_bwd_partials(B, bf16)][3][N] column partials; NULL: only dZ
};
hipError_t launch_ln_swish_fwd(const LnArgs& a, int count, int B, int N, float eps,
                               bool bf16, hipStream_t s);
hipError_t launch_ln_swish_bwd(const LnArgs& a, int count, int B, int N, bool bf16,
                               hipStream_t s);
int ln_bwd_partials(int B, bool bf16_parts);

// column sums of X [B][N] over chunks of 128 rows: part[e][ceil(B/128)][N]
struct ColSumArgs {
  const void* X[2];
  float* part[2];
};
hipError_t launch_colsum_partials(const ColSumArgs& a, int count, int B, int N, int ld,
                                  bool bf16, hipStream_t s);
int colsum_chunks(int B);

// Deferred gradient reductions: g[dst + i] = sum_k part_k[i], part_k at byte
// offset src + 4 k stride in the workspace, i < n, in the order k = 0, 1, ...
// (with four interleaved running sums, combined in a fixed order).  `first`
// is the job's first float4 (few-part jobs) or first block of kManyCols outputs
// (many-part jobs) in the launch's index space.
// Sum of nparts partial blocks (src + k * stride floats, k = 0..nparts-1, in
// that order) into g + dst.  bn == 0: n contiguous floats.  bn > 0: split-K
// partials of an M x N GEMM in fragment order (128 x bn blocks, tiles_n per
// row of blocks), scattered into the row-major
// M x N block at dst.
struct RedJob {
  int64_t src;
  int64_t stride;
  int64_t dst;
  int64_t first;
  int64_t first_chunk;  // few-part jobs with the Adam epilogue: first block, in
                        // chunks of kRedChunk4 float4 outputs
  int32_t nparts, n;
  int32_t M, N, tiles_n, bn;
};
// float4 outputs per block of the reduction with the Adam epilogue: a 64 x 64
// block of a fragment-order tile (two of its waves)
constexpr int kRedChunk4 = 1024;
constexpr int kManyCols = 32;  // outputs per workgroup of a many-part reduction job
struct AdamArgs;
// loss_out = {L_pi, mean log pi, L_alpha, mean f}; *alpha_grad = dL_alpha/dlog alpha:
//   L_pi = alpha mean(log pi) - mean(f),  L_alpha = -log alpha (mean(log pi) + H)
struct ActorLossArgs {
  const float* logpi;
  const float* f;
  int B;
  const float* log_alpha;
  float target_entropy;
  float* loss_out;
  float* alpha_grad;
};
// few-part jobs (total4 float4 outputs) and many-part jobs (nblocks blocks of
// kManyCols outputs) in one launch.  With A, each gradient element goes straight
// into the Adam step of its parameter (g, if not NULL, still receives it).
// With L, one more block reduces the policy's loss.
hipError_t launch_grad_reduce(const char* ws, float* g, const RedJob* few, int nfew,
                              int64_t total4, const RedJob* many, int nmany, int64_t nblocks,
                              double bytes, hipStream_t s, const AdamArgs* A = nullptr,
                              const ActorLossArgs* L = nullptr);

hipError_t launch_cast_bf16(const float* src, bf16_t* dst, int64_t n, hipStream_t s);
// Adam coefficients: 1 - b and log b are formed in double on the host.
struct AdamCoef {
  float lr, b1, b2, omb1, omb2, log_b1, log_b2, eps;
};
hipError_t launch_adam(float* p, const float* g, float* m, float* v, bf16_t* pb,
                       int64_t n, const int64_t* step, const AdamCoef& c, hipStream_t s);
// The optimiser state of a flat vector, for the reduction's Adam epilogue.
struct AdamArgs {
  float* p;
  float* m;
  float* v;
  bf16_t* pb;            // BF16 copy of p, or NULL
  const int64_t* step;   // t (device, read)
  AdamCoef c;
};
hipError_t launch_counter_add(int64_t* c, int64_t inc, hipStream_t s);

// log-sum-exp of (max, sum) partials [nparts][B] per column j, for `count`
// problems in one launch
struct LseMergeArgs {
  const float* pm[2];
  const float* ps[2];
  int nparts[2];
  float* out[2];
};
hipError_t launch_lse_merge(const LseMergeArgs& a, int count, int B, hipStream_t s);
// loss_out[8] from r, c, diag and (pairwise objectives) the per-row terms;
// then *advance += 1 if advance is not NULL (one workgroup, so no fence).
// nparts > 0: c is first formed (and written) from the column partials.
hipError_t launch_loss(const float* r, float* c, const float* diag, const float* term,
                       int B, int loss, float beta, float* loss_out, int64_t* advance,
                       hipStream_t s, const float* col_m = nullptr, const float* col_s = nullptr,
                       int nparts = 0);

// objectives.hip: energies and objectives on the materialised matrix
// unit rows U and norms of phi and psi
hipError_t launch_unit_rows(const float* phi, const float* psi, float* Uphi, float* Upsi,
                            float* nphi, float* npsi, int B, int D, hipStream_t s);
hipError_t launch_l1_energy(const float* phi, const float* psi, float* F, int B, int D, int ld,
                            hipStream_t s);
// partials part[side][split][B][D] of dphi (side 0) and dpsi (1)
int l1_backward_splits(int B, int D);
hipError_t launch_l1_backward(const float* phi, const float* psi, const float* G, int ldg,
                              float* part, int splits, int B, int D, hipStream_t s);
// r, diag, and for the pairwise objectives the row terms and the sums that
// form dL/dF_ii; and the columns' (max, sum) over col_chunks(B) chunks of rows
int col_chunks(int B);
bool col_merge_in_loss(int B);  // few enough columns for the loss kernel to merge the chunks
hipError_t launch_row_col(const float* F, int B, int ld, int loss, float* r, float* diag,
                          float* term, float* aux, float* col_m, float* col_s, hipStream_t s);
// in place F -> dL/dF (or H for the distance energies, with its row sums)
hipError_t launch_grad_obj(float* F, int B, int ld, const float* r, const float* c,
                           const float* diag, const float* aux, int loss, int energy, float beta,
                           float* rowsum, hipStream_t s);
// dphi (side 0) and dpsi (1) from `splits` partials [splits][B][D] (which may
// be the output itself, splits = 1), then the energy's own term:
//   kFixDist: -= (sum of nrs row sums rs[k][row]) X;  kFixCos: X the unit rows,
//   (v - (v . X) X) / nrm.  outb: BF16 copies, or NULL.
enum : int { kFixNone = 0, kFixDist = 1, kFixCos = 2 };
struct ObjFinish {
  const float* part[2];
  float* out[2];
  bf16_t* outb[2];
  const float* X[2];
  const float* rs[2];
  int nrs[2];
  const float* nrm[2];
};
hipError_t launch_obj_finish(const ObjFinish& a, int splits, int fix, int B, int D, hipStream_t s);

// fused InfoNCE (BF16 tiles, FP32 online LSE)
struct FusedArgs {
  const float* phi;
  const float* psi;
  bf16_t* phi_b;      // BF16 copies written by the prep kernel
  bf16_t* psi_b;
  float* nphi;        // squared norms of the BF16-rounded rows (L2)
  float* npsi;
  float* row_m;       // [S][B]
  float* row_s;
  float* col_m;       // [B/64][B]
  float* col_s;
  float* r;
  float* c;
  float* diag;
  float* dX_part;     // [2][S][B][D] backward partials (rows pass, columns pass)
  float* rs_part;     // [2][S][B]   sum_b H_ab (L2)
  float* dphi;        // [B][D] FP32 out
  float* dpsi;
  void* dphi_t;       // storage-type copies for the encoder GEMMs
  void* dpsi_t;
  float* bias_part[2]; // [chunks][D] column sums of dphi / dpsi per 256/D rows, or nullptr
};
int fused_splits(int B);
int fused_bwd_splits(int B);          // splits of the one-pass backward (D = 64)
int fused_bias_chunks(int B, int D);  // row blocks of the backward reduction
// top: the output layer's deferred split-K launch (phi = d[0].C, psi =
// d[1].C), summed with its bias by the prep kernel; nullptr: phi and psi are
// final already.
// energy: CRL_ENERGY_DOT, _L2, _COS (unit rows, dot product) or _L2SQ
hipError_t launch_fused_fwd(const FusedArgs& a, int B, int D, int energy, const GemmParams* top,
                            hipStream_t s);
// Where the backward's partials are those of 256-row blocks, the kernel that
// makes them: by the batch size, or (in tests of their equality) as said.
enum BlockRoute { kRouteAuto, kRouteOnePass, kRouteTwoPasses };
// loss: CRL_LOSS_FWD, _SYM, _BWD, _FLATNCE_FWD or _FLATNCE_BWD
hipError_t launch_fused_bwd(const FusedArgs& a, int B, int D, int energy, int loss, float beta,
                            bool out_bf16, hipStream_t s, BlockRoute route = kRouteAuto);
// whether the backward's partials are those of 256-row blocks (D = 64, at most
// 16 of them), from the one-pass kernel or from the two passes
bool fused_bwd_blocks(int B, int D);

// actor.hip: the policy step's elementwise/row kernels
// Each takes its input either final (top / dx with splits == 1) or as the
// launch's split-K partials, which it sums in split order (plus the bias) and
// also writes out.
hipError_t launch_actor_head_fwd(float* out, const GemmParams& top, int ldo, int A, uint64_t seed,
                                 const int64_t* step, const void* x_sa, void* x_sa2, int ld,
                                 int d_s, float* eps, float* logpi, int B, bool bf16,
                                 hipStream_t s);
// f_b = energy(phi_b, psi_b) (CRL_ENERGY_*) and d(-mean f)/dphi
hipError_t launch_actor_energy(float* phi, float* psi, const GemmParams& top, int D, int energy,
                               float* f, void* dphi, int B, bool bf16, hipStream_t s);
hipError_t launch_actor_head_bwd(const float* out, int ldo, int A, const float* eps,
                                 float* da, int ldd, const GemmParams& dx, const float* log_alpha,
                                 float* dout, void* dout_t, int B, bool bf16, hipStream_t s);
// random goals: xg_out[b] = x_g[j], xsg_out[b] = [x_sg[b][0:d_s], x_g[j], 0...]
// with j the partner drawn for b (j = b when b is not mixed)
hipError_t launch_goal_mix(const void* x_g, int ld_g, const void* x_sg, int ld_sg, int d_s,
                           int d_g, uint64_t seed, const int64_t* step, uint64_t thr53, int B,
                           void* xg_out, void* xsg_out, bool bf16, hipStream_t s);
}  // namespace crl

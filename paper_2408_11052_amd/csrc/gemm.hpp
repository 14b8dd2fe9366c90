// The encoder and logit GEMMs (gfx950): problem descriptions and shared helpers.
//
// C[M][N] = epilogue(alpha * A[M][K] . B[K][N]) for up to two independent
// problems per launch (the phi and psi encoders run side by side).
//
// Operands are either "KC" (the contraction index is contiguous:
// A(m,k) = A[m*lda + k], B(k,n) = B[n*ldb + k]) or "MC" (the row/column index
// is contiguous: A(m,k) = A[k*lda + m], B(k,n) = B[k*ldb + n]).  Pointers are
// 16-byte aligned and leading dimensions whole 16-byte chunks (every caller's
// are multiples of 8 elements); M, N and K are arbitrary.
#pragma once

#include "common.hpp"

namespace crl {

enum : int { LAY_KC = 0, LAY_MC = 1 };
enum : int {
  EPI_NONE = 0,      // v
  EPI_BIAS = 1,      // v + bias[n]
  EPI_BIAS_RELU = 2, // max(v + bias[n], 0)
  EPI_MASK_POS = 3,  // aux(m,n) > 0 ? v : 0      (ReLU backward)
  EPI_L2 = 4,        // -l2_dist(|A(m,.)|^2, |B(.,n)|^2, v)   (FP32 KC x KC,
  EPI_L2SQ = 5       // -l2sq_dist(|A(m,.)|^2, |B(.,n)|^2, v)  unsplit)
};

struct GemmDesc {
  const void* A;
  const void* B;
  void* C;
  const float* bias;
  const void* aux;    // same storage type and leading dim as C
  int M, N, K;
  int lda, ldb, ldc;
  int epi;
  float alpha;
  int kb;             // rows k < kb of an MC-layout B exist (0: all K).  Rows
                      // k >= kb are re-reads of row kb-1; the caller
                      // guarantees A is zero in those columns
  float* asum;        // FP32 MC x MC launches: sum_k A(m,k) to asum[split * M + m], or NULL
  float* bsum;        // FP32 MC x MC launches: sum_k B(k,n) to bsum[split * N + n], or NULL
};

constexpr int kGemmMaxGroup = 2;
enum : int { kTile32 = 0, kTile64x32 = 1, kTile64 = 2, kTile128 = 3 };  // rows x columns

struct GemmParams {
  GemmDesc d[kGemmMaxGroup];
  int count;
  int tile;            // kTile*, chosen by plan_split_k
  int tiles_n[kGemmMaxGroup];
  int tiles[kGemmMaxGroup];
  int splits;          // split-K factor (>= 1)
  int k_chunk;         // K range per split (multiple of the K step)
  float* partial;      // splits > 1: partial[g][s][M][N] (FP32, no epilogue)
  int64_t partial_len; // floats per problem in `partial`
  int defer_reduce;    // splits > 1: leave the partials for a later reduction
  int frag;            // with defer_reduce: > 0 stores the partials in fragment
                       // order of 128 x frag blocks (see frag_partial_floats)
};

// K values of a stage: 128 bytes of every tile row
constexpr int gemm_bk(bool bf16) { return bf16 ? 64 : 32; }

// What the kernel assumes of a launch (every caller provides it); nothing of it
// is checked on the device.
inline bool gemm_operands_ok(const GemmParams& P, bool bf16, int la, int lb) {
  const int v = bf16 ? 8 : 4, BK = gemm_bk(bf16);
  if (P.count < 1 || P.count > kGemmMaxGroup || P.splits < 1 || P.k_chunk < BK || P.k_chunk % BK)
    return false;
  if (P.splits > 1 && !P.partial) return false;
  const bool sums = !bf16 && la == LAY_MC && lb == LAY_MC;
  const bool dist = !bf16 && la == LAY_KC && lb == LAY_KC && P.splits == 1;
  for (int g = 0; g < P.count; ++g) {
    const GemmDesc& d = P.d[g];
    if (d.M < 1 || d.N < 1 || d.K < 1 || d.lda % v || d.ldb % v || d.ldc % 8) return false;
    if ((reinterpret_cast<uintptr_t>(d.A) | reinterpret_cast<uintptr_t>(d.B) |
         reinterpret_cast<uintptr_t>(d.C)) & 15u)
      return false;
    if ((int64_t)P.splits * P.k_chunk < d.K) return false;
    // every stage of B has a row to read: loads past the last are clamped to it
    if (d.kb < 0 || (d.kb > 0 && d.kb <= (d.K - 1) / BK * BK)) return false;
    if (d.N % 8 && (d.epi == EPI_MASK_POS || (P.splits > 1 && P.defer_reduce && P.frag)))
      return false;
    if ((d.asum || d.bsum) && !sums) return false;
    if ((d.epi == EPI_L2 || d.epi == EPI_L2SQ) && !dist) return false;
  }
  return true;
}

// Work item (tile, split, problem) of a workgroup.  Workgroups are dealt to
// the 8 XCDs round-robin by linear id; the linear id is remapped so that each
// XCD gets one contiguous eighth of the (problem, split, tile) order -- a run
// of tiles sharing one K range of one problem, whose operand panels then stay
// in that XCD's L2.
struct WorkItem { int tile, split, prob; };
// lin = launch-order id within a grid of gx tiles x gy splits x problems
// (total ids), whose first id sits on XCD 0
__device__ __forceinline__ WorkItem work_item_of(int lin, int gx, int gy, int total) {
  if ((total & 7) == 0) lin = (lin & 7) * (total >> 3) + (lin >> 3);
  WorkItem w;
  w.tile = lin % gx;
  w.split = (lin / gx) % gy;
  w.prob = lin / (gx * gy);
  return w;
}
__device__ __forceinline__ WorkItem gemm_work_item() {
  const int gx = gridDim.x, gy = gridDim.y;
  return work_item_of(blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z), gx, gy,
                      gx * gy * gridDim.z);
}

// 8 consecutive values as FP32, from/to FP32 or BF16 storage (16-byte aligned)
__device__ inline void load8_any(const float* p, float (&o)[8]) {
  *reinterpret_cast<float4*>(o) = *reinterpret_cast<const float4*>(p);
  *reinterpret_cast<float4*>(o + 4) = *reinterpret_cast<const float4*>(p + 4);
}
__device__ inline void load8_any(const bf16_t* p, float (&o)[8]) {
  u32x4 u = *reinterpret_cast<const u32x4*>(p);
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[2 * i] = __builtin_bit_cast(float, w[i] << 16);
    o[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xffff0000u);
  }
}
__device__ inline void store8_any(float* p, const float (&o)[8]) {
  *reinterpret_cast<float4*>(p) = *reinterpret_cast<const float4*>(o);
  *reinterpret_cast<float4*>(p + 4) = *reinterpret_cast<const float4*>(o + 4);
}
__device__ inline void store8_any(bf16_t* p, const float (&o)[8]) {
  u32x4 u;
  u.x = pack2bf(o[0], o[1]);
  u.y = pack2bf(o[2], o[3]);
  u.z = pack2bf(o[4], o[5]);
  u.w = pack2bf(o[6], o[7]);
  *reinterpret_cast<u32x4*>(p) = u;
}

}  // namespace crl

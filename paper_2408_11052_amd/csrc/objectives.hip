// Energies and contrastive objectives on the materialised critic matrix
// F [B][ld] (FP32): the per-row reductions, the in-place gradient dL/dF, and
// the energy backward passes that are not plain products.
//
// Objectives (Appendix A.2 list of tested objectives, with the logsumexp
// penalty of Section 5.3 on every one): InfoNCE forward / backward /
// symmetric, FlatNCE forward / backward (value 1 per row, the gradient of
// the log of its sum), Forward-Backward, DPO, IPO and SPPO, each averaged
// over the positives i with the sum over j taken over the whole batch.
//
// Energies (Appendix A.2): dot and L2 / L2-without-root come from the logit
// GEMM's epilogue; cosine is the dot product of unit rows (unit_rows_kernel);
// L1 is not a product and has its own vector-ALU kernels here.
#include <algorithm>

#include "internal.hpp"

namespace crl {

__device__ __forceinline__ float softplusf(float x) {
  return fmaxf(x, 0.f) + log1pf(__expf(-fabsf(x)));
}


// U[i] = X[i] / |X[i]| (0 for a zero row) and nrm[i] = |X[i]|, one wave per
// row of phi (blockIdx.y = 0) or psi (1).
__global__ __launch_bounds__(256) void unit_rows_kernel(
    const float* __restrict__ phi, const float* __restrict__ psi, float* __restrict__ Uphi,
    float* __restrict__ Upsi, float* __restrict__ nphi, float* __restrict__ npsi, int B, int D) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= B) return;
  const float* x = (blockIdx.y ? psi : phi) + (int64_t)row * D;
  float* U = (blockIdx.y ? Upsi : Uphi) + (int64_t)row * D;
  float s = 0.f;
  for (int d = lane; d < D; d += 64) s += x[d] * x[d];
  s = wave_sum(s);
  const float n = sqrtf(s);
  const float inv = n > 0.f ? 1.f / n : 0.f;
  for (int d = lane; d < D; d += 64) U[d] = x[d] * inv;
  if (lane == 0) (blockIdx.y ? npsi : nphi)[row] = n;
}
hipError_t launch_unit_rows(const float* phi, const float* psi, float* Uphi, float* Upsi,
                            float* nphi, float* npsi, int B, int D, hipStream_t s) {
  CRL_TIMED("unit_rows_kernel", 6.0 * B * D, 8.0 * B * (2.0 * D + 1.0), s,
            unit_rows_kernel<<<dim3((B + 3) / 4, 2), 256, 0, s>>>(phi, psi, Uphi, Upsi, nphi,
                                                                  npsi, B, D));
  return hipGetLastError();
}

// F_ij = -sum_k |phi_ik - psi_jk| for a 64 x 64 tile per workgroup; each of
// the 256 threads owns a 4 x 4 block.  32-feature slices of both operands go
// through LDS (transposed, so a thread's four rows are one 16-byte read).
constexpr int kL1T = 64, kL1K = 32;
__global__ __launch_bounds__(256) void l1_energy_kernel(const float* __restrict__ phi,
                                                        const float* __restrict__ psi,
                                                        float* __restrict__ F, int B, int D,
                                                        int ld) {
  __shared__ __attribute__((aligned(16))) float As[kL1K][kL1T + 4];
  __shared__ __attribute__((aligned(16))) float Bs[kL1K][kL1T + 4];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int i0 = blockIdx.y * kL1T, j0 = blockIdx.x * kL1T;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < D; k0 += kL1K) {
    __syncthreads();
    // 64 rows x 32 features of each operand: 8 values per thread
    for (int v = tid; v < kL1T * kL1K; v += 256) {
      const int r = v / kL1K, k = v % kL1K;
      const bool kin = k0 + k < D;
      As[k][r] = (i0 + r < B && kin) ? phi[(int64_t)(i0 + r) * D + k0 + k] : 0.f;
      Bs[k][r] = (j0 + r < B && kin) ? psi[(int64_t)(j0 + r) * D + k0 + k] : 0.f;
    }
    __syncthreads();
#pragma unroll 8
    for (int k = 0; k < kL1K; ++k) {
      const float4 a = *reinterpret_cast<const float4*>(&As[k][ty * 4]);
      const float4 b = *reinterpret_cast<const float4*>(&Bs[k][tx * 4]);
      const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[p][q] += fabsf(av[p] - bv[q]);
    }
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int i = i0 + ty * 4 + p;
    if (i >= B) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = j0 + tx * 4 + q;
      if (j < B) F[(int64_t)i * ld + j] = -acc[p][q];
    }
  }
}
hipError_t launch_l1_energy(const float* phi, const float* psi, float* F, int B, int D, int ld,
                            hipStream_t s) {
  const dim3 grid((B + kL1T - 1) / kL1T, (B + kL1T - 1) / kL1T);
  CRL_TIMED("l1_energy_kernel", 3.0 * B * B * D, 4.0 * (2.0 * B * D + (double)B * B), s,
            l1_energy_kernel<<<grid, 256, 0, s>>>(phi, psi, F, B, D, ld));
  return hipGetLastError();
}

// dX_xk = -sum_y C(x, y) sign(X_xk - Y_yk), C(x, y) = G[x][y] (side 0:
// X = phi, Y = psi, giving dphi) or G[y][x] (side 1: X = psi, Y = phi,
// giving dpsi, since dF_ij/dpsi_jk = +sign(phi_ik - psi_jk) =
// -sign(psi_jk - phi_ik)).  Five vector instructions per (x, y, k) bind it.
// A workgroup owns 64 rows x 32 features of one side and one split of y: lane
// l has row l, wave w features 8w..8w+7, so the block of C is read from LDS
// without conflicts and Y as broadcasts, and the splits fill the chip.  One
// thread per row and eight strided features with all of y in one workgroup
// (54 workgroups a side) took 1755 us at B = 1701, D = 40; this takes 74.
constexpr int kL1X = 64, kL1F = 32, kL1Y = 32;
__global__ __launch_bounds__(256) void l1_backward_kernel(const float* __restrict__ phi,
                                                          const float* __restrict__ psi,
                                                          const float* __restrict__ G, int ldg,
                                                          float* __restrict__ part, int splits,
                                                          int ysplit, int B, int D) {
  __shared__ __attribute__((aligned(16))) float Ys[kL1Y][kL1F];
  __shared__ float Cs[kL1Y][kL1X + 1];
  const int side = blockIdx.z & 1, f0 = (blockIdx.z >> 1) * kL1F;
  const float* __restrict__ X = side ? psi : phi;
  const float* __restrict__ Y = side ? phi : psi;
  const int tid = threadIdx.x, xl = tid & 63, fq = (tid >> 6) * 8;
  const int x0 = blockIdx.x * kL1X, x = x0 + xl;
  const int yb = blockIdx.y * ysplit, ye = min(B, yb + ysplit);
  float xv[8], acc[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    xv[m] = (x < B && f0 + fq + m < D) ? X[(int64_t)x * D + f0 + fq + m] : 0.f;
    acc[m] = 0.f;
  }
  for (int y0 = yb; y0 < ye; y0 += kL1Y) {
    __syncthreads();
    for (int v = tid; v < kL1Y * kL1F; v += 256) {
      const int r = v / kL1F, k = v % kL1F;
      Ys[r][k] = (y0 + r < ye && f0 + k < D) ? Y[(int64_t)(y0 + r) * D + f0 + k] : 0.f;
    }
    for (int v = tid; v < kL1Y * kL1X; v += 256) {
      // consecutive threads along G's rows
      const int xi = side ? v % kL1X : v / kL1Y, yi = side ? v / kL1X : v % kL1Y;
      float c = 0.f;
      if (x0 + xi < B && y0 + yi < ye)
        c = side ? G[(int64_t)(y0 + yi) * ldg + x0 + xi] : G[(int64_t)(x0 + xi) * ldg + y0 + yi];
      Cs[yi][xi] = c;
    }
    __syncthreads();
#pragma unroll 4
    for (int y = 0; y < kL1Y; ++y) {  // rows past the split hold C = 0
      const float cf = Cs[y][xl];
      const uint32_t c = __builtin_bit_cast(uint32_t, cf);
      const float none = cf * 0.f;  // c sign(d) where d is 0 or NaN: NaN for a NaN or infinite c
      float yv[8];
      *reinterpret_cast<float4*>(yv) = *reinterpret_cast<const float4*>(&Ys[y][fq]);
      *reinterpret_cast<float4*>(yv + 4) = *reinterpret_cast<const float4*>(&Ys[y][fq + 4]);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        // -c sign(d): c with the opposite of d's sign
        const float d = xv[m] - yv[m];
        const uint32_t t = c ^ (~__builtin_bit_cast(uint32_t, d) & 0x80000000u);
        acc[m] += __builtin_islessgreater(d, 0.f) ? __builtin_bit_cast(float, t) : none;
      }
    }
  }
  if (x >= B) return;
  float* out = part + (((int64_t)side * splits + blockIdx.y) * B + x) * D + f0 + fq;
#pragma unroll
  for (int m = 0; m < 8; ++m)
    if (f0 + fq + m < D) out[m] = acc[m];
}
// Splits of y: about 1024 workgroups (four per CU), each at least 128 rows
// of y deep so that its partial (a B x D block) stays cheap to sum.
int l1_backward_splits(int B, int D) {
  const int tiles = (B + kL1X - 1) / kL1X * ((D + kL1F - 1) / kL1F) * 2;
  int S = 1;
  while (S < 16 && tiles * S * 2 <= 1024 && B / (2 * S) >= 128) S *= 2;
  return S;
}
hipError_t launch_l1_backward(const float* phi, const float* psi, const float* G, int ldg,
                              float* part, int splits, int B, int D, hipStream_t s) {
  const int ysplit = ((B + splits - 1) / splits + kL1Y - 1) / kL1Y * kL1Y;
  const dim3 grid((B + kL1X - 1) / kL1X, splits, (D + kL1F - 1) / kL1F * 2);
  CRL_TIMED("l1_backward_kernel", 6.0 * B * B * D, 8.0 * (2.0 * B * D + (double)B * B), s,
            l1_backward_kernel<<<grid, 256, 0, s>>>(phi, psi, G, ldg, part, splits, ysplit, B, D));
  return hipGetLastError();
}

// Per row i of F: r_i = LSE_j F_ij (max-subtracted), F_ii, and for the
// pairwise objectives the row's term of the objective and the sum that
// forms dL/dF_ii:
//   FB:   term = -exp(F_ii) + sum_{j != i} exp(2 F_ij) / (2 (B - 1))
//   DPO:  term = sum_j softplus(F_ij - F_ii),      aux = sum_{j != i} sigmoid(F_ij - F_ii)
//   IPO:  term = sum_j (F_ii - F_ij - 1)^2,        aux = sum_{j != i} (F_ii - F_ij - 1)
//   SPPO: term = B (F_ii - 1)^2 + sum_j (F_ij + 1)^2
template <int LOSS>
__device__ __forceinline__ void row_obj(const float* __restrict__ row, int i, int B, int lane,
                                        float* __restrict__ r, float* __restrict__ diag,
                                        float* __restrict__ term, float* __restrict__ aux) {
  const float fii = row[i];
  float m = -INFINITY;
  for (int j = lane; j < B; j += 64) m = fmaxf(m, row[j]);
  m = wave_max(m);
  float s = 0.f, t = 0.f, a = 0.f;
  for (int j = lane; j < B; j += 64) {
    const float f = row[j];
    s += __expf(f - m);
    if (LOSS == CRL_LOSS_FB) {
      if (j != i) t += __expf(2.f * f);
    } else if (LOSS == CRL_LOSS_DPO) {
      t += softplusf(f - fii);
      if (j != i) a += sigmoidf_(f - fii);
    } else if (LOSS == CRL_LOSS_IPO) {
      const float e = (fii - f) - 1.f;
      t += e * e;
      if (j != i) a += e;
    } else if (LOSS == CRL_LOSS_SPPO) {
      t += (f + 1.f) * (f + 1.f);
    }
  }
  s = wave_sum(s);
  if (LOSS >= CRL_LOSS_FB) t = wave_sum(t);
  if (LOSS == CRL_LOSS_DPO || LOSS == CRL_LOSS_IPO) a = wave_sum(a);
  if (lane == 0) {
    r[i] = m + __logf(s);
    diag[i] = fii;
    if (LOSS == CRL_LOSS_FB) {
      const float scale = B > 1 ? 0.5f / (float)(B - 1) : 0.f;
      term[i] = -__expf(fii) + scale * t;
    } else if (LOSS == CRL_LOSS_SPPO) {
      term[i] = (float)B * (fii - 1.f) * (fii - 1.f) + t;
    } else if (LOSS >= CRL_LOSS_FB) {
      term[i] = t;
    }
    if (LOSS == CRL_LOSS_DPO || LOSS == CRL_LOSS_IPO) aux[i] = a;
  }
}
// Column chunk: the (max, sum) of 256 columns over rows [i0, i1), eight rows'
// loads in flight before their maximum and then their sum are taken, the sum
// pairwise (an eighth of the roundings that grow with it).
__device__ __forceinline__ void col_lse(const float* __restrict__ F, int ld, int B, int j, int i0,
                                        int i1, float& m, float& s) {
  m = -INFINITY;
  s = 0.f;
  for (int i = i0; i < i1; i += 8) {
    float f[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = i + k < i1 ? F[(int64_t)(i + k) * ld + j] : -INFINITY;
    float mn = m;
#pragma unroll
    for (int k = 0; k < 8; ++k) mn = fmaxf(mn, f[k]);
    s = m == -INFINITY ? 0.f : s * __expf(m - mn);
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = i + k < i1 ? __expf(f[k] - mn) : 0.f;
    s += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
    m = mn;
  }
}

// Rows and columns of F in one launch (both only read it): blocks [0, nrow)
// take four rows each, one per wavefront, the rest one chunk of rows of 256
// columns each.
template <int LOSS>
__global__ __launch_bounds__(256) void row_col_kernel(const float* __restrict__ F, int B, int ld,
                                                      int nrow, int ncol, int rows_per,
                                                      float* __restrict__ r,
                                                      float* __restrict__ diag,
                                                      float* __restrict__ term,
                                                      float* __restrict__ aux,
                                                      float* __restrict__ col_m,
                                                      float* __restrict__ col_s) {
  if ((int)blockIdx.x < nrow) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i < B) row_obj<LOSS>(F + (int64_t)i * ld, i, B, threadIdx.x & 63, r, diag, term, aux);
    return;
  }
  const int blk = blockIdx.x - nrow, chunk = blk / ncol;
  const int j = (blk % ncol) * 256 + threadIdx.x;
  if (j >= B) return;
  float m, s;
  col_lse(F, ld, B, j, chunk * rows_per, min(B, (chunk + 1) * rows_per), m, s);
  col_m[(int64_t)chunk * B + j] = m;
  col_s[(int64_t)chunk * B + j] = s;
}
// Row chunks of the column log-sum-exps (at most 64, the workspace's slots):
// enough blocks beside the rows' and few parts to merge (loss layer, 64 chunks
// against these: B = 512 29.6, 28.8 us; B = 1024 39.1, 38.5; B = 2048 the same).
int col_chunks(int B) { return std::min(B, B <= 1024 ? 16 : B <= 2048 ? 32 : 64); }
// Up to B = 256 the loss kernel itself merges them, a launch less; its one
// workgroup reads all of them, so above lse_merge_kernel does.  Loss layer, D =
// 64, merged in the loss kernel against apart: B = 256 24.3 us both, 384 28.1,
// 25.8; 1024 41.6, 38.5; 1536 74.8, 57.6; 2048 94.7, 74.7.
bool col_merge_in_loss(int B) { return B <= 256; }
hipError_t launch_row_col(const float* F, int B, int ld, int loss, float* r, float* diag,
                          float* term, float* aux, float* col_m, float* col_s, hipStream_t s) {
  const int nrow = (B + 3) / 4, ncol = (B + 255) / 256, chunks = col_chunks(B);
  const int rows_per = (B + chunks - 1) / chunks;
  const dim3 grid(nrow + ncol * chunks);
  const double bytes = 4.0 * (2.0 * B * B + 4.0 * B);
  switch (loss) {
#define CRL_ROW_OBJ(L_, NAME)                                                              \
  CRL_TIMED(NAME, 0.0, bytes, s,                                                           \
            row_col_kernel<L_><<<grid, 256, 0, s>>>(F, B, ld, nrow, ncol, rows_per, r, diag, \
                                                    term, aux, col_m, col_s));             \
  break;
    case CRL_LOSS_FB: CRL_ROW_OBJ(CRL_LOSS_FB, "row_col_kernel<fb>")
    case CRL_LOSS_DPO: CRL_ROW_OBJ(CRL_LOSS_DPO, "row_col_kernel<dpo>")
    case CRL_LOSS_IPO: CRL_ROW_OBJ(CRL_LOSS_IPO, "row_col_kernel<ipo>")
    case CRL_LOSS_SPPO: CRL_ROW_OBJ(CRL_LOSS_SPPO, "row_col_kernel<sppo>")
    // the InfoNCE family needs only r and the diagonal
    default: CRL_ROW_OBJ(CRL_LOSS_FWD, "row_col_kernel<lse>")
#undef CRL_ROW_OBJ
  }
  return hipGetLastError();
}

// In place: F_ij -> G_ij = dL/dF_ij, then through the energy's pointwise
// factor: H_ij = G_ij / d_ij for L2 (d_ij = -F_ij, 0 where d_ij = 0),
// H_ij = 2 G_ij for L2 without the root, G_ij otherwise; rowsum_i = sum_j H_ij
// for the two distance energies.  B G_ij =
//   2 beta r_i Pr_ij                                  (penalty, every objective)
// + wf (Pr_ij - d_ij) + wb (Pc_ij - d_ij)             (InfoNCE, FlatNCE)
// + FB:   -exp(F_ii) d_ij + (1 - d_ij) exp(2 F_ij) / (B - 1)
// + DPO:  (1 - d_ij) sigmoid(F_ij - F_ii) - d_ij aux_i
// + IPO:  -2 (1 - d_ij) (F_ii - F_ij - 1) + 2 d_ij aux_i
// + SPPO: 2 (F_ij + 1) + 2 B d_ij (F_ii - 1)
template <int LOSS, int EN>
__global__ __launch_bounds__(256) void grad_obj_kernel(float* __restrict__ F, int B, int ld,
                                                       const float* __restrict__ r,
                                                       const float* __restrict__ c,
                                                       const float* __restrict__ diag,
                                                       const float* __restrict__ aux,
                                                       float beta, float* __restrict__ rowsum) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= B) return;
  const float inv = 1.f / (float)B;
  const float ri = r[i];
  const float pen = 2.f * beta * ri;
  const float fii = diag[i];
  const float ai = (LOSS == CRL_LOSS_DPO || LOSS == CRL_LOSS_IPO) ? aux[i] : 0.f;
  constexpr bool wf = LOSS == CRL_LOSS_FWD || LOSS == CRL_LOSS_SYM || LOSS == CRL_LOSS_FLATNCE_FWD;
  constexpr bool wb = LOSS == CRL_LOSS_SYM || LOSS == CRL_LOSS_BWD || LOSS == CRL_LOSS_FLATNCE_BWD;
  float* row = F + (int64_t)i * ld;
  float rs = 0.f;
  for (int j = lane; j < B; j += 64) {
    const float f = row[j];
    const bool dg = j == i;
    const float pr = __expf(f - ri);
    float g = pr * pen;
    if (wf) g += pr - (dg ? 1.f : 0.f);
    if (wb) g += __expf(f - c[j]) - (dg ? 1.f : 0.f);
    if (LOSS == CRL_LOSS_FB)
      g += dg ? -__expf(fii) : __expf(2.f * f) / (float)(B - 1);
    if (LOSS == CRL_LOSS_DPO) g += dg ? -ai : sigmoidf_(f - fii);
    if (LOSS == CRL_LOSS_IPO) g += dg ? 2.f * ai : -2.f * ((fii - f) - 1.f);
    if (LOSS == CRL_LOSS_SPPO) g += 2.f * (f + 1.f) + (dg ? 2.f * (float)B * (fii - 1.f) : 0.f);
    g *= inv;
    if (EN == CRL_ENERGY_L2) {
      const float d = -f;
      g = d > 0.f ? g / d : 0.f;
    } else if (EN == CRL_ENERGY_L2SQ) {
      g *= 2.f;
    }
    if (EN == CRL_ENERGY_L2 || EN == CRL_ENERGY_L2SQ) rs += g;
    row[j] = g;
  }
  if (EN == CRL_ENERGY_L2 || EN == CRL_ENERGY_L2SQ) {
    rs = wave_sum(rs);
    if (lane == 0) rowsum[i] = rs;
  }
}

template <int LOSS>
static void grad_obj_launch(float* F, int B, int ld, const float* r, const float* c,
                            const float* diag, const float* aux, int energy, float beta,
                            float* rowsum, hipStream_t s) {
  const dim3 grid((B + 3) / 4);
  switch (energy) {
    case CRL_ENERGY_L2:
      grad_obj_kernel<LOSS, CRL_ENERGY_L2><<<grid, 256, 0, s>>>(F, B, ld, r, c, diag, aux, beta, rowsum);
      break;
    case CRL_ENERGY_L2SQ:
      grad_obj_kernel<LOSS, CRL_ENERGY_L2SQ><<<grid, 256, 0, s>>>(F, B, ld, r, c, diag, aux, beta, rowsum);
      break;
    default:  // dot, cosine and L1 use G itself
      grad_obj_kernel<LOSS, CRL_ENERGY_DOT><<<grid, 256, 0, s>>>(F, B, ld, r, c, diag, aux, beta, rowsum);
  }
}

hipError_t launch_grad_obj(float* F, int B, int ld, const float* r, const float* c,
                           const float* diag, const float* aux, int loss, int energy, float beta,
                           float* rowsum, hipStream_t s) {
  KTimer t = timing_begin("grad_obj_kernel", 0.0, 8.0 * B * B, s);
  switch (loss) {
    case CRL_LOSS_FWD: grad_obj_launch<CRL_LOSS_FWD>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    case CRL_LOSS_SYM: grad_obj_launch<CRL_LOSS_SYM>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    case CRL_LOSS_BWD: grad_obj_launch<CRL_LOSS_BWD>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    case CRL_LOSS_FLATNCE_FWD: grad_obj_launch<CRL_LOSS_FLATNCE_FWD>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    case CRL_LOSS_FLATNCE_BWD: grad_obj_launch<CRL_LOSS_FLATNCE_BWD>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    case CRL_LOSS_FB: grad_obj_launch<CRL_LOSS_FB>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    case CRL_LOSS_DPO: grad_obj_launch<CRL_LOSS_DPO>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    case CRL_LOSS_IPO: grad_obj_launch<CRL_LOSS_IPO>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    case CRL_LOSS_SPPO: grad_obj_launch<CRL_LOSS_SPPO>(F, B, ld, r, c, diag, aux, energy, beta, rowsum, s); break;
    default: return hipErrorInvalidValue;
  }
  timing_end(t);
  return hipGetLastError();
}

// The end of the materialised backward, both sides in one launch (one wave per
// row): the split-K partials' sum in split order, the energy's own term
// (distance: - (sum_j H_ij) x_i; cosine: with dU = G V for the unit rows,
// (dU_i - (dU_i . U_i) U_i) / |X_i|, 0 for a zero row) and the BF16 copies.
// Five launches of 4 to 5 us each before (reductions, row terms, casts).
__global__ __launch_bounds__(256) void obj_finish_kernel(ObjFinish a, int splits, int fix, int B,
                                                         int D) {
  const int side = blockIdx.y, lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= B) return;
  const int64_t n = (int64_t)B * D, o = (int64_t)row * D;
  const float* part = a.part[side] + o;  // may be out itself
  const float* __restrict__ X = a.X[side] + o;
  float* out = a.out[side] + o;
  bf16_t* outb = a.outb[side];
  float rs = 0.f, dot = 0.f, inv = 1.f;
  if (fix == kFixDist) {
    double t = 0.0;  // a rounding a split would add up to more than the splits' own
    for (int k = 0; k < a.nrs[side]; ++k) t += (double)a.rs[side][(int64_t)k * B + row];
    rs = (float)t;
  }
  if (fix == kFixCos) {
    for (int d = lane; d < D; d += 64) {
      float v = 0.f;
      for (int k = 0; k < splits; ++k) v += part[k * n + d];
      dot += v * X[d];
    }
    dot = wave_sum(dot);
    const float nr = a.nrm[side][row];
    inv = nr > 0.f ? 1.f / nr : 0.f;
  }
  for (int d = lane; d < D; d += 64) {
    float v = 0.f;
    for (int k = 0; k < splits; ++k) v += part[k * n + d];
    if (fix == kFixDist) v -= rs * X[d];
    if (fix == kFixCos) v = (v - dot * X[d]) * inv;
    out[d] = v;
    if (outb) outb[o + d] = f2bf(v);
  }
}
hipError_t launch_obj_finish(const ObjFinish& a, int splits, int fix, int B, int D,
                             hipStream_t s) {
  CRL_TIMED("obj_finish_kernel", 0.0, 8.0 * B * D * (splits + 2.0), s,
            obj_finish_kernel<<<dim3((B + 3) / 4, 2), 256, 0, s>>>(a, splits, fix, B, D));
  return hipGetLastError();
}

}  // namespace crl

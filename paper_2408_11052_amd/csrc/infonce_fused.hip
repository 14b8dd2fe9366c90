// Fused InfoNCE over the B x B critic matrix without storing it.
//
// Forward: each workgroup owns 64 rows of phi (4 wavefronts x 16 rows, held
// in registers as MFMA A fragments) and one split of the columns.  For every
// 64-column tile of psi (staged in LDS) it forms the tile F = phi . psi^T with
// v_mfma_f32_16x16x32_bf16, applies the energy, and keeps
//   - per row: an online (max, sum exp) pair over its columns,
//   - per column: the (max, sum exp) over the workgroup's 64 rows,
//   - the diagonal F_ii.
// Row pairs of all splits and column pairs of all row blocks are merged by
// lse_merge_kernel; the loss is then a reduction over r, c and the diagonal.
//
// Backward: G_ij = dL/dF_ij = (1/B)[Pr_ij (wf + 2 beta r_i) - wf d_ij
// + wb (Pc_ij - d_ij)] (wf, wb in {0, 1}: the row and column directions of
// InfoNCE / FlatNCE) is recomputed tile by tile from r and c (never stored)
// and multiplied into the streamed operand with a second MFMA:
// dphi = G psi (row pass) and dpsi = G^T phi (column pass, the same kernel
// with the roles of phi and psi exchanged).  For the L2 energy H = G / d
// replaces G (H = 2 G without the root) and the row sums of H give the
// -(sum_j H_ij) phi_i term.  The cosine energy runs as the dot product of
// unit rows; the reduction then projects out the row's own direction and
// divides by its norm.  Each split writes its own partial, summed in a fixed
// order afterwards (no atomics).
#include <cmath>

#include "internal.hpp"
#include <type_traits>

namespace crl {

constexpr int kFRows = 64;   // rows per workgroup
constexpr int kFCols = 64;   // columns per tile

// Energy applied to a tile value v = <x_i, y_j> (x, y the BF16 rows, or the
// BF16 unit rows for the cosine energy) with squared norms nx, ny.
enum : int { kEnDot = 0, kEnL2 = 1, kEnL2sq = 2 };
static int fused_energy(int energy) {
  return energy == CRL_ENERGY_L2 ? kEnL2 : energy == CRL_ENERGY_L2SQ ? kEnL2sq : kEnDot;
}

// Column splits: enough workgroups for four waves per SIMD (1024 x 4 waves
// over 1024 SIMDs), at most 16 partials per row to merge.
int fused_splits(int B) {
  int nrb = (B + kFRows - 1) / kFRows;
  int S = 1024 / nrb;
  if (S < 1) S = 1;
  if (S > 16) S = 16;
  int cps = (B + S - 1) / S;
  cps = (cps + kFCols - 1) / kFCols * kFCols;
  return (B + cps - 1) / cps;
}
static inline int cols_per_split(int B, int S) {
  int cps = (B + S - 1) / S;
  return (cps + kFCols - 1) / kFCols * kFCols;
}

// BF16 copies of phi, psi and the squared norms of the rounded rows; for the
// cosine energy (unit != 0) the BF16 copies are of the unit rows x / |x| and
// the norm slot holds |x| (FP32).
__device__ __forceinline__ void prep_row(float* X, bf16_t* Xb, float* nrm, int row, int D,
                                         int lane, int unit) {
  float s = 0.f;
  if (unit) {
    for (int d = lane; d < D; d += 64) s += X[d] * X[d];
    s = wave_sum(s);
    const float n = sqrtf(s);
    const float inv = n > 0.f ? 1.f / n : 0.f;
    for (int d = lane; d < D; d += 64) Xb[d] = f2bf(X[d] * inv);
    if (lane == 0) nrm[row] = n;
    return;
  }
  for (int d = lane; d < D; d += 64) {
    const bf16_t h = f2bf(X[d]);
    Xb[d] = h;
    const float v = bf2f(h);
    s += v * v;
  }
  s = wave_sum(s);
  if (lane == 0) nrm[row] = s;
}

__global__ void fused_prep_kernel(FusedArgs a, int B, int D, int unit) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int which = blockIdx.y;
  if (row >= B) return;
  const float* X = (which ? a.psi : a.phi) + (int64_t)row * D;
  bf16_t* Xb = (which ? a.psi_b : a.phi_b) + (int64_t)row * D;
  prep_row(const_cast<float*>(X), Xb, which ? a.npsi : a.nphi, row, D, lane, unit);
}

// The same from the output layer's split-K partials: phi / psi = sum of the
// splits in order + bias (FP32, as the split-K reduction writes them), then
// the BF16 copies and norms.
__global__ void fused_prep_reduce_kernel(FusedArgs a, GemmParams P, int B, int D, int unit) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int which = blockIdx.y;
  if (row >= B) return;
  const GemmDesc& G = P.d[which];
  const int64_t MN = (int64_t)G.M * G.N;
  const float* __restrict__ src = P.partial + (int64_t)which * P.partial_len + (int64_t)row * D;
  float* X = reinterpret_cast<float*>(G.C) + (int64_t)row * G.ldc;
  for (int d = lane; d < D; d += 64) {
    float v = 0.f;
    for (int k = 0; k < P.splits; ++k) v += src[k * MN + d];
    X[d] = v + G.bias[d];
  }
  prep_row(X, (which ? a.psi_b : a.phi_b) + (int64_t)row * D, which ? a.npsi : a.nphi, row, D,
           lane, unit);
}

// A 64-row tile of Y [B][D] (BF16) moves global -> registers -> LDS.  Each
// of the 256 threads holds D/32 16-byte vectors; rows past B are zero.  The
// next tile is fetched into registers while the current one is computed on.
template <int D>
struct TileRegs { u32x4 v[D / 32]; };

// A tile inside the batch (the common case) loads without bounds checks from
// one tile base and per-lane 32-bit offsets; only the last tile of the batch
// checks its rows.
template <int D>
__device__ __forceinline__ void tile_load(TileRegs<D>& t, const bf16_t* __restrict__ Y, int j0,
                                          int B, int tid) {
  constexpr int VPR = D / 8;  // 16-byte vectors per row
  const bf16_t* __restrict__ base = Y + (int64_t)j0 * D;
  if (j0 + kFCols <= B) {
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
      t.v[i] = *reinterpret_cast<const u32x4*>(base + (tid + i * 256) * 8);
    return;
  }
#pragma unroll
  for (int i = 0; i < D / 32; ++i) {
    const int v = tid + i * 256;
    const int r = v / VPR;
    u32x4 val = {0u, 0u, 0u, 0u};
    if (j0 + r < B) val = *reinterpret_cast<const u32x4*>(base + v * 8);
    t.v[i] = val;
  }
}

// LDS rows of D BF16 values are padded to D + 16 (a stride of 2 mod 16 in
// 16-byte bank groups; 64 banks of 4 bytes) and, inside each group of 16
// rows, row r is stored at r with its bits 2 and 3 exchanged.  The three
// accesses to the tile are then free of bank conflicts, given the lane groups
// the LDS serves together (measured on gfx950 with the bank-conflict
// counter): ds_write_b128 serves 8 consecutive lanes, each storing 16
// contiguous bytes of one row here; ds_read_b128 serves the 16 lanes that
// share lane bit 5 and the parity of bits 2..4, which for the MFMA row
// operand (lane (g, j): row j, chunk g) meet 16 distinct bank groups; the
// 8-byte transpose read serves a half-wave, rows c..c+3 and c+8..c+11 with
// 32 bytes each, again 16 distinct groups.  The earlier order (padding 8,
// rows 8a + 4b + t at 8a + 2t + b) left the row operand two-way conflicted.
// Both reads keep one per-lane base plus compile-time offsets: row 16 m + j
// (j < 16) is at 16 m + lds_row(j), and row 32 k + 8 g + 4 q + i (g, i < 4)
// at 32 k + 8 q + lds_row(8 g + i).
__device__ __forceinline__ int lds_row(int r) {
  return (r & ~12) | ((r & 4) << 1) | ((r >> 1) & 4);
}
// element offset of position p (a permuted row), column d
template <int D>
__device__ __forceinline__ int lds_pos(int p, int d) {
  return p * (D + 16) + d;
}
// element offset of row r, column d
template <int D>
__device__ __forceinline__ int lds_at(int r, int d) {
  return lds_pos<D>(lds_row(r), d);
}

// rows layout Ys[r][d] (row order and stride as above)
template <int D, int LDY>
__device__ __forceinline__ void tile_store_rows(bf16_t* __restrict__ Ys, const TileRegs<D>& t,
                                                int tid) {
  constexpr int VPR = D / 8;
#pragma unroll
  for (int i = 0; i < D / 32; ++i) {
    const int v = tid + i * 256;
    const int r = v / VPR, c = v % VPR;
    *reinterpret_cast<u32x4*>(Ys + lds_at<D>(r, c * 8)) = t.v[i];
  }
}

// Exponentials are one v_exp_f32 (2^x) of a scaled argument: exp(x - m) is
// exp2((x - m) * log2(e)) in the forward, where x = m must give exactly 1
// (B = 1 gives r_i = F_ii exactly), and exp2(x * log2(e) - s) with the
// shift s = lse * log2(e) + log2(B) formed once per row or column in the
// backward.
constexpr float kL2E = 1.4426950408889634f;  // log2(e)

// Tile entry of the energy from v = <x_i, y_j> (norms nx, ny for the
// distances), and for L2 the distance d (0 below the norm-expansion noise,
// as l2_dist; the hardware square root, whose 1-ulp error is far below the
// BF16 rounding of the operands).  A NaN operand stays NaN in f and d.
template <int EN>
__device__ __forceinline__ float energy_f(float v, float nx, float ny, float& d) {
  if (EN == kEnL2) {
    const float t = nx + ny;
    const float d2 = __builtin_fmaf(-2.f, v, t);
    d = d2 <= kL2Floor * t ? 0.f : __builtin_amdgcn_sqrtf(d2);
    return -d;
  }
  if (EN == kEnL2sq) {
    const float d2 = __builtin_fmaf(-2.f, v, nx + ny);
    d = d2 < 0.f ? 0.f : d2;
    return -d;
  }
  d = 0.f;
  return v;
}
// The same for the backward, with the factor w that turns the gradient of the
// energy's argument into the tile entry: for L2, 1 / d (0 where d is 0) from
// one reciprocal square root, d = d2 / sqrt(d2) (a NaN operand stays NaN in
// both); 2 for the squared distance; 1 for the product.
template <int EN>
__device__ __forceinline__ float energy_fw(float v, float nx, float ny, float& w) {
  if (EN == kEnL2) {
    const float t = nx + ny;
    const float d2 = __builtin_fmaf(-2.f, v, t);
    // the masked entries take r = 0, so that f = -(d2 r) is a signed zero:
    // only exponentials of f are taken, and those do not see the sign (a
    // squared norm that overflows to inf gives NaN here, as it should)
    const float r = d2 <= kL2Floor * t ? 0.f : __builtin_amdgcn_rsqf(d2);
    w = r;
    return -(d2 * r);
  }
  if (EN == kEnL2sq) {
    const float d2 = __builtin_fmaf(-2.f, v, nx + ny);
    w = 2.f;
    return d2 < 0.f ? -0.f : -d2;
  }
  w = 1.f;
  return v;
}
// The maxima of the online log-sum-exp: IEEE maximum, which returns NaN if
// either operand is NaN and needs no canonicalising of its operands (two
// three-operand instructions for a row's four entries and its running max,
// where fmaxf took seven).  A NaN entry makes its row's and column's LSE NaN
// either way: with fmaxf it was skipped by the max but reached the sum.
__device__ __forceinline__ float max_nan(float a, float b) {
  return __builtin_elementwise_maximum(a, b);
}
__device__ __forceinline__ float exp_diff(float x, float m) {
  return __builtin_amdgcn_exp2f((x - m) * kL2E);
}

// The 16 x 64 tile F = X[16 rows] . Y[64 columns]^T of one wave: four
// 16-column accumulators, the K loop outside, so that the four products of
// a K step are independent and their B fragments can be read together.
template <int KS>
__device__ __forceinline__ void tile_product(floatx4 (&acc)[4], const bf16x8 (&xa)[KS],
                                             const bf16_t* __restrict__ Ys, int r16, int g) {
#pragma unroll
  for (int jb = 0; jb < 4; ++jb) acc[jb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    bf16x8 b[4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
      b[jb] = *reinterpret_cast<const bf16x8*>(Ys + lds_pos<KS * 32>(jb * 16 + lds_row(r16), ks * 32 + g * 8));
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
      acc[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[ks], b[jb], acc[jb], 0, 0, 0);
  }
}

// Tiles of wide representations (D >= 128), loaded straight into LDS.
// A tile row is 2 D bytes unpadded, its 16-byte chunk c in slot c ^ wide_swz(row):
// the row operand's 16-byte reads (16 lanes at a time: rows 0-3 and 12-15 of
// one chunk, 4-11 of the next) and the transpose reads (a half-wave: rows
// 4q..4q+3 and 8 + 4q.., two chunks) each fall on 16 distinct 16-byte banks.
__device__ __forceinline__ int wide_swz(int row) { return 2 * (row & 3) + (row & 8); }

// One wave's share of the 64-row tile at row j0 of Y [B][D] into LDS address
// dst: blocks of 1 KB (NR rows), 16 rows a wave.  Rows past B re-read row B-1;
// the entries they meet are masked.
template <int D>
__device__ __forceinline__ void wide_tile_load(const bf16_t* __restrict__ Y, int j0, int B,
                                               uint32_t dst, int wave, int lane) {
  constexpr int RB = 2 * D, NR = 1024 / RB, NI = 16 / NR;  // row bytes, rows per block, blocks
  constexpr int CPR = RB / 16;                             // chunks per row
  const char* base = reinterpret_cast<const char*>(Y) + (int64_t)j0 * RB;
  const int rl = lane / CPR, c = lane % CPR;
  const int last = B - 1 - j0;  // the tile's last row that exists (>= 0)
  dst = __builtin_amdgcn_readfirstlane(dst + wave * NI * 1024);
  if (last >= kFCols - 1) {
    base += wave * 16 * RB;
    bases_ready(base);
#pragma unroll
    for (int i = 0; i < NI; ++i)
      load_to_lds(base + i * 1024, rl * RB + (c ^ wide_swz(i * NR + rl)) * 16,
                  dst + i * 1024);
  } else {
    bases_ready(base);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = i * NR + rl;
      load_to_lds(base, min(wave * 16 + r, last) * RB + (c ^ wide_swz(r)) * 16,
                  dst + i * 1024);
    }
  }
}

// byte offset in a tile of row r16 (of any 16) and step ks's chunk of lane group
// g, less 256 (ks / 4)
template <int D> __device__ __forceinline__ int wide_at(int r16, int ks, int g) {
  return r16 * 2 * D + (((4 * (ks & 3) + g) ^ wide_swz(r16)) << 4);
}

// tile_product from such a tile, fragments a step ahead of their products (the
// forward's; the backward has the loop in its own body, where it spills nothing)
template <int KS>
__device__ __forceinline__ void wide_product(floatx4 (&acc)[4], const bf16x8 (&xa)[KS],
                                             const char* __restrict__ Yt, const int (&oa)[4]) {
  bf16x8 b[2][4];
  auto frags = [&](int ks) {
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
      b[ks & 1][jb] = *reinterpret_cast<const bf16x8*>(Yt + oa[ks & 3] + (ks >> 2) * 256 +
                                                       jb * 16 * 2 * KS * 32);
  };
#pragma unroll
  for (int jb = 0; jb < 4; ++jb) acc[jb] = floatx4{0.f, 0.f, 0.f, 0.f};
  frags(0);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if (ks + 1 < KS) frags(ks + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
      acc[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[ks], b[ks & 1][jb], acc[jb], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Occupancy targets (wavefronts per SIMD) that the register allocation must
// meet: the forward's LDS holds three workgroups per CU at D = 256, the
// backward's two.
template <int KS> constexpr int fwd_waves() { return KS >= 8 ? 3 : 4; }
template <int KS, int EN> constexpr int wide_waves() { return KS >= 8 || EN != kEnDot ? 2 : 3; }

// Per workgroup: 64 rows (wave w: rows 16w + 4g + r of lane (r16, g), r < 4)
// against the 64-column tiles of one column split.  Tiles inside the batch
// on every side skip the masking, and only the tile that holds a wave's
// diagonal entries looks for them (one wave-uniform branch).
// What binds it is the entries: some 20 vector instructions each beside the two
// MFMAs (D = 256, L2), 3.5 of them exponentials or roots.  At D >= 128 the tile goes from global memory straight
// into the one LDS tile while the entries of the tile before are formed, and
// the tile product reads its fragments a step ahead: staged through registers,
// with a branch for each masked sum, B=16384, D=256, L2 took 305 us, now 278;
// B=8192, D=128, dot 62, now 57.  At D <= 64 the tile is a few registers; there
// the branch-free entries alone gave 201 -> 187 us (B=16384, D=64, L2 without
// the root, prep and merge included).
template <int KS, int EN>
__global__ __launch_bounds__(256, fwd_waves<KS>()) void infonce_fwd_kernel(FusedArgs a, int B, int cps) {
  constexpr bool L2 = EN != kEnDot;
  constexpr int D = KS * 32;
  constexpr int LDY = D + 16;
  constexpr int LDC = kFCols + 16;  // column-partial rows
  constexpr bool WIDE = KS >= 4;
  __shared__ __attribute__((aligned(1024))) bf16_t Ys[kFCols * (WIDE ? D : LDY)];
  // column (max, sum) of each (wave, 4-row group) for the current tile
  __shared__ float cm_s[16][LDC], cs_s[16][LDC];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int rb = blockIdx.x;
  const int row_base = rb * kFRows + wave * 16;
  const int c0 = blockIdx.y * cps, c1 = min(B, c0 + cps);
  const bool rows_full = row_base + 16 <= B;

  bf16x8 xa[KS];
  {
    const int row = row_base + r16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (row < B) xa[ks] = *reinterpret_cast<const bf16x8*>(a.phi_b + (int64_t)row * D + ks * 32 + g * 8);
      else xa[ks] = bf16x8{};
    }
  }
  float nx[4], rm[4], rsum[4];
  bool rvalid[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    int row = row_base + 4 * g + r;
    rvalid[r] = row < B;
    nx[r] = (L2 && rvalid[r]) ? a.nphi[row] : 0.f;
    rm[r] = -INFINITY;
    rsum[r] = 0.f;
  }

  // column (max, sum) partials of a finished tile, merged over the 16
  // (wave, row group) entries: their max first, then the rescaled sums.  Each
  // wave takes 16 of the tile's columns, four lanes per column, each lane four
  // of the entries; the lanes' maxima and sums then meet by butterflies over
  // the lane groups (a fixed order).  Every wave does its share every tile, so
  // no wave arrives at the next barrier with the whole merge.
  auto flush_cols = [&](int jp) {
    const int cl = wave * 16 + r16;
    float mv[4], sv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { mv[i] = cm_s[4 * g + i][cl]; sv[i] = cs_s[4 * g + i][cl]; }
    float cm = max_nan(max_nan(mv[0], mv[1]), max_nan(mv[2], mv[3]));
    cm = max_nan(cm, __shfl_xor(cm, 16, 64));
    cm = max_nan(cm, __shfl_xor(cm, 32, 64));
    float cs = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) cs += sv[i] == 0.f ? 0.f : sv[i] * exp_diff(mv[i], cm);
    cs += __shfl_xor(cs, 16, 64);
    cs += __shfl_xor(cs, 32, 64);
    const int col = jp + cl;
    if (g == 0 && col < c1) {
      a.col_m[(int64_t)rb * B + col] = cm;
      a.col_s[(int64_t)rb * B + col] = cs;
    }
  };
  // The entries of a tile, once F is in acc: the row states, the wave's share of
  // the column partials.  special: the tile touches an edge or the diagonal.
  auto entries = [&](const floatx4 (&acc)[4], const float (&nyv)[4], int j0, bool special) {
    float f[4][4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float d;
        f[jb][r] = energy_f<EN>(acc[jb][r], nx[r], nyv[jb], d);
      }
    if (special && j0 <= row_base && row_base < j0 + kFCols) {  // this wave's diagonal entries
#pragma unroll
      for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = row_base + 4 * g + r;
          if (row == j0 + jb * 16 + r16 && row < c1 && rvalid[r]) a.diag[row] = f[jb][r];
        }
    }
    if (special) {  // entries outside the batch or the split become -inf
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        const bool cv = j0 + jb * 16 + r16 < c1;
#pragma unroll
        for (int r = 0; r < 4; ++r) f[jb][r] = (cv && rvalid[r]) ? f[jb][r] : -INFINITY;
      }
    }
    // rows: online (max, sum)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float nm = max_nan(rm[r], max_nan(max_nan(f[0][r], f[1][r]), max_nan(f[2][r], f[3][r])));
      float sr = rsum[r] * exp_diff(rm[r], nm);
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) sr += exp_diff(f[jb][r], nm);
      if (special) sr = nm == -INFINITY ? 0.f : sr;  // nothing of this row seen yet
      rsum[r] = sr;
      rm[r] = nm;
    }
    // columns: (max, sum) over this lane's 4 rows, one entry per (wave, row
    // group); the merge runs after the next barrier
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      const float cm = max_nan(max_nan(f[jb][0], f[jb][1]), max_nan(f[jb][2], f[jb][3]));
      float cs = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) cs += exp_diff(f[jb][r], cm);
      if (special) cs = cm == -INFINITY ? 0.f : cs;
      cm_s[wave * 4 + g][jb * 16 + r16] = cm;
      cs_s[wave * 4 + g][jb * 16 + r16] = cs;
    }
  };
  // the prefetch is unconditional (clamped to the last tile) so the wait
  // before each LDS store covers exactly the previous fetch
  const int jlast = c0 + ((c1 - c0 - 1) / kFCols) * kFCols;
  TileRegs<D> pf;
  float nypf[4] = {0.f, 0.f, 0.f, 0.f};
  auto ny_load = [&](int j0) {
    if (!L2) return;
    const float* __restrict__ base = a.npsi + j0;
    if (j0 + kFCols <= c1) {
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) nypf[jb] = base[jb * 16 + r16];
      return;
    }
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) nypf[jb] = j0 + jb * 16 + r16 < c1 ? base[jb * 16 + r16] : 0.f;
  };
  const uint32_t lds0 = lds_address(Ys);
  int oa[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) oa[t] = wide_at<D>(r16, t, g);
  if (c0 < c1) {
    if constexpr (WIDE) wide_tile_load<D>(a.psi_b, c0, B, lds0, wave, lane);
    else tile_load<D>(pf, a.psi_b, c0, B, tid);
    ny_load(c0);
  }
  for (int j0 = c0; j0 < c1; j0 += kFCols) {
    floatx4 acc[4];
    float nyv[4];
    if constexpr (WIDE) {
      // the tile has arrived, and so have the previous tile's column partials
      asm volatile("" ::: "memory");
      wait_vm<0>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) nyv[jb] = nypf[jb];
      wide_product<KS>(acc, xa, reinterpret_cast<const char*>(Ys), oa);
      if (j0 > c0) flush_cols(j0 - kFCols);
      // every wave has read both: the next tile loads while this one's entries
      // are formed
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (j0 + kFCols < c1) {
        ny_load(j0 + kFCols);
        wide_tile_load<D>(a.psi_b, j0 + kFCols, B, lds0, wave, lane);
      }
    } else {
      __syncthreads();
      if (j0 > c0) flush_cols(j0 - kFCols);
      tile_store_rows<D, LDY>(Ys, pf, tid);
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) nyv[jb] = nypf[jb];
      tile_load<D>(pf, a.psi_b, min(j0 + kFCols, jlast), B, tid);
      ny_load(min(j0 + kFCols, jlast));
      __syncthreads();
      tile_product<KS>(acc, xa, Ys, r16, g);
    }
    if (!rows_full || j0 + kFCols > c1 || (j0 <= row_base && row_base < j0 + kFCols))
      entries(acc, nyv, j0, true);
    else
      entries(acc, nyv, j0, false);
  }
  if (c0 < c1) {
    __syncthreads();
    flush_cols(jlast);
  }
  // merge the row states across the 16 lanes that share each row: the max
  // by a butterfly, then the sums rescaled to it by a butterfly (every lane
  // ends with the same value: each level adds the same two operands)
  float mrow[4], srow[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) mrow[r] = rm[r];
#pragma unroll
  for (int o = 1; o <= 8; o <<= 1)
#pragma unroll
    for (int r = 0; r < 4; ++r) mrow[r] = max_nan(mrow[r], __shfl_xor(mrow[r], o, 64));
#pragma unroll
  for (int r = 0; r < 4; ++r)
    srow[r] = rsum[r] == 0.f ? 0.f : rsum[r] * exp_diff(rm[r], mrow[r]);
#pragma unroll
  for (int o = 1; o <= 8; o <<= 1)
#pragma unroll
    for (int r = 0; r < 4; ++r) srow[r] += __shfl_xor(srow[r], o, 64);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float m = mrow[r], s = srow[r];
    const int row = row_base + 4 * g + r;
    if (r16 == 0 && row < B) {
      a.row_m[(int64_t)blockIdx.y * B + row] = m;
      a.row_s[(int64_t)blockIdx.y * B + row] = s;
    }
  }
}

// Element offset of (column c, row e) in a wave's transposed G strip: 64
// columns of 16 BF16 rows (32 bytes each).  Inside each group of 16 columns,
// column c8 + 8t (c8 < 8, t = 0 or 1) sits in 32-byte slot (c8 + 4t) mod 8 of
// the group's t-th 256-byte half, its two 16-byte halves swapped when t = 1.
// A half-wave's transpose read (columns c..c+3 and c+8..c+11, 32 bytes each)
// then falls on 64 distinct banks, and a strip store (16 lanes at a time over
// 32 banks, measured) is two-way conflicted; with plain 32-byte rows they
// were two-way and four-way.  Permuting each column's four 8-byte chunks by
// bits 2 and 3 of c as well makes the store conflict-free too, but measured
// about 1% slower at D = 256, so the simpler form stays.
__device__ __forceinline__ int gt_at(int c, int e) {
  const int t = (c >> 3) & 1;
  return (c & ~15) * 16 + t * 128 + (((c & 7) + 4 * t) & 7) * 16 + (e ^ (8 * t));
}

// The two passes at D <= 64, both in one launch (blockIdx.z; each writes its
// own half of the partials): D=32, reduction included, B=65 13.3 -> 8.7 us,
// B=9000 82.9 -> 72.3, D=64 B=8192 87.2 -> 75.7 against a launch each.
// TRANS = 0: rows are phi, streamed operand psi -> partials of dphi.
// TRANS = 1: rows are psi, streamed operand phi -> partials of dpsi.
// Per 64-column tile: F (MFMA), G (or H) into the wave's own LDS strip, then
// dX += G . Y with the Y operand read from the row-major tile by the 16-bit
// transpose read (no transposed copy of the tile is kept).  D <= 64 here: a
// wave reads its own strip back.  The tile's column values (the other side's
// LSE, |y|^2) are fetched together with the tile, one tile ahead.
//
// Entry (i, j) of G (rows pass; the columns pass exchanges the roles) is
//   P^r_ij (wf + 2 beta r_i) / B + wb P^c_ij / B - (wf + wb) delta_ij / B,
// and each P / B is one exp2 of f log2(e) - (lse log2(e) + log2 B), the shifts
// formed once per row and per column: the weight wb (0 or 1) of the other
// direction is folded into its shift (+inf when it is 0).  The strip is kept
// transposed, [column][row], so that each lane stores its four rows of a
// column as one 8-byte write; the transpose read gives back the row-major A
// operand of the product.
template <int KS> constexpr int narrow_ldy() { return KS * 32 + 16; }
constexpr int kStripLd = 16;  // transposed G strip: [64 columns][16 rows]
// Sum over the 16 lanes of a row of 16, each quad's in lane order, then the
// quads' pairwise: the order in which the one-pass kernel sums 16 rows of a
// column (four rows of a lane, then the lane groups).
__device__ __forceinline__ float sum16(float h) {
  auto lane = [](float v, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 decltype(ctrl)::value, 15, 15, true));
  };
  using std::integral_constant;
  const float h0 = lane(h, integral_constant<int, 0x00>{}), h1 = lane(h, integral_constant<int, 0x55>{});
  const float h2 = lane(h, integral_constant<int, 0xAA>{}), h3 = lane(h, integral_constant<int, 0xFF>{});
  float s = ((h0 + h1) + h2) + h3;
  s += lane(s, integral_constant<int, 0x141>{});  // the other quad of 8 lanes
  s += lane(s, integral_constant<int, 0x140>{});  // the other half of 16
  return s;
}

// BLK: partials of 256 columns with the one-pass kernel's sums, to the bit.
template <int KS, int EN, int TRANS, bool BLK>
__device__ __forceinline__ void infonce_bwd_narrow(const FusedArgs& a, int B, int cps, float beta,
                                                   float wf, float wb, float log2b,
                                                   bf16_t (&Ys)[2][kFCols * narrow_ldy<KS>()],
                                                   bf16_t (&Gt)[4][kFCols * kStripLd]) {
  constexpr bool L2 = EN != kEnDot;
  constexpr int D = KS * 32;
  constexpr int LDY = narrow_ldy<KS>();
  constexpr int NB = D / 16;  // 16-wide output blocks of dX
  static_assert(KS <= 2, "wider representations: infonce_bwd_wide_kernel");
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef short v8s __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) v4s lds_v4s;

  const bf16_t* Xb = TRANS ? a.psi_b : a.phi_b;
  const bf16_t* Yb = TRANS ? a.phi_b : a.psi_b;
  const float* nX = TRANS ? a.npsi : a.nphi;
  const float* nY = TRANS ? a.nphi : a.npsi;
  // TRANS=0: rows own r_i (and the penalty), columns own c_j; TRANS=1: swapped
  const float* lseX = TRANS ? a.c : a.r;
  const float* lseY = TRANS ? a.r : a.c;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int rb = blockIdx.x;
  const int row_base = rb * kFRows + wave * 16;
  const int c0 = blockIdx.y * cps, c1 = min(B, c0 + cps);
  const bool rows_full = row_base + 16 <= B;
  const float beta2 = 2.f * beta;
  const float dgv = (wf + wb) / (float)B;  // the diagonal's -delta_ij terms
  // shift and weight of the row direction (the penalty rides on the rows'
  // own LSE r_i) and the shift of the column direction, folded with wb
  auto main_shift = [&](float lse) { return __builtin_fmaf(lse, kL2E, log2b); };
  auto other_shift = [&](float lse) {
    return wb != 0.f ? __builtin_fmaf(lse, kL2E, log2b) : INFINITY;
  };

  bf16x8 xa[KS];
  {
    const int row = row_base + r16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (row < B) xa[ks] = *reinterpret_cast<const bf16x8*>(Xb + (int64_t)row * D + ks * 32 + g * 8);
      else xa[ks] = bf16x8{};
    }
  }
  float nx[4], sh_a[4], k_a[4], hsum[4];
  bool rvalid[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = row_base + 4 * g + r;
    rvalid[r] = row < B;
    nx[r] = (L2 && rvalid[r]) ? nX[row] : 0.f;
    const float l = rvalid[r] ? lseX[row] : 0.f;
    sh_a[r] = TRANS ? other_shift(l) : main_shift(l);
    k_a[r] = wf + beta2 * l;  // used by the rows pass only
    hsum[r] = 0.f;
  }
  floatx4 acc_dx[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc_dx[nb] = floatx4{0.f, 0.f, 0.f, 0.f};

  // per-lane column values of a tile (columns j0 + jb*16 + r16)
  struct ColVals { float lse[4], ny[4]; };
  auto col_load = [&](ColVals& cvv, int j0) {
    if (j0 + kFCols <= c1) {
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        cvv.lse[jb] = lseY[j0 + jb * 16 + r16];
        cvv.ny[jb] = L2 ? nY[j0 + jb * 16 + r16] : 0.f;
      }
      return;
    }
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      const int col = j0 + jb * 16 + r16;
      const bool cv = col < c1;
      cvv.lse[jb] = cv ? lseY[col] : 0.f;
      cvv.ny[jb] = (L2 && cv) ? nY[col] : 0.f;
    }
  };

  // tile j0 sits in Ys[buf]; pf holds tile j0 + 64 (stored into the other
  // buffer at the top of the iteration) and cpf its column values
  const int jlast = c0 + ((c1 - c0 - 1) / kFCols) * kFCols;
  TileRegs<D> pf;
  ColVals cvals, cpf;
  if (c0 < c1) {
    tile_load<D>(pf, Yb, c0, B, tid);
    col_load(cvals, c0);
    tile_store_rows<D, LDY>(Ys[0], pf, tid);
    tile_load<D>(pf, Yb, min(c0 + kFCols, jlast), B, tid);
    col_load(cpf, min(c0 + kFCols, jlast));
  }
  int buf = 0;
  for (int j0 = c0; j0 < c1; j0 += kFCols, buf ^= 1) {
    // Ys[buf] is complete, and every wave is past the previous tile's reads
    // of Ys[buf ^ 1] and of the G strips
    __syncthreads();
    if (j0 + kFCols < c1) {
      tile_store_rows<D, LDY>(Ys[buf ^ 1], pf, tid);
      tile_load<D>(pf, Yb, min(j0 + 2 * kFCols, jlast), B, tid);
    }
    const bf16_t* __restrict__ Yt = Ys[buf];
    floatx4 acc[4];
    tile_product<KS>(acc, xa, Yt, r16, g);
    float sh_b[4], k_b[4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      sh_b[jb] = TRANS ? main_shift(cvals.lse[jb]) : other_shift(cvals.lse[jb]);
      k_b[jb] = wf + beta2 * cvals.lse[jb];  // used by the columns pass only
    }
    const bool edge = !rows_full || j0 + kFCols > c1;
    const bool diag = j0 <= row_base && row_base < j0 + kFCols;
    // one 16-column block at a time: its four rows' G, the diagonal and edge
    // terms, H, the rows' sums and the strip store
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      float h[4], wv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float fv = energy_fw<EN>(acc[jb][r], nx[r], cvals.ny[jb], wv[r]);
        const float pa = __builtin_amdgcn_exp2f(__builtin_fmaf(fv, kL2E, -sh_a[r]));
        const float pb = __builtin_amdgcn_exp2f(__builtin_fmaf(fv, kL2E, -sh_b[jb]));
        h[r] = TRANS ? __builtin_fmaf(pb, k_b[jb], pa) : __builtin_fmaf(pa, k_a[r], pb);
      }
      if (diag) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row_base + 4 * g + r == j0 + jb * 16 + r16) h[r] -= dgv;
      }
      if (edge) {
        const bool cv = j0 + jb * 16 + r16 < c1;
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = (cv && rvalid[r]) ? h[r] : 0.f;
      }
      // H = G / d (L2; 0 where d = 0) or 2 G (L2 without the root)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (EN != kEnDot) h[r] *= wv[r];
        if (BLK) asm("" : "+v"(h[r]));  // the sums take the rounded H: no contraction
        hsum[r] += BLK && TRANS ? sum16(h[r]) : h[r];
      }
      uint2 w;
      w.x = pack2bf(h[0], h[1]);
      w.y = pack2bf(h[2], h[3]);
      *reinterpret_cast<uint2*>(&Gt[wave][gt_at(jb * 16 + r16, 4 * g)]) = w;
    }
    // only this wave reads its strip back: a wave-local LDS wait suffices
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
    // dX[16 rows][D] += G[16][64] . Y[64][D]; lane (g, j) needs G[j][8g + 0..7]
    // and Y[8g + 0..7][d] of column d = nb*16 + j: transpose reads of 4 rows
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      v4s gq[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int krow = kk * 32 + 8 * g + 4 * q + (r16 >> 2);
        gq[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_v4s*)(&Gt[wave][gt_at(krow, 4 * (r16 & 3))]));
      }
      v8s gv8 = {gq[0][0], gq[0][1], gq[0][2], gq[0][3], gq[1][0], gq[1][1], gq[1][2], gq[1][3]};
      const bf16x8 ga = __builtin_bit_cast(bf16x8, gv8);
      // up to four output blocks at a time: their B fragments read together
      constexpr int NU = NB < 4 ? NB : 4;
#pragma unroll
      for (int nb0 = 0; nb0 < NB; nb0 += NU) {
        v4s hq[NU][2];
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int jpos = kk * 32 + 8 * q + lds_row(8 * g + (r16 >> 2));
            const int dcol = (nb0 + u) * 16 + 4 * (r16 & 3);
            hq[u][q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(Yt + lds_pos<D>(jpos, dcol)));
          }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          v8s yv = {hq[u][0][0], hq[u][0][1], hq[u][0][2], hq[u][0][3],
                    hq[u][1][0], hq[u][1][1], hq[u][1][2], hq[u][1][3]};
          acc_dx[nb0 + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              ga, __builtin_bit_cast(bf16x8, yv), acc_dx[nb0 + u], 0, 0, 0);
        }
      }
    }
    cvals = cpf;
    col_load(cpf, min(j0 + 2 * kFCols, jlast));
  }
  // write this split's partials (the two passes use separate halves)
  float* dst = a.dX_part + ((int64_t)TRANS * gridDim.y + blockIdx.y) * B * D;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row_base + 4 * g + r;
      if (row < B) dst[(int64_t)row * D + nb * 16 + r16] = acc_dx[nb][r];
    }
  if (L2) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float s = hsum[r];
      if (!(BLK && TRANS))
#pragma unroll
        for (int o = 1; o <= 8; o <<= 1) s += __shfl_xor(s, o, 64);
      const int row = row_base + 4 * g + r;
      if (r16 == 0 && row < B) a.rs_part[((int64_t)TRANS * gridDim.y + blockIdx.y) * B + row] = s;
    }
  }
}

template <int KS, int EN, bool BLK>
__global__ __launch_bounds__(256, 4) void infonce_bwd_kernel(FusedArgs a, int B, int cps,
                                                          float beta, float wf, float wb,
                                                          float log2b) {
  // two tile buffers: the next tile is stored while this one is in use
  __shared__ __attribute__((aligned(16))) bf16_t Ys[2][kFCols * narrow_ldy<KS>()];
  __shared__ __attribute__((aligned(16))) bf16_t Gt[4][kFCols * kStripLd];
  if (blockIdx.z) infonce_bwd_narrow<KS, EN, 1, BLK>(a, B, cps, beta, wf, wb, log2b, Ys, Gt);
  else infonce_bwd_narrow<KS, EN, 0, BLK>(a, B, cps, beta, wf, wb, log2b, Ys, Gt);
}

// The two passes at D >= 128, both in one launch (blockIdx.z; each writes its
// own half of the partials).  As infonce_bwd_kernel, but the dX product is
// split over D instead of rows: after a workgroup barrier each wave multiplies
// all four G strips (64 rows) by its quarter of the tile's columns, so the
// tile is read once per workgroup in that product rather than once per wave.
//
// What binds it is the mix per 64 x 64 tile: 64 MFMAs a wave, some 18 vector
// instructions an entry (of 13 that an L2 entry itself takes) and 192 KB of LDS
// reads a workgroup, with two workgroups on a CU.  Vector instructions and
// MFMAs of a SIMD's two waves overlap only in part (a wave of FMAs beside one
// that keeps the matrix core busy runs at half its rate), and their times
// added, 390 and 250 us at B=16384, D=256, are about the time measured.  Four
// waves on a SIMD (workgroups of eight, half the columns each) or one tile's
// product, another's entries and a third's dX interleaved in one wave took as
// long or longer.
// Tiles go from global memory straight into LDS, one ahead: staged through
// registers they held 32 of a lane's 256, which spilled, and left each step
// waiting for its own fragments.  Fragments are read a step ahead of the tile
// product and two ahead of the dX product, the first of them before the
// barrier; the tile and column loads, and the entries of a tile that touches
// neither an edge nor the diagonal, run without branches.
// B=16384, D=256, L2: 703 -> 625 us for both passes; B=8192, D=256, dot: 150;
// B=8192, D=128, dot: 115 -> 90; B=1500, D=128: 23 -> 15, one launch instead of
// two.
template <int KS, int EN, int TRANS>
__device__ __forceinline__ void infonce_bwd_wide(const FusedArgs& a, int B, int cps, float beta,
                                                 float wf, float wb, float log2b,
                                                 bf16_t* __restrict__ Ys,
                                                 bf16_t* __restrict__ Gt) {
  constexpr bool L2 = EN != kEnDot;
  constexpr int D = KS * 32;
  constexpr int NB = D / 16;  // 16-wide output blocks of dX
  constexpr int NW = NB / 4;  // ... per wave: columns [w D/4, (w+1) D/4) of all 64 rows
  constexpr int TILE = kFCols * D;  // elements of a tile
  constexpr int STRIP = kFCols * 16;
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef short v8s __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) v4s lds_v4s;

  const bf16_t* Xb = TRANS ? a.psi_b : a.phi_b;
  const bf16_t* Yb = TRANS ? a.phi_b : a.psi_b;
  const float* nX = TRANS ? a.npsi : a.nphi;
  const float* nY = TRANS ? a.nphi : a.npsi;
  // TRANS=0: rows own r_i (and the penalty), columns own c_j; TRANS=1: swapped
  const float* lseX = TRANS ? a.c : a.r;
  const float* lseY = TRANS ? a.r : a.c;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int rb = blockIdx.x;
  const int row_base = rb * kFRows + wave * 16;
  const int c0 = blockIdx.y * cps, c1 = min(B, c0 + cps);
  const bool rows_full = row_base + 16 <= B;
  const float beta2 = 2.f * beta;
  const float dgv = (wf + wb) / (float)B;  // the diagonal's -delta_ij terms
  auto main_shift = [&](float lse) { return __builtin_fmaf(lse, kL2E, log2b); };
  auto other_shift = [&](float lse) {
    return wb != 0.f ? __builtin_fmaf(lse, kL2E, log2b) : INFINITY;
  };
  const uint32_t lds0 = lds_address(Ys);
  if (c0 < c1) wide_tile_load<D>(Yb, c0, B, lds0, wave, lane);

  bf16x8 xa[KS];
  {
    const int row = row_base + r16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (row < B) xa[ks] = *reinterpret_cast<const bf16x8*>(Xb + (int64_t)row * D + ks * 32 + g * 8);
      else xa[ks] = bf16x8{};
    }
  }
  float nx[4], sh_a[4], k_a[4], hsum[4];
  bool rvalid[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = row_base + 4 * g + r;
    rvalid[r] = row < B;
    nx[r] = (L2 && rvalid[r]) ? nX[row] : 0.f;
    const float l = rvalid[r] ? lseX[row] : 0.f;
    sh_a[r] = TRANS ? other_shift(l) : main_shift(l);
    k_a[r] = wf + beta2 * l;  // used by the rows pass only
    hsum[r] = 0.f;
  }
  floatx4 acc_dx[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc_dx[nb] = floatx4{0.f, 0.f, 0.f, 0.f};

  // per-lane column values of a tile (columns j0 + jb*16 + r16)
  struct ColVals { float lse[4], ny[4]; };
  auto col_load = [&](ColVals& cvv, int j0) {
    if (j0 + kFCols <= B) {
      const float* __restrict__ lp = lseY + j0;
      const float* __restrict__ np = nY + j0;
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        cvv.lse[jb] = lp[jb * 16 + r16];
        cvv.ny[jb] = L2 ? np[jb * 16 + r16] : 0.f;
      }
      return;
    }
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      const int col = min(j0 + jb * 16 + r16, B - 1);  // past the edge: masked
      cvv.lse[jb] = lseY[col];
      cvv.ny[jb] = L2 ? nY[col] : 0.f;
    }
  };
  ColVals cvals, cpf;
  if (c0 < c1) col_load(cvals, c0);
  // byte offsets in a tile: row operand chunk (t ^ (its row's swizzle)), t the
  // step's low two bits; transpose read of output block u
  int oa[4], ot[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    oa[t] = wide_at<D>(r16, t, g);
    const int tr = 8 * g + (r16 >> 2);  // + 4 q + 32 kk: the same swizzle
    const int ch = (wave * NW + (t < NW ? t : 0)) * 2 + ((r16 & 3) >> 1);
    ot[t] = tr * 2 * D + ((ch ^ wide_swz(tr)) << 4) + (r16 & 1) * 8;
  }

  int buf = 0;
  for (int j0 = c0; j0 < c1; j0 += kFCols, buf ^= 1) {
    // this tile has arrived (its loads were issued a tile ago), and every wave
    // is past the previous tile's reads of the other buffer and of the strips
    asm volatile("" ::: "memory");
    wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const char* __restrict__ Yt = reinterpret_cast<const char*>(Ys + buf * TILE);
    floatx4 acc[4];
    {
      // fragments a step ahead of their products (two ahead spills)
      bf16x8 b[2][4];
      auto frags = [&](int ks) {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
          b[ks & 1][jb] = *reinterpret_cast<const bf16x8*>(Yt + oa[ks & 3] + (ks >> 2) * 256 +
                                                           jb * 16 * 2 * D);
      };
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) acc[jb] = floatx4{0.f, 0.f, 0.f, 0.f};
      frags(0);
      if (j0 + kFCols < c1) {
        col_load(cpf, j0 + kFCols);
        wide_tile_load<D>(Yb, j0 + kFCols, B, lds0 + (buf ^ 1) * TILE * 2, wave, lane);
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + 1 < KS) frags(ks + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
          acc[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[ks], b[ks & 1][jb], acc[jb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    float sh_b[4], k_b[4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      sh_b[jb] = TRANS ? main_shift(cvals.lse[jb]) : other_shift(cvals.lse[jb]);
      k_b[jb] = wf + beta2 * cvals.lse[jb];  // used by the columns pass only
    }
    const bool edge = !rows_full || j0 + kFCols > c1;
    const bool diag = j0 <= row_base && row_base < j0 + kFCols;
    // one 16-column block at a time: its four rows' G, the diagonal and edge
    // terms, H, the rows' sums and the strip store
    auto entries = [&](bool special) {
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        float h[4], wv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float fv = energy_fw<EN>(acc[jb][r], nx[r], cvals.ny[jb], wv[r]);
          const float pa = __builtin_amdgcn_exp2f(__builtin_fmaf(fv, kL2E, -sh_a[r]));
          const float pb = __builtin_amdgcn_exp2f(__builtin_fmaf(fv, kL2E, -sh_b[jb]));
          h[r] = TRANS ? __builtin_fmaf(pb, k_b[jb], pa) : __builtin_fmaf(pa, k_a[r], pb);
        }
        if (special) {
          const bool cv = j0 + jb * 16 + r16 < c1;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (row_base + 4 * g + r == j0 + jb * 16 + r16) h[r] -= dgv;
            h[r] = (cv && rvalid[r]) ? h[r] : 0.f;
          }
        }
        // H = G / d (L2; 0 where d = 0) or 2 G (L2 without the root)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (EN != kEnDot) {
            h[r] *= wv[r];
            asm("" : "+v"(h[r]));  // the sum takes the rounded H: no contraction
          }
          hsum[r] += h[r];
        }
        uint2 w;
        w.x = pack2bf(h[0], h[1]);
        w.y = pack2bf(h[2], h[3]);
        *reinterpret_cast<uint2*>(Gt + wave * STRIP + gt_at(jb * 16 + r16, 4 * g)) = w;
      }
    };
    if (edge || diag) entries(true);
    else entries(false);
    // dX[64 rows][this wave's D/4 columns] += G[64][64] . Y[64][D/4 columns];
    // the A fragments of the four strips are read once and each used NW times,
    // the B fragments two steps ahead
    bf16x8 y[3], ga[2][4];
    auto yread = [&](int i) {
      const int kk = i / NW, u = i % NW;
      v4s hq[2];
#pragma unroll
      for (int q = 0; q < 2; ++q)
        hq[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_v4s*)(Yt + ot[u] + (kk * 32 + 4 * q) * 2 * D));
      v8s yv = {hq[0][0], hq[0][1], hq[0][2], hq[0][3], hq[1][0], hq[1][1], hq[1][2], hq[1][3]};
      y[i % 3] = __builtin_bit_cast(bf16x8, yv);
    };
    auto gread = [&](int kk) {
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        v4s gq[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int krow = kk * 32 + 8 * g + 4 * q + (r16 >> 2);
          gq[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_v4s*)(Gt + st * STRIP + gt_at(krow, 4 * (r16 & 3))));
        }
        v8s gv8 = {gq[0][0], gq[0][1], gq[0][2], gq[0][3], gq[1][0], gq[1][1], gq[1][2], gq[1][3]};
        ga[kk][st] = __builtin_bit_cast(bf16x8, gv8);
      }
    };
    yread(0);
    yread(1);
    // every wave reads all four strips: a workgroup barrier (LDS only)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    gread(0);
#pragma unroll
    for (int i = 0; i < 2 * NW; ++i) {
      if (i + 2 < 2 * NW) yread(i + 2);
      if (i == (NW > 2 ? NW - 2 : 0)) gread(1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < 4; ++st)
        acc_dx[st * NW + i % NW] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            ga[i / NW][st], y[i % 3], acc_dx[st * NW + i % NW], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    cvals = cpf;
  }
  // write this split's partials (the two passes use separate halves)
  float* dst = a.dX_part + ((int64_t)TRANS * gridDim.y + blockIdx.y) * B * D;
#pragma unroll
  for (int st = 0; st < 4; ++st)
#pragma unroll
    for (int u = 0; u < NW; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = rb * kFRows + st * 16 + 4 * g + r;
        if (row < B) dst[(int64_t)row * D + (wave * NW + u) * 16 + r16] = acc_dx[st * NW + u][r];
      }
  if (L2) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float s = hsum[r];
#pragma unroll
      for (int o = 1; o <= 8; o <<= 1) s += __shfl_xor(s, o, 64);
      const int row = row_base + 4 * g + r;
      if (r16 == 0 && row < B) a.rs_part[((int64_t)TRANS * gridDim.y + blockIdx.y) * B + row] = s;
    }
  }
}
template <int KS, int EN>
__global__ __launch_bounds__(256, (wide_waves<KS, EN>())) void infonce_bwd_wide_kernel(
    FusedArgs a, int B, int cps, float beta, float wf, float wb, float log2b) {
  // two tiles and the four G strips
  __shared__ __attribute__((aligned(1024))) bf16_t sm[2 * kFCols * KS * 32 + 4 * kFCols * 16];
  bf16_t* Gt = sm + 2 * kFCols * KS * 32;
  if (blockIdx.z) infonce_bwd_wide<KS, EN, 1>(a, B, cps, beta, wf, wb, log2b, sm, Gt);
  else infonce_bwd_wide<KS, EN, 0>(a, B, cps, beta, wf, wb, log2b, sm, Gt);
}

// Both gradients in one pass (D = 64): a workgroup of 16 wavefronts owns 256
// rows and 256 columns of the critic matrix, computes each 64-column tile of
// G once, and uses it twice:
//   dphi[rows] += G . psi[tile]        (wave w: its 16 rows, as in the row pass)
//   dpsi[tile]  = G^T . phi[rows]      (wave w: 16 columns x 16 features, K = 256)
// phi's 256 rows and the G tile stay in LDS, the tile transposed
// ([column][row]: each lane stores its four rows of a column as one 8-byte
// write); G^T rows are then plain 16-byte reads and the G strip of the first
// product a transpose read, as is phi in the second.  dphi partials go to
// split blockIdx.y (the column block), dpsi partials to split blockIdx.x (the
// row block); for L2 the row and column sums of H go with them.  The entries
// of G are formed as in infonce_bwd_kernel.
// 16 waves and one workgroup a CU move in step, so phases add up (vector
// instructions of the entries, then MFMAs, then stores of the partials: 33 MB
// at B=4096): with one barrier a tile instead of two, the G tile and its column
// sums in two buffers, part of the waves multiply while others form entries,
// and entries off the edges and the diagonal take no branches.  B=4096, D=64,
// reduction included: dot 35.4 -> 34.3 us, L2 46.5 -> 44.8; B=333 17.4 -> 16.5.
constexpr int kBRows = 256;  // rows (and columns) per workgroup of the one-pass backward
int fused_bwd_splits(int B) { return (B + kBRows - 1) / kBRows; }

template <int EN>
__global__ __launch_bounds__(1024) void infonce_bwd_both_kernel(FusedArgs a, int B, float beta,
                                                               float wf, float wb, float log2b) {
  constexpr bool L2 = EN != kEnDot;
  constexpr int D = 64, KS = 2, NB = 4;
  constexpr int LDX = D + 16;          // phi / psi rows in LDS (160 B, lds_at order)
  constexpr int LDGT = kBRows + 16;    // transposed G rows (one per column of the tile, lds_row order)
  // for the product energy, columns with bit 3 set swap adjacent 16-byte
  // chunks: the 8-byte G stores (16 lanes over 32 banks) are then two-way
  // instead of four-way conflicted, with both reads of the tile still
  // conflict-free (the distance energies have no registers to spare for it)
  const int hsw = EN == kEnDot ? 8 * ((threadIdx.x >> 3) & 1) : 0;  // column r16 + 16 m
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef short v8s __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) v4s lds_v4s;
  __shared__ __attribute__((aligned(16))) bf16_t Xs[kBRows * LDX];
  __shared__ __attribute__((aligned(16))) bf16_t Ys[2][kFCols * LDX];  // this tile and the next
  __shared__ __attribute__((aligned(16))) bf16_t Gts[2][kFCols * LDGT];
  __shared__ float csums[2][16][kFCols];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int r0 = blockIdx.x * kBRows, cb0 = blockIdx.y * kBRows;
  const int row_base = r0 + wave * 16;
  const bool rows_full = row_base + 16 <= B;
  const float beta2 = 2.f * beta;
  const float dgv = (wf + wb) / (float)B;

  // phi rows of the block -> LDS (rows past B are zero)
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int v = tid + i * 1024;     // 16-byte vector: row v / 8, chunk v % 8
    const int r = v >> 3, c = v & 7;
    u32x4 val = {0u, 0u, 0u, 0u};
    if (r0 + r < B) val = *reinterpret_cast<const u32x4*>(a.phi_b + (int64_t)(r0 + r) * D + c * 8);
    *reinterpret_cast<u32x4*>(Xs + lds_at<D>(r, c * 8)) = val;
  }
  bf16x8 xa[KS];
  {
    const int row = row_base + r16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (row < B) xa[ks] = *reinterpret_cast<const bf16x8*>(a.phi_b + (int64_t)row * D + ks * 32 + g * 8);
      else xa[ks] = bf16x8{};
    }
  }
  float nx[4], sh_r[4], k_r[4], hrow[4];
  bool rvalid[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = row_base + 4 * g + r;
    rvalid[r] = row < B;
    nx[r] = (L2 && rvalid[r]) ? a.nphi[row] : 0.f;
    const float lr = rvalid[r] ? a.r[row] : 0.f;
    sh_r[r] = __builtin_fmaf(lr, kL2E, log2b);
    k_r[r] = wf + beta2 * lr;
    hrow[r] = 0.f;
  }
  floatx4 acc_dx[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc_dx[nb] = floatx4{0.f, 0.f, 0.f, 0.f};

  // psi tile loader: threads 0..511 move one 16-byte vector each
  auto y_load = [&](int j0) {
    u32x4 val = {0u, 0u, 0u, 0u};
    const int r = (tid & 511) >> 3, c = tid & 7;
    if (tid < 512 && j0 + r < B) val = *reinterpret_cast<const u32x4*>(a.psi_b + (int64_t)(j0 + r) * D + c * 8);
    return val;
  };
  const int ntiles = min(kBRows, B - cb0 + kFCols - 1) / kFCols;
  // tile t sits in Ys[t & 1]; ypf holds tile t + 1, stored into the other
  // buffer at the top of iteration t
  u32x4 ypf = y_load(cb0);
  if (tid < 512) *reinterpret_cast<u32x4*>(Ys[0] + lds_at<D>(tid >> 3, (tid & 7) * 8)) = ypf;
  if (ntiles > 1) ypf = y_load(cb0 + kFCols);
  __syncthreads();  // Ys[0] and Xs are written
  for (int t = 0; t < ntiles; ++t) {
    // One barrier a tile, between G and its second product: every wave is past
    // the tile before's then, so past its reads of Ys[(t + 1) & 1], of the G
    // tile before that and its column sums; and while some waves still multiply
    // others form the next tile's entries.
    const int j0 = cb0 + t * kFCols;
    bf16_t* __restrict__ Gt = Gts[t & 1];
    float (*csum)[kFCols] = csums[t & 1];
    if (t + 1 < ntiles) {
      if (tid < 512) *reinterpret_cast<u32x4*>(Ys[(t + 1) & 1] + lds_at<D>(tid >> 3, (tid & 7) * 8)) = ypf;
      if (t + 2 < ntiles) ypf = y_load(j0 + 2 * kFCols);
    }
    const bf16_t* __restrict__ Yt = Ys[t & 1];
    float sh_c[4], ny[4];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
      const int col = j0 + jb * 16 + r16;
      const bool cv = col < B;
      sh_c[jb] = (wb != 0.f && cv) ? __builtin_fmaf(a.c[col], kL2E, log2b) : INFINITY;
      ny[jb] = (L2 && cv) ? a.npsi[col] : 0.f;
    }
    floatx4 acc[4];
    tile_product<KS>(acc, xa, Yt, r16, g);
    // G (or H = G / d) of the wave's 16 rows, one 16-column block at a time;
    // row and column sums of H for L2
    const bool edge = !rows_full || j0 + kFCols > B;
    const bool diag = j0 <= row_base && row_base < j0 + kFCols;
    float hcol[4] = {0.f, 0.f, 0.f, 0.f};
    auto entries = [&](bool special) {
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        float h[4], wv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float fv = energy_fw<EN>(acc[jb][r], nx[r], ny[jb], wv[r]);
          const float pa = __builtin_amdgcn_exp2f(__builtin_fmaf(fv, kL2E, -sh_r[r]));
          const float pb = __builtin_amdgcn_exp2f(__builtin_fmaf(fv, kL2E, -sh_c[jb]));
          h[r] = __builtin_fmaf(pa, k_r[r], pb);
        }
        if (special) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (row_base + 4 * g + r == j0 + jb * 16 + r16) h[r] -= dgv;
        }
        if (special) {
          const bool cv = j0 + jb * 16 + r16 < B;
#pragma unroll
          for (int r = 0; r < 4; ++r) h[r] = (cv && rvalid[r]) ? h[r] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (EN != kEnDot) {
            h[r] *= wv[r];
            asm("" : "+v"(h[r]));  // the sums take the rounded H: no contraction
          }
          hrow[r] += h[r];
          hcol[jb] += h[r];
        }
        uint2 w;
        w.x = pack2bf(h[0], h[1]);
        w.y = pack2bf(h[2], h[3]);
        *reinterpret_cast<uint2*>(&Gt[(jb * 16 + lds_row(r16)) * LDGT + ((wave * 16 + 4 * g) ^ hsw)]) = w;
      }
    };
    if (edge || diag) entries(true);
    else entries(false);
    if (L2) {
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        float hc = hcol[jb];
        hc += __shfl_xor(hc, 16, 64);
        hc += __shfl_xor(hc, 32, 64);
        if (g == 0) csum[wave][jb * 16 + r16] = hc;
      }
    }
    // dphi[16 rows][D] += G[16][64] . Y[64][D] from the wave's own rows of
    // the tile (only this wave wrote them: a wave-local LDS wait suffices)
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      v4s gq[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int kpos = kk * 32 + 8 * q + lds_row(8 * g + (r16 >> 2));
        gq[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_v4s*)(&Gt[kpos * LDGT + ((wave * 16 + 4 * (r16 & 3)) ^ (EN == kEnDot ? 8 * (g & 1) : 0))]));
      }
      v8s gv8 = {gq[0][0], gq[0][1], gq[0][2], gq[0][3], gq[1][0], gq[1][1], gq[1][2], gq[1][3]};
      const bf16x8 ga = __builtin_bit_cast(bf16x8, gv8);
      // up to four output blocks at a time: their B fragments read together
      constexpr int NU = NB < 4 ? NB : 4;
#pragma unroll
      for (int nb0 = 0; nb0 < NB; nb0 += NU) {
        v4s hq[NU][2];
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int jpos = kk * 32 + 8 * q + lds_row(8 * g + (r16 >> 2));
            const int dcol = (nb0 + u) * 16 + 4 * (r16 & 3);
            hq[u][q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(Yt + lds_pos<D>(jpos, dcol)));
          }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          v8s yv = {hq[u][0][0], hq[u][0][1], hq[u][0][2], hq[u][0][3],
                    hq[u][1][0], hq[u][1][1], hq[u][1][2], hq[u][1][3]};
          acc_dx[nb0 + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              ga, __builtin_bit_cast(bf16x8, yv), acc_dx[nb0 + u], 0, 0, 0);
        }
      }
    }
    __syncthreads();  // the whole G tile (and csum) is in LDS
    {
      // dpsi[16 columns cb16][16 features nb] = G^T . phi over the 256 rows:
      // A = G^T (lane (g, j): rows 32kk + 8g..+7 of column j, one 16-byte
      // read of the transposed tile), B = phi (rows 32kk + 8g..+7 of feature
      // j, transpose reads)
      const int cb16 = wave >> 2, nb = wave & 3;
      floatx4 acc_dy = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < kBRows / 32; ++kk) {
        const bf16x8 av =
            *reinterpret_cast<const bf16x8*>(&Gt[(cb16 * 16 + lds_row(r16)) * LDGT + ((kk * 32 + 8 * g) ^ hsw)]);
        v4s hb[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int kpos = kk * 32 + 8 * q + lds_row(8 * g + (r16 >> 2));
          hb[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_v4s*)(Xs + lds_pos<D>(kpos, nb * 16 + 4 * (r16 & 3))));
        }
        v8s bv = {hb[0][0], hb[0][1], hb[0][2], hb[0][3], hb[1][0], hb[1][1], hb[1][2], hb[1][3]};
        acc_dy = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bv),
                                                         acc_dy, 0, 0, 0);
      }
      float* dst = a.dX_part + ((int64_t)gridDim.y + blockIdx.x) * B * D;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = j0 + cb16 * 16 + 4 * g + r;
        if (col < B) dst[(int64_t)col * D + nb * 16 + r16] = acc_dy[r];
      }
      if (L2 && tid < kFCols && j0 + tid < B) {
        float hs = 0.f;
#pragma unroll
        for (int w = 0; w < 16; ++w) hs += csum[w][tid];
        a.rs_part[((int64_t)gridDim.y + blockIdx.x) * B + j0 + tid] = hs;
      }
    }
  }
  // dphi partial of column block blockIdx.y
  float* dst = a.dX_part + (int64_t)blockIdx.y * B * D;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row_base + 4 * g + r;
      if (row < B) dst[(int64_t)row * D + nb * 16 + r16] = acc_dx[nb][r];
    }
  if (L2) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float hr = hrow[r];
#pragma unroll
      for (int o = 1; o <= 8; o <<= 1) hr += __shfl_xor(hr, o, 64);
      const int row = row_base + 4 * g + r;
      if (r16 == 0 && row < B) a.rs_part[(int64_t)blockIdx.y * B + row] = hr;
    }
  }
}

// dphi and dpsi (blockIdx.y) from the S split partials:
//   dX = sum_s part[s]  (- (sum_s rs[s]) * X_bf16 for the distance energies;
//   for the cosine energy, with U the BF16 unit rows: (dX - (dX . U) U) / |X|),
// FP32 and storage copies, four consecutive columns per thread (16-byte
// loads and stores); with bias_part set, also the column sums of each
// block's rows (the output layer's bias-gradient partials).  en: 0 dot,
// 1 distance, 2 cosine.  NT threads per block: red_threads(D).
constexpr int kRedVec = 4;  // columns per thread
template <typename OutT, int D, int NT>
__global__ __launch_bounds__(NT) void bwd_reduce_kernel(FusedArgs a, int S, int B, int en, int rounds) {
  constexpr int TPR = D / kRedVec;  // threads per row
  constexpr int TR = NT / TPR;      // rows per round; a block takes `rounds` rounds
  __shared__ float red[NT];
  __shared__ float4 redv[NT];
  const int side = blockIdx.y;
  const int c = threadIdx.x % TPR;
  const int64_t n = (int64_t)B * D;
  const bf16_t* __restrict__ Xb = side ? a.psi_b : a.phi_b;
  float4 bsum = make_float4(0.f, 0.f, 0.f, 0.f);  // this thread's columns over the block's rows
#pragma unroll 2
  for (int rd = 0; rd < rounds; ++rd) {
    const int row = (blockIdx.x * rounds + rd) * TR + threadIdx.x / TPR;
    const int64_t idx = (int64_t)row * D + c * kRedVec;
    float v[kRedVec] = {0.f, 0.f, 0.f, 0.f}, u[kRedVec] = {0.f, 0.f, 0.f, 0.f};
    if (row < B) {
      const float* __restrict__ part = a.dX_part + (int64_t)side * S * n + idx;
#pragma unroll 2
      for (int i = 0; i < S; ++i) {
        const float4 p = *reinterpret_cast<const float4*>(part + i * n);
        v[0] += p.x; v[1] += p.y; v[2] += p.z; v[3] += p.w;
      }
      if (en != 0) {
        const uint2 xw = *reinterpret_cast<const uint2*>(Xb + idx);
        u[0] = __builtin_bit_cast(float, xw.x << 16);
        u[1] = __builtin_bit_cast(float, xw.x & 0xffff0000u);
        u[2] = __builtin_bit_cast(float, xw.y << 16);
        u[3] = __builtin_bit_cast(float, xw.y & 0xffff0000u);
      }
      if (en == 1) {
        const float* __restrict__ rs = a.rs_part + (int64_t)side * S * B + row;
        float h = 0.f;
        for (int i = 0; i < S; ++i) h += rs[(int64_t)i * B];
#pragma unroll
        for (int k = 0; k < kRedVec; ++k) v[k] -= h * u[k];
      }
    }
    if (en == 2) {  // the row's dot product with its unit vector, a tree over its TPR threads
      red[threadIdx.x] = (v[0] * u[0] + v[1] * u[1]) + (v[2] * u[2] + v[3] * u[3]);
      __syncthreads();
      for (int o = TPR / 2; o > 0; o >>= 1) {
        if (c < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
      }
      const float dot = red[threadIdx.x - c];
      __syncthreads();
      if (row < B) {
        const float nr = (side ? a.npsi : a.nphi)[row];
#pragma unroll
        for (int k = 0; k < kRedVec; ++k) v[k] = nr > 0.f ? (v[k] - dot * u[k]) / nr : 0.f;
      }
    }
    if (row < B) {
      *reinterpret_cast<float4*>((side ? a.dpsi : a.dphi) + idx) = make_float4(v[0], v[1], v[2], v[3]);
      OutT* t = reinterpret_cast<OutT*>(side ? a.dpsi_t : a.dphi_t) + idx;
      if constexpr (sizeof(OutT) == 2)
        *reinterpret_cast<uint2*>(t) = make_uint2(pack2bf(v[0], v[1]), pack2bf(v[2], v[3]));
      else
        *reinterpret_cast<float4*>(t) = make_float4(v[0], v[1], v[2], v[3]);
      bsum.x += v[0]; bsum.y += v[1]; bsum.z += v[2]; bsum.w += v[3];  // rows past B add nothing
    }
  }
  float* bias = a.bias_part[side];
  if (bias == nullptr) return;
  redv[threadIdx.x] = bsum;
  __syncthreads();
  if (threadIdx.x < TPR) {
    float4 t = redv[threadIdx.x];
#pragma unroll
    for (int q = 1; q < TR; ++q) {
      const float4 w = redv[q * TPR + threadIdx.x];
      t.x += w.x; t.y += w.y; t.z += w.z; t.w += w.w;
    }
    *reinterpret_cast<float4*>(bias + (int64_t)blockIdx.x * D + threadIdx.x * kRedVec) = t;
  }
}

// Threads per block of the backward reduction: 1024 at D >= 128, so that a
// block's rounds (below) stay few and each SIMD holds eight wavefronts of
// them; 256 below.
static constexpr int red_threads(int D) { return D >= 128 ? 1024 : 256; }

// Rounds of red_threads(D) * kRedVec / D rows per block of the backward reduction:
// enough that the output layer's bias keeps at most 512 partial rows.  With
// one round it had 16384 at B = 16384, D = 256, which the gradient reduction
// sums serially per column (103 us for the reduction, 43.7 us with 512);
// capped at 256 the rounds left this kernel too few blocks (91 us against 56).
static int fused_bias_rounds(int B, int D) {
  const int tr = red_threads(D) * kRedVec / D;
  const int blocks = (B + tr - 1) / tr;
  return std::max(1, (blocks + 511) / 512);
}
int fused_bias_chunks(int B, int D) {
  const int rows = (red_threads(D) * kRedVec / D) * fused_bias_rounds(B, D);
  return (B + rows - 1) / rows;
}

#define CRL_FUSED_DISPATCH(KS_, BODY)                      \
  switch (D) {                                              \
    case 32:  { constexpr int KS_ = 1; BODY; } break;      \
    case 64:  { constexpr int KS_ = 2; BODY; } break;      \
    case 128: { constexpr int KS_ = 4; BODY; } break;      \
    case 256: { constexpr int KS_ = 8; BODY; } break;      \
    default: return hipErrorInvalidValue;                   \
  }

// Workgroups of the forward kernel for (D, energy) that the device holds at
// once (its register and LDS use decide how many fit on a CU), or 0 if unknown.
static int fwd_resident_wgs(int D, int en) {
  const void* k = nullptr;
#define CRL_FWD_PTR(KS_)                                                           \
  k = en == kEnL2 ? reinterpret_cast<const void*>(&infonce_fwd_kernel<KS_, kEnL2>)   \
    : en == kEnL2sq ? reinterpret_cast<const void*>(&infonce_fwd_kernel<KS_, kEnL2sq>) \
                    : reinterpret_cast<const void*>(&infonce_fwd_kernel<KS_, kEnDot>)
  switch (D) {
    case 32: CRL_FWD_PTR(1); break;
    case 64: CRL_FWD_PTR(2); break;
    case 128: CRL_FWD_PTR(4); break;
    case 256: CRL_FWD_PTR(8); break;
    default: return 0;
  }
#undef CRL_FWD_PTR
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, 256, 0) != hipSuccess)
    return 0;
  return std::min(per_cu, D >= 256 ? fwd_waves<8>() : fwd_waves<4>()) * cus;
}

// Column splits of the forward: fused_splits(B), or fewer where the kernel's
// resident capacity takes the launch in one round that way (D = 256 holds
// three workgroups per CU: 3 splits at B=16384 run in one round, 4 in two).
// The count returned is that of the non-empty splits once each split's
// columns are rounded up to whole 64-column tiles.
static int fused_fwd_splits(int B, int D, int en) {
  const int S = fused_splits(B);
  const int nrb = (B + kFRows - 1) / kFRows;
  const int cap = fwd_resident_wgs(D, en);
  if (cap <= 0 || (int64_t)nrb * S <= cap) return S;
  const int S1 = std::max(1, cap / nrb);
  // one round of S1 splits against ceil(nrb S / cap) rounds of S splits
  const int64_t rounds = ((int64_t)nrb * S + cap - 1) / cap;
  if ((int64_t)S1 * rounds <= S) return S;
  const int cps = cols_per_split(B, S1);
  return (B + cps - 1) / cps;
}

// Workgroups of one of the two backward passes that the device holds at once,
// for the split rule: the waves on a SIMD (one of each workgroup on its CU) that
// each kernel's registers leave, which is part of the rule (the splits decide
// the order of the partial sums) and so stated here.
static int bwd_resident_wgs(int D, int en) {
  const int per_cu = D >= 256 ? 2 : D >= 128 ? (en == kEnDot ? 3 : 2) : D >= 64 ? 4 : (en == kEnDot ? 6 : 4);
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  return per_cu * cus;
}

// Column splits of the two backward passes: each split writes a B x D
// partial of dX that bwd_reduce_kernel reads back, so take the fewest splits
// (at most fused_splits(B)) whose busiest workgroup slot carries no more
// 64-column tiles than with fused_splits(B): rounds of resident workgroups
// times tiles per workgroup (B=16384, D=256: 2 splits and not 4, half the
// partials).  The rounds are those of one pass, as when each had a launch of its
// own; the one grid of both has twice the workgroups (there 1024, two rounds of
// 512), and a count over it would come to fewer splits still.  It stays because
// the splits decide the order of the partial sums, which BF16 training keeps.
static int fused_bwd2_splits(int B, int D, int en) {
  const int S = fused_splits(B);
  const int nrb = (B + kFRows - 1) / kFRows;
  const int cap = bwd_resident_wgs(D, en);
  if (cap <= 0) return S;
  auto load = [&](int s) {
    const int64_t rounds = ((int64_t)nrb * s + cap - 1) / cap;
    return rounds * (cols_per_split(B, s) / kFCols);
  };
  const int64_t target = load(S);
  int best = S;
  for (int s = S - 1; s >= 1; --s)
    if (load(s) <= target) best = s;
  const int cps = cols_per_split(B, best);
  return (B + cps - 1) / cps;
}

#define CRL_EN_DISPATCH(EN_, BODY)                                  \
  switch (en) {                                                      \
    case kEnL2:   { constexpr int EN_ = kEnL2; BODY; } break;        \
    case kEnL2sq: { constexpr int EN_ = kEnL2sq; BODY; } break;      \
    default:      { constexpr int EN_ = kEnDot; BODY; } break;       \
  }

static const char* fused_name(const char* const names[3], int en) { return names[en]; }

hipError_t launch_fused_fwd(const FusedArgs& a, int B, int D, int energy, const GemmParams* top,
                            hipStream_t s) {
  const int en = fused_energy(energy);
  const int unit = energy == CRL_ENERGY_COS;
  if (top)
    CRL_TIMED("fused_prep_reduce_kernel", 0.0, 2.0 * B * D * (4.0 * top->splits + 10.0), s,
              fused_prep_reduce_kernel<<<dim3((B + 3) / 4, 2), 256, 0, s>>>(a, *top, B, D, unit));
  else
    CRL_TIMED("fused_prep_kernel", 0.0, 2.0 * B * D * 6.0, s,
              fused_prep_kernel<<<dim3((B + 3) / 4, 2), 256, 0, s>>>(a, B, D, unit));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int S = fused_fwd_splits(B, D, en), cps = cols_per_split(B, S);
  const int nrb = (B + kFRows - 1) / kFRows;
  dim3 grid(nrb, S);
  const double fw_flops = 2.0 * B * B * D;
  const double fw_bytes = 2.0 * 2.0 * B * D + 4.0 * 2.0 * ((double)S * B + (double)nrb * B);
  static const char* const names[3] = {"infonce_fwd_kernel<dot>", "infonce_fwd_kernel<l2>",
                                       "infonce_fwd_kernel<l2sq>"};
  KTimer t = timing_begin(fused_name(names, en), fw_flops, fw_bytes, s);
  CRL_EN_DISPATCH(EN, CRL_FUSED_DISPATCH(KS, (infonce_fwd_kernel<KS, EN><<<grid, 256, 0, s>>>(a, B, cps))))
  timing_end(t);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  LseMergeArgs m{};  // row LSEs over the column splits, column LSEs over the row blocks
  m.pm[0] = a.row_m; m.ps[0] = a.row_s; m.nparts[0] = S; m.out[0] = a.r;
  m.pm[1] = a.col_m; m.ps[1] = a.col_s; m.nparts[1] = nrb; m.out[1] = a.c;
  return launch_lse_merge(m, 2, B, s);
}

// At D = 64 the partials of dphi and of dpsi are those of 256-row blocks,
// ceil(B / 256) of B x 64 floats each; above kBothMaxSplits of them the passes
// choose their splits, at most 16 (fused_splits).
constexpr int kBothMaxSplits = 16;
bool fused_bwd_blocks(int B, int D) { return D == 64 && fused_bwd_splits(B) <= kBothMaxSplits; }

// Such partials come from the one-pass kernel, a 256 x 256 block per workgroup
// of a whole CU, or, equal to the bit, from the two passes with 256 columns a
// workgroup: twice the entries, but 8 times the workgroups, each with a
// quarter of the waves.  The passes are faster while the device holds all of
// their workgroups at once (B up to 2816 on 256 CUs).  Reduction included, one
// pass against two: dot B=333 16.7, 9.8 us; B=1000 18.5, 11.7; B=2048 20.9, 15.3;
// B=2816 23.9, 23.5; B=4096 33.9, 34.4.  L2 B=333 23.0, 13.8; B=2048 29.1, 21.2;
// B=3072 35.8, 36.6.
static bool blocks_by_passes(int B, int en) {
  const int64_t nrb = (B + kFRows - 1) / kFRows;
  return 2 * nrb * fused_bwd_splits(B) <= bwd_resident_wgs(64, en);
}

hipError_t launch_fused_bwd(const FusedArgs& a, int B, int D, int energy, int loss, float beta,
                            bool out_bf16, hipStream_t s, BlockRoute route) {
  const int en = fused_energy(energy);
  const float wf = (loss == CRL_LOSS_FWD || loss == CRL_LOSS_SYM || loss == CRL_LOSS_FLATNCE_FWD) ? 1.f : 0.f;
  const float wb = (loss == CRL_LOSS_SYM || loss == CRL_LOSS_BWD || loss == CRL_LOSS_FLATNCE_BWD) ? 1.f : 0.f;
  const int64_t n = (int64_t)B * D;
  const float l2b = (float)std::log2((double)B);
  const bool blocks = fused_bwd_blocks(B, D);
  const bool one = blocks && (route == kRouteAuto ? !blocks_by_passes(B, en) : route == kRouteOnePass);
  const int S = blocks ? fused_bwd_splits(B) : fused_bwd2_splits(B, D, en);
  if (one) {  // one pass for both gradients
    const dim3 grid(S, S);
    const double flops = 4.0 * B * B * D;  // G . psi and G^T . phi; the tile recompute is not counted
    const double bytes = 2.0 * 2.0 * B * D + 4.0 * 2.0 * B + 2.0 * 4.0 * (double)S * B * (D + 1.0);
    static const char* const names[3] = {"infonce_bwd_both_kernel<dot>",
                                         "infonce_bwd_both_kernel<l2>",
                                         "infonce_bwd_both_kernel<l2sq>"};
    KTimer t = timing_begin(fused_name(names, en), flops, bytes, s);
    CRL_EN_DISPATCH(EN, (infonce_bwd_both_kernel<EN><<<grid, 1024, 0, s>>>(a, B, beta, wf, wb, l2b)))
    timing_end(t);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int cps = blocks ? kBRows : cols_per_split(B, S);
  const int nrb = (B + kFRows - 1) / kFRows;
  const double bw_flops = 2.0 * B * B * D;  // G . Y per pass; the tile recompute is not counted
  const double bw_bytes = 2.0 * 2.0 * B * D + 4.0 * 2.0 * B + 4.0 * (double)S * B * (D + 1.0);
  if (!one) {  // both passes in one launch
    const dim3 grid(nrb, S, 2);
    KTimer t = timing_begin(D >= 128 ? "infonce_bwd_wide_kernel" : "infonce_bwd_kernel",
                            2.0 * bw_flops, 2.0 * bw_bytes, s);
    switch (D) {
      case 32: CRL_EN_DISPATCH(EN, (infonce_bwd_kernel<1, EN, false><<<grid, 256, 0, s>>>(a, B, cps, beta, wf, wb, l2b))) break;
      case 64:
        if (blocks) {
          CRL_EN_DISPATCH(EN, (infonce_bwd_kernel<2, EN, EN != kEnDot><<<grid, 256, 0, s>>>(a, B, cps, beta, wf, wb, l2b)))
        } else {
          CRL_EN_DISPATCH(EN, (infonce_bwd_kernel<2, EN, false><<<grid, 256, 0, s>>>(a, B, cps, beta, wf, wb, l2b)))
        }
        break;
      case 128: CRL_EN_DISPATCH(EN, (infonce_bwd_wide_kernel<4, EN><<<grid, 256, 0, s>>>(a, B, cps, beta, wf, wb, l2b))) break;
      default: CRL_EN_DISPATCH(EN, (infonce_bwd_wide_kernel<8, EN><<<grid, 256, 0, s>>>(a, B, cps, beta, wf, wb, l2b)))
    }
    timing_end(t);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int ren = energy == CRL_ENERGY_COS ? 2 : (en != kEnDot ? 1 : 0);
  const dim3 rgrid(fused_bias_chunks(B, D), 2);
  const int rounds = fused_bias_rounds(B, D);
  const double rb = 2.0 * (4.0 * (double)n * (S + 1.0) + (double)n * (out_bf16 ? 2 : 4));
  if (out_bf16) {
    CRL_TIMED("bwd_reduce_kernel", 0.0, rb, s,
              CRL_FUSED_DISPATCH(KS, (bwd_reduce_kernel<bf16_t, KS * 32, red_threads(KS * 32)>
                                      <<<rgrid, red_threads(KS * 32), 0, s>>>(a, S, B, ren, rounds))));
  } else {
    CRL_TIMED("bwd_reduce_kernel", 0.0, rb, s,
              CRL_FUSED_DISPATCH(KS, (bwd_reduce_kernel<float, KS * 32, red_threads(KS * 32)>
                                      <<<rgrid, red_threads(KS * 32), 0, s>>>(a, S, B, ren, rounds))));
  }
  return hipGetLastError();
}

}  // namespace crl

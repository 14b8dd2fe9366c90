// Instantiations, launch planning and host dispatch of the MFMA GEMM.
#include "internal.hpp"
#include "gemm_lds.hpp"

namespace crl {

// Sum of split-K partials: C[m][n] (+)= sum_s partial[s][m][n] (+ bias[n]),
// FP32 out; the only epilogues used with split-K are none and bias.
__global__ void splitk_reduce_kernel(GemmParams P) {
  const int g = blockIdx.y;
  const GemmDesc& D = P.d[g];
  const int64_t MN = (int64_t)D.M * D.N;
  const float* src = P.partial + (int64_t)g * P.partial_len;
  float* C = reinterpret_cast<float*>(D.C);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < MN;
       i += (int64_t)gridDim.x * blockDim.x) {
    float s = 0.f;
    for (int k = 0; k < P.splits; ++k) s += src[k * MN + i];
    int64_t row = i / D.N, col = i % D.N;
    int64_t o = row * D.ldc + col;
    if (D.epi == EPI_BIAS) s += D.bias[col];
    C[o] = s;
  }
}

// by storage type, layouts (those of run_layout) and output type
template <typename T, int LA, int LB, typename OutT>
static const char* lds_kernel_name() {
  static const char* names[2][3][2] = {
      {{"gemm_lds_kernel<f32,KC,KC,f32>", nullptr},
       {"gemm_lds_kernel<f32,KC,MC,f32>", nullptr},
       {"gemm_lds_kernel<f32,MC,MC,f32>", nullptr}},
      {{"gemm_lds_kernel<KC,KC,f32>", "gemm_lds_kernel<KC,KC,bf16>"},
       {"gemm_lds_kernel<KC,MC,f32>", "gemm_lds_kernel<KC,MC,bf16>"},
       {"gemm_lds_kernel<MC,MC,f32>", nullptr}}};
  static_assert(LA <= LB, "layouts in use: KC x KC, KC x MC, MC x MC");
  return names[sizeof(T) == 2][LA + LB][sizeof(OutT) == 2];
}

int frag_bn(const GemmParams& P) {
  int nmax = 0;
  for (int g = 0; g < P.count; ++g) nmax = P.d[g].N > nmax ? P.d[g].N : nmax;
  return nmax > 64 ? 128 : 64;
}

int64_t frag_partial_floats(const GemmParams& P, int g, int bn) {
  const GemmDesc& d = P.d[g];
  return (int64_t)((d.M + 127) / 128) * ((d.N + bn - 1) / bn) * 128 * bn;
}

// algorithmic FLOPs and bytes of one launch (the unpadded K)
static void algo_counts(const GemmParams& P, double esize, double osize, double& flops,
                        double& bytes) {
  for (int g = 0; g < P.count; ++g) {
    const GemmDesc& d = P.d[g];
    const double k = d.kb > 0 ? d.kb : d.K;
    flops += 2.0 * d.M * d.N * k;
    bytes += esize * ((double)d.M * k + k * d.N) + (P.splits > 1 ? 4.0 : osize) * d.M * d.N;
  }
}

static int max_tiles(const GemmParams& P) {
  int maxt = 0;
  for (int g = 0; g < P.count; ++g) maxt = P.tiles[g] > maxt ? P.tiles[g] : maxt;
  return maxt;
}

static int64_t tiles_of(const GemmDesc& d, int tile) {
  static const int rows[4] = {32, 64, 64, 128}, cols[4] = {32, 32, 64, 128};
  return (int64_t)((d.M + rows[tile] - 1) / rows[tile]) *
         ((d.N + cols[tile] - 1) / cols[tile]);
}
static int64_t tiles_of(const GemmParams& P, int tile) {
  int64_t n = 0;
  for (int g = 0; g < P.count; ++g) n += tiles_of(P.d[g], tile);
  return n;
}
int64_t gemm_tiles128(const GemmDesc& d) { return tiles_of(d, kTile128); }

void set_tile(GemmParams& P, int tile) {
  static const int cols[4] = {32, 32, 64, 128};
  P.tile = tile;
  for (int g = 0; g < P.count; ++g) {
    P.tiles_n[g] = (P.d[g].N + cols[tile] - 1) / cols[tile];
    P.tiles[g] = (int)tiles_of(P.d[g], tile);
  }
}

// Tile of a launch with n[tile] work items in each: the one with the least
// time, taken as (work items of the busiest of 256 CUs) x (a work item's
// time).  A small tile spreads a small launch and shortens its longest chain;
// a large one reads its operands from LDS less often.  The times are measured
// per K of 1024, launch overhead off, in us; the first number is that of a CU
// with one work item, whose latencies nothing hides, the second that of each
// of several.  (FP32, 2 x 600 x 1024 x 1024: 33.4 us in 32, 28.8 in 64 x 32,
// 35.6 in 64 tiles; 2 x 256: 15.4, 17.9, 25.4; 2 x 4096: 161, 140, 133, and
// 126 in 128 tiles.  BF16, 2 x 512: 12.5 us in 32, 8.5 in 64, 11.6 in 128
// tiles; 2 x 2048: 43, 18.5, 13.4.)
static int pick_tile(const int64_t (&n)[4], bool bf16) {
  static const double one[2][4] = {{5.7, 13.9, 21.3, 66.0}, {2.1, 1e9, 4.4, 8.0}};
  static const double more[2][4] = {{5.6, 8.2, 16.0, 61.0}, {2.1, 1e9, 3.4, 8.7}};
  int best = kTile128;
  double least = 1e300;
  for (int t = kTile128; t >= kTile32; --t) {
    const int64_t rounds = (n[t] + 255) / 256;
    const double us = rounds <= 1 ? one[bf16][t] : more[bf16][t] * (double)rounds;
    if (us < least) {
      least = us;
      best = t;
    }
  }
  return best;
}
static int pick_tile(const GemmParams& P, int splits, bool bf16) {
  int64_t n[4];
  for (int t = 0; t < 4; ++t) n[t] = tiles_of(P, t) * splits;
  return pick_tile(n, bf16);
}

// BF16 launches with a K that is no whole number of stages run in the other k
// order (see fragment).  That order keeps their bits; the tile would not matter
// to them, but 64 is the only one built in it (critic forward and backward, 3 x
// 1024 layers: B = 4097 535 us on the earlier register-staged kernel, 419 here;
// B = 4096 326).
template <typename T> static bool alt_order(const GemmParams& P) {
  bool alt = false;
  if (sizeof(T) == 2)
    for (int g = 0; g < P.count; ++g) alt = alt || P.d[g].K % lds::bk<T>() != 0;
  return alt;
}

template <typename T, int LA, int LB, typename OutT, int TILE, bool ALT>
static void run_tile(const GemmParams& P, hipStream_t s) {
  typedef typename lds::TileOf<T, TILE>::type C;
  const dim3 grid(max_tiles(P), P.splits, P.count);
  gemm_lds_kernel<T, LA, LB, OutT, C, ALT><<<grid, C::NT, 0, s>>>(P);
}

template <typename T, int LA, int LB, typename OutT>
static hipError_t run(GemmParams& P, hipStream_t s) {
  if (max_tiles(P) == 0) return hipSuccess;
  if (!gemm_operands_ok(P, sizeof(T) == 2, LA, LB)) return hipErrorInvalidValue;
  double flops = 0.0, bytes = 0.0;
  algo_counts(P, sizeof(T), sizeof(OutT), flops, bytes);
  const bool alt = alt_order<T>(P);
  if (alt) set_tile(P, kTile64);
  KTimer t = timing_begin(lds_kernel_name<T, LA, LB, OutT>(), flops, bytes, s);
  if constexpr (sizeof(T) == 2) {
    if (alt) run_tile<T, LA, LB, OutT, kTile64, true>(P, s);
  }
  if (!alt) {
    if (P.tile == kTile128) run_tile<T, LA, LB, OutT, kTile128, false>(P, s);
    else if (P.tile == kTile64) run_tile<T, LA, LB, OutT, kTile64, false>(P, s);
    else if (P.tile == kTile32) run_tile<T, LA, LB, OutT, kTile32, false>(P, s);
    else if constexpr (sizeof(T) == 4) run_tile<T, LA, LB, OutT, kTile64x32, false>(P, s);
  }
  timing_end(t);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || P.splits <= 1 || P.defer_reduce) return e;
  int64_t mn = 0;
  for (int g = 0; g < P.count; ++g) {
    int64_t v = (int64_t)P.d[g].M * P.d[g].N;
    mn = v > mn ? v : mn;
  }
  int64_t blocks = (mn + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  KTimer tr = timing_begin("splitk_reduce_kernel", 0.0, (double)(P.splits + 1) * 4.0 * mn * P.count, s);
  splitk_reduce_kernel<<<dim3((unsigned)blocks, P.count), 256, 0, s>>>(P);
  timing_end(tr);
  return hipGetLastError();
}

// The layouts in use: KC x MC (forward products, G . psi), KC x KC (input
// gradients, logits), MC x MC (weight gradients, G^T . phi).
template <typename T, typename OutT>
static hipError_t run_layout(GemmParams& P, int la, int lb, hipStream_t s) {
  if (la == LAY_KC && lb == LAY_KC) return run<T, LAY_KC, LAY_KC, OutT>(P, s);
  if (la == LAY_KC && lb == LAY_MC) return run<T, LAY_KC, LAY_MC, OutT>(P, s);
  if constexpr (sizeof(OutT) == 4)
    if (la == LAY_MC && lb == LAY_MC) return run<T, LAY_MC, LAY_MC, float>(P, s);
  return hipErrorInvalidValue;
}

bool gemm_pair_ok(const GemmParams& Pw, const GemmParams& Px, bool bf16) {
  // a BF16 input gradient keeps its own k order where K is ragged
  for (int g = 0; g < Px.count; ++g)
    if (bf16 && Px.d[g].K % lds::bk<bf16_t>()) return false;
  return (Pw.splits == 1 || Pw.defer_reduce) && Px.splits == 1 && max_tiles(Pw) > 0 &&
         max_tiles(Px) > 0;
}

// Tile of a pair of launches, and the grid that holds both.
static PairGrid plan_pair(GemmParams& P1, GemmParams& P2, bool bf16, bool alt) {
  int64_t n[4];
  for (int t = 0; t < 4; ++t) n[t] = tiles_of(P1, t) * P1.splits + tiles_of(P2, t) * P2.splits;
  const int tile = alt ? kTile64 : pick_tile(n, bf16);
  set_tile(P1, tile);
  set_tile(P2, tile);
  PairGrid G;
  G.gx1 = max_tiles(P1);
  G.gy1 = P1.splits;
  G.n1 = G.gx1 * G.gy1 * P1.count;
  G.gx2 = max_tiles(P2);
  G.gy2 = P2.splits;
  G.n2 = G.gx2 * G.gy2 * P2.count;
  return G;
}

template <typename T, int TILE, int LA2, int LB2, bool ALT1>
static void run_pair_tile(const GemmParams& P1, const GemmParams& P2, const PairGrid& G,
                          hipStream_t s) {
  typedef typename lds::TileOf<T, TILE>::type C;
  gemm_lds_pair_kernel<T, LAY_MC, LAY_MC, float, LA2, LB2, T, C, ALT1>
      <<<G.n1 + G.n2, C::NT, 0, s>>>(P1, P2, G);
}
template <typename T, int LA2, int LB2>
static void run_pair(GemmParams& P1, GemmParams& P2, hipStream_t s) {
  const bool alt = alt_order<T>(P1);
  const PairGrid G = plan_pair(P1, P2, sizeof(T) == 2, alt);
  if constexpr (sizeof(T) == 2) {
    if (alt) {
      run_pair_tile<T, kTile64, LA2, LB2, true>(P1, P2, G, s);
      return;
    }
  }
  if (P1.tile == kTile128) run_pair_tile<T, kTile128, LA2, LB2, false>(P1, P2, G, s);
  else if (P1.tile == kTile64) run_pair_tile<T, kTile64, LA2, LB2, false>(P1, P2, G, s);
  else if (P1.tile == kTile32) run_pair_tile<T, kTile32, LA2, LB2, false>(P1, P2, G, s);
  else if constexpr (sizeof(T) == 4) run_pair_tile<T, kTile64x32, LA2, LB2, false>(P1, P2, G, s);
}

hipError_t launch_gemm_dw_dx(GemmParams& Pw, GemmParams& Px, bool bf16, hipStream_t s) {
  if (!gemm_pair_ok(Pw, Px, bf16) || !gemm_operands_ok(Pw, bf16, LAY_MC, LAY_MC) ||
      !gemm_operands_ok(Px, bf16, LAY_KC, LAY_KC))
    return hipErrorInvalidValue;
  double flops = 0.0, bytes = 0.0;
  const double es = bf16 ? 2.0 : 4.0;
  algo_counts(Pw, es, 4.0, flops, bytes);
  algo_counts(Px, es, es, flops, bytes);
  KTimer t = timing_begin(bf16 ? "gemm_lds_pair_kernel<dW,dX>" : "gemm_lds_pair_kernel<f32,dW,dX>",
                          flops, bytes, s);
  if (bf16) run_pair<bf16_t, LAY_KC, LAY_KC>(Pw, Px, s);
  else run_pair<float, LAY_KC, LAY_KC>(Pw, Px, s);
  timing_end(t);
  return hipGetLastError();
}

hipError_t launch_gemm_obj(GemmParams& Pc, GemmParams& Pr, hipStream_t s) {
  if (!gemm_operands_ok(Pc, false, LAY_MC, LAY_MC) || !gemm_operands_ok(Pr, false, LAY_KC, LAY_MC))
    return hipErrorInvalidValue;
  if ((Pc.splits > 1 && !Pc.defer_reduce) || (Pr.splits > 1 && !Pr.defer_reduce))
    return hipErrorInvalidValue;
  double flops = 0.0, bytes = 0.0;
  algo_counts(Pc, 4.0, 4.0, flops, bytes);
  algo_counts(Pr, 4.0, 4.0, flops, bytes);
  KTimer t = timing_begin("gemm_lds_pair_kernel<f32,dpsi,dphi>", flops, bytes, s);
  run_pair<float, LAY_KC, LAY_MC>(Pc, Pr, s);
  timing_end(t);
  return hipGetLastError();
}

void plan_split_k(GemmParams& P, bool bf16, int target_wgs, int min_steps) {
  const int BK = bf16 ? lds::bk<bf16_t>() : lds::bk<float>();
  int kmax = 0;
  for (int g = 0; g < P.count; ++g) kmax = P.d[g].K > kmax ? P.d[g].K : kmax;
  // BF16 splits are counted in 128 tiles whatever tile runs (the split decides
  // how a sum that is later rounded to BF16 is formed).  An FP32 step of K is
  // half as deep and four times as slow in MFMAs, so its tiles are chosen
  // first; a reduction launch of its own (4.7 us) pays from 32 steps per split
  // on (a 32-tile work item takes 0.33 us a step).
  int64_t tiles = tiles_of(P, kTile128);
  if (!bf16) {
    tiles = tiles_of(P, pick_tile(P, 1, false));
    if (min_steps < 8) min_steps = 32;
  }
  int splits = 1;
  if (tiles > 0 && P.partial != nullptr) {
    int max_splits = kmax / (min_steps * BK);
    while (splits * 2 <= max_splits && tiles * splits * 2 <= target_wgs) splits *= 2;
  }
  int kc = (kmax + splits - 1) / splits;
  kc = (kc + BK - 1) / BK * BK;
  if (kc == 0) kc = BK;
  P.splits = splits;
  P.k_chunk = kc;
  set_tile(P, pick_tile(P, splits, bf16));
}

hipError_t launch_gemm(GemmParams& P, bool bf16, int la, int lb, bool out_bf16, hipStream_t s) {
  if (bf16) {
    if (out_bf16) return run_layout<bf16_t, bf16_t>(P, la, lb, s);
    return run_layout<bf16_t, float>(P, la, lb, s);
  }
  if (out_bf16) return hipErrorInvalidValue;
  return run_layout<float, float>(P, la, lb, s);
}

}  // namespace crl

// MFMA GEMM whose operand tiles go from global memory straight into LDS
// (global_load_lds_dwordx4: no staging registers), for BF16 and FP32 storage.
//
// A stage is 128 bytes of K of every tile row (64 BF16 or 32 FP32 values);
// ST stages ring through LDS, so ST - 1 of them are in flight while one is
// multiplied (BF16: software-pipelined by half a stage of fragments as well).
// Tiles that are contiguous along K (KC) are read with ds_read_b128 through an
// XOR swizzle of their 16-byte chunks; tiles contiguous along M or N (MC) are
// read with the 16-bit transpose read ds_read_b64_tr_b16 (BF16), which turns
// four rows of 4 x 16-bit chunks into the per-lane K runs the MFMA wants, or
// as single floats (FP32).
//   BF16: v_mfma_f32_16x16x32_bf16, FP32 accumulation.
//   FP32: v_mfma_f32_16x16x4_f32.
// Every result is the same chain of MFMAs in K order whatever the tile, so all
// tiles give the same bits.
//
// The loads are issued with explicit counted waits (load_to_lds): with the
// compiler's own waits the prefetch overlapped nothing.  One 2 x (4096 x 1024
// x 1024) BF16 forward launch went from 25.0 to 21.7 us, one 2 x (1024 x 1024 x
// 4096, two splits) dW launch from 36.7 to 24.7 us (794 and 695 TFLOP/s; a
// 64-deep step of a resident pair of workgroups takes 0.93 us, 86% of the
// 1.25-1.35 PFLOP/s that large library products reach on this card; 7 us of a
// launch are its fixed cost).
#pragma once
#include "gemm.hpp"

namespace crl {
namespace lds {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4s lds_v4s;

template <typename T> constexpr int bk() { return gemm_bk(sizeof(T) == 2); }  // K per stage
template <typename T> constexpr int vec() { return 16 / (int)sizeof(T); }   // values per chunk

// BM x BN tile, WM x WN waves, ST stages, OCC waves per SIMD to compile for
template <int BM_, int BN_, int WM_, int WN_, int ST_, int OCC_> struct Tile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, ST = ST_, OCC = OCC_;
  static constexpr int NW = WM * WN, NT = 64 * NW;
  static constexpr int MI = BM / WM / 16, NJ = BN / WN / 16;  // 16 x 16 blocks per wave
  static constexpr int STAGE = (BM + BN) * 128;
  static constexpr int EPI = 4 * BM * (BN + 4);  // FP32 epilogue tile, shares the stages' space
  static constexpr int SMEM = ST * STAGE > EPI ? ST * STAGE : EPI;
};
// The tiles of each storage type.  Two 128-tile workgroups fit a CU (64 KB of
// stages each); a third stage would leave one, which measured slower (26.5
// against 20.7 us for the 2 x 4096 x 1024 x 1024 input gradient), as did
// 256 x 128 tiles with eight waves (22.1 us) and sixteen (20.5; no gain).
template <typename T, int TILE> struct TileOf;
template <> struct TileOf<bf16_t, kTile128> { typedef Tile<128, 128, 2, 4, 2, 4> type; };
template <> struct TileOf<bf16_t, kTile64> { typedef Tile<64, 64, 2, 2, 3, 2> type; };
template <> struct TileOf<bf16_t, kTile32> { typedef Tile<32, 32, 2, 2, 4, 2> type; };
template <> struct TileOf<float, kTile128> { typedef Tile<128, 128, 2, 2, 2, 2> type; };
template <> struct TileOf<float, kTile64> { typedef Tile<64, 64, 2, 2, 2, 2> type; };
template <> struct TileOf<float, kTile64x32> { typedef Tile<64, 32, 2, 2, 3, 2> type; };
template <> struct TileOf<float, kTile32> { typedef Tile<32, 32, 2, 2, 4, 2> type; };

// KC tile: row r holds 128 bytes of K (8 chunks of 16 B); logical chunk c sits
// in slot c ^ kc_swz(r).  A ds_read_b128 pass of 16 rows then touches 16
// distinct (bank window, slot) pairs.
__device__ __forceinline__ int kc_swz(int r) { return (r >> 1) & 7; }

// MC tile of W columns: k-row kr holds W values; chunk c sits in slot
// c ^ mc_swz(kr).  BF16: a half-wave of transpose reads covers 8 k-rows x 2
// adjacent chunks, FP32: a wave reads 16 columns (4 chunks) of 4 k-rows that
// are 8 apart; the swizzle gives those 16 chunks distinct banks (FP32, W = 32:
// two rows meet, a row being half the banks).
template <typename T, int W> __device__ __forceinline__ int mc_swz(int kr) {
  if (sizeof(T) == 4) return W >= 64 ? 4 * ((kr >> 3) & 3) : 4 * ((kr >> 3) & 1);
  if (W >= 128) return 2 * ((kr & 3) + 4 * ((kr >> 3) & 1));
  if (W == 64) return 2 * (((kr >> 1) & 1) + 2 * ((kr >> 3) & 1));
  return 2 * ((kr >> 3) & 1);
}

// One operand's stages.  One wave instruction fills one 1 KB block of the
// tile; the NW waves take blocks wave, wave + NW, ...  W = extent of the tile
// along M or N; R = extent of the operand along it; kv = K values (KC) or
// k-rows (MC) of the operand that exist.  A KC row past R re-reads row R-1, an
// MC chunk past the row stride the last chunk, a KC chunk or MC k-row past kv
// the last one: all in bounds.  Rows and columns past the edge only feed
// outputs that are not stored; K past the end is zeroed in LDS (zero_tail) or
// meets zeros of the other operand (GemmDesc::kb).
template <typename T, int LAY, int W, int NW> struct Operand {
  static constexpr int NB = W / 8 / NW;
  static constexpr int LPR = W * (int)sizeof(T) / 16;  // lanes (chunks) per MC k-row
  static_assert(NB >= 1 && W % (8 * NW) == 0, "whole blocks per wave");
  const char* base;   // the next stage's first byte
  int64_t step;       // bytes from one stage to the next
  uint32_t off[NB];   // this lane's offsets inside a whole stage
  int ld, r0, R, kv;

  // offset of this lane's chunk of block i in a stage with `lim` K values left
  __device__ __forceinline__ uint32_t offset(int i, int lim, int wave, int lane) const {
    constexpr int es = (int)sizeof(T);
    const int blk = wave + NW * i;
    if (LAY == LAY_KC) {  // 8 rows of 128 B per block
      const int r = blk * 8 + (lane >> 3);
      const int c = min((lane & 7) ^ kc_swz(r), (lim - 1) / vec<T>());
      return (uint32_t)((min(r0 + r, R - 1) - r0) * ld * es + 16 * c);
    }
    const int kr = blk * (64 / LPR) + lane / LPR;
    const int c = (lane % LPR) ^ mc_swz<T, W>(kr);
    return (uint32_t)(min(kr, lim - 1) * ld * es + min(r0 + vec<T>() * c, ld - vec<T>()) * es);
  }
  __device__ __forceinline__ void init(const void* X, int ld_, int r0_, int R_, int kv_, int kbeg,
                                       int wave, int lane) {
    ld = ld_; r0 = r0_; R = R_; kv = kv_;
    const char* x = reinterpret_cast<const char*>(X);
    if (LAY == LAY_KC) {
      base = x + ((int64_t)r0 * ld + kbeg) * (int)sizeof(T);
      step = 128;
    } else {
      base = x + (int64_t)kbeg * ld * (int)sizeof(T);
      step = (int64_t)bk<T>() * ld * (int)sizeof(T);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) off[i] = offset(i, bk<T>(), wave, lane);
  }
  // the stage that starts at k0 (stages come in order), into LDS address dst
  __device__ __forceinline__ void issue(int k0, uint32_t dst, int wave, int lane) {
    if (k0 + bk<T>() <= kv) {
#pragma unroll
      for (int i = 0; i < NB; ++i) load_to_lds(base, off[i], dst + (wave + NW * i) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        load_to_lds(base, offset(i, kv - k0, wave, lane), dst + (wave + NW * i) * 1024);
    }
    base += step;
  }
};

// Zeroes K values valid..bk-1 of a stage's tile (1 <= valid < bk).
template <typename T, int LAY, int W, int NT>
__device__ __forceinline__ void zero_tail(char* tile, int valid, int tid) {
  if (LAY == LAY_KC) {
    const int n = bk<T>() - valid;
    for (int idx = tid; idx < W * n; idx += NT) {
      const int row = idx / n, k = valid + idx % n;
      reinterpret_cast<T*>(tile + row * 128 + (((k / vec<T>()) ^ kc_swz(row)) << 4))[k % vec<T>()] =
          T(0);
    }
  } else {
    for (int o = valid * W * (int)sizeof(T) + tid * 16; o < W * 128; o += NT * 16)
      *reinterpret_cast<u32x4*>(tile + o) = u32x4{0, 0, 0, 0};
  }
}

// Half a stage's fragments of one 16-row (or 16-column) block at mb; lane
// (g, j) = (lane / 16, lane % 16).  BF16: 8 consecutive k of row j, starting
// at 8 c with c = 4 hh + g, or (ALT) 2 g + hh.  ALT is the order of launches
// whose K is not a whole number of stages; it is kept because BF16 outputs of
// such launches round differently in another order (and weights that such a
// weight gradient has moved).
template <int LAY, int W, bool ALT>
__device__ __forceinline__ bf16x8 fragment(const char* tile, int mb, int hh, int g, int j,
                                           bf16_t*) {
  const int c = ALT ? 2 * g + hh : 4 * hh + g;
  if (LAY == LAY_KC) {
    const int row = mb + j;
    return *reinterpret_cast<const bf16x8*>(tile + row * 128 + ((c ^ kc_swz(row)) << 4));
  }
  // In a 16-lane group, lane j addresses k-row 8 c + 4 t + j/4 at columns
  // 4 (j%4)..+3; the transpose read hands lane j the column-j values of those
  // four rows.
  v4s h[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int kr = 8 * c + 4 * t + (j >> 2);
    const int m = mb + 4 * (j & 3);
    const int off = kr * (2 * W) + (((m >> 3) ^ mc_swz<bf16_t, W>(kr)) << 4) + (m & 7) * 2;
    h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(tile + off));
  }
  v8s r = {h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]};
  return __builtin_bit_cast(bf16x8, r);
}
// FP32: k = 8 g + 4 hh + 0..3 of row j, one MFMA each.
template <int LAY, int W, bool ALT>
__device__ __forceinline__ floatx4 fragment(const char* tile, int mb, int hh, int g, int j,
                                            float*) {
  if (LAY == LAY_KC) {
    const int row = mb + j;
    return *reinterpret_cast<const floatx4*>(tile + row * 128 +
                                             (((2 * g + hh) ^ kc_swz(row)) << 4));
  }
  floatx4 r;
  const int m = mb + j;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int kr = 8 * g + 4 * hh + i;
    r[i] = *reinterpret_cast<const float*>(tile + kr * (4 * W) +
                                           (((m >> 2) ^ mc_swz<float, W>(kr)) << 4) + (m & 3) * 4);
  }
  return r;
}
template <typename T> struct Frag { typedef bf16x8 type; };
template <> struct Frag<float> { typedef floatx4 type; };

template <typename T, int LA, int LB, typename C, bool ALT>
__device__ __forceinline__ void load_half(typename Frag<T>::type (&a)[C::MI],
                                          typename Frag<T>::type (&b)[C::NJ], const char* st,
                                          int hh, int wm, int wn, int lane) {
  const int g = lane >> 4, j = lane & 15;
#pragma unroll
  for (int i = 0; i < C::NJ; ++i)
    b[i] = fragment<LB, C::BN, ALT>(st + C::BM * 128, (wn * C::NJ + i) * 16, hh, g, j, (T*)nullptr);
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
    a[i] = fragment<LA, C::BM, ALT>(st, (wm * C::MI + i) * 16, hh, g, j, (T*)nullptr);
}
template <typename C>
__device__ __forceinline__ void mma_half(floatx4 (&acc)[C::MI][C::NJ], const bf16x8 (&a)[C::MI],
                                         const bf16x8 (&b)[C::NJ]) {
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
#pragma unroll
    for (int j = 0; j < C::NJ; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
}
template <typename C>
__device__ __forceinline__ void mma_half(floatx4 (&acc)[C::MI][C::NJ], const floatx4 (&a)[C::MI],
                                         const floatx4 (&b)[C::NJ]) {
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int j = 0; j < C::NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][q], b[j][q], acc[i][j], 0, 0, 0);
}
__device__ __forceinline__ float sum4(floatx4 x) { return (x[0] + x[1]) + (x[2] + x[3]); }
__device__ __forceinline__ float square_sum(floatx4 x) {
  return __builtin_fmaf(x[1], x[1], x[0] * x[0]) + __builtin_fmaf(x[3], x[3], x[2] * x[2]);
}
}  // namespace lds

// Wait states between MFMAs and the first vector instruction that reads their
// results, where a branch may lie between.  (The compiler inserts them, but
// counts back along one path into a block: behind a skipped branch it left 5
// or 6 of the 10 that a 16x16x4 FP32 MFMA needs, and 3 gave wrong sums.)
template <typename A> __device__ __forceinline__ void settle(A& acc) {
  floatx4* v = reinterpret_cast<floatx4*>(&acc);
  asm volatile("s_nop 15" : "+v"(v[0]));
#pragma unroll
  for (int i = 1; i < (int)(sizeof(A) / sizeof(floatx4)); ++i) asm volatile("" : "+v"(v[i]));
}

// One workgroup's work item wi of launch P; smem holds C::SMEM bytes.
template <typename T, int LA, int LB, typename OutT, typename C, bool ALT>
__device__ __forceinline__ void gemm_lds_tile(const GemmParams& P, const WorkItem wi, char* smem) {
  using namespace lds;
  constexpr int BK = bk<T>(), MI = C::MI, NJ = C::NJ;
  const int gi = wi.prob;
  const GemmDesc& D = P.d[gi];
  const int pid = wi.tile;
  if (pid >= P.tiles[gi]) return;
  const int tm = pid / P.tiles_n[gi], tn = pid % P.tiles_n[gi];
  const int m0 = tm * C::BM, n0 = tn * C::BN;
  const int K = D.K, kbeg = wi.split * P.k_chunk;
  const int nk = (min(K, kbeg + P.k_chunk) - kbeg + BK - 1) / BK;  // <= 0: empty split
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  const uint32_t lds0 = lds_address(smem);
  floatx4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // FP32 MC x MC launches may ask for an operand's sums over K (wave-uniform):
  // each lane's quarter of K, four values at a time added in 64 bits.  (Products
  // with ones, four MFMAs a fragment, were chains of 128 rounded sums: at
  // B = 1024, D = 64 the L2 energy's dpsi was 4.0e-7 off what its own matrix
  // gives, against 3.2e-7 with a column-sum kernel and 2.8e-7 now.)
  constexpr bool SUMS = sizeof(T) == 4 && LA == LAY_MC && LB == LAY_MC;
  const bool want_a = SUMS && D.asum != nullptr && tn == 0 && wn == 0;
  const bool want_b = SUMS && D.bsum != nullptr && tm == 0 && wm == 0;
  double ka[MI], kb[NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i) ka[i] = 0.0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) kb[j] = 0.0;
  // distance energies (FP32 KC x KC): the rows' squared norms, four squares at
  // a time added in 64 bits: a lane has a quarter of K, and a running FP32 sum
  // that long errs by more than a tree over 64 lanes (RMS in 2^-24 at K = 64
  // 0.81 against 0.69, at K = 256 1.16 against 0.70; this way 0.47 and 0.45)
  constexpr bool DIST = LA == LAY_KC && LB == LAY_KC && sizeof(T) == 4;
  const bool dist = DIST && (D.epi == EPI_L2 || D.epi == EPI_L2SQ);
  double na[MI], nb[NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i) na[i] = 0.0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) nb[j] = 0.0;

  if (nk > 0) {
    typedef Operand<T, LA, C::BM, C::NW> OpA;
    typedef Operand<T, LB, C::BN, C::NW> OpB;
    constexpr int LPS = OpA::NB + OpB::NB;  // loads of one wave per stage
    OpA oa;
    OpB ob;
    oa.init(D.A, D.lda, m0, D.M, K, kbeg, wave, lane);
    ob.init(D.B, D.ldb, n0, D.N, D.kb > 0 ? D.kb : K, kbeg, wave, lane);
    int head = 0, tail = 0;  // ring slots: the next to fill, the one in use
    auto issue = [&](int t) {
      const uint32_t st = lds0 + head * C::STAGE;
      bases_ready(oa.base, ob.base);
      oa.issue(kbeg + t * BK, st, wave, lane);
      ob.issue(kbeg + t * BK, st + C::BM * 128, wave, lane);
      head = head + 1 == C::ST ? 0 : head + 1;
    };
    // Stage kt complete for the whole workgroup, with `later` <= ST - 1 of
    // the following stages issued already: this wave's part has arrived once
    // at most their loads are outstanding, the barrier covers the others'.
    // It also means that every wave has its fragments of stage kt - 1 in
    // registers (its LDS reads are done), so that stage's slot is free.
    auto arrive = [&](int kt, int later) {
      if (later >= 3 && C::ST >= 4) wait_vm<(C::ST >= 4 ? 3 : 0) * LPS>();
      else if (later >= 2 && C::ST >= 3) wait_vm<(C::ST >= 3 ? 2 : 0) * LPS>();
      else if (later >= 1) wait_vm<LPS>();
      else wait_vm<0>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    // the last stage's K values past the end
    auto finish = [&](int kt, char* st) {
      const int valid = K - (kbeg + kt * BK);
      if (valid < BK) {
        zero_tail<T, LA, C::BM, C::NT>(st, valid, tid);
        zero_tail<T, LB, C::BN, C::NT>(st + C::BM * 128, valid, tid);
        __syncthreads();
      }
    };
    // FP32: the running sums are added into `sum` every 128 of K, so that a
    // long K rounds like the short chains of a split one
    floatx4 sum[MI][NJ];
    // the operands' own sums over K, in the first tile row (B) or column (A) of
    // the launch
    auto sum_k = [&](const typename Frag<T>::type (&a)[MI], const typename Frag<T>::type (&b)[NJ]) {
      if constexpr (SUMS) {
        if (want_a)
#pragma unroll
          for (int i = 0; i < MI; ++i) ka[i] += (double)sum4(a[i]);
        if (want_b)
#pragma unroll
          for (int j = 0; j < NJ; ++j) kb[j] += (double)sum4(b[j]);
      }
    };
    // squared norms of the operands' rows, from the fragments as they pass
    auto norms = [&](const typename Frag<T>::type (&a)[MI], const typename Frag<T>::type (&b)[NJ]) {
      if constexpr (DIST) {
        if (dist) {
#pragma unroll
          for (int i = 0; i < MI; ++i) na[i] += (double)square_sum(a[i]);
#pragma unroll
          for (int j = 0; j < NJ; ++j) nb[j] += (double)square_sum(b[j]);
        }
      }
    };
    auto flush = [&]() {
      settle(acc);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          sum[i][j] += acc[i][j];
          acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
    };
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) sum[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    auto multiply = [&](const typename Frag<T>::type (&a)[MI],
                        const typename Frag<T>::type (&b)[NJ]) {
      mma_half<C>(acc, a, b);
      sum_k(a, b);
      norms(a, b);
    };
    typename Frag<T>::type a0[MI], b0[NJ], a1[MI], b1[NJ];
    if constexpr (sizeof(T) == 4) {
      // FP32: the MFMAs of a half (32 cycles each) outlast its LDS reads, and
      // holding the next half's fragments measured 7 to 15% slower
#pragma unroll
      for (int s = 0; s < C::ST - 1; ++s)
        if (s < nk) issue(s);
      for (int kt = 0; kt < nk; ++kt) {
        arrive(kt, min(nk - 1 - kt, C::ST - 2));
        if (kt + C::ST - 1 < nk) issue(kt + C::ST - 1);
        char* st = smem + tail * C::STAGE;
        tail = tail + 1 == C::ST ? 0 : tail + 1;
        finish(kt, st);
        load_half<T, LA, LB, C, ALT>(a0, b0, st, 0, wm, wn, lane);
        multiply(a0, b0);
        load_half<T, LA, LB, C, ALT>(a1, b1, st, 1, wm, wn, lane);
        multiply(a1, b1);
        if ((kt & 3) == 3) flush();
      }
    } else {
      // BF16: one half's fragments are read while the other half multiplies
#pragma unroll
      for (int s = 0; s < C::ST; ++s)
        if (s < nk) issue(s);
      arrive(0, min(nk, (int)C::ST) - 1);
      finish(0, smem);
      load_half<T, LA, LB, C, ALT>(a0, b0, smem, 0, wm, wn, lane);
      for (int kt = 0; kt < nk; ++kt) {
        load_half<T, LA, LB, C, ALT>(a1, b1, smem + tail * C::STAGE, 1, wm, wn, lane);
        __builtin_amdgcn_sched_barrier(0);
        multiply(a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        if (kt + 1 < nk) {
          tail = tail + 1 == C::ST ? 0 : tail + 1;
          // issued by now: stages up to kt + ST - 1
          arrive(kt + 1, min(nk - 2 - kt, C::ST - 2));
          if (kt + C::ST < nk) issue(kt + C::ST);
          char* st = smem + tail * C::STAGE;
          finish(kt + 1, st);
          load_half<T, LA, LB, C, ALT>(a0, b0, st, 0, wm, wn, lane);
        }
        __builtin_amdgcn_sched_barrier(0);
        multiply(a1, b1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (sizeof(T) == 4) {
      flush();
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = sum[i][j];
    }
  }
  if constexpr (SUMS) {
    // the four quarters of K; then lane (g, j) has row / column j's sum
    if (want_a) {
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        ka[i] += __shfl_xor(ka[i], 16, 64);
        ka[i] += __shfl_xor(ka[i], 32, 64);
        const int row = m0 + (wm * MI + i) * 16 + lane;
        if (lane < 16 && row < D.M) D.asum[(int64_t)wi.split * D.M + row] = (float)ka[i];
      }
    }
    if (want_b) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        kb[j] += __shfl_xor(kb[j], 16, 64);
        kb[j] += __shfl_xor(kb[j], 32, 64);
        const int col = n0 + (wn * NJ + j) * 16 + lane;
        if (lane < 16 && col < D.N) D.bsum[(int64_t)wi.split * D.N + col] = (float)kb[j];
      }
    }
  }
  const bool split = P.splits > 1;
  if (split && P.defer_reduce && P.frag) {
    // deferred split-K partial in fragment order of 128 x frag blocks: the
    // 16 x 16 block (rb, cb) is fragment (rb % 4, cb % 2) of the 64 x 32 wave
    // block it lies in, 256 floats, one 1 KB store per wave
    const int bn = P.frag, nwc = bn / 32, cpb = bn / 16;
    const int tn_l = (D.N + bn - 1) / bn, nblk = (D.M + 127) / 128 * tn_l;
    float* out = P.partial + (int64_t)gi * P.partial_len + (int64_t)wi.split * nblk * 128 * bn;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int rb = m0 / 16 + wm * MI + i, cb = n0 / 16 + wn * NJ + j;
        const int blk = (rb >> 3) * tn_l + cb / cpb;
        const int w = ((rb & 7) >> 2) * nwc + (cb % cpb >> 1);
        if (rb * 16 < D.M && cb * 16 < D.N)
          *reinterpret_cast<floatx4*>(
              out + (((int64_t)blk * 2 * nwc + w) * 8 + (rb & 3) * 2 + (cb & 1)) * 256 + lane * 4) =
              acc[i][j];
      }
    return;
  }
  __syncthreads();

  // Epilogue: row/column-only operations in registers, then the FP32 tile is
  // staged in LDS so that global memory sees 16-byte row stores.
  const int r16 = lane & 15, gq = lane >> 4;
  constexpr int kLdc = C::BN + 4;
  float* Cs = reinterpret_cast<float*>(smem);
  const int epi = split ? EPI_NONE : D.epi;
  const bool has_bias = epi == EPI_BIAS || epi == EPI_BIAS_RELU;
  if constexpr (DIST) {
    if (dist) {  // each lane's quarter of K; then lane (g, j) has row / column j's norm
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        na[i] += __shfl_xor(na[i], 16, 64);
        na[i] += __shfl_xor(na[i], 32, 64);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        nb[j] += __shfl_xor(nb[j], 16, 64);
        nb[j] += __shfl_xor(nb[j], 32, 64);
      }
    }
  }
  const float alpha = split ? 1.f : D.alpha;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int cl = (wn * NJ + j) * 16 + r16;
    const int col = min(n0 + cl, D.N - 1);  // past-the-edge values are not stored
    const float bcol = has_bias ? D.bias[col] : 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rl = (wm * MI + i) * 16 + gq * 4 + r;
        float v = acc[i][j][r] * alpha + bcol;
        if (epi == EPI_BIAS_RELU) v = fmaxf(v, 0.f);
        if constexpr (DIST) {
          if (dist) {
            const float rv = __shfl((float)na[i], gq * 4 + r, 64), cv = (float)nb[j];
            v = epi == EPI_L2 ? -l2_dist(rv, cv, v) : -l2sq_dist(rv, cv, v);
          }
        }
        Cs[rl * kLdc + cl] = v;
      }
  }
  __syncthreads();
  // BN/8 threads per row, 8 values each; with N a multiple of 8 a chunk is
  // either wholly inside or wholly past the edge
  constexpr int TPR = C::BN / 8, RSTEP = C::NT / TPR;
  const int ch = tid % TPR;
  const int col0 = n0 + ch * 8;
  const int rows = min(C::BM, D.M - m0);
  if (col0 >= D.N) return;
  const int nc = min(8, D.N - col0);
  const bool ragged = (D.N & 7) != 0;  // unrolled element stores: no private-memory array
  if (split) {
    float* out = P.partial + (int64_t)gi * P.partial_len + (int64_t)wi.split * D.M * D.N;
    for (int rl = tid / TPR; rl < rows; rl += RSTEP) {
      const float* src = Cs + rl * kLdc + ch * 8;
      float* dst = out + (int64_t)(m0 + rl) * D.N + col0;
      if (ragged) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (k < nc) dst[k] = src[k];
        continue;
      }
      *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(src);
      *reinterpret_cast<float4*>(dst + 4) = *reinterpret_cast<const float4*>(src + 4);
    }
    return;
  }
  OutT* __restrict__ Cg = reinterpret_cast<OutT*>(D.C);
  const OutT* __restrict__ aux = reinterpret_cast<const OutT*>(D.aux);
  for (int rl = tid / TPR; rl < rows; rl += RSTEP) {
    const float* src = Cs + rl * kLdc + ch * 8;
    const int64_t o = (int64_t)(m0 + rl) * D.ldc + col0;
    float v[8];
    *reinterpret_cast<float4*>(v) = *reinterpret_cast<const float4*>(src);
    *reinterpret_cast<float4*>(v + 4) = *reinterpret_cast<const float4*>(src + 4);
    if (epi == EPI_MASK_POS) {  // only with N a multiple of 8 (hidden widths)
      float a8[8];
      load8_any(aux + o, a8);
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = a8[k] > 0.f ? v[k] : 0.f;
    }
    if (ragged) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k < nc) Cg[o + k] = Store<OutT>::from_f(v[k]);
      continue;
    }
    store8_any(Cg + o, v);
  }
}

template <typename T, int LA, int LB, typename OutT, typename C, bool ALT>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::OCC)))
void gemm_lds_kernel(GemmParams P) {
  __shared__ __attribute__((aligned(1024))) char smem[C::SMEM];
  gemm_lds_tile<T, LA, LB, OutT, C, ALT>(P, gemm_work_item(), smem);
}

// Two independent launches in one grid: ids [0, n1) take launch P1 (grid g1 =
// tiles x splits x problems), the rest launch P2.  One launch instead of two
// saves a launch's fixed cost (first stage, epilogue, ramp) and lets the
// second launch's tiles fill the first one's tail.
struct PairGrid { int n1, gx1, gy1, gx2, gy2, n2; };
// ALT1: the first launch in the other k order (see fragment).
template <typename T, int LA1, int LB1, typename Out1, int LA2, int LB2, typename Out2, typename C,
          bool ALT1>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::OCC)))
void gemm_lds_pair_kernel(GemmParams P1, GemmParams P2, PairGrid G) {
  __shared__ __attribute__((aligned(1024))) char smem[C::SMEM];
  const int id = blockIdx.x;
  if (id < G.n1)
    gemm_lds_tile<T, LA1, LB1, Out1, C, ALT1>(P1, work_item_of(id, G.gx1, G.gy1, G.n1), smem);
  else
    gemm_lds_tile<T, LA2, LB2, Out2, C, false>(P2, work_item_of(id - G.n1, G.gx2, G.gy2, G.n2),
                                               smem);
}

}  // namespace crl

// Relabel/gather, LayerNorm+Swish, column reductions, materialised InfoNCE,
// Adam and small utility kernels (gfx950, wave64).
#include "internal.hpp"
#include "relabel.hpp"

namespace crl {

// S samples per wavefront: draw (e, t, k), then copy the rows.
template <typename T, int S>
__global__ __launch_bounds__(256) void relabel_kernel(
    const float* __restrict__ obs, const float* __restrict__ act, int E, int T_,
    int d_s, int d_a, int d_g, int goal_lo, uint64_t seed, const int64_t* __restrict__ step,
    const uint64_t* __restrict__ thr, int B, int32_t* __restrict__ idx,
    T* __restrict__ x_sa, int ld_sa, T* __restrict__ x_g, int ld_g,
    T* __restrict__ x_sg, int ld_sg) {
  const int lane = threadIdx.x & 63;
  const int b0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * S;
  if (b0 >= B) return;
  const int n = min(S, B - b0);
  const GeomProbe probe = geom_prefetch(thr, T_ - 2, lane);
  uint64_t x[4] = {(uint64_t)(b0 + min(lane, S - 1)), (uint64_t)(*step), 0ull, 0ull};
  philox4x64_10(x, seed, 0ull);
  const int el = (int)__umul64hi(x[0], (uint64_t)E);
  const int tl = (int)__umul64hi(x[1], (uint64_t)(T_ - 1));
  uint64_t w2[S];
  int km1[S];  // k - 1
#pragma unroll
  for (int s = 0; s < S; ++s) w2[s] = lane_value(x[2], s);
  geom_counts<S>(thr, probe, w2, lane, km1);
  const float *s_row[S], *a_row[S], *g_row[S];
  int gl = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int t = lane_value(tl, s);
    const int tg = min(t + 1 + km1[s], T_ - 1);
    const int64_t ep = (int64_t)lane_value(el, s) * T_;
    s_row[s] = obs + (ep + t) * d_s;
    a_row[s] = act + (ep + t) * d_a;
    g_row[s] = obs + (ep + tg) * d_s + goal_lo;
    gl = lane == s ? tg : gl;
  }
  if (lane < n) {
    idx[3 * (b0 + lane) + 0] = el;
    idx[3 * (b0 + lane) + 1] = tl;
    idx[3 * (b0 + lane) + 2] = gl;
  }
  write_inputs<T, S>(s_row, a_row, g_row, d_s, d_a, d_g, b0, n, lane, x_sa, ld_sa, x_g,
                     ld_g, x_sg, ld_sg);
}

hipError_t launch_relabel(const float* obs, const float* act, int E, int T, int d_s,
                          int d_a, int d_g, int goal_lo, uint64_t seed,
                          const int64_t* step, const uint64_t* thr, int B,
                          int32_t* idx, void* x_sa, int ld_sa, void* x_g, int ld_g,
                          void* x_sg, int ld_sg, bool bf16, hipStream_t s) {
  const int per = relabel_samples(B);
  dim3 grid((B + 4 * per - 1) / (4 * per)), block(256);
  const double es = bf16 ? 2.0 : 4.0;
  const double bytes = (double)B * (4.0 * (d_s + d_a + d_g + (x_sg ? d_s + d_g : 0)) +
                                    es * (ld_sa + ld_g + (x_sg ? ld_sg : 0)) + 12.0);
#define CRL_RELABEL(T_, S_)                                                              \
  CRL_TIMED("relabel_kernel", 0.0, bytes, s,                                             \
            relabel_kernel<T_, S_><<<grid, block, 0, s>>>(                               \
                obs, act, E, T, d_s, d_a, d_g, goal_lo, seed, step, thr, B, idx, (T_*)x_sa, \
                ld_sa, (T_*)x_g, ld_g, (T_*)x_sg, ld_sg))
  if (bf16) {
    if (per == 1) CRL_RELABEL(bf16_t, 1);
    else if (per == 2) CRL_RELABEL(bf16_t, 2);
    else CRL_RELABEL(bf16_t, 4);
  } else {
    if (per == 1) CRL_RELABEL(float, 1);
    else if (per == 2) CRL_RELABEL(float, 2);
    else CRL_RELABEL(float, 4);
  }
#undef CRL_RELABEL
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 8-element row chunks
// ---------------------------------------------------------------------------
__device__ inline void load8(const float* p, float (&o)[8]) {
  float4 a = *reinterpret_cast<const float4*>(p);
  float4 b = *reinterpret_cast<const float4*>(p + 4);
  o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
  o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}
__device__ inline void load8(const bf16_t* p, float (&o)[8]) {
  uint4 u = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[2 * i] = __builtin_bit_cast(float, w[i] << 16);
    o[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xffff0000u);
  }
}
__device__ inline void store8(float* p, const float (&o)[8]) {
  *reinterpret_cast<float4*>(p) = make_float4(o[0], o[1], o[2], o[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(o[4], o[5], o[6], o[7]);
}
__device__ inline void store8(bf16_t* p, const float (&o)[8]) {
  uint4 u;
  u.x = pack2bf(o[0], o[1]);
  u.y = pack2bf(o[2], o[3]);
  u.z = pack2bf(o[4], o[5]);
  u.w = pack2bf(o[6], o[7]);
  *reinterpret_cast<uint4*>(p) = u;
}

// ---------------------------------------------------------------------------
// LayerNorm (biased variance over the N features) -> affine -> Swish.
// One wavefront per row; lane owns chunks lane, lane+64, ... of 8 features.
// ---------------------------------------------------------------------------
// 16-byte raw chunk of a row (8 BF16 or 4 FP32 values; FP32 rows use two)
template <typename T> struct RawChunk;
template <> struct RawChunk<bf16_t> {
  u32x4 w;
  __device__ inline void load(const bf16_t* p) { w = *reinterpret_cast<const u32x4*>(p); }
  __device__ inline void get(float (&o)[8]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __builtin_bit_cast(float, w[i] << 16);
      o[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xffff0000u);
    }
  }
};
template <> struct RawChunk<float> {
  float4 a, b;
  __device__ inline void load(const float* p) {
    a = *reinterpret_cast<const float4*>(p);
    b = *reinterpret_cast<const float4*>(p + 4);
  }
  __device__ inline void get(float (&o)[8]) const {
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
  }
};

// FULL: N = 512 CH, every lane owns a chunk of each of the CH.  Elsewhere the
// lanes past the row's end load its last chunk and leave it unused: a load
// under a branch makes the compiler wait for every load in flight where the
// branches meet.  (Forward, two encoders of 4096 rows of 1024: 11.5 -> 10.9 us.)
template <bool FULL>
__device__ inline int ln_chunk(int ch, int nch) { return FULL ? ch : min(ch, nch - 1); }

template <typename T, int CH, bool FULL>
__global__ __launch_bounds__(256) void ln_swish_fwd_kernel(LnArgs a, int B, int N, float eps) {
  const int e = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= B) return;  // whole wavefronts: the row sums below see all 64 lanes
  const int nch = N >> 3;
  const T* z = reinterpret_cast<const T*>(a.Z[e]) + (int64_t)row * N;
  T* h = reinterpret_cast<T*>(a.H[e]) + (int64_t)row * N;
  // every load of the wave is issued before the first value is used
  RawChunk<T> zr[CH];
  float v[CH][8], gv[CH][8], bv[CH][8];
#pragma unroll
  for (int c = 0; c < CH; ++c) zr[c].load(z + ln_chunk<FULL>(lane + 64 * c, nch) * 8);
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ch = ln_chunk<FULL>(lane + 64 * c, nch);
    load8(a.g[e] + ch * 8, gv[c]);
    load8(a.b[e] + ch * 8, bv[c]);
  }
#pragma unroll
  for (int c = 0; c < CH; ++c) zr[c].get(v[c]);
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (FULL || lane + 64 * c < nch)
#pragma unroll
      for (int i = 0; i < 8; ++i) s += v[c][i];
  const float inv_n = 1.f / (float)N;  // exact for the power-of-two widths
  const float mean = wave_sum_full(s) * inv_n;
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (FULL || lane + 64 * c < nch)
#pragma unroll
      for (int i = 0; i < 8; ++i) { float d = v[c][i] - mean; q += d * d; }
  const float var = wave_sum_full(q) * inv_n;
  const float rstd = __builtin_amdgcn_rsqf(var + eps);  // hardware 1/sqrt (1 ulp)
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ch = lane + 64 * c;
    if (FULL || ch < nch) {
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float y = gv[c][i] * ((v[c][i] - mean) * rstd) + bv[c][i];
        o[i] = y * sigmoidf_(y);
      }
      store8(h + ch * 8, o);
    }
  }
  if (lane == 0) { a.mu[e][row] = mean; a.rstd[e][row] = rstd; }
}

hipError_t launch_ln_swish_fwd(const LnArgs& a, int count, int B, int N, float eps,
                               bool bf16, hipStream_t s) {
  dim3 grid((B + 3) / 4, count), block(256);
  int ch = (N / 8 + 63) / 64;
  const double lnf_bytes = (double)count * B * N * 2.0 * (bf16 ? 2 : 4);
#define LNF(T, C) CRL_TIMED("ln_swish_fwd_kernel", 0.0, lnf_bytes, s, \
                            N == 512 * C                                                \
                                ? ln_swish_fwd_kernel<T, C, true><<<grid, block, 0, s>>>(a, B, N, eps) \
                                : ln_swish_fwd_kernel<T, C, false><<<grid, block, 0, s>>>(a, B, N, eps))
  // hidden widths are at most 1024 (checked at context creation): CH <= 2
  if (bf16) { if (ch <= 1) LNF(bf16_t, 1); else LNF(bf16_t, 2); }
  else      { if (ch <= 1) LNF(float, 1);  else LNF(float, 2); }
#undef LNF
  return hipGetLastError();
}

// Backward of h = Swish(g * zhat + b), zhat = (z - mu) * rstd.  Each
// workgroup owns `rows` rows (a multiple of 4 R, taken 4 R at a time, R per
// wavefront, one row at a time):
//   dy = dh * Swish'(y), dzhat = g * dy,
//   dz = rstd * (dzhat - mean(dzhat) - zhat * mean(dzhat * zhat)),
// and it accumulates the column sums dg = sum dy*zhat, db_ln = sum dy,
// db_linear = sum dz of its rows; the four wavefronts' sums are added in LDS
// in a fixed order and written as one partial row per workgroup (PARTS = 0:
// no parameter gradients are wanted, only dz).
// Bound by HBM (3 N values a row in T) and by the latency of one round: at
// B = 4096 two workgroups a CU pass through it once, so what counts is that
// every row is requested at once and the first is worked on when it arrives.
// With the loads under branches each row waited for all of them: 17.3 -> 15.3
// us by events for two encoders of 4096 rows of 1024 in BF16 (57 MB), 43.6 ->
// 40.5 at 16384 rows.
template <typename T, int CH, int R, int PARTS, bool FULL>
__global__ __launch_bounds__(256) void ln_swish_bwd_kernel(LnArgs a, int B, int N, int rows) {
  extern __shared__ float red[];  // [4 waves][3][N]
  constexpr int kRound = 4 * R;   // rows of a round
  const int e = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // rows, row sums: scalar
  const int nch = N >> 3;
  const T* Zb = reinterpret_cast<const T*>(a.Z[e]);
  const T* dHb = reinterpret_cast<const T*>(a.dH[e]);
  T* dZb = reinterpret_cast<T*>(a.dZ[e]);
  float gv[CH][8], bv[CH][8], cg[CH][8], cb[CH][8], cz[CH][8];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ch = ln_chunk<FULL>(lane + 64 * c, nch);
#pragma unroll
    for (int i = 0; i < 8; ++i) cg[c][i] = cb[c][i] = cz[c][i] = 0.f;
    load8(a.g[e] + ch * 8, gv[c]);
    load8(a.b[e] + ch * 8, bv[c]);
  }
  const float inv_n = 1.f / (float)N;
  // rounds of 4 R rows (R per wavefront) over the workgroup's rows; the column
  // sums run on across the rounds
  const int wg_end = min(B, (blockIdx.x + 1) * rows);
  auto round = [&](int base) __attribute__((always_inline)) {
    const int r0 = base + wave * R;
    const int nr = max(0, min(R, B - r0));
    // all rows of this wavefront are requested before any is used, those past
    // the batch as its last row (unused), so that no load is under a branch
    // and the first row is worked on while the others are on their way
    RawChunk<T> zr[R][CH], hr[R][CH];
    float mu[R], rs[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      mu[j] = a.mu[e][min(r0 + j, B - 1)];
      rs[j] = a.rstd[e][min(r0 + j, B - 1)];
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int row = min(r0 + j, B - 1);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int64_t at = (int64_t)row * N + ln_chunk<FULL>(lane + 64 * c, nch) * 8;
        zr[j][c].load(Zb + at);
        hr[j][c].load(dHb + at);
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // left to itself the compiler sinks the later rows' loads
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j >= nr) break;  // uniform over the wavefront, as the row sums need
      const int row = r0 + j;
      float zh[CH][8], dzh[CH][8];
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = lane + 64 * c;
        if (FULL || ch < nch) {
          float z[8], dh[8];
          zr[j][c].get(z);
          hr[j][c].get(dh);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float xh = (z[i] - mu[j]) * rs[j];
            const float y = __builtin_fmaf(gv[c][i], xh, bv[c][i]);
            const float sg = sigmoidf_(y);
            // Swish'(y) = sg (1 + y (1 - sg)) = sg + y sg (1 - sg)
            const float q = __builtin_fmaf(-sg, sg, sg);
            const float dy = dh[i] * __builtin_fmaf(y, q, sg);
            if (PARTS) {
              cg[c][i] += dy * xh;
              cb[c][i] += dy;
            }
            const float d = dy * gv[c][i];
            zh[c][i] = xh;
            dzh[c][i] = d;
            s1 += d;
            s2 += d * xh;
          }
        }
      }
      // dz = rstd (dzhat - m1 - zhat m2) = rstd dzhat + (e zhat + k),
      // e = -rstd m2, k = -rstd m1
      const float k = -rs[j] * (wave_sum_full(s1) * inv_n);
      const float e = -rs[j] * (wave_sum_full(s2) * inv_n);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int ch = lane + 64 * c;
        if (FULL || ch < nch) {
          float o[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            o[i] = __builtin_fmaf(rs[j], dzh[c][i], __builtin_fmaf(e, zh[c][i], k));
            if (PARTS) cz[c][i] += o[i];
          }
          store8(dZb + (int64_t)row * N + ch * 8, o);
        }
      }
    }
  };
  // The first round stands before the loop: rows past the batch leave loads
  // that nothing waited for, and one loop's head would wait for them, in the
  // first round for g and b, before the rows are requested.
  int base = blockIdx.x * rows;  // the grid starts no workgroup past B
  round(base);
  for (base += kRound; base < wg_end; base += kRound) round(base);
  if (!PARTS) return;
  float* mine = red + (int64_t)wave * 3 * N;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int ch = lane + 64 * c;
    if (FULL || ch < nch) {
      store8(mine + ch * 8, cg[c]);
      store8(mine + N + ch * 8, cb[c]);
      store8(mine + 2 * N + ch * 8, cz[c]);
    }
  }
  __syncthreads();
  // N is a multiple of 8: the four wave rows and the partial row in float4s
  const float4* r4 = reinterpret_cast<const float4*>(red);
  float4* p4 = reinterpret_cast<float4*>(a.part[e] + (int64_t)blockIdx.x * 3 * N);
  const int n4 = 3 * N / 4;
  for (int k = threadIdx.x; k < n4; k += 256) {
    const float4 w0 = r4[k], w1 = r4[n4 + k], w2 = r4[2 * n4 + k], w3 = r4[3 * n4 + k];
    float4 o;
    o.x = (w0.x + w1.x) + (w2.x + w3.x);
    o.y = (w0.y + w1.y) + (w2.y + w3.y);
    o.z = (w0.z + w1.z) + (w2.z + w3.z);
    o.w = (w0.w + w1.w) + (w2.w + w3.w);
    p4[k] = o;
  }
}

// Rows of a wavefront at a time.  Up to B = 2048 one or two, so that the
// launch has four times or twice the workgroups and each its chain of rows
// shortened (one encoder at B = 1000: 63 workgroups and 7.2 us with four rows,
// 250 and 5.0 us with one); above, four: a workgroup's 256 column partials
// are then paid for by 16 rows.  The number of partial rows is at most 256
// either way.  BF16 parameter gradients always take four: in another order
// they differ in the last bit, the next step's BF16 weights then now and then
// in theirs, and that step's result at 1e-4.
int ln_bwd_r(int B, bool bf16_parts) {
  return bf16_parts ? 4 : B <= 1024 ? 1 : B <= 2048 ? 2 : 4;
}
// Rows per workgroup: one round up to B = 4096 (at most 512 workgroups for two
// encoders), then more rounds per workgroup instead of more workgroups, so the
// column partials (3 N floats per workgroup, summed again in the gradient
// reduction) stop growing with B.
int ln_bwd_rows(int B, bool bf16_parts) {
  return 4 * ln_bwd_r(B, bf16_parts) * std::max(1, (B + 4095) / 4096);
}
int ln_bwd_partials(int B, bool bf16_parts) {
  const int rows = ln_bwd_rows(B, bf16_parts);
  return (B + rows - 1) / rows;
}

template <typename T, int CH, int R>
static void ln_bwd_run(const LnArgs& a, int count, int B, int N, hipStream_t s) {
  const bool bp = sizeof(T) == 2 && a.part[0];
  const int rows = ln_bwd_rows(B, bp);
  const dim3 grid(ln_bwd_partials(B, bp), count);
  const size_t lds = (size_t)4 * 3 * N * sizeof(float);
  const bool full = N == 512 * CH;
  if (!a.part[0]) {
    if (full) ln_swish_bwd_kernel<T, CH, R, 0, true><<<grid, 256, 0, s>>>(a, B, N, rows);
    else ln_swish_bwd_kernel<T, CH, R, 0, false><<<grid, 256, 0, s>>>(a, B, N, rows);
  } else if constexpr (sizeof(T) == 4 || R == 4) {
    if (full) ln_swish_bwd_kernel<T, CH, R, 1, true><<<grid, 256, lds, s>>>(a, B, N, rows);
    else ln_swish_bwd_kernel<T, CH, R, 1, false><<<grid, 256, lds, s>>>(a, B, N, rows);
  }
}
template <typename T, int CH>
static void ln_bwd_rows_run(const LnArgs& a, int count, int B, int N, hipStream_t s) {
  const int r = ln_bwd_r(B, sizeof(T) == 2 && a.part[0]);
  if (r == 1) ln_bwd_run<T, CH, 1>(a, count, B, N, s);
  else if (r == 2) ln_bwd_run<T, CH, 2>(a, count, B, N, s);
  else ln_bwd_run<T, CH, 4>(a, count, B, N, s);
}
hipError_t launch_ln_swish_bwd(const LnArgs& a, int count, int B, int N, bool bf16,
                               hipStream_t s) {
  const int ch = (N / 8 + 63) / 64;
  const double bytes = (double)count * ((double)B * N * 3.0 * (bf16 ? 2 : 4) +
                                        (a.part[0] ? 12.0 * ln_bwd_partials(B, bf16) * N : 0.0));
  KTimer t = timing_begin("ln_swish_bwd_kernel", 0.0, bytes, s);
  // hidden widths are at most 1024 (checked at context creation): CH <= 2
  if (bf16) { if (ch <= 1) ln_bwd_rows_run<bf16_t, 1>(a, count, B, N, s); else ln_bwd_rows_run<bf16_t, 2>(a, count, B, N, s); }
  else      { if (ch <= 1) ln_bwd_rows_run<float, 1>(a, count, B, N, s);  else ln_bwd_rows_run<float, 2>(a, count, B, N, s); }
  timing_end(t);
  return hipGetLastError();
}

// 4-element chunks for the column kernels
__device__ inline void load4(const float* p, float (&o)[4]) {
  float4 a = *reinterpret_cast<const float4*>(p);
  o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
}
__device__ inline void load4(const bf16_t* p, float (&o)[4]) {
  uint2 u = *reinterpret_cast<const uint2*>(p);
  o[0] = __builtin_bit_cast(float, u.x << 16);
  o[1] = __builtin_bit_cast(float, u.x & 0xffff0000u);
  o[2] = __builtin_bit_cast(float, u.y << 16);
  o[3] = __builtin_bit_cast(float, u.y & 0xffff0000u);
}
constexpr int kColRows = 128;  // rows per chunk of the column-sum kernel

// Column sums of X [B][ld] over one chunk of rows, 256 columns per workgroup.
template <typename T>
__global__ __launch_bounds__(256) void colsum_partial_kernel(ColSumArgs a, int B, int N, int ld) {
  __shared__ float red[4][256];
  const int e = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = blockIdx.x * 256 + lane * 4;
  const int r0 = blockIdx.y * kColRows, r1 = min(B, r0 + kColRows);
  float acc[4] = {0, 0, 0, 0};
  if (n0 < N) {
    const T* X = reinterpret_cast<const T*>(a.X[e]);
    // the wavefront's rows r0 + wave, + 4, + 8, ... in that order, eight
    // rows' loads in flight before they are added
    int row = r0 + wave;
    for (; row + 28 < r1; row += 32) {
      float v[8][4];
#pragma unroll
      for (int k = 0; k < 8; ++k) load4(X + (int64_t)(row + 4 * k) * ld + n0, v[k]);
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += v[k][i];
    }
    for (; row < r1; row += 4) {
      float v[4];
      load4(X + (int64_t)row * ld + n0, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] += v[i];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) red[wave][lane * 4 + i] = acc[i];
  __syncthreads();
  const int t = threadIdx.x;
  const int n = blockIdx.x * 256 + t;
  if (n < N)
    a.part[e][(int64_t)blockIdx.y * N + n] = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
}

int colsum_chunks(int B) { return (B + kColRows - 1) / kColRows; }

hipError_t launch_colsum_partials(const ColSumArgs& a, int count, int B, int N, int ld,
                                  bool bf16, hipStream_t s) {
  // N and ld must be multiples of 4 (vector loads of 4 elements)
  const int nrb = colsum_chunks(B);
  dim3 grid((N + 255) / 256, nrb, count), block(256);
  const double cs_bytes = (double)count * B * N * (bf16 ? 2 : 4);
  if (bf16) CRL_TIMED("colsum_partial_kernel", 0.0, cs_bytes, s,
                      colsum_partial_kernel<bf16_t><<<grid, block, 0, s>>>(a, B, N, ld));
  else      CRL_TIMED("colsum_partial_kernel", 0.0, cs_bytes, s,
                      colsum_partial_kernel<float><<<grid, block, 0, s>>>(a, B, N, ld));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------
// One Adam update, written with explicit fused multiply-adds so that every
// kernel that applies it rounds the same way:
//   m = b1 m + (1-b1) g,  v = b2 v + (1-b2) g^2,
//   p -= lr (m c1) / (sqrt(v c2) + eps),  c1 = 1/(1 - b1^t), c2 = 1/(1 - b2^t).
__device__ __forceinline__ float adam_update(float& p, float g, float& m, float& v, float c1,
                                             float c2, const AdamCoef& c) {
  m = __builtin_fmaf(c.b1, m, c.omb1 * g);
  v = __builtin_fmaf(c.b2, v, (c.omb2 * g) * g);
  p = p - (c.lr * (m * c1)) / (sqrtf(v * c2) + c.eps);
  return p;
}
// bias-correction factors 1 / (1 - b^t) = -1 / expm1(t log b): full FP32
// relative accuracy (no cancellation in 1 - b^t)
__device__ __forceinline__ void adam_factors(const AdamCoef& c, const int64_t* step, float& c1,
                                             float& c2) {
  const float t = (float)(*step);
  c1 = 1.f / (-expm1f(t * c.log_b1));
  c2 = 1.f / (-expm1f(t * c.log_b2));
}
// Adam on parameter k with gradient gk
__device__ __forceinline__ void adam_at(const AdamArgs& A, float c1, float c2, int64_t k,
                                        float gk) {
  float pk = A.p[k], mk = A.m[k], vk = A.v[k];
  adam_update(pk, gk, mk, vk, c1, c2, A.c);
  A.p[k] = pk;
  A.m[k] = mk;
  A.v[k] = vk;
  if (A.pb) A.pb[k] = f2bf(pk);
}
// ... on the four parameters k4 * 4 + 0..3 (16-byte aligned)
__device__ __forceinline__ void adam_at4(const AdamArgs& A, float c1, float c2, int64_t k4,
                                         float4 gg) {
  float4 pp = reinterpret_cast<float4*>(A.p)[k4];
  float4 mm = reinterpret_cast<float4*>(A.m)[k4];
  float4 vv = reinterpret_cast<float4*>(A.v)[k4];
  adam_update(pp.x, gg.x, mm.x, vv.x, c1, c2, A.c);
  adam_update(pp.y, gg.y, mm.y, vv.y, c1, c2, A.c);
  adam_update(pp.z, gg.z, mm.z, vv.z, c1, c2, A.c);
  adam_update(pp.w, gg.w, mm.w, vv.w, c1, c2, A.c);
  reinterpret_cast<float4*>(A.p)[k4] = pp;
  reinterpret_cast<float4*>(A.m)[k4] = mm;
  reinterpret_cast<float4*>(A.v)[k4] = vv;
  if (A.pb) {
    uint2 u;
    u.x = pack2bf(pp.x, pp.y);
    u.y = pack2bf(pp.z, pp.w);
    reinterpret_cast<uint2*>(A.pb)[k4] = u;
  }
}

// last job whose `first` is <= v (jobs sorted by `first`)
__device__ inline int find_job(const RedJob* __restrict__ jobs, int njobs, int64_t v) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].first <= v) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// sum of a float4 over the job's parts, in part order (four running sums)
__device__ __forceinline__ float4 sum_parts(const float4* __restrict__ p, int64_t st,
                                            int nparts) {
  float4 s[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) s[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  int k = 0;
  for (; k + 3 < nparts; k += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 t = p[(k + q) * st];
      s[q].x += t.x; s[q].y += t.y; s[q].z += t.z; s[q].w += t.w;
    }
  }
  for (; k < nparts; ++k) {
    const float4 t = p[k * st];
    s[0].x += t.x; s[0].y += t.y; s[0].z += t.z; s[0].w += t.w;
  }
  float4 r;
  r.x = (s[0].x + s[1].x) + (s[2].x + s[3].x);
  r.y = (s[0].y + s[1].y) + (s[2].y + s[3].y);
  r.z = (s[0].z + s[1].z) + (s[2].z + s[3].z);
  r.w = (s[0].w + s[1].w) + (s[2].w + s[3].w);
  return r;
}

// last job whose first_chunk is <= v
__device__ inline int find_job_chunk(const RedJob* __restrict__ jobs, int njobs, int64_t v) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].first_chunk <= v) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Few parts with the Adam epilogue: block blk takes chunk c of one job
// (kRedChunk4 float4 outputs, 4 per thread).  Dense jobs step their float4s
// in place.  Fragment-order jobs hold each tile wave by wave (64 x 32 per
// wave, bn / 32 waves per 64-row half); a chunk is two consecutive waves, a
// 64 x 64 block of the tile, whose partials are summed into an LDS copy of
// the block and then stepped row by row, so that p, m, v move in 256-byte
// row runs.  (Half-tile chunks took half the blocks, too few to fill the
// chip when the vector is small.)
constexpr int kRedWaves = kRedChunk4 * 4 / 2048;  // waves of a tile per chunk
constexpr int kRedCols = 32 * kRedWaves;          // block columns
constexpr int kRedLdsFloats = 64 * (kRedCols + 4);
static_assert(kRedWaves == 2, "a chunk is two waves: a 64 x 64 block of a 64- or 128-wide tile");
__device__ __forceinline__ void reduce_few_adam(const char* __restrict__ ws,
                                                float* __restrict__ g,
                                                const RedJob* __restrict__ jobs, int njobs,
                                                int64_t blk, const AdamArgs& A, float c1,
                                                float c2, float* __restrict__ T) {
  const RedJob J = jobs[find_job_chunk(jobs, njobs, blk)];
  const int64_t c = blk - J.first_chunk;
  const float4* src = reinterpret_cast<const float4*>(ws + J.src);
  const int64_t st = J.stride / 4, n4 = J.n / 4;
  const int tid = threadIdx.x;
  if (J.bn == 0) {
#pragma unroll
    for (int k = 0; k < kRedChunk4 / 256; ++k) {
      const int64_t i4 = c * kRedChunk4 + k * 256 + tid;
      if (i4 < n4) {
        const float4 r = sum_parts(src + i4, st, J.nparts);
        if (g) reinterpret_cast<float4*>(g + J.dst)[i4] = r;
        adam_at4(A, c1, c2, J.dst / 4 + i4, r);
      }
    }
    return;
  }
  // the chunk: tile t, waves [w0, w0 + 2): rows [R0, R0 + 64), columns
  // [C0, C0 + 64) of the tile
  const int bn = J.bn, wpr = bn / 32, ld = kRedCols + 4;
  const int64_t tsz4 = 32 * (int64_t)bn;  // float4s per tile
  const int t = (int)((c * kRedChunk4) / tsz4);
  const int w0 = (int)(((c * kRedChunk4) % tsz4) / kRedChunk4) * kRedWaves;
  const int R0 = (w0 / wpr) * 64, C0 = (w0 % wpr) * 32;
#pragma unroll
  for (int k = 0; k < kRedChunk4 / 256; ++k) {
    const int64_t i4 = c * kRedChunk4 + k * 256 + tid;
    const float4 r = sum_parts(src + i4, st, J.nparts);
    // float4 i4 = lane's 4 accumulator rows of fragment f of wave w of tile t
    const int rem = (int)(i4 * 4 - (int64_t)t * tsz4 * 4);
    const int w = rem >> 11, f = (rem >> 8) & 7, lane = (rem >> 2) & 63;
    const int rl = (w / wpr) * 64 + (f >> 1) * 16 + (lane >> 4) * 4 - R0;
    const int cl = (w % wpr) * 32 + (f & 1) * 16 + (lane & 15) - C0;
    T[rl * ld + cl] = r.x;
    T[(rl + 1) * ld + cl] = r.y;
    T[(rl + 2) * ld + cl] = r.z;
    T[(rl + 3) * ld + cl] = r.w;
  }
  __syncthreads();
  constexpr int q4 = kRedCols / 4;  // float4s per block row
  const int row0 = (t / J.tiles_n) * 128 + R0, col0 = (t % J.tiles_n) * bn + C0;
#pragma unroll
  for (int k = 0; k < kRedChunk4 / 256; ++k) {
    const int v = k * 256 + tid;
    const int rl = v / q4, cq = v % q4;
    const int row = row0 + rl, col = col0 + 4 * cq;
    if (row < J.M && col < J.N) {  // N is a multiple of 8: whole float4s
      const float4 r = *reinterpret_cast<const float4*>(T + rl * ld + 4 * cq);
      const int64_t k0 = J.dst + (int64_t)row * J.N + col;
      if (g) *reinterpret_cast<float4*>(g + k0) = r;
      adam_at4(A, c1, c2, k0 / 4, r);
    }
  }
}

// few parts (split-K partials): one float4 of one job per thread
template <bool ADAM>
__device__ __forceinline__ void reduce_few(const char* __restrict__ ws, float* __restrict__ g,
                                           const RedJob* __restrict__ jobs, int njobs,
                                           int64_t total4, int64_t blk, const AdamArgs& A,
                                           float c1, float c2) {
  const int64_t v = blk * 256ll + threadIdx.x;
  if (v >= total4) return;
  const RedJob J = jobs[find_job(jobs, njobs, v)];
  const int64_t i4 = v - J.first;
  int64_t o0 = -1;  // fragment order: row-major offset of this float4's first row
  if (J.bn > 0) {
    // float4 i4 = lane's 4 accumulator rows of fragment (i, j) of wave w of
    // tile t (the direct-to-LDS kernel's 64 x 32 wave blocks)
    const int64_t e = i4 * 4;
    const int64_t tsz = (int64_t)128 * J.bn;
    const int t = (int)(e / tsz);
    const int rem = (int)(e - (int64_t)t * tsz);
    const int w = rem >> 11, f = (rem >> 8) & 7, lane = (rem >> 2) & 63;
    const int wpr = J.bn / 32;  // waves per row of wave blocks
    const int row = (t / J.tiles_n) * 128 + (w / wpr) * 64 + (f >> 1) * 16 + (lane >> 4) * 4;
    const int col = (t % J.tiles_n) * J.bn + (w % wpr) * 32 + (f & 1) * 16 + (lane & 15);
    if (row >= J.M || col >= J.N) return;
    o0 = (int64_t)row * J.N + col;
  }
  const float4* p = reinterpret_cast<const float4*>(ws + J.src) + i4;
  const int64_t st = J.stride / 4;
  float4 s[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) s[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  int k = 0;
  for (; k + 3 < J.nparts; k += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 t = p[(k + q) * st];
      s[q].x += t.x; s[q].y += t.y; s[q].z += t.z; s[q].w += t.w;
    }
  }
  for (; k < J.nparts; ++k) {
    const float4 t = p[k * st];
    s[0].x += t.x; s[0].y += t.y; s[0].z += t.z; s[0].w += t.w;
  }
  float4 r;
  r.x = (s[0].x + s[1].x) + (s[2].x + s[3].x);
  r.y = (s[0].y + s[1].y) + (s[2].y + s[3].y);
  r.z = (s[0].z + s[1].z) + (s[2].z + s[3].z);
  r.w = (s[0].w + s[1].w) + (s[2].w + s[3].w);
  if (o0 < 0) {
    if (!ADAM || g) reinterpret_cast<float4*>(g + J.dst)[i4] = r;
    if (ADAM) adam_at4(A, c1, c2, J.dst / 4 + i4, r);
  } else {  // rows past M inside the last tile are not stored
    const int64_t k = J.dst + o0;
    const int nrow = min(4, J.M - (int)(o0 / J.N));
    if (!ADAM || g) {
      float* q = g + k;
      q[0] = r.x;
      if (nrow > 1) q[J.N] = r.y;
      if (nrow > 2) q[2 * (int64_t)J.N] = r.z;
      if (nrow > 3) q[3 * (int64_t)J.N] = r.w;
    }
    if (ADAM) {
      adam_at(A, c1, c2, k, r.x);
      if (nrow > 1) adam_at(A, c1, c2, k + J.N, r.y);
      if (nrow > 2) adam_at(A, c1, c2, k + 2 * (int64_t)J.N, r.z);
      if (nrow > 3) adam_at(A, c1, c2, k + 3 * (int64_t)J.N, r.w);
    }
  }
}

// many parts (per-chunk column partials): kManyCols = 32 outputs per
// workgroup (a wavefront reads two whole 128-byte lines per load), the parts
// over 8 groups, then a fixed-order tree in LDS.  A job with no parts writes
// zeros (the padding between parameter tensors).
template <bool ADAM>
__device__ __forceinline__ void reduce_many(const char* __restrict__ ws, float* __restrict__ g,
                                            const RedJob* __restrict__ jobs, int njobs,
                                            int64_t blk, const AdamArgs& A, float c1, float c2) {
  constexpr int NG = 256 / kManyCols;  // groups
  __shared__ float red[NG][kManyCols + 1];
  const RedJob J = jobs[find_job(jobs, njobs, blk)];
  const int col = threadIdx.x % kManyCols, grp = threadIdx.x / kManyCols;
  const int64_t i = (blk - J.first) * kManyCols + col;
  // eight running sums: eight loads in flight per thread
  float sk[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) sk[q] = 0.f;
  if (i < J.n) {
    const float* p = reinterpret_cast<const float*>(ws + J.src) + i;
    int k = grp;
    for (; k + 7 * NG < J.nparts; k += 8 * NG) {
#pragma unroll
      for (int q = 0; q < 8; ++q) sk[q] += p[(k + NG * q) * J.stride];
    }
    for (; k < J.nparts; k += NG) sk[0] += p[k * J.stride];
  }
  red[grp][col] = ((sk[0] + sk[1]) + (sk[2] + sk[3])) + ((sk[4] + sk[5]) + (sk[6] + sk[7]));
  __syncthreads();
  for (int h = NG / 2; h >= 1; h >>= 1) {
    if (grp < h) red[grp][col] += red[grp + h][col];
    __syncthreads();
  }
  if (grp == 0 && i < J.n) {
    const float r = red[0][col];
    if (!ADAM || g) g[J.dst + i] = r;
    if (ADAM) adam_at(A, c1, c2, J.dst + i, r);
  }
}

// The policy step's loss (see ActorLossArgs) by one workgroup of 256 threads:
// 1024 Kahan sums over the samples (four per thread, so that the sums are those
// of 1024 threads), then an ordered tree.
__device__ void actor_loss(const ActorLossArgs& L, float* __restrict__ sh) {
  const int tid = threadIdx.x;
  for (int v = tid; v < 1024; v += 256) {
    float s0 = 0.f, c0 = 0.f, s1 = 0.f, c1 = 0.f;
    for (int i = v; i < L.B; i += 1024) {
      kahan_add(s0, c0, L.logpi[i]);
      kahan_add(s1, c1, L.f[i]);
    }
    sh[v] = s0 - c0;
    sh[1024 + v] = s1 - c1;
  }
  __syncthreads();
  for (int w = 512; w >= 1; w >>= 1) {
    for (int v = tid; v < w; v += 256) {
      sh[v] += sh[v + w];
      sh[1024 + v] += sh[1024 + v + w];
    }
    __syncthreads();
  }
  if (tid == 0) {
    const float la = *L.log_alpha;
    const float mlp = sh[0] / (float)L.B, mf = sh[1024] / (float)L.B;
    L.loss_out[0] = expf(la) * mlp - mf;
    L.loss_out[1] = mlp;
    L.loss_out[2] = -la * (mlp + L.target_entropy);
    L.loss_out[3] = mf;
    *L.alpha_grad = -(mlp + L.target_entropy);
  }
}

// Both reductions in one launch: blocks [0, nbf) take the few-part jobs,
// the rest the many-part jobs, and one more block the policy's loss where
// L.loss_out is set (a launch of its own took 4.8 us).  ADAM: each reduced
// element goes into the Adam step of its parameter (the jobs then cover the
// whole vector).
template <bool ADAM>
__global__ __launch_bounds__(256) void grad_reduce_kernel(const char* __restrict__ ws,
                                                          float* __restrict__ g,
                                                          const RedJob* __restrict__ few,
                                                          int nfew, int64_t total4,
                                                          const RedJob* __restrict__ many,
                                                          int nmany, int64_t nbf, AdamArgs A,
                                                          ActorLossArgs L) {
  constexpr int kLds = ADAM ? kRedLdsFloats : 2048;
  __shared__ __attribute__((aligned(16))) float T[kLds];
  static_assert(kLds >= 2048, "the policy loss takes 2048 floats");
  if (L.loss_out && blockIdx.x == gridDim.x - 1) {
    actor_loss(L, T);
    return;
  }
  if constexpr (ADAM) {
    float c1, c2;
    adam_factors(A.c, A.step, c1, c2);
    if (blockIdx.x < nbf) reduce_few_adam(ws, g, few, nfew, blockIdx.x, A, c1, c2, T);
    else reduce_many<true>(ws, g, many, nmany, blockIdx.x - nbf, A, c1, c2);
  } else {
    if (blockIdx.x < nbf) reduce_few<false>(ws, g, few, nfew, total4, blockIdx.x, A, 0.f, 0.f);
    else reduce_many<false>(ws, g, many, nmany, blockIdx.x - nbf, A, 0.f, 0.f);
  }
}

hipError_t launch_grad_reduce(const char* ws, float* g, const RedJob* few, int nfew,
                              int64_t total4, const RedJob* many, int nmany, int64_t nblocks,
                              double bytes, hipStream_t s, const AdamArgs* A,
                              const ActorLossArgs* L) {
  // with Adam, total4 counts chunks of kRedChunk4 float4s
  const int64_t nbf = nfew > 0 ? (A ? total4 : (total4 + 255) / 256) : 0;
  const int64_t nbm = nmany > 0 ? nblocks : 0;
  if (nbf + nbm == 0) return L ? hipErrorInvalidValue : hipSuccess;
  const dim3 grid((unsigned)(nbf + nbm + (L ? 1 : 0)));
  const ActorLossArgs la = L ? *L : ActorLossArgs{};
  if (A)
    CRL_TIMED("grad_reduce_adam_kernel", 0.0, bytes, s,
              grad_reduce_kernel<true><<<grid, 256, 0, s>>>(ws, g, few, nfew, total4, many,
                                                            nmany, nbf, *A, la));
  else
    CRL_TIMED("grad_reduce_kernel", 0.0, bytes, s,
              grad_reduce_kernel<false><<<grid, 256, 0, s>>>(ws, g, few, nfew, total4, many,
                                                             nmany, nbf, AdamArgs{}, la));
  return hipGetLastError();
}

__global__ void cast_bf16_kernel(const float* __restrict__ src, bf16_t* __restrict__ dst, int64_t n) {
  int64_t i = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) * 4;
  for (; i < n; i += (int64_t)gridDim.x * blockDim.x * 4) {
    if (i + 4 <= n) {
      float4 v = *reinterpret_cast<const float4*>(src + i);
      uint2 u;
      u.x = pack2bf(v.x, v.y);
      u.y = pack2bf(v.z, v.w);
      *reinterpret_cast<uint2*>(dst + i) = u;
    } else {
      for (int64_t j = i; j < n; ++j) dst[j] = f2bf(src[j]);
    }
  }
}
hipError_t launch_cast_bf16(const float* src, bf16_t* dst, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 1023) / 1024;
  if (blocks > 8192) blocks = 8192;
  CRL_TIMED("cast_bf16_kernel", 0.0, 6.0 * n, s,
            cast_bf16_kernel<<<(int)blocks, 256, 0, s>>>(src, dst, n));
  return hipGetLastError();
}

// Adam on a flat vector (adam_update on every element).
__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v,
                                                   bf16_t* __restrict__ pb, int64_t n,
                                                   const int64_t* __restrict__ step, AdamCoef c) {
  float c1, c2;
  adam_factors(c, step, c1, c2);
  const AdamArgs A{p, m, v, pb, step, c};
  const int64_t n4 = n >> 2;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n4;
       i += (int64_t)gridDim.x * blockDim.x)
    adam_at4(A, c1, c2, i, reinterpret_cast<const float4*>(g)[i]);
  if (blockIdx.x == 0 && threadIdx.x < (n & 3)) {
    const int64_t k = n4 * 4 + threadIdx.x;
    adam_at(A, c1, c2, k, g[k]);
  }
}
hipError_t launch_adam(float* p, const float* g, float* m, float* v, bf16_t* pb, int64_t n,
                       const int64_t* step, const AdamCoef& c, hipStream_t s) {
  int64_t blocks = (n / 4 + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 16384) blocks = 16384;
  CRL_TIMED("adam_kernel", 0.0, (28.0 + (pb ? 2.0 : 0.0)) * n, s,
            adam_kernel<<<(int)blocks, 256, 0, s>>>(p, g, m, v, pb, n, step, c));
  return hipGetLastError();
}

__global__ void counter_add_kernel(int64_t* c, int64_t inc) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *c += inc;
}
hipError_t launch_counter_add(int64_t* c, int64_t inc, hipStream_t s) {
  counter_add_kernel<<<1, 64, 0, s>>>(c, inc);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// log-sum-exp merge and loss
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void lse_merge_kernel(LseMergeArgs a, int B) {
  // problem blockIdx.y; 64 columns per workgroup (a wavefront reads 256
  // contiguous bytes of one part), the parts split over the 16 wavefronts
  // (p = grp, grp + 16, ...), then a fixed-order tree over them in LDS
  __shared__ float sm[16][65], ss[16][65];
  const int e = blockIdx.y;
  const float* __restrict__ pm = a.pm[e];
  const float* __restrict__ ps = a.ps[e];
  const int nparts = a.nparts[e];
  const int col = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + col;
  float m = -INFINITY, s = 0.f;
  if (j < B)
    for (int p = grp; p < nparts; p += 16)
      lse_merge(m, s, pm[(int64_t)p * B + j], ps[(int64_t)p * B + j]);
  sm[grp][col] = m;
  ss[grp][col] = s;
  __syncthreads();
  for (int h = 8; h >= 1; h >>= 1) {
    if (grp < h) {
      float mm = sm[grp][col], s2 = ss[grp][col];
      lse_merge(mm, s2, sm[grp + h][col], ss[grp + h][col]);
      sm[grp][col] = mm;
      ss[grp][col] = s2;
    }
    __syncthreads();
  }
  if (grp == 0 && j < B) a.out[e][j] = sm[0][col] + __logf(ss[0][col]);
}
hipError_t launch_lse_merge(const LseMergeArgs& a, int count, int B, hipStream_t s) {
  double parts = 0.0;
  for (int e = 0; e < count; ++e) parts += a.nparts[e];
  CRL_TIMED("lse_merge_kernel", 0.0, 4.0 * B * (2.0 * parts + count), s,
            lse_merge_kernel<<<dim3((B + 63) / 64, count), 1024, 0, s>>>(a, B));
  return hipGetLastError();
}
// Loss from r, c, diag (and the per-row objective terms of the pairwise
// objectives) in one workgroup: per-thread Kahan sums, then an ordered
// pairwise tree over the threads (deterministic).
//   loss_out = {L_obj + L_pen, mean(r - diag), mean(c - diag), L_pen,
//               mean r, mean c, #non-finite rows, L_obj}
// with L_obj the objective `loss` (CRL_LOSS_*): the two InfoNCE directions,
// their sum, FlatNCE (exp(x - x) per row, x = r - diag or c - diag), or the
// mean of term[] (Forward-Backward, DPO, IPO, SPPO).
// With nparts > 0 each thread first merges its columns' (max, sum) partials in
// part order into c: one launch less where the columns are few (at B = 2000 the
// merge takes 24 us of this one workgroup).  The order is serial, so the sum is
// compensated (without, c was up to 1.1 times as far off as lse_merge_kernel's
// tree leaves it).
// Latency is all it costs: four rows' loads go out together, and the last six
// levels of the tree run inside a wavefront (B=16384 9.8 -> 8.4 us, B=4096 4.6
// -> 4.2).  Joined to lse_merge_kernel (its last workgroup takes the loss) it
// cost as much as the two launches from B=1500 on: 8.9 us at B=4096, 23 at
// B=16384, mostly the workgroups' counting.
__global__ __launch_bounds__(1024) void loss_kernel(const float* __restrict__ r,
                                                    float* __restrict__ c,
                                                    const float* __restrict__ diag,
                                                    const float* __restrict__ term, int B,
                                                    int loss, float beta,
                                                    float* __restrict__ loss_out,
                                                    int64_t* __restrict__ advance,
                                                    const float* __restrict__ col_m,
                                                    const float* __restrict__ col_s, int nparts) {
  __shared__ float sh[7][1024];
  constexpr int NR = 4;  // rows in flight per thread
  const int tid = threadIdx.x;
  float acc[6] = {0, 0, 0, 0, 0, 0}, cmp[6] = {0, 0, 0, 0, 0, 0};
  float bad = 0.f;
  const bool pairwise = loss >= CRL_LOSS_FB;
  for (int i0 = tid; i0 < B; i0 += NR * 1024) {
    float rv[NR], cv[NR], dv[NR], tv[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int i = min(i0 + k * 1024, B - 1);
      rv[k] = r[i];
      dv[k] = diag[i];
      cv[k] = nparts > 0 ? 0.f : c[i];
      tv[k] = pairwise ? term[i] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int i = i0 + k * 1024;
      if (i >= B) break;
      const float ri = rv[k], di = dv[k];
      float ci = cv[k];
      if (nparts > 0) {
        float m = -INFINITY, sum = 0.f, low = 0.f;
#pragma unroll 4
        for (int p = 0; p < nparts; ++p)
          lse_merge_kahan(m, sum, low, col_m[(int64_t)p * B + i], col_s[(int64_t)p * B + i]);
        ci = m + __logf(sum - low);
        c[i] = ci;
      }
      float o = tv[k];
      if (loss == CRL_LOSS_FLATNCE_FWD) { const float x = ri - di; o = __expf(x - x); }
      else if (loss == CRL_LOSS_FLATNCE_BWD) { const float x = ci - di; o = __expf(x - x); }
      const float t[6] = {ri - di, ci - di, ri * ri, ri, ci, o};
#pragma unroll
      for (int q = 0; q < 6; ++q) kahan_add(acc[q], cmp[q], t[q]);
      if (!isfinite(ri) || !isfinite(ci) || !isfinite(di) || !isfinite(o)) bad += 1.f;
    }
  }
  float v[7];
#pragma unroll
  for (int q = 0; q < 6; ++q) v[q] = acc[q] - cmp[q];
  v[6] = bad;
#pragma unroll
  for (int q = 0; q < 7; ++q) sh[q][tid] = v[q];
  __syncthreads();
  for (int w = 512; w >= 64; w >>= 1) {
    if (tid < w)
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        v[q] += sh[q][tid + w];
        sh[q][tid] = v[q];
      }
    __syncthreads();
  }
  if (tid >= 64) return;
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1)
#pragma unroll
    for (int q = 0; q < 7; ++q) v[q] += __shfl_down(v[q], w, 64);
  if (tid == 0) {
    const float inv = 1.f / (float)B;
    const float lf = v[0] * inv, lb = v[1] * inv, lp = beta * v[2] * inv;
    float obj;
    if (loss == CRL_LOSS_FWD) obj = lf;
    else if (loss == CRL_LOSS_SYM) obj = lf + lb;
    else if (loss == CRL_LOSS_BWD) obj = lb;
    else obj = v[5] * inv;
    loss_out[0] = obj + lp;
    loss_out[1] = lf;
    loss_out[2] = lb;
    loss_out[3] = lp;
    loss_out[4] = v[3] * inv;
    loss_out[5] = v[4] * inv;
    loss_out[6] = v[6];
    loss_out[7] = obj;
    if (advance) *advance += 1;
  }
}
hipError_t launch_loss(const float* r, float* c, const float* diag, const float* term,
                       int B, int loss, float beta, float* loss_out, int64_t* advance,
                       hipStream_t s, const float* col_m, const float* col_s, int nparts) {
  CRL_TIMED("loss_kernel", 0.0, 16.0 * B + 8.0 * B * nparts, s,
            loss_kernel<<<1, 1024, 0, s>>>(r, c, diag, term, B, loss, beta, loss_out, advance,
                                           col_m, col_s, nparts));
  return hipGetLastError();
}

}  // namespace crl

// The replay buffer as a ring of steps per environment: the insert of a
// chunk of time-major steps and the sampler that relabels goals inside the
// trajectory of the drawn step (gfx950, wave64).
#include "internal.hpp"
#include "relabel.hpp"

namespace crl {

// n consecutive elements (pieces of V) of rows of d elements, from src to the
// rows dst[k] of a buffer: element q belongs to row q / d < kInsRows.  UN loads
// of a lane are in flight before the first store.
constexpr int kInsRows = 4;
template <int UN, typename V>
__device__ __forceinline__ void scatter_rows(V* __restrict__ buf, const V* __restrict__ src,
                                             const int64_t (&dst)[kInsRows], int d, int n,
                                             int lane) {
  for (int q0 = lane; q0 < n; q0 += 64 * UN) {
    V v[UN];
#pragma unroll
    for (int i = 0; i < UN; ++i)
      v[i] = q0 + 64 * i < n ? src[q0 + 64 * i] : V{};
#pragma unroll
    for (int i = 0; i < UN; ++i) {
      const int q = q0 + 64 * i;
      int64_t to = dst[0] * d + q;
#pragma unroll
      for (int k = 1; k < kInsRows; ++k) to = q >= k * d ? (dst[k] - k) * d + q : to;
      if (q < n) buf[to] = v[i];
    }
  }
}

// n mod C, in 32 bits where they hold n (the 64-bit remainder takes longer than
// the rest of a row's arithmetic)
__device__ __forceinline__ int ring_first(int64_t n, int C) {
  return n >> 31 ? (int)(n % C) : (int)((uint32_t)n % (uint32_t)C);
}

// kInsRows consecutive (step u, env e) rows of the chunk per wavefront: a row's
// obs and act words go to ring row (count + u) mod C of env e, its trajectory
// id beside them.  The chunk is read in order (rows of one step are
// contiguous), the ring is written in whole rows; with V4 (d_s a multiple of
// 4, both obs buffers 16-byte aligned) the obs rows move in 16-byte pieces.
// Bound by HBM once enough loads are in flight: a wavefront that took one row
// at a time, each piece's store before the next load, took 36 us for 62 x 1024
// rows of 268 + 17 floats out of HBM; four rows take 29 (146 MB: 5 TB/s).
template <bool V4>
__global__ __launch_bounds__(256) void replay_insert_kernel(
    float* __restrict__ obs, float* __restrict__ act, int32_t* __restrict__ traj, int E, int C,
    int d_s, int d_a, const float* __restrict__ nobs, const float* __restrict__ nact,
    const int32_t* __restrict__ ntraj, int U, const int64_t* __restrict__ count) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = (blockIdx.x * 4 + wave) * kInsRows;  // u * E + e
  const int nr = min(kInsRows, U * E - r0);
  if (nr <= 0) return;
  const int id = lane < nr ? ntraj[r0 + lane] : 0;
  const int first = ring_first(*count, C);
  int64_t dst[kInsRows];
  int u = r0 / E, e = r0 - u * E;
#pragma unroll
  for (int k = 0; k < kInsRows; ++k) {
    int row = first + u;  // u < C, so one wrap at most
    if (row >= C) row -= C;
    dst[k] = (int64_t)e * C + row;
    if (++e == E) {
      e = 0;
      ++u;
    }
  }
  if (V4)
    scatter_rows<5>(reinterpret_cast<floatx4*>(obs),
                    reinterpret_cast<const floatx4*>(nobs + (int64_t)r0 * d_s), dst, d_s >> 2,
                    nr * (d_s >> 2), lane);
  else
    scatter_rows<5>(obs, nobs + (int64_t)r0 * d_s, dst, d_s, nr * d_s, lane);
  scatter_rows<2>(act, nact + (int64_t)r0 * d_a, dst, d_a, nr * d_a, lane);
  if (lane < nr) {
    int64_t row = dst[0];
#pragma unroll
    for (int k = 1; k < kInsRows; ++k) row = lane == k ? dst[k] : row;
    traj[row] = id;
  }
}

// S samples per wavefront.  size = min(count, C) steps are stored, logical
// index i (0 = oldest) at ring row (count - size + i) mod C.  Draw e, i and
// the offset k, then clip i + k to the last step of i's trajectory: the
// lanes compare 64 ids at a time against i's, and the first differing one
// ends the run.  k averages 1 / (1 - gamma), so this is one or two probes of
// 256 contiguous bytes for most samples; the first of each goes out with its
// own id.
template <typename T, int S>
__global__ __launch_bounds__(256) void ring_relabel_kernel(
    const float* __restrict__ obs, const float* __restrict__ act,
    const int32_t* __restrict__ traj, int E, int C, const int64_t* __restrict__ count,
    int d_s, int d_a, int d_g, int goal_lo, uint64_t seed, const int64_t* __restrict__ step,
    const uint64_t* __restrict__ thr, int n_thr, int B, int32_t* __restrict__ idx,
    T* __restrict__ x_sa, int ld_sa, T* __restrict__ x_g, int ld_g,
    T* __restrict__ x_sg, int ld_sg) {
  const int lane = threadIdx.x & 63;
  const int b0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * S;
  if (b0 >= B) return;
  const int n = min(S, B - b0);
  const int64_t cnt = *count;
  const int size = (int)(cnt < (int64_t)C ? cnt : (int64_t)C);
  if (size < 2) {  // nothing to draw: (-1, -1, -1) and zero rows
    if (lane < 3 * n) idx[3 * b0 + lane] = -1;
    const int64_t b = b0;
    for (int c = lane; c < n * ld_sa; c += 64) x_sa[b * ld_sa + c] = T(0);
    for (int c = lane; c < n * ld_g; c += 64) x_g[b * ld_g + c] = T(0);
    if (x_sg)
      for (int c = lane; c < n * ld_sg; c += 64) x_sg[b * ld_sg + c] = T(0);
    return;
  }
  const GeomProbe probe = geom_prefetch(thr, n_thr, lane);
  const int base = ring_first(cnt - size, C);  // ring row of logical index 0
  uint64_t x[4] = {(uint64_t)(b0 + min(lane, S - 1)), (uint64_t)(*step), 0ull, 0ull};
  philox4x64_10(x, seed, 0ull);
  const int el = (int)__umul64hi(x[0], (uint64_t)E);
  const int il = (int)__umul64hi(x[1], (uint64_t)(size - 1));
  auto ring_row = [&](int j) { int q = base + j; return q >= C ? q - C : q; };
  uint64_t w2[S];
  int km1[S];  // k - 1
#pragma unroll
  for (int s = 0; s < S; ++s) w2[s] = lane_value(x[2], s);
  geom_counts<S>(thr, probe, w2, lane, km1);
  const float *s_row[S], *a_row[S], *g_row[S];
  int32_t tid[S], ids[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int i = lane_value(il, s), lim = min(i + 1 + km1[s], size - 1);
    const int32_t* __restrict__ tr = traj + (int64_t)lane_value(el, s) * C;
    tid[s] = tr[ring_row(i)];
    ids[s] = tr[ring_row(min(i + 1 + lane, lim))];
  }
  int rl = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int e = lane_value(el, s), i = lane_value(il, s);
    const int32_t* __restrict__ tr = traj + (int64_t)e * C;
    const int lim = min(i + 1 + km1[s], size - 1);
    int tg = lim;
    int32_t id = ids[s];
    for (int j0 = i + 1;;) {
      const uint64_t m = __ballot(j0 + lane <= lim && id != tid[s]);
      if (m) {
        tg = j0 + (int)__builtin_ctzll(m) - 1;
        break;
      }
      j0 += 64;
      if (j0 > lim) break;
      id = tr[ring_row(min(j0 + lane, lim))];
    }
    const int ri = ring_row(i), rg = ring_row(tg);
    rl = lane == 2 * s ? ri : lane == 2 * s + 1 ? rg : rl;
    s_row[s] = obs + ((int64_t)e * C + ri) * d_s;
    a_row[s] = act + ((int64_t)e * C + ri) * d_a;
    g_row[s] = obs + ((int64_t)e * C + rg) * d_s + goal_lo;
  }
  const int ri = __shfl(rl, 2 * (lane & (S - 1)), 64), rg = __shfl(rl, 2 * (lane & (S - 1)) + 1, 64);
  if (lane < n) {
    idx[3 * (b0 + lane) + 0] = el;
    idx[3 * (b0 + lane) + 1] = ri;
    idx[3 * (b0 + lane) + 2] = rg;
  }
  write_inputs<T, S>(s_row, a_row, g_row, d_s, d_a, d_g, b0, n, lane, x_sa, ld_sa, x_g,
                     ld_g, x_sg, ld_sg);
}

hipError_t launch_replay_insert(float* obs, float* act, int32_t* traj, int E, int C, int d_s,
                                int d_a, const float* nobs, const float* nact,
                                const int32_t* ntraj, int U, int64_t* count, hipStream_t s) {
  const int64_t rows = (int64_t)U * E;
  dim3 grid((unsigned)((rows + 4 * kInsRows - 1) / (4 * kInsRows))), block(256);
  const double bytes = 2.0 * (double)rows * (4.0 * (d_s + d_a) + 4.0);
  const bool v4 = (d_s & 3) == 0 && ((reinterpret_cast<uintptr_t>(obs) |
                                       reinterpret_cast<uintptr_t>(nobs)) & 15u) == 0;
  if (v4)
    CRL_TIMED("replay_insert_kernel", 0.0, bytes, s,
      replay_insert_kernel<true><<<grid, block, 0, s>>>(obs, act, traj, E, C, d_s, d_a, nobs,
                                                        nact, ntraj, U, count));
  else
    CRL_TIMED("replay_insert_kernel", 0.0, bytes, s,
      replay_insert_kernel<false><<<grid, block, 0, s>>>(obs, act, traj, E, C, d_s, d_a, nobs,
                                                         nact, ntraj, U, count));
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  return launch_counter_add(count, U, s);
}

hipError_t launch_ring_relabel(const float* obs, const float* act, const int32_t* traj, int E,
                               int C, const int64_t* count, int d_s, int d_a, int d_g,
                               int goal_lo, uint64_t seed, const int64_t* step,
                               const uint64_t* thr, int n_thr, int B, int32_t* idx, void* x_sa,
                               int ld_sa, void* x_g, int ld_g, void* x_sg, int ld_sg, bool bf16,
                               hipStream_t s) {
  const int per = relabel_samples(B);
  dim3 grid((B + 4 * per - 1) / (4 * per)), block(256);
  const double es = bf16 ? 2.0 : 4.0;
  const double bytes = (double)B * (4.0 * (d_s + d_a + d_g + (x_sg ? d_s + d_g : 0)) +
                                    es * (ld_sa + ld_g + (x_sg ? ld_sg : 0)) + 12.0);
#define CRL_RING_RELABEL(T_, S_)                                                          \
  CRL_TIMED("ring_relabel_kernel", 0.0, bytes, s,                                         \
            ring_relabel_kernel<T_, S_><<<grid, block, 0, s>>>(                           \
                obs, act, traj, E, C, count, d_s, d_a, d_g, goal_lo, seed, step, thr, n_thr, B, \
                idx, (T_*)x_sa, ld_sa, (T_*)x_g, ld_g, (T_*)x_sg, ld_sg))
  if (bf16) {
    if (per == 1) CRL_RING_RELABEL(bf16_t, 1);
    else if (per == 2) CRL_RING_RELABEL(bf16_t, 2);
    else CRL_RING_RELABEL(bf16_t, 4);
  } else {
    if (per == 1) CRL_RING_RELABEL(float, 1);
    else if (per == 2) CRL_RING_RELABEL(float, 2);
    else CRL_RING_RELABEL(float, 4);
  }
#undef CRL_RING_RELABEL
  return hipGetLastError();
}

}  // namespace crl

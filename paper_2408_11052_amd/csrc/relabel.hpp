// The geometric goal offset shared by the episode-row and ring samplers.
#pragma once

#include "common.hpp"

namespace crl {

// Samples of a wavefront of the samplers.  A sample's Philox block is some 600
// vector instructions whether one lane or 64 compute it (lane s computes sample
// s's), which is most of the time of a full chip; a small launch is three
// dependent loads (threshold, own row's ids, rows) and is shortest with a
// wavefront a sample.  Measured with 1, 2, 4 samples, rows of 67 + 8 floats:
// B=1024 3.2, 3.8, 4.7 us; B=2048 4.2, 3.9, 4.7; B=4096 6.2, 4.7, 4.9; B=8192
// 10.4, 6.7, 6.2; B=16384 18.7, 10.5, 8.9 (before, one sample and its loads one
// after the other: 3.8, 4.3, 5.8, 8.7, 14.4; out of the ring 5.4, 5.8, 7.7, 10.6,
// 17.8, now 4.4, 5.4, 6.6, 9.1, 12.4).
inline int relabel_samples(int B) { return B < 2048 ? 1 : B < 8192 ? 2 : 4; }

// lane s's value of v, uniform
__device__ __forceinline__ int lane_value(int v, int s) { return __builtin_amdgcn_readlane(v, s); }
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int s) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, s);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), s);
  return (uint64_t)hi << 32 | lo;
}

// First level of the threshold search, issued before Philox runs: the probes
// of the first level are the same 64 entries for every sample.
struct GeomProbe {
  int n_thr, step0, q0;
  uint64_t thr0;
};
__device__ inline GeomProbe geom_prefetch(const uint64_t* __restrict__ thr, int n_thr, int lane) {
  GeomProbe p;
  p.n_thr = n_thr;
  p.step0 = (n_thr + 63) >> 6;
  p.q0 = lane * p.step0;
  p.thr0 = (n_thr > 64 && p.q0 < n_thr) ? thr[p.q0] : 0ull;
  return p;
}

// k - 1 = #{m in [1, n_thr] : w2 < thr[m]} (thr[m] stored at index m - 1).
// The table is non-increasing, so the count is the length of its prefix that
// exceeds w2.  64-way search: the lanes probe 64 evenly spaced entries of the
// remaining range at once, and the number of probes above w2 narrows the
// prefix end to one gap between probes.  Every lane of the wave must call it
// with the same w2; every lane returns the same count.
__device__ inline int geom_count(const uint64_t* __restrict__ thr, const GeomProbe& p,
                                 uint64_t w2, int lane) {
  int lo = 0, hi = p.n_thr;  // count in [lo, hi]
  if (hi - lo > 64) {
    const bool above = p.q0 < hi && p.thr0 > w2;
    const int c = __popcll(__ballot(above));
    const int nlo = c > 0 ? (c - 1) * p.step0 + 1 : 0;
    hi = min(hi, c * p.step0);
    lo = nlo;
  }
  while (hi - lo > 64) {
    const int step = (hi - lo + 63) >> 6;
    const int q = lo + lane * step;
    const bool above = q < hi && thr[q] > w2;
    const int c = __popcll(__ballot(above));  // probes 0..c-1 are above w2
    const int nlo = c > 0 ? lo + (c - 1) * step + 1 : lo;
    const int qc = lo + c * step;             // first probe not above (or past hi)
    hi = min(hi, qc);
    lo = nlo;
  }
  const int q = lo + lane;
  const bool above = q < hi && thr[q] > w2;
  return lo + __popcll(__ballot(above));
}

// The counts of S samples, their table reads in flight together where two
// levels cover the table.
template <int S>
__device__ __forceinline__ void geom_counts(const uint64_t* __restrict__ thr, const GeomProbe& p,
                                            const uint64_t (&w2)[S], int lane, int (&out)[S]) {
  if (S == 1 || p.n_thr > 64 * 64 || p.n_thr < 1) {
#pragma unroll
    for (int s = 0; s < S; ++s) out[s] = geom_count(thr, p, w2[s], lane);
    return;
  }
  uint64_t t[S];
  int lo[S], hi[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    lo[s] = 0;
    hi[s] = p.n_thr;
    if (p.n_thr > 64) {
      const int c = __popcll(__ballot(p.q0 < p.n_thr && p.thr0 > w2[s]));
      lo[s] = c > 0 ? (c - 1) * p.step0 + 1 : 0;
      hi[s] = min(p.n_thr, c * p.step0);
    }
    t[s] = thr[min(lo[s] + lane, p.n_thr - 1)];
  }
#pragma unroll
  for (int s = 0; s < S; ++s)
    out[s] = lo[s] + __popcll(__ballot(lo[s] + lane < hi[s] && t[s] > w2[s]));
}

// The encoder inputs of samples b0 .. b0 + n - 1 (n <= S) from their rows (one
// wavefront, lane-strided): x_sa = [s, a, 0...], x_g = [g, 0...], x_sg = [s, g,
// 0...] (x_sg optional).  The copy is bound by latency: the loads of 128
// columns of all samples go out together, without branches (a column past the
// end reads the row's first word), and the state's are shared by x_sa and x_sg.
template <typename T, int S>
__device__ __forceinline__ void write_inputs(const float* const (&s_row)[S],
                                             const float* const (&a_row)[S],
                                             const float* const (&g_row)[S], int d_s, int d_a,
                                             int d_g, int64_t b0, int n, int lane,
                                             T* __restrict__ x_sa, int ld_sa, T* __restrict__ x_g,
                                             int ld_g, T* __restrict__ x_sg, int ld_sg) {
  constexpr int UN = 2;
  if (!x_sg) ld_sg = 0;
  float g0[S];
#pragma unroll
  for (int s = 0; s < S; ++s) g0[s] = g_row[s][lane < d_g ? lane : 0];
  for (int c0 = lane; c0 < max(ld_sa, ld_sg); c0 += 64 * UN) {
    float sa[S][UN], sg[S][UN];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int i = 0; i < UN; ++i) {
        const int c = c0 + 64 * i, k = c - d_s;
        const float* from = k >= 0 && k < d_a ? a_row[s] + k : s_row[s] + (k < 0 ? c : 0);
        sa[s][i] = *from;
        sg[s][i] = g_row[s][k >= 0 && k < d_g ? k : 0];
      }
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (s < n)
#pragma unroll
        for (int i = 0; i < UN; ++i) {
          const int c = c0 + 64 * i, k = c - d_s;
          if (c < ld_sa) x_sa[(b0 + s) * ld_sa + c] = Store<T>::from_f(k < d_a ? sa[s][i] : 0.f);
          if (c < ld_sg)
            x_sg[(b0 + s) * ld_sg + c] =
                Store<T>::from_f(k < 0 ? sa[s][i] : k < d_g ? sg[s][i] : 0.f);
        }
  }
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (s < n) {
      if (lane < ld_g) x_g[(b0 + s) * ld_g + lane] = Store<T>::from_f(lane < d_g ? g0[s] : 0.f);
      for (int c = lane + 64; c < ld_g; c += 64)
        x_g[(b0 + s) * ld_g + c] = Store<T>::from_f(c < d_g ? g_row[s][c] : 0.f);
    }
}

}  // namespace crl

// The internal launches whose route a dispatch rule chooses, with the route as
// an argument, for the tests that compare the routes (test_gpu_routes.py).
#include "internal.hpp"

using namespace crl;

namespace {
struct Carve {
  char* at;
  int64_t left;
  void* take(int64_t bytes) {
    bytes = (bytes + 255) & ~(int64_t)255;
    left -= bytes;
    void* p = at;
    at += bytes;
    return p;
  }
  float* floats(int64_t n) { return (float*)take(4 * n); }
};
}  // namespace

// The fused critic matrix, forward then backward.  route: BlockRoute.
extern "C" __attribute__((visibility("default"))) int routes_fused(
    int B, int D, int energy, int loss, float beta, int route, const float* phi, const float* psi,
    float* dphi, float* dpsi, char* ws, int64_t bytes, void* stream) {
  const int S = fused_splits(B) > fused_bwd_splits(B) ? fused_splits(B) : fused_bwd_splits(B);
  const int64_t nrb = (B + 63) / 64, n = (int64_t)B * D;
  Carve w{ws, bytes};
  FusedArgs a{};
  a.phi = phi; a.psi = psi;
  a.phi_b = (bf16_t*)w.take(2 * n); a.psi_b = (bf16_t*)w.take(2 * n);
  a.nphi = w.floats(B); a.npsi = w.floats(B);
  a.row_m = w.floats(S * (int64_t)B); a.row_s = w.floats(S * (int64_t)B);
  a.col_m = w.floats(nrb * B); a.col_s = w.floats(nrb * B);
  a.r = w.floats(B); a.c = w.floats(B); a.diag = w.floats(B);
  a.dX_part = w.floats(2 * S * n); a.rs_part = w.floats(2 * S * (int64_t)B);
  a.dphi = dphi; a.dpsi = dpsi;
  a.dphi_t = dphi; a.dpsi_t = dpsi;
  if (w.left < 0) return hipErrorOutOfMemory;
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = launch_fused_fwd(a, B, D, energy, nullptr, s);
  if (e != hipSuccess) return e;
  return launch_fused_bwd(a, B, D, energy, loss, beta, false, s, (BlockRoute)route);
}

// C = A . B (layouts la, lb) in tiles `tile`; partial: split K where the plan
// says so, summed by the reduction launch.
extern "C" __attribute__((visibility("default"))) int routes_gemm(
    int bf16, int la, int lb, int out_bf16, int M, int N, int K, const void* A, int lda,
    const void* Bm, int ldb, void* C, int ldc, int epi, float* asum, float* bsum, float* partial,
    int64_t partial_floats, int tile, int* splits, void* stream) {
  GemmParams P{};
  P.count = 1;
  GemmDesc& d = P.d[0];
  d.A = A; d.B = Bm; d.C = C;
  d.M = M; d.N = N; d.K = K;
  d.lda = lda; d.ldb = ldb; d.ldc = ldc;
  d.epi = epi;
  d.alpha = 1.f;
  d.asum = asum; d.bsum = bsum;
  P.partial = partial;
  plan_split_k(P, bf16, 512);
  P.partial_len = (int64_t)P.splits * M * N;
  if (P.splits > 1 && P.partial_len > partial_floats) return hipErrorOutOfMemory;
  if (tile == kTile64x32 && bf16) return hipErrorInvalidValue;
  set_tile(P, tile);
  *splits = P.splits;
  return launch_gemm(P, bf16, la, lb, out_bf16, (hipStream_t)stream);
}

// One launch of a layer's dW (MC x MC) and dX (KC x KC), both unsplit.
extern "C" __attribute__((visibility("default"))) int routes_pair(
    int bf16, int B, int I, int O, const void* x, const void* w, const void* dz, float* dw, void* dx,
    void* stream) {
  GemmParams Pw{}, Px{};
  Pw.count = Px.count = 1;
  GemmDesc& d = Pw.d[0];
  d.A = x; d.B = dz; d.C = dw;
  d.M = I; d.N = O; d.K = B;
  d.lda = I; d.ldb = O; d.ldc = O;
  d.alpha = 1.f;
  GemmDesc& q = Px.d[0];
  q.A = dz; q.B = w; q.C = dx;
  q.M = B; q.N = I; q.K = O;
  q.lda = O; q.ldb = O; q.ldc = I;
  q.alpha = 1.f;
  plan_split_k(Pw, bf16, 0);
  plan_split_k(Px, bf16, 0);
  return launch_gemm_dw_dx(Pw, Px, bf16, (hipStream_t)stream);
}

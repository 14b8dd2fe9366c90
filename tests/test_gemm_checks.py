"""Launches that the GEMM kernel's indexing does not hold for are refused on the
host (gemm_operands_ok in csrc/gemm.hpp), each taken from one that is accepted.
A host program built from the header; no GPU needed."""
import os
import shutil
import subprocess

import pytest

from paper_2408_11052_amd import build as B

SOURCE = r'''
#include <cstdio>
#include <functional>
#include "gemm.hpp"
using namespace crl;
static GemmParams good(bool bf16) {
  GemmParams P{};
  P.count = 2;
  P.splits = 2;
  P.k_chunk = 128;
  P.partial = reinterpret_cast<float*>(64);
  for (int g = 0; g < 2; ++g) {
    GemmDesc& d = P.d[g];
    d.A = d.B = reinterpret_cast<void*>(256);
    d.C = reinterpret_cast<void*>(512);
    d.M = 33; d.N = 40; d.K = 256;
    d.lda = d.ldb = 256; d.ldc = 40;
  }
  return P;
}
static void check(const char* name, bool bf16, int la, int lb, std::function<void(GemmParams&)> f) {
  GemmParams P = good(bf16);
  f(P);
  std::printf("%s %d\n", name, (int)gemm_operands_ok(P, bf16, la, lb));
}
int main() {
  const int KC = LAY_KC, MC = LAY_MC;
  check("plain_bf16", true, KC, MC, [](GemmParams&) {});
  check("plain_fp32", false, KC, KC, [](GemmParams&) {});
  check("kb_in_the_last_stage_bf16", true, KC, MC, [](GemmParams& P) { P.d[1].kb = 193; });
  check("kb_in_the_last_stage_fp32", false, KC, MC, [](GemmParams& P) { P.d[1].kb = 225; });
  check("both_sums", false, MC, MC, [](GemmParams& P) {
    P.d[0].asum = P.d[0].bsum = reinterpret_cast<float*>(64); });
  check("distance", false, KC, KC, [](GemmParams& P) {
    P.splits = 1; P.k_chunk = 256; P.d[0].epi = EPI_L2; P.d[1].epi = EPI_L2SQ; });
  check("not:kb_a_stage_short_bf16", true, KC, MC, [](GemmParams& P) { P.d[1].kb = 192; });
  check("not:kb_a_stage_short_fp32", false, KC, MC, [](GemmParams& P) { P.d[1].kb = 224; });
  check("not:negative_kb", true, KC, MC, [](GemmParams& P) { P.d[0].kb = -1; });
  check("not:chunk_no_whole_stages", true, KC, MC, [](GemmParams& P) { P.k_chunk = 160; });
  check("not:chunks_short_of_k", true, KC, MC, [](GemmParams& P) { P.k_chunk = 64; });
  check("not:splits_without_partials", true, KC, MC, [](GemmParams& P) { P.partial = nullptr; });
  check("not:no_rows", true, KC, MC, [](GemmParams& P) { P.d[1].M = 0; });
  check("not:row_stride", true, KC, MC, [](GemmParams& P) { P.d[1].lda = 260; });
  check("not:alignment", false, KC, MC, [](GemmParams& P) { P.d[1].B = reinterpret_cast<void*>(264); });
  check("not:sums_in_bf16", true, MC, MC, [](GemmParams& P) { P.d[0].bsum = reinterpret_cast<float*>(64); });
  check("not:sums_of_rows", false, KC, MC, [](GemmParams& P) { P.d[0].asum = reinterpret_cast<float*>(64); });
  check("not:distance_split", false, KC, KC, [](GemmParams& P) { P.d[0].epi = EPI_L2; });
  check("not:distance_in_bf16", true, KC, KC, [](GemmParams& P) {
    P.splits = 1; P.k_chunk = 256; P.d[0].epi = EPI_L2SQ; });
  check("not:ragged_columns_in_fragment_order", true, MC, MC, [](GemmParams& P) {
    P.d[0].N = 41; P.defer_reduce = 1; P.frag = 64; });
}
'''


def test_the_launch_checks(tmp_path):
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("no hipcc")
    (tmp_path / "main.hip").write_text(SOURCE)
    subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-host-only", str(tmp_path / "main.hip"), "-o", str(tmp_path / "main")],
                   check=True, capture_output=True)
    out = subprocess.run([str(tmp_path / "main")], check=True, capture_output=True, text=True).stdout
    lines = [l.split() for l in out.splitlines()]
    assert len(lines) == 20
    assert [n for n, ok in lines if ok != ("0" if n.startswith("not:") else "1")] == []

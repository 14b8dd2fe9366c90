"""Routes that a dispatch rule chooses between and that are to give the same bits:
the one-pass kernel and the two passes of the fused backward of 64-wide
representations, the GEMM's tiles, and its paired and single launches.
Through tests/libroutes.so, which the build links from the library's objects.
"""
import ctypes as C

import pytest
import torch

from paper_2408_11052_amd import build
from paper_2408_11052_amd._lib import ENERGY, LOSS

pytestmark = pytest.mark.gpu

KC, MC = 0, 1
TILES = {"32": 0, "64x32": 1, "64": 2, "128": 3}
EPI_NONE, EPI_L2 = 0, 4


@pytest.fixture(scope="module")
def routes():
    lib = C.CDLL(build.ROUTES)
    p, i = C.c_void_p, C.c_int
    lib.routes_fused.argtypes = [i, i, i, i, C.c_float, i, p, p, p, p, p, C.c_int64, p]
    lib.routes_gemm.argtypes = [i] * 7 + [p, i, p, i, p, i, i, p, p, p, C.c_int64, i, C.POINTER(i), p]
    lib.routes_pair.argtypes = [i, i, i, i, p, p, p, p, p, p]
    return lib


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _randn(gen, *shape, dtype=torch.float32):
    return torch.randn(*shape, generator=gen, device="cuda").to(dtype)


@pytest.mark.parametrize("energy", ["dot", "l2", "l2sq", "cos"])
@pytest.mark.parametrize("loss", ["symmetric_infonce", "bwd_infonce"])
@pytest.mark.parametrize("B", [1, 63, 65, 256, 300, 1023, 2817, 4096])
def test_one_pass_and_two_passes(routes, B, energy, loss):
    gen = torch.Generator(device="cuda").manual_seed(B)
    scale = {"dot": 0.3, "cos": 1.0, "l2": 0.5, "l2sq": 0.2}[energy]
    x = _randn(gen, B, 64)
    y = 0.6 * x + 0.8 * _randn(gen, B, 64)
    x, y = scale * x, scale * y
    if B > 1:
        y[B // 2] = x[B // 2]  # a distance of zero
    ws = torch.empty((64 << 20) + 20000 * B, dtype=torch.uint8, device="cuda")
    out = []
    for route in (1, 2):
        print(f"B={B} {energy} {loss} route {route}", flush=True)
        ws.fill_(255)
        g = [torch.full_like(x, float("nan")) for _ in range(2)]
        assert routes.routes_fused(B, 64, ENERGY[energy], LOSS[loss], 0.1, route, x.data_ptr(), y.data_ptr(),
                                   g[0].data_ptr(), g[1].data_ptr(), ws.data_ptr(), ws.numel(), _stream()) == 0
        torch.cuda.synchronize()
        out.append(g)
    assert torch.isfinite(out[0][0]).all() and torch.isfinite(out[0][1]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def _gemm(routes, bf16, la, lb, out_bf16, M, N, K, A, Bm, tile, epi=EPI_NONE, sums=False, partial=None):
    ldc = -(-N // 8) * 8
    c = torch.zeros(M, ldc, device="cuda", dtype=torch.bfloat16 if out_bf16 else torch.float32)
    extra = torch.zeros(2, 64 * max(M, N), device="cuda")
    splits = C.c_int()
    rc = routes.routes_gemm(bf16, la, lb, out_bf16, M, N, K, A.data_ptr(), A.stride(0), Bm.data_ptr(), Bm.stride(0),
                            c.data_ptr(), ldc, epi, extra[0].data_ptr() if sums else None,
                            extra[1].data_ptr() if sums else None, None if partial is None else partial.data_ptr(),
                            0 if partial is None else partial.numel(), tile, C.byref(splits), _stream())
    assert rc == 0
    torch.cuda.synchronize()
    return c[:, :N], extra, splits.value


# (storage, la, lb, output, M, N, K, epilogue, sums, split)
GEMMS = [("fp32", KC, MC, "fp32", 130, 72, 100, EPI_NONE, False, False),
         ("fp32", KC, KC, "fp32", 257, 96, 1030, EPI_NONE, False, False),
         ("fp32", KC, KC, "fp32", 250, 250, 72, EPI_L2, False, False),
         ("fp32", MC, MC, "fp32", 136, 104, 1001, EPI_NONE, True, False),
         ("fp32", KC, MC, "fp32", 70, 64, 4096, EPI_NONE, False, True),
         ("fp32", MC, MC, "fp32", 64, 40, 2100, EPI_NONE, True, True),
         ("bf16", KC, MC, "bf16", 130, 72, 192, EPI_NONE, False, False),
         ("bf16", KC, KC, "bf16", 257, 96, 1024, EPI_NONE, False, False),
         ("bf16", KC, MC, "fp32", 70, 64, 2048, EPI_NONE, False, True),
         ("bf16", MC, MC, "fp32", 136, 104, 1088, EPI_NONE, False, False)]


@pytest.mark.parametrize("store,la,lb,to,M,N,K,epi,sums,split", GEMMS)
def test_gemm_tiles(routes, store, la, lb, to, M, N, K, epi, sums, split):
    bf16, dt = store == "bf16", torch.bfloat16 if store == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    up = lambda n: -(-n // 8) * 8
    A = _randn(gen, *((M, up(K)) if la == KC else (K, up(M))), dtype=dt)
    Bm = _randn(gen, *((N, up(K)) if lb == KC else (K, up(N))), dtype=dt)
    partial = torch.empty(1 << 22, device="cuda") if split else None
    ref = None
    for name, tile in TILES.items():
        if bf16 and name == "64x32":
            continue
        print(store, la, lb, M, N, K, "tile", name, flush=True)
        got = _gemm(routes, bf16, la, lb, to == "bf16", M, N, K, A, Bm, tile, epi, sums, partial)
        assert (got[2] > 1) == split
        if ref is None:
            ref = got
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), name
    a = (A[:, :K] if la == KC else A[:, :M].T).double()
    b = (Bm[:, :K].T if lb == KC else Bm[:, :N]).double()
    want = a @ b
    if epi == EPI_L2:
        want = -((a * a).sum(1)[:, None] + (b * b).sum(0) - 2 * want).sqrt()
    # FP32 chains of 128 products, or one BF16 rounding of the output
    assert (ref[0].double() - want).norm() <= (1e-5 if to == "fp32" else 4e-3) * want.norm()


@pytest.mark.parametrize("store", ["fp32", "bf16"])
@pytest.mark.parametrize("B,I,O", [(64, 64, 64), (130, 72, 64), (1000, 256, 128), (1025, 1024, 512), (4096, 512, 512)])
def test_paired_and_single_launches(routes, store, B, I, O):
    bf16, dt = store == "bf16", torch.bfloat16 if store == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(B)
    x, w, dz = _randn(gen, B, I, dtype=dt), _randn(gen, I, O, dtype=dt), _randn(gen, B, O, dtype=dt)
    dw, dx = torch.zeros(I, O, device="cuda"), torch.zeros(B, I, device="cuda", dtype=dt)
    print(store, B, I, O, flush=True)
    assert routes.routes_pair(bf16, B, I, O, x.data_ptr(), w.data_ptr(), dz.data_ptr(), dw.data_ptr(),
                              dx.data_ptr(), _stream()) == 0
    torch.cuda.synchronize()
    # a ragged BF16 batch takes one tile and k order wherever it runs
    one = _gemm(routes, bf16, MC, MC, False, I, O, B, x, dz, TILES["64"])[0]
    two = _gemm(routes, bf16, KC, KC, bf16, B, I, O, dz, w, TILES["64"])[0]
    assert torch.equal(dw, one) and torch.equal(dx, two)

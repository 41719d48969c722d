"""The 4-bit strip kernels called for by name (decode4_tile_kernel: mask tile 128, up to 8 rows; decode4_kernel otherwise) against the float64
product of the dequantized weight: one to many tiles per wavefront, odd counts and remainders, one to three strips per workgroup with a
part-filled last one, every block count of rows and its edges, sets whose weights meet inside a workgroup, guard regions around Y.  Element bound
as in test_gpu_batch4 (products are exact in fp32)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def _weight(N, K, tile, f, seed):
    c = synth.make_case("strip4", N, K, 1, tile, f, seed=seed)
    W = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(W, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, W, stream)
    P = B.patch_pack4(W, N, K, c.tile_map, tile, stream)
    B.patch_unpack4(P, W_deq=W, stream=stream)
    return W.double(), P


def _strip4(X, M, Ps, Ys):
    vp, n = ctypes.c_void_p, len(Ps)
    st = B.lib().patch_test_gemm4(vp(X.data_ptr()), ctypes.c_int64(M), (vp * n)(*[p.handle for p in Ps]), (vp * n)(*[y.data_ptr() for y in Ys]), n, 0, 1, vp(0),
                                  ctypes.c_size_t(0), vp(torch.cuda.current_stream().cuda_stream))
    assert st == B.OK, st


def _check(Y, X, W, what):
    ref, bound = X @ W.T, 2 * X.shape[1] ** 0.5 * 2.0 ** -24 * X.norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
    worst = ((Y.double() - ref).abs() / bound).max().item()
    assert worst <= 1.0, (what, worst)       # (NaN, an output never written, fails too)


@pytest.mark.parametrize("tile,N,K,f", [(128, 128, 128, 1.0), (128, 256, 384, 0.5), (128, 128, 8960, 0.5), (128, 5504, 640, 0.4), (128, 12160, 256, 0.6),
                                        (128, 12288, 2176, 0.0), (64, 64, 64, 1.0), (64, 192, 1088, 0.5), (64, 5504, 320, 0.5), (64, 12224, 192, 0.3)])
def test_strip4(tile, N, K, f):
    print(f"strip4 tile={tile} N={N} K={K} f={f}", flush=True)
    (W, P), (W2, P2) = _weight(N, K, tile, f, 1), _weight(tile, K, tile, 1 - f, 2)
    for M in (1, 2, 4, 5, 8, 9, 16, 17, 32, 33, 48, 49, 64, 69):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        buf = torch.full((M * N + 2048,), 7.0, device="cuda")
        Y = buf[1024:1024 + M * N].view(M, N)
        Y.fill_(float("nan"))
        _strip4(X, M, [P], [Y])
        _check(Y, X.double(), W, f"M={M}")
        assert bool((buf[:1024] == 7.0).all()) and bool((buf[1024 + M * N:] == 7.0).all()), "wrote outside Y"
        Ys = [torch.full((M, n), float("nan"), device="cuda") for n in (N, tile, N)]
        _strip4(X, M, [P, P2, P], Ys)
        for y, w in zip(Ys, (W, W2, W)):
            _check(y, X.double(), w, f"set M={M}")
        again = torch.empty_like(Ys[0])
        _strip4(X, M, [P, P2, P], [again, Ys[1], Ys[2]])
        assert torch.equal(again, Ys[0]), "not reproducible"


@pytest.mark.parametrize("tile,N,K,f", [(128, [256, 128, 128, 384], 384, 0.5), (128, [2560] * 4, 640, 0.5), (128, [128] * 8, 1152, 1.0), (64, [64, 192, 64, 64, 128], 320, 0.4)])
def test_strip4_set_of_more_than_three(tile, N, K, f):
    """2560: three strips per workgroup, which then hold strips of two weights (2560 / 16 = 160 strips each)"""
    print(f"strip4 set tile={tile} N={N} K={K} f={f}", flush=True)
    weights = [_weight(n, K, tile, f, 1 + i) for i, n in enumerate(N)]
    for M in (1, 8, 9, 16, 17, 32, 33, 48, 49, 64):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        Ys = [torch.full((M, n), float("nan"), device="cuda") for n in N]
        _strip4(X, M, [p for _, p in weights], Ys)
        for i, (y, (w, _)) in enumerate(zip(Ys, weights)):
            _check(y, X.double(), w, f"M={M} weight {i}")


@pytest.mark.parametrize("tile,N,K,f", [(64, 64, 4160, 0.0), (64, 192, 4672, 0.5), (64, 12352, 2176, 0.5), (128, 128, 4480, 1.0), (128, 256, 4736, 0.4)])
def test_strip4_long_runs(tile, N, K, f):
    """one weight, more than four 64-column steps per wavefront: dense codes by one load behind a branch"""
    print(f"strip4 long tile={tile} N={N} K={K} f={f}", flush=True)
    W, P = _weight(N, K, tile, f, 1)
    for M in (1, 9, 16, 17, 33, 49, 64):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        Y = torch.full((M, N), float("nan"), device="cuda")
        _strip4(X, M, [P], [Y])
        _check(Y, X.double(), W, f"M={M}")

"""The 4-bit batched-decoding kernel (batch4_kernel, 128 features x up to 64 rows per workgroup) called for by name - the dispatch takes
it at larger sizes only - against the float64 product of the dequantized weight: every count of 16-row blocks and its edges, one to five
128-column units (two wavefront groups take them in turn), a last unit of one 64-column step, a last feature group of 64, K in chunks
over a workspace that ends in a guard region, sets in one launch.  Then the interface itself, whichever kernel it takes.  Element bound as in test_gpu_prefill64 (the dequantized weight is a bf16 matrix, so products are exact
in fp32)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def _weight(N, K, tile, f, seed):
    c = synth.make_case("batch4", N, K, 1, tile, f, seed=seed)
    W = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(W, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, W, stream)
    P = B.patch_pack4(W, N, K, c.tile_map, tile, stream)
    B.patch_unpack4(P, W_deq=W, stream=stream)
    return W.double(), P


def _check(Y, X, W, what):
    ref, bound = X @ W.T, 2 * X.shape[1] ** 0.5 * 2.0 ** -24 * X.norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
    worst = ((Y.double() - ref).abs() / bound).max().item()
    assert worst <= 1.0, (what, worst)       # (NaN, an output never written, fails too)


def _x(M, K):
    return torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)


def _batch4(X, M, Ps, Ys, chunks=1, workspace=None):
    """batch4_kernel in passes of 64 rows (kernel 1 of the test hook)."""
    vp, n = ctypes.c_void_p, len(Ps)
    st = B.lib().patch_test_gemm4(vp(X.data_ptr()), ctypes.c_int64(M), (vp * n)(*[p.handle for p in Ps]), (vp * n)(*[y.data_ptr() for y in Ys]), n, 1, chunks,
                                  vp(workspace.data_ptr() if workspace is not None else 0), ctypes.c_size_t(4 * workspace.numel() if workspace is not None else 0),
                                  vp(torch.cuda.current_stream().cuda_stream))
    assert st == B.OK, st


@pytest.mark.parametrize("tile,N,K,f", [(64, 64, 64, 1.0), (64, 192, 192, 0.5), (64, 320, 576, 0.6), (128, 128, 128, 0.0), (128, 384, 640, 0.5), (128, 256, 2048, 1.0)])
def test_batch4(tile, N, K, f):
    print(f"batch4 tile={tile} N={N} K={K} f={f}", flush=True)
    (W, P), (W2, P2) = _weight(N, K, tile, f, 1), _weight(tile, K, tile, 1 - f, 2)
    for M in (1, 8, 16, 17, 32, 33, 48, 49, 64, 70):
        X, rows = _x(M, K), min(M, 64)
        for chunks in sorted({1, min(2, (K + 127) // 128), min(5, (K + 127) // 128)}):
            need = chunks * rows * N
            buf = torch.full((need + 1024,), float("nan"), device="cuda")
            buf[need:] = 7.0
            Y = torch.full((M, N), float("nan"), device="cuda")
            _batch4(X, M, [P], [Y], chunks, buf[:need])
            _check(Y, X.double(), W, f"M={M} chunks={chunks}")
            assert bool((buf[need:] == 7.0).all()), "wrote behind the workspace"
        Ys = [torch.full((M, n), float("nan"), device="cuda") for n in (N, tile, N)]
        _batch4(X, M, [P, P2, P], Ys)
        for y, w in zip(Ys, (W, W2, W)):
            _check(y, X.double(), w, f"set M={M}")
    P.close()
    P2.close()


@pytest.mark.parametrize("tile,N,K,f", [(128, 384, 4096, 0.5), (64, 320, 4160, 0.6), (64, 64, 2112, 1.0), (128, 128, 6144, 0.0)])
def test_workspaces_of_gemm4(tile, N, K, f):
    """patch_gemm4_ex at any size of workspace, whatever kernel it takes: nothing is written behind it."""
    print(f"gemm4 workspace tile={tile} N={N} K={K} f={f}", flush=True)
    stream = torch.cuda.current_stream().cuda_stream
    W, P = _weight(N, K, tile, f, 1)
    for M in (16, 17, 33, 48, 49, 64):
        X = _x(M, K)
        for slices in (2, 3, 8):
            need = slices * M * N
            buf = torch.full((need + 1024,), float("nan"), device="cuda")
            buf[need:] = 7.0
            Y = torch.full((M, N), float("nan"), device="cuda")
            B.patch_gemm4(X, M, P, Y, stream, workspace=buf[:need])
            _check(Y, X.double(), W, f"M={M} workspace for {slices}")
            assert bool((buf[need:] == 7.0).all()), "wrote behind the workspace"
    P.close()


@pytest.mark.parametrize("tile,K", [(128, 4096), (64, 4160)])
def test_set_of_gemm4(tile, K):
    print(f"gemm4 set tile={tile} K={K}", flush=True)
    stream = torch.cuda.current_stream().cuda_stream
    (W, P), (W2, P2) = _weight(8192 + tile, K, tile, 0.5, 1), _weight(8192, K, tile, 0.7, 2)
    for M in (17, 33, 64, 70):
        X = _x(M, K)
        Ys = [torch.full((M, n), float("nan"), device="cuda") for n in (8192 + tile, 8192)]
        B.patch_gemm4_many(X, M, [P, P2], Ys, stream)
        for y, w in zip(Ys, (W, W2)):
            _check(y, X.double(), w, f"set M={M}")
    P.close()
    P2.close()

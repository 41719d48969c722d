"""The last steps of a product: the sum over K slices at every number of slices (2 - 8 by name, more by a loop), for one weight and for a set, and
the rounding of a bf16 output at ties, range ends, denormals, infinities and NaN, against the float64 product and torch's rounding on the CPU."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def _check(Y, X, W, what):
    """products are exact in fp32; K additions, as in test_gpu_batch"""
    ref, bound = X @ W.T, 2 * X.shape[1] ** 0.5 * 2.0 ** -24 * X.norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
    worst = ((Y.double() - ref).abs() / bound).max().item()
    assert worst <= 1.0, (what, worst)       # (NaN, an output never written, fails too)


@pytest.mark.parametrize("path,variant,M", [(B.PATH_DECODE, 7, 1), (B.PATH_DECODE, 7, 100), (B.PATH_PREFILL, 0, 100)])
def test_every_number_of_slices(path, variant, M):
    N, K, tile = 384, 2048, 128
    c = synth.make_case("slices", N, K, 1, tile, 0.5, seed=3)
    stream = torch.cuda.current_stream().cuda_stream
    Wd = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    B.patch_apply_mask(Wd, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, Wd, stream)
    P, W = B.patch_pack(Wd, N, K, c.tile_map, tile, stream), Wd.double()
    X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    for split in range(2, 17):
        print(f"slices path={path} variant={variant} M={M} split={split}", flush=True)
        ws = torch.full((2 * split * M * N,), float("nan"), device="cuda")
        kw = dict(path=path, variant=variant, split_k=split, workspace=ws)
        Y, Yb = torch.full((M, N), float("nan"), device="cuda"), torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
        B.patch_gemm(X, M, P, Y, stream, **kw)
        _check(Y, X.double(), W, f"split={split}")
        B.patch_gemm(X, M, P, Yb, stream, y_bf16=True, **kw)
        assert torch.equal(Yb, Y.to(torch.bfloat16)), "bf16 output is the fp32 sum rounded once"
        if path == B.PATH_DECODE:
            Ys = [torch.full((M, N), float("nan"), device="cuda") for _ in range(2)]
            B.patch_gemm_many(X, M, [P, P], Ys, stream, **kw)
            assert torch.equal(Ys[0], Y) and torch.equal(Ys[1], Y), f"set split={split}"
    P.close()


@pytest.mark.parametrize("path,variant", [(B.PATH_DECODE, 0), (B.PATH_DECODE, 4), (B.PATH_DECODE, 7), (B.PATH_PREFILL, 0)])
def test_bf16_rounding_at_the_edges(path, variant):
    """Y = a + b, two terms of a row, both exact in fp32 except where noted: ties to even and odd, either side of a tie, overflow by rounding, denormal
    results, infinities, NaN."""
    N, K, tile = 128, 128, 128
    u, top = 2.0 ** -8, 255 * 2.0 ** 120             # half a unit of 1.0; the largest bf16
    pairs = [(1.0, u), (1.0 + 2 * u, u), (1.0, u * (1 + 2 * u)), (1.0, u * (1 - u)), (top, 2.0 ** 119), (top, 2.0 ** 118), (2.0 ** -126, 0.0),
             (2.0 ** -130, 2.0 ** -133), (2.0 ** -120, 2.0 ** -128), (float("inf"), 1.0), (float("inf"), float("-inf")), (float("nan"), 1.0), (0.0, 0.0)]
    pairs += [(-a, -b) for a, b in pairs]
    M = len(pairs)
    X = torch.zeros(M, K)
    X[:, :2] = torch.tensor(pairs, dtype=torch.float64).float()
    X = X.to(torch.bfloat16).cuda()
    W = torch.zeros(N, K, dtype=torch.bfloat16)
    W[:, :2] = 1.0
    stream = torch.cuda.current_stream().cuda_stream
    P = B.patch_pack(W.cuda(), N, K, synth.make_case("edges", N, K, 1, tile, 0.0, seed=1).tile_map, tile, stream)
    print(f"edges path={path} variant={variant}", flush=True)
    Y, Yb = torch.full((M, N), 7.0, device="cuda"), torch.full((M, N), 7.0, device="cuda", dtype=torch.bfloat16)
    B.patch_gemm(X, M, P, Y, stream, path=path, variant=variant)
    B.patch_gemm(X, M, P, Yb, stream, path=path, variant=variant, y_bf16=True)
    want, got = Y.cpu().to(torch.bfloat16), Yb.cpu()
    nan = want.isnan()
    assert torch.equal(nan, got.isnan())
    assert torch.equal(want.view(torch.int16)[~nan], got.view(torch.int16)[~nan])
    exact = [i for i, (a, b) in enumerate(pairs) if abs(a) >= 1.0 and a == a and a + b == a + b]
    ref = (X[:, 0].cpu().float() + X[:, 1].cpu().float()).to(torch.bfloat16)[:, None].expand(M, N)
    assert torch.equal(ref[exact], got[exact])
    P.close()


def test_bf16_conversion_of_every_pattern():
    bad = torch.zeros(1, device="cuda", dtype=torch.int32)
    st = B.lib().patch_test_bf16_mismatches(ctypes.c_void_p(bad.data_ptr()), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == B.OK and bad.item() == 0

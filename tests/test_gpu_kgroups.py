"""The 4-bit prefill-shaped kernel with two K groups per workgroup, called for by name: one to fourteen K-steps (fewer than its three units in
flight, odd counts, every place in its rotation of three buffers), all-dense, mixed and all-2:4 maps, missing tile rows, part-filled row blocks, more
than 64 tiles along K, K in slices over a workspace with a guard region behind it, against the float64 product of the dequantized weight.
Element bound as in test_gpu_strip4; repeated launches bit-equal."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("tile,N,K", [(128, 128, 128), (128, 384, 384), (128, 640, 896), (128, 256, 8448), (64, 64, 64), (64, 192, 192), (64, 320, 832), (64, 256, 4224)])
def test_two_k_groups(tile, N, K, f):
    vp = ctypes.c_void_p
    c = synth.make_case("kgroups", N, K, 1, tile, f, seed=3)
    Wd = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(Wd, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, Wd, stream)
    P = B.patch_pack4(Wd, N, K, c.tile_map, tile, stream)
    B.patch_unpack4(P, W_deq=Wd, stream=stream)
    W = Wd.double()
    for M in (1, 32, 33, 127, 128, 129, 300):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        ref, bound = X.double() @ W.T, 2 * K ** 0.5 * 2.0 ** -24 * X.double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
        for chunks in sorted({1, 2, 3, K // tile} & set(range(1, min(8, K // tile) + 1))):
            print(f"kgroups tile={tile} N={N} K={K} f={f} M={M} chunks={chunks}", flush=True)
            buf = torch.full((M * N + 2048,), 7.0, device="cuda")
            Y = buf[1024:1024 + M * N].view(M, N)
            first = None
            for _ in range(2):
                Y.fill_(float("nan"))
                ws = torch.full((chunks * M * N + 1024,), 7.0, device="cuda")
                st = B.lib().patch_test_gemm4(vp(X.data_ptr()), ctypes.c_int64(M), (vp * 1)(P.handle), (vp * 1)(Y.data_ptr()), 1, 4, chunks, vp(ws.data_ptr()),
                                              ctypes.c_size_t(4 * chunks * M * N), vp(stream))
                assert st == B.OK, st
                worst = ((Y.double() - ref).abs() / bound).max().item()
                assert worst <= 1.0, (M, chunks, worst)       # (NaN, an output never written, fails too)
                assert bool((buf[:1024] == 7.0).all()) and bool((buf[1024 + M * N:] == 7.0).all()), "wrote outside Y"
                assert bool((ws[chunks * M * N:] == 7.0).all()), "wrote behind the workspace"
                assert first is None or torch.equal(Y, first), "launches of one configuration must be bit-equal"
                first = Y.clone()
    P.close()


@pytest.mark.parametrize("tile,N,K", [(128, 384, 512), (128, 128, 896), (64, 320, 192), (64, 192, 832)])
def test_last_round_in_slices(tile, N, K):
    """The blocks beyond 256 of a launch in K slices over slots of the workspace: part-filled last rows, a feature block that lacks tile rows."""
    vp = ctypes.c_void_p
    c = synth.make_case("kgroups", N, K, 1, tile, 0.5, seed=7)
    Wd = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(Wd, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, Wd, stream)
    P = B.patch_pack4(Wd, N, K, c.tile_map, tile, stream)
    B.patch_unpack4(P, W_deq=Wd, stream=stream)
    W, units = Wd.double(), -(-N // 256)
    M = 128 * -(-259 // units) - 40
    tail = units * -(-M // 128) - 256
    X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    ref, bound = X.double() @ W.T, 2 * K ** 0.5 * 2.0 ** -24 * X.double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
    for chunks in (2, 3, min(7, K // tile)):
        print(f"kgroups last round tile={tile} N={N} K={K} M={M} tail={tail} chunks={chunks}", flush=True)
        buf = torch.full((M * N + 2048,), 7.0, device="cuda")
        Y = buf[1024:1024 + M * N].view(M, N)
        Y.fill_(float("nan"))
        ws = torch.full((chunks * tail * 32768 + 1024,), float("nan"), device="cuda")
        ws[chunks * tail * 32768:] = 7.0
        st = B.lib().patch_test_gemm4(vp(X.data_ptr()), ctypes.c_int64(M), (vp * 1)(P.handle), (vp * 1)(Y.data_ptr()), 1, 5, chunks, vp(ws.data_ptr()),
                                      ctypes.c_size_t(4 * chunks * tail * 32768), vp(stream))
        assert st == B.OK, st
        assert ((Y.double() - ref).abs() / bound).max().item() <= 1.0
        assert bool((buf[:1024] == 7.0).all()) and bool((buf[1024 + M * N:] == 7.0).all()), "wrote outside Y"
        assert bool((ws[chunks * tail * 32768:] == 7.0).all()), "wrote behind the workspace"
    P.close()


@pytest.mark.parametrize("tile,N,K,M,kernel", [(128, 640, 4224, 1112, 4), (128, 1408, 4224, 600, 4), (64, 640, 4160, 1112, 4), (64, 1344, 4224, 600, 4),
                                               (128, 640, 4096, 10968, 5), (128, 1408, 4224, 5464, 5), (64, 640, 4160, 10968, 5), (64, 1344, 4160, 5464, 5)])
def test_the_default_choice_in_slices(tile, N, K, M, kernel):
    """Through the public call, where it takes this kernel with K in slices (4) and with the last round alone in slices (5): equal to the launch called for by
    name, and nothing written behind a workspace of just the size that allows it."""
    vp = ctypes.c_void_p
    c = synth.make_case("kgroups", N, K, 1, tile, 0.5, seed=9)
    Wd = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(Wd, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, Wd, stream)
    P = B.patch_pack4(Wd, N, K, c.tile_map, tile, stream)
    B.patch_unpack4(P, W_deq=Wd, stream=stream)
    W, floats = Wd.double(), (4 if kernel == 4 else 2) * M * N
    X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    which, chunks = (ctypes.c_int * 8)(), (ctypes.c_int * 8)()
    pct = round(100 * (c.tile_map == 0).sum() / c.tile_map.size)
    assert B.lib().patch_test_schedule4(ctypes.c_int64(M), 1, (ctypes.c_int64 * 1)(N), ctypes.c_int64(K), tile, pct, ctypes.c_size_t(4 * floats), which, chunks) == 1
    assert which[0] == kernel and chunks[0] > 1, (which[0], chunks[0])
    ws = torch.full((floats + 1024,), float("nan"), device="cuda")
    ws[floats:] = 7.0
    Y, Z = (torch.full((M, N), float("nan"), device="cuda") for _ in range(2))
    B.patch_gemm4(X, M, P, Y, stream, workspace=ws[:floats])
    assert bool((ws[floats:] == 7.0).all()), "wrote behind the workspace"
    for m in range(0, M, 4096):
        ref, bound = X[m:m + 4096].double() @ W.T, 2 * K ** 0.5 * 2.0 ** -24 * X[m:m + 4096].double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
        assert ((Y[m:m + 4096].double() - ref).abs() / bound).max().item() <= 1.0
    named = torch.full((max(floats, chunks[0] * M * N),), float("nan"), device="cuda")
    assert B.lib().patch_test_gemm4(vp(X.data_ptr()), ctypes.c_int64(M), (vp * 1)(P.handle), (vp * 1)(Z.data_ptr()), 1, kernel, chunks[0], vp(named.data_ptr()),
                                    ctypes.c_size_t(4 * named.numel()), vp(stream)) == B.OK
    assert torch.equal(Y, Z)
    P.close()


@pytest.mark.parametrize("tile,N,K,chunks", [(128, 384, 640, 1), (128, 384, 640, 3), (64, 320, 448, 1), (64, 320, 448, 2)])
def test_infinities_and_nan_in_x(tile, N, K, chunks):
    """Infinities and NaN in X reach the outputs of their rows that they reach in the kernel with one K group, and no others."""
    vp = ctypes.c_void_p
    c = synth.make_case("kgroups", N, K, 1, tile, 0.5, seed=13)
    Wd = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(Wd, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, Wd, stream)
    P = B.patch_pack4(Wd, N, K, c.tile_map, tile, stream)
    B.patch_unpack4(P, W_deq=Wd, stream=stream)
    M, W = 200, Wd.double()
    X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    clean = X.clone()
    X[3, 5], X[64, K - 1], X[64, 1], X[130, K // 2], X[M - 1, 7] = float("inf"), float("inf"), float("-inf"), float("nan"), float("-inf")
    out = []
    for kernel in (4, 2):
        Y, ws = torch.zeros(M, N, device="cuda"), torch.full((chunks * M * N,), float("nan"), device="cuda")
        assert B.lib().patch_test_gemm4(vp(X.data_ptr()), ctypes.c_int64(M), (vp * 1)(P.handle), (vp * 1)(Y.data_ptr()), 1, kernel, chunks, vp(ws.data_ptr()),
                                        ctypes.c_size_t(4 * ws.numel()), vp(stream)) == B.OK
        out.append(Y)
    Y, Z = out
    assert torch.equal(torch.isnan(Y), torch.isnan(Z)) and torch.equal(torch.isinf(Y), torch.isinf(Z)) and torch.equal(Y[torch.isinf(Y)], Z[torch.isinf(Z)])
    assert bool(torch.isnan(Y[130]).any()) and bool((~torch.isfinite(Y[3])).any()) and bool((~torch.isfinite(Y[M - 1])).any())
    rows = [m for m in range(M) if m not in (3, 64, 130, M - 1)]
    ref, bound = clean.double() @ W.T, 2 * K ** 0.5 * 2.0 ** -24 * clean.double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
    assert ((Y.double() - ref).abs() / bound)[rows].max().item() <= 1.0
    P.close()

"""The prefill-shaped product from the 4-bit storage called for by name (blocks of 128 and 256 rows): one
to ten steps, odd counts, all-dense, mixed and all-2:4 maps, part-filled blocks, K in slices over a workspace with a guard region behind
it, against the float64 product of the dequantized weight.  Element bound as in test_gpu_strip4."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("tile,N,K", [(128, 128, 128), (128, 384, 640), (128, 512, 256), (64, 64, 64), (64, 320, 320), (64, 256, 128)])
def test_prefill4(tile, N, K, f):
    vp = ctypes.c_void_p
    c = synth.make_case("prefill4", N, K, 1, tile, f, seed=1)
    Wd = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(Wd, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, Wd, stream)
    P = B.patch_pack4(Wd, N, K, c.tile_map, tile, stream)
    B.patch_unpack4(P, W_deq=Wd, stream=stream)
    W = Wd.double()
    for M in (1, 65, 128, 129, 256, 300):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        ref, bound = X.double() @ W.T, 2 * K ** 0.5 * 2.0 ** -24 * X.double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
        for kernel in (2, 3):
            for chunks in range(1, min(3, K // tile) + 1):
                print(f"prefill4 tile={tile} N={N} K={K} f={f} M={M} kernel={kernel} chunks={chunks}", flush=True)
                buf = torch.full((M * N + 2048,), 7.0, device="cuda")
                Y = buf[1024:1024 + M * N].view(M, N)
                Y.fill_(float("nan"))
                ws = torch.full((chunks * M * N + 1024,), 7.0, device="cuda")
                st = B.lib().patch_test_gemm4(vp(X.data_ptr()), ctypes.c_int64(M), (vp * 1)(P.handle), (vp * 1)(Y.data_ptr()), 1, kernel, chunks, vp(ws.data_ptr()),
                                              ctypes.c_size_t(4 * chunks * M * N), vp(stream))
                assert st == B.OK, st
                worst = ((Y.double() - ref).abs() / bound).max().item()
                assert worst <= 1.0, (M, kernel, chunks, worst)       # (NaN, an output never written, fails too)
                assert bool((buf[:1024] == 7.0).all()) and bool((buf[1024 + M * N:] == 7.0).all()), "wrote outside Y"
                assert bool((ws[chunks * M * N:] == 7.0).all()), "wrote behind the workspace"
    P.close()

"""Batched decoding from the 4-bit storage at sizes whose passes take the kernel with 128 features per workgroup, against the
float64 product of the dequantized weight: counts of 16-row blocks and their edges, a last unit of one 64-column step, a last
feature group of 64, K in chunks over a workspace that ends in a guard region, sets in one launch.  Element bound as in
test_gpu_prefill64 (the dequantized weight is a bf16 matrix, so products are exact in fp32)."""
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


@pytest.mark.parametrize("tile,N,K,f", [(128, 384, 4096, 0.5), (64, 320, 4160, 0.6), (64, 64, 2112, 1.0), (128, 128, 6144, 0.0)])
def test_batch4_split(tile, N, K, f):
    print(f"batch4 tile={tile} N={N} K={K} f={f}", flush=True)
    stream = torch.cuda.current_stream().cuda_stream
    W, P = _weight(N, K, tile, f, 1)
    for M in (16, 17, 33, 48, 49, 64):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
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
def test_batch4_set(tile, K):
    print(f"batch4 set tile={tile} K={K}", flush=True)
    stream = torch.cuda.current_stream().cuda_stream
    (W, P), (W2, P2) = _weight(8192 + tile, K, tile, 0.5, 1), _weight(8192, K, tile, 0.7, 2)
    for M in (17, 33, 64, 70):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        Ys = [torch.full((M, n), float("nan"), device="cuda") for n in (8192 + tile, 8192)]
        B.patch_gemm4_many(X, M, [P, P2], Ys, stream)
        for y, w in zip(Ys, (W, W2)):
            _check(y, X.double(), w, f"set M={M}")
    P.close()
    P2.close()

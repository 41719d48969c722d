"""The batched-decoding kernel (128 features x up to 128 rows per workgroup, decode variant 7) where it can go wrong, against the
float64 product of the same bf16 values: every count of 16-row blocks and its edges, one to five 128-column units (two wavefront
groups take them in turn), a last unit of one 64-column step, a last feature group of 64, K in chunks over a workspace that ends in a
guard region, sets of weights in one launch, bf16 output.  Element bound as in test_gpu_prefill64."""
import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def _weight(N, K, tile, f, seed):
    c = synth.make_case("batch", N, K, 1, tile, f, seed=seed)
    W = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(W, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, W, stream)
    return W.double(), B.patch_pack(W, N, K, c.tile_map, tile, stream)


def _check(Y, X, W, what):
    ref, bound = X @ W.T, 2 * X.shape[1] ** 0.5 * 2.0 ** -24 * X.norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
    worst = ((Y.double() - ref).abs() / bound).max().item()
    assert worst <= 1.0, (what, worst)       # (NaN, an output never written, fails too)


@pytest.mark.parametrize("tile,N,K,f", [(64, 64, 64, 1.0), (64, 192, 192, 0.5), (64, 320, 576, 0.6), (128, 128, 128, 0.0), (128, 384, 640, 0.5),
                                        (128, 256, 2048, 1.0)])
def test_batch(tile, N, K, f):
    print(f"batch tile={tile} N={N} K={K} f={f}", flush=True)
    stream = torch.cuda.current_stream().cuda_stream
    (W, P), (W2, P2) = _weight(N, K, tile, f, 1), _weight(tile, K, tile, 1 - f, 2)
    for M in (1, 8, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 128, 130):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        for split in (1, 2, 3, 0):
            rows = min(M, 128)
            need = max(1, split) * rows * N if split else B.patch_gemm_workspace_bytes(M, P, path=B.PATH_DECODE, variant=7) // 4
            buf = torch.full((need + 1024,), float("nan"), device="cuda")
            buf[need:] = 7.0
            kw = dict(path=B.PATH_DECODE, variant=7, split_k=split, workspace=buf[:need] if need else None)
            Y, Yb = torch.full((M, N), float("nan"), device="cuda"), torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
            B.patch_gemm(X, M, P, Y, stream, **kw)
            _check(Y, X.double(), W, f"M={M} split={split}")
            B.patch_gemm(X, M, P, Yb, stream, y_bf16=True, **kw)
            assert torch.equal(Yb, Y.to(torch.bfloat16)), "bf16 output is the fp32 sum rounded once"
            assert bool((buf[need:] == 7.0).all()), "wrote behind the workspace"
        ws = torch.full((8 * M * (2 * N + tile),), float("nan"), device="cuda")
        for kw in (dict(), dict(workspace=ws), dict(path=B.PATH_DECODE), dict(path=B.PATH_DECODE, variant=7), dict(path=B.PATH_DECODE, variant=7, workspace=ws)):
            Ys = [torch.full((M, n), float("nan"), device="cuda") for n in (N, tile, N)]
            B.patch_gemm_many(X, M, [P, P2, P], Ys, stream, **kw)
            for y, w in zip(Ys, (W, W2, W)):
                _check(y, X.double(), w, f"set M={M}")
    P.close()
    P2.close()


@pytest.mark.parametrize("tile,N,K", [(128, 384, 640), (64, 192, 576)])
def test_set_takes_the_chunks_asked_for(tile, N, K):
    """split_k of variant 7 counts K chunks over the workspace for a set too: its first split_k x M x (sum of N) floats are written, nothing
    behind them."""
    print(f"batch set chunks tile={tile} N={N} K={K}", flush=True)
    stream = torch.cuda.current_stream().cuda_stream
    (W, P), (W2, P2) = _weight(N, K, tile, 0.5, 1), _weight(tile, K, tile, 0.5, 2)
    for M, split in ((5, 2), (64, 3), (100, 5)):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        Ys = [torch.full((M, n), float("nan"), device="cuda") for n in (N, tile)]
        need = split * M * (N + tile)
        ws = torch.full((need + 4096,), float("nan"), device="cuda")
        B.patch_gemm_many(X, M, [P, P2], Ys, stream, path=B.PATH_DECODE, variant=7, split_k=split, workspace=ws)
        for y, w in zip(Ys, (W, W2)):
            _check(y, X.double(), w, f"set M={M} split={split}")
        assert bool(torch.isfinite(ws[:need]).all()) and bool(ws[need:].isnan().all()), f"M={M} split={split}: not {split} chunks"
    P.close()
    P2.close()

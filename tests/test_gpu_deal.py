"""17 - 64 rows whose blocks of 16 are dealt over several workgroups per feature group (strip kernel and mid_kernel, K whole or in chunks; the
dispatch takes what it estimates fastest): every block count and its edges, sets, fp32 and bf16 output, guard regions around Y and behind the workspace,
against the float64 product.  Element bound as in test_gpu_batch (products are exact in fp32); a bf16 output is that sum rounded once."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def _weight(N, K, tile, f, seed):
    c = synth.make_case("deal", N, K, 1, tile, f, seed=seed)
    W = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(W, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, W, stream)
    return W.double(), B.patch_pack(W, N, K, c.tile_map, tile, stream)


def _plan(M, N, K, tile, f, ws_bytes):
    """kernel (0 strip, 1 mid), K chunks and deals of the rows of the pass the dispatch takes"""
    kernel, chunks, deals = (ctypes.c_int * 8)(), (ctypes.c_int * 8)(), (ctypes.c_int * 8)()
    assert B.lib().patch_test_schedule_deals(ctypes.c_int64(M), len(N), (ctypes.c_int64 * len(N))(*N), ctypes.c_int64(K), tile, round(100 * f), ctypes.c_size_t(ws_bytes), kernel, chunks, deals) == 1
    return kernel[0], chunks[0], deals[0]


# takes: (kernel, K in chunks or not, deals) that have to be among the passes; 1472 and 1088 + 64 + 320 features are 92 strips, 5504 are 86 groups of 64
@pytest.mark.parametrize("tile,N,K,f,ws,takes", [
    (128, [896] * 3, 896, 0.5, 0, {(1, False, 3), (1, False, 4)}), (128, [896], 4864, 0.5, 0, {(0, False, 2), (0, False, 3), (0, False, 4)}),
    (64, [896], 4864, 1.0, 32 << 20, {(1, True, 2), (1, True, 3)}), (128, [2048], 2048, 0.0, 0, {(0, False, 2)}), (64, [2048] * 3, 2048, 0.5, 0, {(1, False, 2)}),
    (128, [4096], 4096, 0.5, 0, {(1, False, 3), (1, False, 4)}), (64, [512], 13824, 0.5, 32 << 20, {(1, True, 2), (1, True, 3), (1, True, 4)}),
    (64, [1088, 64, 320], 1088, 0.4, 32 << 20, {(0, False, 2)}), (64, [1472], 1472, 0.5, 32 << 20, {(0, False, 2)}), (128, [5504], 2048, 0.5, 0, {(1, False, 2)})])
def test_rows_dealt_over_workgroups(tile, N, K, f, ws, takes):
    weights = [_weight(n, K, tile, f, 1 + i) for i, n in enumerate(N)]
    taken = set()
    for M in (17, 31, 32, 33, 47, 48, 49, 63, 64):
        kernel, chunks, deals = _plan(M, N, K, tile, f, ws)
        taken.add((kernel, chunks > 1, deals))
        print(f"deal tile={tile} N={N} K={K} M={M} kernel={kernel} chunks={chunks} deals={deals}", flush=True)
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        for dtype in (torch.float32, torch.bfloat16):
            bufs = [torch.full((M * n + 2048,), 7.0, device="cuda", dtype=dtype) for n in N]
            Ys = [b[1024:1024 + M * n].view(M, n) for b, n in zip(bufs, N)]
            for y in Ys:
                y.fill_(float("nan"))
            work = torch.full((ws // 4 + 1024,), 7.0, device="cuda") if ws else None
            kw = dict(workspace=work[:ws // 4]) if ws else {}
            if len(N) > 1:
                B.patch_gemm_many(X, M, [p for _, p in weights], Ys, torch.cuda.current_stream().cuda_stream, y_bf16=dtype == torch.bfloat16, **kw)
            else:
                B.patch_gemm(X, M, weights[0][1], Ys[0], torch.cuda.current_stream().cuda_stream, y_bf16=dtype == torch.bfloat16, **kw)
            for (W, _), y, b, n in zip(weights, Ys, bufs, N):
                ref = X.double() @ W.T
                bound = 2 * K ** 0.5 * 2.0 ** -24 * X.double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
                if dtype == torch.bfloat16:
                    bound = bound + ref.abs() * 2.0 ** -8
                worst = ((y.double() - ref).abs() / bound).max().item()
                assert worst <= 1.0, (M, dtype, worst)       # (NaN, an output never written, fails too)
                assert bool((b[:1024] == 7.0).all()) and bool((b[1024 + M * n:] == 7.0).all()), "wrote outside Y"
            if ws:
                assert bool((work[ws // 4:] == 7.0).all()), "wrote behind the workspace"
    assert takes <= taken, (takes, taken)


@pytest.mark.parametrize("M", [12, 17, 40, 64])
def test_tuner_times_what_an_untuned_call_runs(M):
    """512 x 13824 with a workspace: from 17 rows on mid_kernel in chunks with its rows dealt, which no single variant stands for"""
    tile, N, K, f = 64, 512, 13824, 0.5
    _, P = _weight(N, K, tile, f, 1)
    X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    Y, work, stream = torch.empty(M, N, device="cuda"), torch.empty(8 << 20, device="cuda"), torch.cuda.current_stream().cuda_stream
    print(f"tune M={M}", flush=True)
    timed = B.patch_tune_all(X, M, P, Y, work, stream=stream, reps=2)
    assert len(timed) < 64 and dict(path=B.PATH_DECODE, split_k=0, variant=0, uses_workspace=True) in [sched for sched, _ in timed]
    _, chunks, deals = _plan(M, [N], K, tile, f, 4 * work.numel())
    assert (chunks > 1 and deals > 1) or M < 17
    B.patch_gemm(X, M, P, Y, stream, path=B.PATH_DECODE, workspace=work)
    auto = torch.empty_like(Y)
    B.patch_gemm(X, M, P, auto, stream, workspace=work)
    assert torch.equal(Y, auto)

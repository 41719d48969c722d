"""The 256 x 256 prefill kernel of mask tile 64 (prefill_kernel_w64) where its step loop, its list of table entries and its
launches can go wrong, against the float64 product of the same bf16 values: one to three K-steps (fewer than the loop
looks ahead), the 256 tiles its entry list holds at most, one to three tile rows in the last feature block, ragged rows,
K in slices, a set of weights in one launch, a part-filled last round in slices.

Element bound (as in test_gpu_parity): products of two bf16 are exact in fp32, so an element is off by the rounding of K
additions whose partial sums do not exceed |x_m| |w_n|: at most 2 sqrt(K) 2^-24 |x_m| |w_n|."""
import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def _weight(N, K, f, seed):
    c = synth.make_case("w64", N, K, 1, 64, f, seed=seed)
    W = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(W, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, 64, W, stream)
    return W.double(), B.patch_pack(W, N, K, c.tile_map, 64, stream)


def _check(Y, X, W, what):
    ref, bound = X @ W.T, 2 * X.shape[1] ** 0.5 * 2.0 ** -24 * X.norm(dim=1)[:, None] * W.norm(dim=1)[None, :]
    worst = ((Y.double() - ref).abs() / bound).max().item()
    print(f"  {what}: worst error / bound {worst:.3f}", flush=True)
    assert worst <= 1.0, what       # (NaN, an output never written, fails too)


@pytest.mark.parametrize("N,K,M,f", [(64, 64, 5, 1.0), (128, 128, 256, 0.5), (320, 192, 257, 1.0), (448, 448, 130, 0.0), (192, 16384, 70, 0.5),
                                     (2112, 2048, 7400, 0.6)])
def test_prefill64(N, K, M, f):
    print(f"prefill64 N={N} K={K} M={M} f={f}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    X = torch.randn(M, K, device="cuda", generator=gen).to(torch.bfloat16)
    (W, P), (W2, P2) = _weight(N, K, f, 1), _weight(64, K, f, 2)
    ws = torch.empty(max(9 * M * (N + 64), 64 << 18), device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for kw in (dict(variant=3), dict(variant=3, workspace=ws), dict(variant=3, workspace=ws, split_k=min(5, K // 64))):
        Y, Yb = torch.full((M, N), float("nan"), device="cuda"), torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
        ws.fill_(float("nan"))
        B.patch_gemm(X, M, P, Y, stream, path=B.PATH_PREFILL, **kw)
        _check(Y, X.double(), W, f"split_k={kw.get('split_k', 0)} workspace={'workspace' in kw}")
        B.patch_gemm(X, M, P, Yb, stream, path=B.PATH_PREFILL, y_bf16=True, **kw)
        assert torch.equal(Yb, Y.to(torch.bfloat16)), "bf16 output is the fp32 sum rounded once"
    for kw in (dict(), dict(workspace=ws)):
        Ys = [torch.full((M, n), float("nan"), device="cuda") for n in (N, 64, N)]
        ws.fill_(float("nan"))
        B.patch_gemm_many(X, M, [P, P2, P], Ys, stream, path=B.PATH_PREFILL, **kw)
        for y, w in zip(Ys, (W, W2, W)):
            _check(y, X.double(), w, f"set of {len(Ys)}, workspace={'workspace' in kw}")
    P.close()
    P2.close()

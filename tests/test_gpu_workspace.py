"""patch_gemm_workspace_bytes against what the launch does: given any amount of workspace a product writes no further than the query
says (nothing where it says 0), and given exactly that amount it runs the same schedule - the same split of K, hence the same
bits."""
import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu
PATTERN = 0x7FC0BEEF


def _weight(N, K, tile, f):
    c = synth.make_case("workspace", N, K, 1, tile, f, seed=5)
    W = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(W, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, W, stream)
    return B.patch_pack(W, N, K, c.tile_map, tile, stream)


def _check(P, N, K, M, kw, big):
    """-> bytes the query asks for; `big`: int32 scratch of more than any schedule wants."""
    stream = torch.cuda.current_stream().cuda_stream
    X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    need = B.patch_gemm_workspace_bytes(M, P, **kw)
    what = f"{N}x{K} M={M} {kw}: {need} bytes asked for"
    print(what, flush=True)
    big.fill_(PATTERN)
    Y, E = torch.full((M, N), float("nan"), device="cuda"), torch.full((M, N), float("nan"), device="cuda")
    B.patch_gemm(X, M, P, Y, stream, workspace=big.view(torch.float32), **kw)
    kept = bool((big[need // 4:] == PATTERN).all())
    assert kept, what + ", more written"
    if need:
        B.patch_gemm(X, M, P, E, stream, workspace=big[:need // 4].view(torch.float32), **kw)
        assert torch.equal(Y, E), what + ", another schedule with exactly that"
    return need


@pytest.mark.parametrize("tile,N,K,f", [(128, 640, 4096, 0.5), (64, 448, 4160, 0.5)])
def test_query_of_decode_passes(tile, N, K, f):
    P = _weight(N, K, tile, f)
    big = torch.empty(16 * 256 * N, device="cuda", dtype=torch.int32)
    asked = []
    for kw in (dict(), dict(path=B.PATH_DECODE), dict(path=B.PATH_DECODE, variant=4), dict(path=B.PATH_DECODE, variant=7),
               dict(path=B.PATH_DECODE, variant=7, split_k=2), dict(path=B.PATH_DECODE, variant=7, split_k=5)):
        for M in (1, 8, 12, 16, 17, 33, 64, 65, 100, 128, 130, 200):
            need = _check(P, N, K, M, kw, big)
            asked.append(need)
            if kw.get("split_k"):
                assert need == kw["split_k"] * min(M, 128) * N * 4, "the requested chunks of the largest pass"
    assert max(asked) > 0
    P.close()


@pytest.mark.parametrize("N,K,M", [(2112, 2048, 7400), (320, 4160, 300), (4096, 1024, 513), (192, 16448, 300)])
def test_query_of_prefill_launches_of_mask_tile_64(N, K, M):
    """A part-filled last round in slices, whole launches in slices in either block height, and a K beyond the register-weight kernel."""
    P = _weight(N, K, 64, 0.6)
    big = torch.empty(max(9 * M * N, 64 << 18), device="cuda", dtype=torch.int32)
    asked = [_check(P, N, K, M, kw, big) for kw in (dict(), dict(path=B.PATH_PREFILL), dict(path=B.PATH_PREFILL, variant=3),
                                                    dict(path=B.PATH_PREFILL, variant=6), dict(path=B.PATH_PREFILL, split_k=3))]
    assert max(asked) > 0
    P.close()


def test_static_scratch_takes_a_part_filled_last_round_of_mask_tile_64():
    """306 blocks of 256 x 256: the 50 of the last round would like 62 MB in slices; patch_gemm_static runs with what its array holds."""
    N, K, M = 2112, 5120, 8700
    P = _weight(N, K, 64, 0.5)
    assert B.patch_gemm_workspace_bytes(M, P) > B.STATIC_SCRATCH_BYTES
    stream = torch.cuda.current_stream().cuda_stream
    X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    Y, E = torch.full((M, N), float("nan"), device="cuda"), torch.full((M, N), float("nan"), device="cuda")
    B.patch_gemm_static(X, M, P, Y, stream)
    B.patch_gemm(X, M, P, E, stream, workspace=torch.empty(B.STATIC_SCRATCH_BYTES // 4, device="cuda"))
    assert torch.equal(Y, E)
    P.close()


def test_static_scratch_and_last_rounds_of_mask_tile_128():
    """324 tiles, the last 68 in slices of 51 MB where there is a workspace for them: accepted, since slices of 256-row tiles alone would not be made, and run in
    what the array holds.  384 tiles of a longer K, whose last 128 would be 64 MB in two slices: refused, though the launch takes halves and writes no
    scratch; the size asked for is those 64 MB."""
    stream = torch.cuda.current_stream().cuda_stream
    P, M = _weight(4608, 4096, 128, 0.0), 4608
    assert B.patch_gemm_workspace_bytes(M, P) == 3 * 68 * (256 << 10) > B.STATIC_SCRATCH_BYTES
    X = torch.randn(M, 4096, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    Y, E = (torch.full((M, 4608), float("nan"), device="cuda") for _ in range(2))
    B.patch_gemm_static(X, M, P, Y, stream)
    B.patch_gemm(X, M, P, E, stream, workspace=torch.empty(B.STATIC_SCRATCH_BYTES // 4, device="cuda"))
    assert torch.equal(Y, E)
    P.close()
    P, M = _weight(4096, 11008, 128, 0.5), 6144
    assert B.patch_gemm_workspace_bytes(M, P) == 2 * 128 * (256 << 10)
    X = torch.randn(M, 11008, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
    Y, ws = torch.full((M, 4096), 7.0, device="cuda"), torch.full((16 << 20,), 7.0, device="cuda")
    with pytest.raises(B.PatchError) as e:
        B.patch_gemm_static(X, M, P, Y, stream)
    assert e.value.status == B.ERR_SIZE and bool((Y == 7.0).all())
    B.patch_gemm(X, M, P, Y, stream, workspace=ws)
    assert bool((ws == 7.0).all())
    P.close()


@pytest.mark.parametrize("tile,N,K,f", [(128, 640, 4096, 0.5), (64, 448, 4160, 0.5)])
def test_sets_write_what_the_header_says(tile, N, K, f):
    """patch_gemm_many at any M, few rows included: at most max(8, split_k) x M x (sum of N) floats of the workspace, or 64 MB where the
    last round of a prefill launch is split."""
    Ps = [_weight(N, K, tile, f), _weight(tile, K, tile, f)]
    total, stream = N + tile, torch.cuda.current_stream().cuda_stream
    big = torch.empty(16 * 300 * total + (16 << 20), device="cuda", dtype=torch.int32)
    used = []
    for M in (1, 8, 12, 16, 17, 33, 64, 65, 100, 128, 130, 300):
        X = torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)
        for kw in (dict(), dict(path=B.PATH_DECODE), dict(path=B.PATH_DECODE, variant=4), dict(path=B.PATH_DECODE, variant=7, split_k=12)):
            big.fill_(PATTERN)
            Ys = [torch.full((M, n), float("nan"), device="cuda") for n in (N, tile)]
            B.patch_gemm_many(X, M, Ps, Ys, stream, workspace=big.view(torch.float32), **kw)
            touched = torch.nonzero(big != PATTERN)
            used.append(int(touched[-1]) + 1 if len(touched) else 0)
            assert used[-1] <= max(max(8, kw.get("split_k", 0)) * M * total, 16 << 20 if M > 128 else 0), (M, kw)
    assert max(used) > 0
    for P in Ps:
        P.close()

"""Mask merge and packing, whose tile map travels as kernel arguments: maps of more tiles than one launch takes (whole tile rows, and a single row that is
longer), rows that are no multiple of a wavefront's 512 columns, any nonzero byte as "dense"; and calls from more threads than there are words to report in."""
import threading
import time

import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,N,K", [(64, 64, 64), (64, 192, 576), (128, 384, 896), (128, 128, 1408), (64, 4224, 19584), (64, 128, 64 * 19500), (128, 128, 128 * 9800)])
def test_maps_of_any_size(tile, N, K):
    stream = torch.cuda.current_stream().cuda_stream
    g = torch.Generator(device="cuda").manual_seed(N + K)
    W = torch.randn(N, K, device="cuda", generator=g).to(torch.bfloat16)
    first = torch.randint(0, 3, (N, K // 4), device="cuda", generator=g)     # two of four kept: `first` and a later one
    mask = torch.zeros(N, K // 4, 4, device="cuda", dtype=torch.uint8)
    mask.scatter_(2, first[..., None], 1)
    mask.scatter_(2, torch.full_like(first[..., None], 3), 1)
    mask = mask.view(N, K)
    tm = np.random.default_rng(N + K).integers(0, 2, (N // tile, K // tile)).astype(np.uint8) * 3
    keep = mask.bool() | torch.from_numpy(tm != 0).cuda().repeat_interleave(tile, 0).repeat_interleave(tile, 1)
    want = torch.where(keep, W, torch.zeros_like(W))
    del keep
    out = torch.full((N * K + 64,), 7.0, device="cuda", dtype=torch.bfloat16)
    B.patch_apply_mask(W, mask, tm, N, K, tile, out, stream)
    assert torch.equal(out[:N * K].view(N, K), want) and bool((out[N * K:] == 7.0).all())
    B.patch_apply_mask(W, mask, tm, N, K, tile, W, stream)      # in place
    assert torch.equal(W, want)
    P = B.patch_pack(want, N, K, tm, tile, stream)
    back = torch.full_like(want, float("nan"))
    B.patch_unpack(P, back, stream)
    torch.cuda.synchronize()
    assert torch.equal(back, want)
    P.close()
    # 4-bit: the whole matrix as its parts, each packed by itself
    P4 = B.patch_pack4(want, N, K, tm, tile, stream)
    B.patch_unpack4(P4, W_deq=back, stream=stream)
    P4.close()
    for r0, r1, c0, c1 in ((0, tile, 0, min(K, 1024 // tile * tile)), (N - tile, N, K - min(K, 1024 // tile * tile), K)):
        part, tp = want[r0:r1, c0:c1].contiguous(), np.ascontiguousarray(tm[r0 // tile:r1 // tile, c0 // tile:c1 // tile])
        P4 = B.patch_pack4(part, r1 - r0, c1 - c0, tp, tile, stream)
        alone = torch.full_like(part, float("nan"))
        B.patch_unpack4(P4, W_deq=alone, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(back[r0:r1, c0:c1], alone)
        P4.close()


def _pruned(N, K, tile):
    """(W, keep bytes, tile map, expected W_hat) on the GPU; every third byte of the keep mask is zero."""
    g = torch.Generator(device="cuda").manual_seed(N + K)
    W = torch.randn(N, K, device="cuda", generator=g).to(torch.bfloat16)
    mask = (torch.arange(N * K, device="cuda") % 3 != 0).to(torch.uint8).view(N, K)
    tm = np.random.default_rng(N + K).integers(0, 2, (N // tile, K // tile)).astype(np.uint8)
    dense = torch.from_numpy(tm != 0).cuda().repeat_interleave(tile, 0).repeat_interleave(tile, 1)
    return W, mask, tm, torch.where(mask.bool() | dense, W, torch.zeros_like(W))


@pytest.mark.parametrize("tile,N,K", [(64, 64, 64), (64, 4160, 64), (64, 192, 128), (64, 128, 192), (64, 320, 256), (64, 64, 320), (64, 128, 448), (64, 192, 512),
                                      (128, 128, 128), (128, 4224, 128), (128, 384, 256), (128, 128, 384), (64, 64 * 19500, 64)])
def test_mask_merge_of_short_rows(tile, N, K):
    """Rows that share a wavefront with others (up to 256 columns), and the next longer ones."""
    stream = torch.cuda.current_stream().cuda_stream
    W, mask, tm, want = _pruned(N, K, tile)
    out = torch.full((N * K + 64,), 7.0, device="cuda", dtype=torch.bfloat16)
    B.patch_apply_mask(W, mask, tm, N, K, tile, out, stream)
    assert torch.equal(out[:N * K].view(N, K), want) and bool((out[N * K:] == 7.0).all())
    B.patch_apply_mask(W, mask, tm, N, K, tile, W, stream)      # in place
    assert torch.equal(W, want)


def test_short_rows_cost_what_long_ones_do():
    """The same bytes as rows of 64 and of 4096 columns: the calls take about the same time (2.2 times as long with a wavefront per row)."""
    stream, us = torch.cuda.current_stream().cuda_stream, []
    for N, K in ((2 ** 20, 64), (2 ** 14, 4096)):
        W, mask, tm, _ = _pruned(N, K, 64)
        out, best = torch.empty_like(W), []
        for _ in range(20):
            torch.cuda.synchronize()
            t = time.perf_counter()
            B.patch_apply_mask(W, mask, tm, N, K, 64, out, stream)
            best.append(time.perf_counter() - t)
        us.append(min(best))
    assert us[0] < 1.6 * us[1], us


def test_every_thread_gets_its_own_report():
    """80 threads pack at once, every third a matrix that is not 2:4: each call reports on its own matrix, first and second time."""
    good = torch.zeros(256, 256, device="cuda", dtype=torch.bfloat16)
    good.view(256, 64, 4)[:, :, :2] = 1.0
    bad = good.clone()
    bad[200, 130:133] = 1.0
    torch.cuda.synchronize()
    tm, results = np.zeros((2, 2), np.uint8), [[] for _ in range(80)]

    def work(i):
        for pack in (B.patch_pack, B.patch_pack4):
            try:
                pack(bad if i % 3 == 0 else good, 256, 256, tm, 128, 0).close()
                results[i].append(B.OK)
            except B.PatchError as e:
                results[i].append(e.status)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(80)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert results == [[B.ERR_NOT_24] * 2 if i % 3 == 0 else [B.OK] * 2 for i in range(80)]

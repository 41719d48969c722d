"""The bf16 prefill kernel in blocks of 128 rows (prefill_kernel_r128), called for by name and as the default choice takes it: one to fourteen K-steps
(fewer than its four stages, odd counts), all-dense, mixed and all-2:4 maps, missing tile rows, part-filled row blocks, more than 64 tiles along K, K in
slices over a workspace with a guard region behind it, sets of weights, both output types, against the float64 product.  Element bound as in
test_gpu_parity (bf16 output: its rounding on top); repeated launches bit-equal."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu

vp = ctypes.c_void_p


def _weight(N, K, tile, f, seed):
    c = synth.make_case("rows128", N, K, 1, tile, f, seed=seed)
    Wd = torch.from_numpy(c.W.view(np.int16)).cuda().view(torch.bfloat16)
    stream = torch.cuda.current_stream().cuda_stream
    B.patch_apply_mask(Wd, torch.from_numpy(c.mask24).cuda(), c.tile_map, N, K, tile, Wd, stream)
    return B.patch_pack(Wd, N, K, c.tile_map, tile, stream), Wd.double()


def _x(M, K):
    return torch.randn(M, K, device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)).to(torch.bfloat16)


def _ref(X, W):
    ref = X.double() @ W.T
    return ref, 2 * X.shape[1] ** 0.5 * 2.0 ** -24 * X.double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :]


@pytest.mark.parametrize("f", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("tile,Ns,K", [(128, [128], 128), (128, [384], 384), (128, [640, 128], 896), (128, [256], 8448), (64, [64], 64), (64, [192], 192),
                                       (64, [320, 64, 192], 832), (64, [256], 4224)])
def test_rows128(tile, Ns, K, f):
    stream = torch.cuda.current_stream().cuda_stream
    Ps, Ws = zip(*[_weight(N, K, tile, f, 3 + i) for i, N in enumerate(Ns)])
    for M in (1, 32, 33, 127, 128, 129, 300):
        X = _x(M, K)
        refs = [_ref(X, W) for W in Ws]
        for split in sorted({1, 2, 3, K // tile} & set(range(1, min(8, K // tile) + 1))):
            for dt in (torch.float32, torch.bfloat16):
                print(f"rows128 tile={tile} N={Ns} K={K} f={f} M={M} split={split} {dt}", flush=True)
                first, ends = None, np.cumsum([1024] + [M * N + 1024 for N in Ns])
                for _ in range(2):
                    buf = torch.full((int(ends[-1]),), 7.0, device="cuda", dtype=dt)
                    Ys = [buf[e:e + M * N].view(M, N) for e, N in zip(ends, Ns)]
                    for Y in Ys:
                        Y.fill_(float("nan"))
                    ws = torch.full((split * M * sum(Ns) + 1024,), float("nan"), device="cuda")
                    ws[split * M * sum(Ns):] = 7.0
                    st = B.lib().patch_test_prefill128(vp(X.data_ptr()), ctypes.c_int64(M), (vp * len(Ns))(*[P.handle for P in Ps]),
                                                       (vp * len(Ns))(*[Y.data_ptr() for Y in Ys]), len(Ns), split, int(dt == torch.bfloat16),
                                                       vp(ws.data_ptr()), ctypes.c_size_t(4 * split * M * sum(Ns)), vp(stream))
                    assert st == B.OK, st
                    for Y, (ref, bound) in zip(Ys, refs):
                        allowed = bound if dt == torch.float32 else bound + 2.0 ** -8 * (ref.abs() + bound)
                        worst = ((Y.double() - ref).abs() / allowed).max().item()
                        assert worst <= 1.0, (M, split, worst)       # (NaN, an output never written, fails too)
                    guards = torch.cat([buf[e - 1024:e] for e in ends])
                    assert bool((guards == 7.0).all()), "wrote outside Y"
                    assert bool((ws[split * M * sum(Ns):] == 7.0).all()), "wrote behind the workspace"
                    assert first is None or all(torch.equal(Y, Z) for Y, Z in zip(Ys, first)), "launches of one configuration must be bit-equal"
                    first = Ys
    for P in Ps:
        P.close()


@pytest.mark.parametrize("tile,Ns,K,M,workspace", [(128, [2176], 4096, 400, True), (64, [2112], 4160, 400, True), (128, [2176, 640], 4096, 384, True), (128, [2176, 640], 1024, 384, False),
                                                   (64, [1344, 1344, 64], 1088, 513, False), (64, [2048], 16448, 129, True)])
def test_the_default_choice_takes_it(tile, Ns, K, M, workspace):
    """Through the public calls: equal to the kernel called for by name, whatever is behind the workspace stays, and a workspace of the size the library
    asks for gives what a larger one gives."""
    stream = torch.cuda.current_stream().cuda_stream
    Ps, Ws = zip(*[_weight(N, K, tile, 0.5, 11 + i) for i, N in enumerate(Ns)])
    X = _x(M, K)
    pct = 100 * sum(P.dims()[3] for P in Ps) // sum((N // tile) * (K // tile) for N in Ns)
    ws_bytes = 64 << 20 if workspace else 0
    split = B.lib().patch_test_prefill128_split(ctypes.c_int64(M), len(Ns), (ctypes.c_int64 * len(Ns))(*Ns), ctypes.c_int64(K), tile, pct, ctypes.c_size_t(ws_bytes))
    assert split >= 1 and (workspace or split == 1)
    sizes = [ws_bytes]
    if workspace and len(Ns) == 1:
        sizes.append(B.patch_gemm_workspace_bytes(M, Ps[0], path=B.PATH_PREFILL))
        assert sizes[1] >= (4 * split * M * Ns[0] if split > 1 else 0)
    outs = []
    for size in sizes:
        ws = torch.full((size // 4 + 1024,), 7.0, device="cuda") if workspace else None
        Ys = [torch.full((M, N), float("nan"), device="cuda") for N in Ns]
        kw = dict(path=B.PATH_PREFILL, workspace=ws[:size // 4] if size else None) if workspace else dict(path=B.PATH_PREFILL)
        if len(Ns) == 1:
            B.patch_gemm(X, M, Ps[0], Ys[0], stream, **kw)
        else:
            B.patch_gemm_many(X, M, Ps, Ys, stream, **kw)
        assert ws is None or bool((ws[size // 4:] == 7.0).all()), "wrote behind the workspace"
        outs.append(Ys)
    named = [torch.full((M, N), float("nan"), device="cuda") for N in Ns]
    ws = torch.empty(split * M * sum(Ns), device="cuda")
    assert B.lib().patch_test_prefill128(vp(X.data_ptr()), ctypes.c_int64(M), (vp * len(Ns))(*[P.handle for P in Ps]), (vp * len(Ns))(*[Y.data_ptr() for Y in named]),
                                         len(Ns), split, 0, vp(ws.data_ptr()), ctypes.c_size_t(4 * ws.numel()), vp(stream)) == B.OK
    for Ys in outs:
        for Y, Z, W in zip(Ys, named, Ws):
            ref, bound = _ref(X, W)
            assert ((Y.double() - ref).abs() / bound).max().item() <= 1.0
            assert torch.equal(Y, Z)
    for P in Ps:
        P.close()


@pytest.mark.parametrize("tile,Ns,K", [(128, [384], 384), (128, [128, 256], 640), (64, [320], 192), (64, [320, 64], 448)])
def test_last_round_in_halves(tile, Ns, K):
    """The tiles beyond 256 of a launch over 256 x 256 tiles, 128 rows a workgroup: whole K and slices in workspace slots, last row blocks whose second half
    is part-filled or empty, feature blocks that lack tile rows, sets."""
    stream = torch.cuda.current_stream().cuda_stream
    Ps, Ws = zip(*[_weight(N, K, tile, 0.5, 5 + i) for i, N in enumerate(Ns)])
    units = sum(-(-N // 256) for N in Ns)
    for missing in (200, 40):
        M = 256 * (-(-258 // units)) - missing
        tail = units * -(-M // 256) - 256
        X = _x(M, K)
        refs = [_ref(X, W) for W in Ws]
        for slices in sorted({1, 2, 3, K // tile} & set(range(1, min(8, K // tile) + 1))):
            for dt in (torch.float32, torch.bfloat16):
                print(f"last round tile={tile} N={Ns} K={K} M={M} tail={tail} slices={slices} {dt}", flush=True)
                ends = np.cumsum([1024] + [M * N + 1024 for N in Ns])
                buf = torch.full((int(ends[-1]),), 7.0, device="cuda", dtype=dt)
                Ys = [buf[e:e + M * N].view(M, N) for e, N in zip(ends, Ns)]
                for Y in Ys:
                    Y.fill_(float("nan"))
                ws = torch.full((slices * tail * 65536 + 1024,), float("nan"), device="cuda")
                ws[slices * tail * 65536:] = 7.0
                st = B.lib().patch_test_prefill_last_round(vp(X.data_ptr()), ctypes.c_int64(M), (vp * len(Ns))(*[P.handle for P in Ps]),
                                                           (vp * len(Ns))(*[Y.data_ptr() for Y in Ys]), len(Ns), 1, slices, int(dt == torch.bfloat16),
                                                           vp(ws.data_ptr()), ctypes.c_size_t(4 * slices * tail * 65536), vp(stream))
                assert st == B.OK, st
                for Y, (ref, bound) in zip(Ys, refs):
                    allowed = bound if dt == torch.float32 else bound + 2.0 ** -8 * (ref.abs() + bound)
                    assert ((Y.double() - ref).abs() / allowed).max().item() <= 1.0
                assert bool((torch.cat([buf[e - 1024:e] for e in ends]) == 7.0).all()), "wrote outside Y"
                assert bool((ws[slices * tail * 65536:] == 7.0).all()), "wrote behind the workspace"
    for P in Ps:
        P.close()


@pytest.mark.parametrize("workspace", [False, True])
def test_the_last_round_of_the_default_choice(workspace):
    N, K, M = 640, 2048, 256 * 86 - 100     # 258 tiles
    stream = torch.cuda.current_stream().cuda_stream
    P, W = _weight(N, K, 128, 0.5, 21)
    X = _x(M, K)
    ws = torch.full((8 * 2 * 65536,), float("nan"), device="cuda")
    Y = torch.full((M, N), float("nan"), device="cuda")

    def forced(halves, slices):
        Z = torch.full((M, N), float("nan"), device="cuda")
        assert B.lib().patch_test_prefill_last_round(vp(X.data_ptr()), ctypes.c_int64(M), (vp * 1)(P.handle), (vp * 1)(Z.data_ptr()), 1, halves, slices, 0,
                                                     vp(ws.data_ptr()), ctypes.c_size_t(4 * ws.numel()), vp(stream)) == B.OK
        return Z

    B.patch_gemm(X, M, P, Y, stream, path=B.PATH_PREFILL, workspace=ws if workspace else None)
    ref, bound = _ref(X, W)
    assert ((Y.double() - ref).abs() / bound).max().item() <= 1.0
    assert any(torch.equal(Y, forced(1, n)) for n in (range(2, 5) if workspace else [1]))
    # whole K in halves adds up in the order of the 256-row kernel; slices do not
    assert torch.equal(Y, forced(-1, 1)) != workspace
    need = B.patch_gemm_workspace_bytes(M, P, path=B.PATH_PREFILL)
    if workspace:
        Z = torch.full((M, N), float("nan"), device="cuda")
        B.patch_gemm(X, M, P, Z, stream, path=B.PATH_PREFILL, workspace=torch.full((need // 4,), float("nan"), device="cuda"))
        assert torch.equal(Y, Z)
    P.close()


@pytest.mark.parametrize("tile,N,K,split", [(128, 384, 640, 1), (128, 384, 640, 3), (64, 320, 448, 1), (64, 320, 448, 2)])
def test_infinities_and_nan_in_x(tile, N, K, split):
    """Infinities and NaN in X reach the outputs of their rows that they reach in the earlier kernel of 128 rows, and no others."""
    stream = torch.cuda.current_stream().cuda_stream
    P, W = _weight(N, K, tile, 0.5, 17)
    M = 200
    X = _x(M, K)
    clean = X.clone()
    X[3, 5], X[64, K - 1], X[64, 1], X[130, K // 2], X[M - 1, 7] = float("inf"), float("inf"), float("-inf"), float("nan"), float("-inf")
    Y, Z, ws = torch.zeros(M, N, device="cuda"), torch.zeros(M, N, device="cuda"), torch.full((split * M * N,), float("nan"), device="cuda")
    assert B.lib().patch_test_prefill128(vp(X.data_ptr()), ctypes.c_int64(M), (vp * 1)(P.handle), (vp * 1)(Y.data_ptr()), 1, split, 0, vp(ws.data_ptr()),
                                         ctypes.c_size_t(4 * ws.numel()), vp(stream)) == B.OK
    B.patch_gemm(X, M, P, Z, stream, path=B.PATH_PREFILL, variant=5)
    assert torch.equal(torch.isnan(Y), torch.isnan(Z)) and torch.equal(torch.isinf(Y), torch.isinf(Z)) and torch.equal(Y[torch.isinf(Y)], Z[torch.isinf(Z)])
    assert bool(torch.isnan(Y[130]).any()) and bool(torch.isinf(Y[3]).any()) and bool(torch.isinf(Y[M - 1]).any())
    rows = [m for m in range(M) if m not in (3, 64, 130, M - 1)]
    ref, bound = _ref(clean, W)
    assert ((Y.double() - ref).abs() / bound)[rows].max().item() <= 1.0
    P.close()


def test_x_of_more_than_4_gb():
    """Rows of X beyond 32-bit byte offsets, through the public call: the first, the last and those around the middle and each 4 GB."""
    stream = torch.cuda.current_stream().cuda_stream
    N, K, M = 128, 65664, 32768
    P, W = _weight(N, K, 128, 0.5, 19)
    pct = 100 * P.dims()[3] // (K // 128)
    assert B.lib().patch_test_prefill128_split(ctypes.c_int64(M), 1, (ctypes.c_int64 * 1)(N), ctypes.c_int64(K), 128, pct, ctypes.c_size_t(0)) == 1
    X = torch.randn(M, K, device="cuda", dtype=torch.bfloat16, generator=torch.Generator(device="cuda").manual_seed(1))
    Y = torch.full((M, N), float("nan"), device="cuda")
    B.patch_gemm(X, M, P, Y, stream, path=B.PATH_PREFILL)
    edge = 2 ** 32 // (2 * K)
    for r in (0, M // 2 - 32, edge - 32, M - 64):
        ref, bound = _ref(X[r:r + 64], W)
        assert ((Y[r:r + 64].double() - ref).abs() / bound).max().item() <= 1.0, r
    assert bool(torch.isfinite(Y).all())
    P.close()

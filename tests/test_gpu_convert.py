"""Conversion kernels where they can go wrong, bit for bit against the oracle: quotients that are exact half-integers, scales
at both ends of the exponent range, all-zero rows, kept positions of every kind of group, and pointers that only
have the alignment the interface asks for."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2509_23410_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def _bits(x):
    return (np.asarray(x, np.float32).view(np.uint32) >> 16).astype(np.uint16)


def _dev(bits):
    return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)


@pytest.mark.parametrize("tile,N,K", [(64, 64, 64), (128, 128, 128), (64, 192, 448), (128, 384, 640)])
def test_pack4_codes_scales_and_outputs_of_any_alignment(tile, N, K):
    print(f"pack4 tile={tile} {N}x{K}", flush=True)
    rng = np.random.default_rng(N + K)
    c = synth.make_case("conv4", N, K, 1, tile, 0.5, seed=3)
    W = synth.bf16_bits_to_f64(oracle.apply_mask(c.W, c.tile_map, c.mask24, tile))
    W[1::8] = np.round(rng.uniform(-7, 7, W[1::8].shape) * 2) / 2 * (W[1::8] != 0)       # ties: s = 1 where a row holds 7,
    W[1::8, ::tile] = 7 * (W[1::8, ::tile] != 0)
    W[2::8] *= 2.0 ** -115                                                               # scales outside the range of the fast quotient,
    W[3::8] *= 2.0 ** 120
    W[4::8] = 0                                                                          # no scale at all,
    W[5::8] = np.sign(W[5::8]) * (W[5::8] != 0)                                          # one magnitude
    Wb = _bits(W)
    stream = torch.cuda.current_stream().cuda_stream
    P = B.patch_pack4(_dev(Wb), N, K, c.tile_map, tile, stream)
    codes_o, scales_o = oracle.quantize4(Wb, tile)
    deq_o = oracle.dequantize4(codes_o, scales_o, tile)
    for off in (0, 8, 1, 5):                                                             # codes: no alignment of their own
        buf = torch.full((N * K + 16,), 99, dtype=torch.int8, device="cuda")
        deq = torch.empty(N, K, dtype=torch.bfloat16, device="cuda")
        scales = torch.empty(N, K // tile, dtype=torch.int16, device="cuda")
        B.patch_unpack4(P, W_deq=deq, codes=buf[off:off + N * K], scales=scales, stream=stream)
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert np.array_equal(got[off:off + N * K].reshape(N, K), codes_o)
        assert (got[:off] == 99).all() and (got[off + N * K:] == 99).all(), "wrote outside the codes"
        assert np.array_equal(deq.view(torch.int16).cpu().numpy().view(np.uint16), deq_o)
        assert np.array_equal(scales.cpu().numpy().view(np.uint16), scales_o)
    only = torch.empty(N, K, dtype=torch.int8, device="cuda")
    B.patch_unpack4(P, codes=only, stream=stream)
    assert np.array_equal(only.cpu().numpy(), codes_o)
    P.close()


@pytest.mark.parametrize("tile,N,K", [(64, 64, 64), (128, 256, 384)])
def test_pack_of_every_kind_of_group_and_masks_of_any_alignment(tile, N, K):
    print(f"pack tile={tile} {N}x{K}", flush=True)
    rng = np.random.default_rng(N + K)
    T = (N // tile, K // tile)
    tm = np.zeros(T, np.uint8)
    keep = rng.permuted(np.tile(np.array([1, 1, 0, 0], np.uint8), (N * K // 4, 1)), axis=1) & rng.integers(0, 2, (N * K // 4, 4), dtype=np.uint8)
    Wb = (_bits(rng.standard_normal((N, K))) * keep.reshape(N, K)).astype(np.uint16)     # none, one or two of four, everywhere
    stream = torch.cuda.current_stream().cuda_stream
    P = B.patch_pack(_dev(Wb), N, K, tm, tile, stream)
    vals, meta = B.patch_export_canonical(P)
    vals_o, meta_o = oracle.pack(Wb, tm, tile)
    assert np.array_equal(vals, vals_o) and np.array_equal(meta, meta_o)
    P.close()
    logits = rng.standard_normal((6, N * K // 4)).astype(np.float32)
    logits[rng.integers(0, 6, 40), rng.integers(0, N * K // 4, 40)] = np.nan
    logits[:, :8] = 0                                                                    # ties: the first candidate
    want = oracle.hard_masks(np.ones(T, np.float32), logits, N, K, tile)
    want = next(a for a in want if a.size == N * K).reshape(-1)
    for src, dst in ((0, 0), (1, 0), (0, 8), (2, 8)):                                    # 4-byte logits, 8-byte masks
        lb = torch.zeros(logits.size + 4, device="cuda")
        lb[src:src + logits.size] = torch.from_numpy(logits.reshape(-1)).cuda()
        mb = torch.full((N * K + 16,), 9, dtype=torch.uint8, device="cuda")
        B.patch_hard_masks(np.ones(T, np.float32), lb[src:src + logits.size], N, K, tile, mb[dst:dst + N * K], stream)
        torch.cuda.synchronize()
        got = mb.cpu().numpy()
        assert np.array_equal(got[dst:dst + N * K], want) and (got[:dst] == 9).all() and (got[dst + N * K:] == 9).all()

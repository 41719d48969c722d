"""The tile map as kernel arguments: a bit per tile, any nonzero byte is dense, and the dense tiles in front of every 64 (host only)."""
import ctypes
import time

import numpy as np

from paper_2509_23410_amd import binding as B


def _fill(tiles, before=0):
    fn = B.lib().patch_test_map_args
    fn.restype = ctypes.c_int64
    out = np.full(3 * -(-len(tiles) // 64), 7, np.uint32)
    args, best = (ctypes.c_void_p(tiles.ctypes.data), len(tiles), ctypes.c_uint32(before), ctypes.c_void_p(out.ctypes.data)), 1.0
    for _ in range(100):
        t = time.perf_counter()
        total = fn(*args)
        best = min(best, time.perf_counter() - t)
    return out.reshape(-1, 3), total, best


def test_bits_and_counts():
    rng = np.random.default_rng(5)
    for n in [1, 7, 8, 9, 63, 64, 65, 72, 127, 128, 191, 1000, 19455, 19456]:
        for tiles in (rng.integers(0, 2, n, dtype=np.uint8), rng.integers(0, 256, n, dtype=np.uint8), np.full(n, 255, np.uint8), np.full(n, 128, np.uint8), np.zeros(n, np.uint8),
                      (rng.integers(0, 256, n) * (rng.random(n) < 0.1)).astype(np.uint8)):
            got, total, _ = _fill(tiles, before=11)
            bits = np.zeros(64 * len(got), np.uint8)
            bits[:n] = tiles != 0
            words = np.packbits(bits.reshape(-1, 64), axis=1, bitorder="little").view(np.uint32)
            dense = bits.reshape(-1, 64).sum(axis=1, dtype=np.int64)
            assert np.array_equal(got[:, :2], words) and total == 11 + dense.sum()
            assert np.array_equal(got[:, 2], 11 + np.cumsum(dense) - dense)


def test_tiles_are_taken_eight_at_a_time():
    """The mask merge and the packing of a weight wait for this: 19456 tiles in less than half the 18.5 us that a loop over bytes takes (3.6)."""
    assert _fill(np.random.default_rng(6).integers(0, 2, 19456, dtype=np.uint8))[2] < 9e-6

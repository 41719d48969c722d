"""What AUTO chooses against what was measured, without a device: the estimates behind the choice hold constants fitted to measurements,
and a change of one of them must not send a call to a kernel that is slower there.  A row: features of the weights that share X, their
K, mask tile, share of 2:4 tiles, rows of X, workspace or not, and microseconds of the kernels that come into question - strip, mid (mid*
with K in chunks), both with /<deals> where the rows are dealt over several workgroups per feature group, b<chunks> = the kernel with 128 features in
one pass, two passes = of 64 rows and the rest, prefill (MI355X, fp32 output, launches back to back)."""
import ctypes

import pytest

from paper_2509_23410_amd import binding as B

MEASURED = [
    ([896] * 3, 896, 128, 0.0, 20, False, {'mid': 6.2, 'strip': 4.9}),
    ([896] * 3, 896, 64, 0.5, 20, False, {'mid': 5.7, 'strip': 4.8}),
    ([896] * 3, 896, 64, 1.0, 20, False, {'mid': 5.5, 'strip': 4.7}),
    ([28672] * 2, 4096, 128, 1.0, 72, False, {'b1': 72.8, 'prefill': 64.5}),
    ([896] * 3, 896, 64, 0.0, 20, True, {'mid': 5.9, 'strip': 4.8}),
    ([896] * 3, 896, 128, 0.0, 17, True, {'mid': 6.1, 'strip': 4.8}),
    ([896] * 3, 896, 128, 0.5, 17, True, {'mid': 5.7, 'strip': 4.6}),
    ([896] * 3, 896, 64, 1.0, 17, True, {'mid': 5.4, 'strip': 4.5}),
    ([28672] * 2, 4096, 128, 1.0, 65, True, {'prefill': 63.8, 'b1': 70.7}),
    ([11008] * 2, 4096, 64, 1.0, 81, True, {'prefill': 35.1, 'b1': 38.5}),
    ([4096], 4096, 128, 0.0, 20, False, {'mid': 17.2, 'strip': 10.6}),
    ([4096], 4096, 64, 0.5, 17, False, {'mid': 14.6, 'strip': 8.9}),
    ([4096], 4096, 128, 1.0, 20, False, {'mid': 12.4, 'strip': 9.1}),
    ([4096], 4096, 128, 1.0, 17, False, {'mid': 12.0, 'strip': 8.5}),
    ([896], 896, 128, 0.0, 112, False, {'two passes': 13.1, 'prefill': 15.2}),
    ([4096], 11008, 64, 0.0, 96, False, {'two passes': 72.8, 'b1': 86.0}),
    ([4096], 11008, 128, 0.5, 96, False, {'two passes': 70.5, 'b1': 90.7}),
    ([5120], 13824, 64, 1.0, 72, False, {'two passes': 89.5, 'b1': 98.1}),
    ([32896], 4096, 128, 0.5, 16, False, {'b1': 47.9, 'mid': 42.9}),
    ([36864], 4096, 64, 0.5, 16, False, {'b1': 48.1, 'mid': 44.5}),
    ([36864], 4096, 128, 1.0, 16, False, {'b1': 37.9, 'mid': 34.5}),
    ([896], 896, 128, 0.0, 17, True, {'mid': 5.0, 'strip': 4.0, 'strip/2': 3.5}),
    ([896], 896, 64, 0.5, 17, True, {'mid': 5.0, 'strip': 3.9, 'strip/2': 3.5}),
    ([896], 896, 128, 0.5, 20, True, {'mid': 5.1, 'strip': 4.1, 'strip/2': 3.5}),
    ([896], 896, 64, 1.0, 17, True, {'mid': 4.8, 'strip': 3.9, 'strip/2': 3.4}),
    ([13824], 5120, 128, 0.0, 56, True, {'b2': 29.3, 'prefill': 31.0, 'mid': 34.8}),
    ([128256], 1024, 128, 0.5, 56, True, {'prefill': 39.3, 'b1': 48.8}),
    ([32896], 4096, 128, 0.5, 33, True, {'prefill': 46.4, 'b1': 52.2}),
    ([2048], 2048, 64, 1.0, 49, True, {'mid*': 9.0, 'strip': 9.6, 'b4': 8.3, 'mid/4': 6.2}),
    ([13824], 5120, 64, 0.5, 96, True, {'b2': 33.1, 'prefill': 30.0}),
    ([32000], 4096, 64, 1.0, 81, True, {'prefill': 34.8, 'b1': 39.0}),
    ([32000], 4096, 128, 1.0, 96, True, {'prefill': 35.7, 'b1': 39.9}),
    ([36864], 4096, 64, 0.5, 16, True, {'b1': 48.1, 'mid': 44.5}),
    ([36864], 4096, 128, 1.0, 16, True, {'b1': 37.9, 'mid': 34.5}),
    ([28672] * 2, 4096, 128, 0.0, 20, False, {'b1': 69.0, 'mid': 84.5}),
    ([13824] * 2, 5120, 64, 0.0, 56, False, {'b1': 45.1, 'mid': 71.4}),
    ([4096, 1024, 1024], 4096, 128, 0.0, 96, False, {'two passes': 46.9, 'b1': 36.4}),
    ([11008] * 2, 4096, 128, 0.0, 8, False, {'b1': 28.0, 'mid': 35.2}),
    ([13824] * 2, 5120, 64, 0.0, 24, True, {'b1': 42.0, 'mid': 50.4}),
    ([3456] * 3, 3456, 128, 0.0, 48, True, {'b2': 19.8, 'mid': 23.6}),
    ([896] * 3, 896, 64, 0.0, 128, True, {'prefill': 20.6, 'b1': 13.5}),
    ([11008] * 2, 4096, 128, 0.0, 9, True, {'b1': 28.1, 'mid': 34.6}),
    ([128256], 1024, 64, 0.0, 20, False, {'b1': 45.7, 'mid': 57.6}),
    ([32000], 4096, 64, 0.0, 56, False, {'b1': 41.4, 'prefill': 67.2}),
    ([32000], 4096, 128, 0.0, 112, False, {'b1': 52.6, 'prefill': 74.4}),
    ([20480], 4096, 64, 0.0, 12, False, {'b1': 27.4, 'mid': 35.9}),
    ([128256], 1024, 64, 0.5, 20, True, {'b1': 37.9, 'mid': 50.9}),
    ([256], 1024, 64, 0.5, 56, True, {'mid*': 8.8, 'strip': 6.5, 'strip/4': 3.6}),
    ([512], 13824, 128, 0.5, 96, True, {'b8': 21.9, 'prefill': 28.8}),
    ([512], 13824, 128, 0.5, 16, True, {'b8': 14.1, 'strip': 18.3}),
    # launches of many rounds over a short K, and weights beyond the last-level cache
    ([128256], 1024, 64, 1.0, 12, False, {'b1': 24.6, 'mid': 34.7, 'strip': 38.9}),
    ([128256], 1024, 128, 0.5, 16, True, {'b1': 35.8, 'mid': 43.4, 'strip': 43.7}),
    ([36864], 4096, 128, 0.0, 56, True, {'b1': 66.0, 'prefill': 82.7}),
    ([32000], 4096, 128, 0.5, 112, True, {'b1': 50.9, 'prefill': 43.3}),
    # rows dealt over workgroups: few feature groups, K whole and in chunks
    ([896] * 3, 896, 128, 0.5, 40, False, {'strip': 6.3, 'mid': 7.8, 'b1': 8.2, 'mid/3': 4.9}),
    ([896] * 3, 896, 128, 0.5, 64, False, {'strip': 7.2, 'mid': 8.7, 'b1': 8.8, 'mid/4': 4.8}),
    ([896], 4864, 128, 0.5, 64, False, {'strip': 21.3, 'mid': 28.5, 'strip/4': 8.6}),
    ([896], 4864, 128, 0.5, 24, True, {'strip': 11.5, 'mid*': 7.8, 'b8': 8.6, 'mid*/2': 6.8}),
    ([896], 4864, 128, 0.5, 40, True, {'strip': 16.8, 'mid*': 9.7, 'b8': 9.5, 'mid*/3': 7.7}),
    ([512], 13824, 64, 0.5, 64, True, {'mid*': 17.6, 'b8': 15.5, 'mid*/4': 9.7}),
    ([4096], 4096, 128, 0.5, 64, False, {'strip': 20.1, 'mid': 25.8, 'b1': 27.1, 'mid/4': 13.1}),
    ([2048] * 3, 2048, 64, 0.5, 48, True, {'strip': 18.9, 'mid': 14.2, 'b1': 14.1, 'mid/2': 10.4}),
    ([4864], 13824, 128, 0.5, 40, False, {'strip': 80.4, 'mid': 59.6, 'b1': 74.9, 'mid/3': 39.9}),
    ([1472], 1472, 64, 0.5, 33, False, {'strip': 6.8, 'mid': 8.6, 'b1': 8.8, 'strip/2': 5.8}),
]


def _schedule(N, K, tile, f, M, workspace):
    """-> [(kernel, K chunks, deals of the rows) of every pass]; kernel 0 strip, 1 mid, 2 batch, 3 / 4 prefill (4: in blocks of 128 rows)."""
    kernel, chunks, deals = (ctypes.c_int * 8)(), (ctypes.c_int * 8)(), (ctypes.c_int * 8)()
    n = B.lib().patch_test_schedule_deals(ctypes.c_int64(M), len(N), (ctypes.c_int64 * len(N))(*N), ctypes.c_int64(K), tile, round(100 * f),
                                    ctypes.c_size_t(384 << 20 if workspace else 0), kernel, chunks, deals)
    assert n > 0
    return [(kernel[i], chunks[i], deals[i]) for i in range(n)]


@pytest.mark.parametrize("N,K,tile,f,M,workspace,us", MEASURED)
def test_choice_is_no_slower_than_what_was_measured(N, K, tile, f, M, workspace, us):
    passes = _schedule(N, K, tile, f, M, workspace)
    (k, c, deals), *rest = passes
    chosen = "two passes" if rest else ("strip", "mid" if c == 1 else "mid*", f"b{c}", "prefill", "prefill")[k] + (f"/{deals}" if deals > 1 else "")
    assert chosen in us, (chosen, us)
    assert us[chosen] <= 1.03 * min(us.values()) + 0.3, (chosen, us)


@pytest.mark.parametrize("deals", [1, 2, 3, 4])
def test_deals_of_a_feature_group_meet_in_one_die(deals):
    """256 compute units on eight dies that take workgroups in turn: a dealt launch over `units` feature groups is made a multiple of 8 wide, so that
    a group's workgroups are multiples of 8 apart, unless the fullest die would then need more rounds than the launch as it is."""
    for units in range(1, 300):
        width = B.lib().patch_test_deal_units(units, deals, 256)
        fullest = max(deals * len(range(die, units, 8)) for die in range(8))
        rounds, fits = -(-units * deals // 256), -(-fullest // 32)
        assert width == (units if deals == 1 or fits > rounds else -(-units // 8) * 8), (units, deals)


@pytest.mark.parametrize("N,K,M,us", [
    (5120, 5120, 129, {128: 22.6, 256: 27.0}), (5120, 5120, 160, {128: 23.2, 256: 27.7}), (6912, 3456, 192, {128: 23.3, 256: 27.3}),
    (4096, 4096, 1003, {128: 43.0, 256: 46.2}), (11008, 4096, 300, {128: 52.8, 256: 48.1}), (13824, 5120, 300, {128: 65.6, 256: 60.6}),
    (11008, 4096, 1003, {128: 106.7, 256: 67.9}),
])
def test_block_height_of_mask_tile_64(N, K, M, us):
    """A prefill launch on mask tile 64, f = 1/2, with a workspace: blocks of 128 rows or the 256-row register-weight kernel."""
    (k, _, _), = _schedule([N], K, 64, 0.5, M, True)
    assert us[{4: 128, 3: 256}[k]] == min(us.values())


# the 4-bit storage: patch_gemm4_ex (one weight), patch_gemm4_many; the passes of a call joined by "+"
MEASURED4 = [
    ([49152], 2048, 64, 0.0, 12, False, {'strip': 17.1, 'b1': 19.3}),
    ([36864], 4096, 128, 0.0, 16, False, {'strip': 22.3, 'b1': 29.9}),
    ([1024], 8192, 128, 0.0, 193, False, {'strip+strip+strip+strip': 100.8, 'prefill': 120.5}),
    ([128256], 1024, 64, 1.0, 64, False, {'prefill': 33.3, 'b1': 36.8}),
    ([36864], 4096, 128, 0.0, 32, False, {'strip': 40.3, 'b1': 34.5}),
    ([5120], 13824, 128, 1.0, 193, False, {'prefill': 148.3, 'strip+strip+strip+strip': 169.6}),
    ([512], 13824, 64, 0.0, 9, True, {'strip': 12.6, 'b8': 12.7}),
    ([32000], 4096, 64, 0.0, 2, True, {'strip': 18.0, 'b1': 22.6}),
    ([256], 1024, 128, 0.0, 96, True, {'strip+strip': 10.3, 'prefill': 13.4}),
    ([512], 13824, 64, 0.5, 9, True, {'strip': 11.9, 'b8': 12.3}),
    ([32000], 4096, 128, 1.0, 80, True, {'prefill': 34.8, 'b1+b1': 42.7}),
    ([11008] * 2, 4096, 128, 0.0, 12, False, {'strip': 16.6, 'b1': 20.0}),
    ([11008] * 2, 4096, 64, 0.0, 16, False, {'strip': 17.4, 'b1': 21.8}),
    ([49152], 2048, 128, 0.0, 17, False, {'strip': 23.5, 'b1': 18.6}),
    ([896], 896, 64, 0.0, 256, False, {'strip+strip+strip+strip': 22.6, 'prefill': 17.3}),
    ([32000], 4096, 128, 0.5, 64, False, {'prefill': 58.1, 'b1': 29.3}),
    ([32000], 4096, 64, 0.5, 65, False, {'prefill': 62.2, 'b1+strip': 48.4}),
    ([128256], 1024, 64, 1.0, 16, False, {'strip': 18.1, 'b1': 17.1}),
    ([13824], 5120, 64, 1.0, 80, False, {'strip+strip': 54.7, 'b1+strip': 46.3}),
    ([5120], 13824, 128, 0.0, 16, True, {'strip': 21.0, 'b6': 15.6}),
    ([896], 896, 64, 0.0, 256, True, {'strip+strip+strip+strip': 22.7, 'prefill': 17.5}),
    ([896], 4864, 128, 0.5, 33, True, {'strip': 12.5, 'b8': 9.3}),
    ([256], 1024, 64, 0.5, 160, True, {'strip+strip+strip': 16.1, 'prefill': 13.5}),
    ([896], 4864, 128, 1.0, 33, True, {'strip': 12.2, 'b8': 8.8}),
    ([4864], 896, 64, 1.0, 129, True, {'strip+strip+strip': 15.7, 'prefill': 14.5}),
    ([13824] * 2, 5120, 128, 0.0, 48, False, {'strip': 59.6, 'b1': 32.4}),
    ([13824] * 2, 5120, 128, 0.5, 16, False, {'strip': 26.3, 'b1': 23.2}),
    ([28672] * 2, 4096, 64, 1.0, 64, False, {'strip': 90.0, 'b1': 53.9}),
    # launches just past or just below a whole number of workgroups per compute unit, and K chunks at 11 - 36 rows
    ([32896], 4096, 128, 0.5, 24, False, {'strip': 34.6, 'b1': 30.0}),
    ([24576], 4096, 64, 1.0, 20, False, {'strip': 16.7, 'b1': 21.4}),
    ([49152], 2048, 64, 0.0, 14, False, {'strip': 16.9, 'b1': 19.0}),
    ([49152], 2048, 64, 0.0, 20, False, {'strip': 24.2, 'b1': 20.8}),
    ([28672] * 2, 4096, 64, 0.5, 1, False, {'strip': 25.5, 'b1': 33.8}),
    ([16384], 4096, 64, 0.0, 33, False, {'strip': 24.0, 'b1': 27.2}),
    ([512], 13824, 128, 1.0, 11, True, {'strip': 13.1, 'b8': 10.4}),
    ([4096], 11008, 128, 1.0, 12, True, {'strip': 13.0, 'b8': 10.8}),
    ([4096], 4096, 64, 1.0, 36, True, {'strip': 12.1, 'b8': 10.1}),
]


@pytest.mark.parametrize("N,K,tile,f,M,workspace,us", MEASURED4)
def test_choice_from_the_4_bit_storage(N, K, tile, f, M, workspace, us):
    kernel, chunks = (ctypes.c_int * 8)(), (ctypes.c_int * 8)()
    n = B.lib().patch_test_schedule4(ctypes.c_int64(M), len(N), (ctypes.c_int64 * len(N))(*N), ctypes.c_int64(K), tile, round(100 * f),
                                     ctypes.c_size_t(384 << 20 if workspace else 0), kernel, chunks)
    assert n > 0
    chosen = "prefill" if kernel[0] > 1 else "+".join("strip" if kernel[i] == 0 else f"b{chunks[i]}" for i in range(n))
    assert chosen in us, (chosen, us)
    assert us[chosen] <= 1.03 * min(us.values()) + 0.3, (chosen, us)


def test_limits_of_the_4_bit_prefill_choice():
    """K slices: at most 8 of at least 512 columns, partial sums that the workspace holds; of the last round alone, blocks that fill the chip at most once behind
    one to four full rounds, slots of 128 KB."""
    kernel, chunks, taken = (ctypes.c_int * 8)(), (ctypes.c_int * 8)(), set()
    for tile in (64, 128):
        for N in (640, 1024, 4096, 11008):
            for K in (384, 1024, 4096, 13824):
                for M in (129, 300, 600, 800, 1536, 2100, 4096, 10968, 20000):
                    for f in (0.0, 0.5, 1.0):
                        for slices in (0, 2, 5):
                            ws = 4 * slices * M * N
                            n = B.lib().patch_test_schedule4(ctypes.c_int64(M), 1, (ctypes.c_int64 * 1)(N), ctypes.c_int64(K), tile, round(100 * f), ctypes.c_size_t(ws), kernel, chunks)
                            if n != 1 or kernel[0] < 2:
                                continue
                            k, c = kernel[0], chunks[0]
                            assert 1 <= c <= 8 and (c == 1 or (512 * c <= K and ws > 0))
                            if k == 5:
                                blocks = -(-N // 256) * -(-M // 128)
                                assert c > 1 and 256 < blocks < 5 * 256 and 2 * (blocks % 256) <= 256 and c * (blocks % 256) <= 256
                                assert c * (blocks % 256) * (128 << 10) <= ws
                            else:
                                assert c == 1 or 4 * c * M * N <= ws
                            taken.add((k, c > 1))
    assert {(2, False), (2, True), (4, False), (4, True), (5, True)} <= taken, taken

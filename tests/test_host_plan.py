"""Host logic of the library without a GPU: which chunks of a streamed pass cross the link as tiles."""
import ctypes as C

import pytest


def plan(channels, blocks, H, W, tile, used, num_cu=256, chunk=1024):
    from paper_2509_02447_amd import binding as b
    first, rest, lent = C.c_int32(), C.c_int32(), C.c_int32()
    assert b.load_library().qrm_diag_host_plan(channels, blocks, H, W, tile, chunk, used, num_cu, C.byref(first), C.byref(rest),
                                               C.byref(lent)) == 0
    return first.value, rest.value, lent.value


@pytest.mark.parametrize("channels,blocks,side,tile,rest", [
    (64, 8, 256, 32, 1), (64, 8, 256, 64, 1), (32, 4, 256, 64, 1), (32, 4, 256, 128, 1), (64, 2, 256, 96, 1), (64, 8, 512, 128, 1),
    # the kernels of a chunk take longer than its copy: 4.2 .. 7.3 ms against 3.5 per 1024 images
    (64, 8, 256, 80, 0), (64, 8, 256, 96, 0), (64, 8, 256, 128, 0), (64, 8, 512, 192, 0), (64, 8, 512, 256, 0)])
def test_later_chunks_are_gathered_only_where_the_link_is_the_bound(channels, blocks, side, tile, rest):
    first, got, lent = plan(channels, blocks, side, side, tile, 3)
    assert first == 1 and got == rest
    assert lent in (8, 16) if rest else lent == 0       # kernels keep every compute unit beside a copy


def test_alone_on_the_device_every_chunk_is_gathered():
    for tile in (32, 64, 96, 128):
        assert plan(64, 8, 256, 256, tile, 1) == (1, 1, 0)


def test_large_tiles_are_copied():
    for used in (1, 2, 3):
        assert plan(64, 8, 256, 256, 192, used) == (0, 0, 0) and plan(32, 4, 100, 100, 64, used) == (0, 0, 0)


def test_small_devices_lend_nothing():
    """A device partition of few compute units cannot spare any: only the first chunk, beside which nothing runs, is gathered."""
    for num_cu in (32, 63):
        assert plan(64, 8, 256, 256, 64, 3, num_cu) == (1, 0, 0) and plan(64, 8, 256, 256, 64, 1, num_cu) == (1, 1, 0)
    assert plan(64, 8, 256, 256, 64, 3, 64)[1] == 1


def strips(N, T):
    from paper_2509_02447_amd import binding as b
    got = C.c_int32()
    assert b.load_library().qrm_diag_preprocess_strips(N, T, C.byref(got)) == 0
    return got.value


def test_small_windows_are_not_cut_for_more_than_one_wave():
    """Where cutting further was measured slower: 1024 windows of 64 (2 strips 13.7 us, 8 14.8), 3000 of 30 (1 strip 10.4 us, 2 12.0)."""
    for N, T in ((1024, 64), (3000, 30), (3000, 48), (1000, 32), (2048, 64), (5000, 17)):
        assert strips(N, T) <= max(1, 2048 // N), (N, T)


def test_large_windows_get_several_waves_of_strips():
    for N, T, least in ((600, 256, 12), (300, 256, 14), (700, 256, 10), (150, 384, 24), (1, 256, 32), (20000, 32, 1)):
        assert least <= strips(N, T) <= (T + 7) // 8, (N, T)
    for N in (1, 7, 255, 256, 300, 1024, 2047, 2048, 2049, 8192, 8193, 1 << 31):      # no strip is empty
        for T in (1, 2, 3, 4, 7, 8, 9, 17, 31, 32, 33, 100, 255, 256, 1000, 1024):
            c = strips(N, T)
            rows = -(-T // c)
            assert 1 <= c <= (T + 7) // 8 and (c - 1) * rows < T <= c * rows, (N, T)


@pytest.mark.parametrize("n,k,few,many", [
    (255, 251, 32, 16), (255, 253, 32, 16), (255, 247, 32, 16), (129, 121, 32, 16), (128, 120, 16, 16), (63, 55, 16, 16),
    (15, 7, 16, 16), (255, 239, 32, 32), (31, 15, 32, 32), (12, 8, 1, 1), (15, 13, 1, 1), (17, 13, 16, 16)])
def test_few_long_words_are_dealt_to_more_lanes(n, k, few, many):
    """10240 words of RS(255,247) take 10.2 us on 16 lanes a word and 9.8 on 32; 16000 take 10.7 and 12.2."""
    from paper_2509_02447_amd import binding as b
    lanes = C.c_int32()
    for N, want in ((1, few), (300, few), (4096, few), (10240, few), (10241, many), (20000, many), (1 << 20, many)):
        assert b.load_library().qrm_diag_rs_lanes(n, k, N, C.byref(lanes)) == 0
        assert lanes.value == want, N

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

"""Which batches go through all blocks in one launch (qrm_diag_chain_rule): host code, no device needed."""
import ctypes as C

import pytest

from paper_2509_02447_amd import binding


def rule(channels, blocks, n, h, w, num_cu=256):
    fits, taken = C.c_int32(), C.c_int32()
    assert binding.load_library().qrm_diag_chain_rule(channels, blocks, n, h, w, num_cu, fits, taken) == 0
    return bool(fits.value), bool(taken.value)


@pytest.mark.parametrize("case,taken", [
    ((32, 4, 16, 32, 32), True), ((32, 4, 256, 32, 32), True), ((32, 4, 390, 29, 12), True), ((64, 8, 7, 128, 128), True),
    ((32, 4, 2, 128, 128), False), ((64, 8, 4, 128, 128), False),   # an XCD has one image or none, of many items
    ((64, 8, 1, 64, 64), False), ((64, 8, 300, 16, 33), False),     # narrow tiles of 64 channels: fused pairs
    ((32, 2, 272, 29, 12), False), ((32, 2, 147, 207, 10), False), ((32, 3, 139, 43, 13), False), ((32, 3, 22, 192, 82), False),  # 1.03 .. 1.1 times as long
    ((64, 8, 2048, 64, 64), False), ((32, 4, 4096, 32, 32), False), ((32, 2, 4, 250, 250), False)])
def test_the_rule_takes_what_is_faster_so(case, taken):
    assert rule(*case)[1] == taken
    if taken:
        assert rule(*case)[0]


@pytest.mark.parametrize("channels", [32, 64])
def test_what_does_not_fit_is_not_taken(channels):
    """Counters for 2048 images times blocks, a workgroup of the head per image up to 512, lines in the place of an image's activations,
    at least two blocks."""
    assert rule(channels, 4, 512, 32, 32)[0] and not rule(channels, 4, 513, 32, 32)[0]
    assert rule(channels, 8, 256, 32, 32)[0] and not rule(channels, 8, 257, 32, 32)[0]
    assert not rule(channels, 1, 16, 32, 32)[0]
    assert not rule(channels, 65, 16, 32, 32)[0]
    assert not rule(channels, 4, 16, 2, 2)[0]
    for n in range(1, 600, 7):
        for side in (3, 5, 16, 33, 64, 100, 256):
            fits, taken = rule(channels, 4, n, side, side)
            assert fits or not taken


def test_bad_arguments_are_refused():
    f, t = C.c_int32(), C.c_int32()
    lib = binding.load_library()
    assert lib.qrm_diag_chain_rule(48, 4, 1, 8, 8, 256, f, t) != 0 and lib.qrm_diag_chain_rule(32, 0, 1, 8, 8, 256, f, t) != 0
    assert lib.qrm_diag_chain_rule(32, 4, 1, 8, 8, 0, f, t) != 0 and lib.qrm_diag_chain_rule(32, 4, 1, 8, 8, 256, None, t) != 0

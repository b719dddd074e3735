"""Host logic of the library without a GPU: how a fused launch deals its row pairs to workgroups, and which schedule wide
tiles take."""
import ctypes as C
import random

import pytest

CU = 256


@pytest.fixture(scope="module")
def split():
    from paper_2509_02447_amd import binding as b
    lib = b.load_library()

    def call(n, h, w, last):
        part, per, cost = C.c_int32(), C.c_int32(), C.c_int32()
        assert lib.qrm_diag_pair_split(n, h, w, last, CU, C.byref(part), C.byref(per), C.byref(cost)) == 0
        return part.value, per.value, cost.value
    return call


def longest_walk(n_img, h, w, last, per):
    """Cost of the longest workgroup, counted by walking through its stream of positions one at a time."""
    S, J, quant = (h + 1) // 2, -(-w // 64), 4 if last else 1
    ppi = -(-S // quant)
    longest = 0
    for q0 in range(0, n_img * ppi, per):
        q1 = min(n_img * ppi, q0 + per)
        units = []                                # (first, behind the last row pair) of each unit of the run
        for n in range(q0 // ppi, (q1 - 1) // ppi + 1):
            lo, hi = max(q0, n * ppi) - n * ppi, min(q1, (n + 1) * ppi) - n * ppi
            units += [(lo * quant, min(S, hi * quant))] * J
        steps = 2                                 # the second block and its epilogue run two positions behind
        pairs = 0                                 # row pairs multiplied by the first and by the second block
        for lo, hi in units:
            steps += 1                            # opening position (of the first unit: the one behind the last unit)
            for j in range(lo - (lo > 0), hi + (hi < S)):
                steps += 1
                pairs += 2 if lo <= j < hi else 1  # a halo pair is not the second block's
        longest = max(longest, 8 * steps + pairs)
    return longest


def runs_per(n_img, h, last):
    pieces = n_img * -(-((h + 1) // 2) // (4 if last else 1))
    return -(-pieces // CU)


def whole_per(n_img, h, last):
    return -(-n_img // CU) * -(-((h + 1) // 2) // (4 if last else 1))


def check(split, n, h, w, last):
    part, per, cost = split(n, h, w, last)
    whole, runs = (longest_walk(n, h, w, last, f(n, h, last)) for f in (whole_per, runs_per))
    assert per == (runs_per if part else whole_per)(n, h, last)
    assert cost == (runs if part else whole), (n, h, w, last)
    assert bool(part) == (103 * runs < 100 * whole), (n, h, w, last, whole, runs)
    assert cost <= whole


@pytest.mark.parametrize("n,h,w", [(192, 8, 64), (224, 16, 64), (240, 32, 64), (480, 16, 128), (245, 64, 64)])
def test_whole_images_where_runs_would_be_longer(split, n, h, w):
    for last in (0, 1):
        assert split(n, h, w, last)[0] == 0
        check(split, n, h, w, last)


@pytest.mark.parametrize("n,h,w", [(1, 64, 64), (7, 128, 128), (300, 64, 64), (333, 64, 64), (140, 32, 64), (40, 5, 64), (160, 16, 64), (200, 128, 128)])
def test_runs_where_whole_images_leave_compute_units_idle(split, n, h, w):
    assert split(n, h, w, 0)[0] == 1
    for last in (0, 1):
        check(split, n, h, w, last)


def test_cost_of_the_longest_workgroup(split):
    rng = random.Random(5)
    for _ in range(300):
        check(split, rng.choice([1, 2, rng.randint(1, 40), rng.randint(1, 1200)]), rng.randint(1, 140), rng.randint(1, 260),
              rng.randint(0, 1))
    check(split, 5, 1, 1, 0)
    check(split, 5, 2, 1, 1)


def schedule(n, h, w, num_cu=256):
    fused, single_us, fused_us = C.c_int32(), C.c_double(), C.c_double()
    from paper_2509_02447_amd import binding as b
    st = b.load_library().qrm_diag_wide_schedule(n, h, w, num_cu, C.byref(fused), C.byref(single_us), C.byref(fused_us))
    assert st == 0
    return bool(fused.value), single_us.value, fused_us.value


# microseconds of eight blocks on a chip of 256 compute units, measured at commit eefb1c9, whose kernels the estimates are fitted to:
# (tiles, height, width, single blocks, fused)
SCHEDULES = [(256, 8, 100, 191, 144), (256, 4, 160, 166, 128), (256, 12, 80, 233, 186), (256, 16, 66, 274, 225),
             (256, 20, 200, 621, 540), (200, 4, 200, 185, 154), (200, 30, 200, 741, 681), (200, 30, 160, 576, 516),
             (700, 4, 100, 259, 216), (700, 8, 256, 798, 704), (400, 4, 100, 186, 158),
             (128, 24, 66, 203, 216), (128, 20, 66, 183, 192), (128, 36, 66, 268, 278), (160, 20, 128, 254, 265)]


@pytest.mark.parametrize("n,h,w,single_us,fused_us", SCHEDULES)
def test_wide_tiles_take_the_faster_schedule(n, h, w, single_us, fused_us):
    """Tiles wider than 64 columns: the estimates are near what they are fitted to (their standard deviation is 3.5 %, twice
    of which is the largest seen; shapes further off are not listed) and pick the way that was the faster one there."""
    fused, est_single, est_fused = schedule(n, h, w)
    assert fused == (fused_us < single_us)
    assert abs(est_single / single_us - 1) < 0.15 and abs(est_fused / fused_us - 1) < 0.1


def test_wide_tiles_schedule_limits():
    for h, w in ((5, 66), (30, 128), (128, 200), (256, 256)):
        assert not schedule(1, h, w)[0] and not schedule(127, h, w)[0]    # fewer images than half the compute units
        n = -(-12 * 256 // ((h + 1) // 2))                                # from 12 row pairs per compute unit on
        assert schedule(max(128, n), h, w)[0] and schedule(5000, h, w)[0]
    f, s, u = C.c_int32(), C.c_double(), C.c_double()
    from paper_2509_02447_amd import binding as b
    assert b.load_library().qrm_diag_wide_schedule(10, 10, 64, 256, C.byref(f), C.byref(s), C.byref(u)) != 0


def last_lines(n, h, w, blocks=4):
    from paper_2509_02447_amd import binding as b
    pairs, size = C.c_int32(), C.c_int64()
    assert b.load_library().qrm_diag_last_lines(n, h, w, blocks, CU, C.byref(pairs), C.byref(size)) == 0
    return pairs.value, size.value


@pytest.mark.parametrize("w", [1, 2, 3, 4, 5, 6, 8, 16, 33, 64])
@pytest.mark.parametrize("h", [1, 2, 7, 16, 33, 64, 75, 128])
def test_a_smaller_batch_needs_no_larger_workspace(h, w):
    """Launches of few tiles leave four times as many lines of sums; a stream that has served a batch serves every smaller one
    without a new workspace."""
    sizes = [last_lines(n, h, w)[1] for n in range(1, 300)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:])), (h, w)


def test_a_line_per_row_pair_means_runs(split):
    """Launches that leave a line per row pair deal their row pairs in runs: there is no kernel for whole images with such lines."""
    fine = 0
    for h in range(1, 200):
        for n in range(1, 256):
            if n * -(-((h + 1) // 2) // 4) < CU and last_lines(n, h, 64)[0] == 1:
                fine += 1
                assert split(n, h, 64, 0)[0] == 1, (n, h)
    assert fine > 1000

"""The benchmark's recorded traffic figures: they hold for the kernels and launch sizes that they were taken on, no others."""
import os

import bench


def test_a_record_holds_for_its_kernels_and_launch_size_only():
    for key in [k for k in bench.RECORDED_TRAFFIC if isinstance(k, tuple)]:
        images, nbytes = bench.RECORDED_TRAFFIC[key]
        assert bench.recorded_traffic(*key, images, bench.RECORDED_TRAFFIC["kernels"]) == nbytes
        assert bench.recorded_traffic(*key, images + 1, bench.RECORDED_TRAFFIC["kernels"]) is None
        assert bench.recorded_traffic(*key, images, "000000000000") is None
    assert bench.recorded_traffic("C2", "head", 1024, bench.RECORDED_TRAFFIC["kernels"]) is None


def test_the_kernels_key_follows_the_code_and_not_its_comments():
    path = os.path.join(bench.ROOT, "paper_2509_02447_amd", "csrc", "extractor.hip")
    texts = [open(path).read(), "int a;"]
    key = bench.kernel_source_key(texts)
    assert bench.kernel_source_key([texts[0] + "\n// a remark\n", texts[1]]) == key
    assert bench.kernel_source_key([texts[0].replace("kChunk = 4", "kChunk = 8"), texts[1]]) != key
    assert bench.kernel_source_key([texts[0], "int b;"]) != key
    assert len(bench.kernel_source_key()) == 12

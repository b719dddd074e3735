"""The benchmark's recorded traffic figures: they hold for the kernels and launch sizes that they were taken on, no others."""
import os
import subprocess

import pytest

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


def test_the_record_names_the_commit_whose_kernels_it_was_taken_on():
    """The key is that of the sources at the commit named, and the summary names the same commit."""
    commit, csrc = bench.RECORDED_TRAFFIC["commit"], "paper_2509_02447_amd/csrc/"
    path = os.path.join(bench.ROOT, bench.RECORDED_TRAFFIC["source"])
    if os.path.exists(path):
        assert f"sources at commit {commit}" in open(path).readline()
    git = ["git", "-C", bench.ROOT]
    if subprocess.run(git + ["cat-file", "-e", commit], capture_output=True).returncode:
        pytest.skip("the history is not here")
    texts = [subprocess.run(git + ["show", f"{commit}:{csrc}{f}"], capture_output=True, text=True, check=True).stdout
             for f in ("extractor.hip", "qrm_internal.h")]
    assert bench.kernel_source_key(texts) == bench.RECORDED_TRAFFIC["kernels"]

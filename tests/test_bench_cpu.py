"""bench.py's own rules: which kernel a class runs, and when a committed counter summary is out of date."""
import dataclasses
import os
import shutil

import pytest

import bench
from paper_2206_09878_amd.workloads import workload


def grid(n1, n2, n3, order=8):
    return dataclasses.replace(workload("small", n=n1, n2=n2), n3=n3, m3=3 * n3 // 2, order=order)


@pytest.mark.parametrize("name", ["lmvd.hip", "tile.h", "fft_reg.h", "fft_lds.h", "substep_adjoint.h"])
def test_digest_covers_the_device_code(tmp_path, name):
    src = os.path.join(os.path.dirname(bench.__file__), "paper_2206_09878_amd", "csrc")
    shutil.copytree(src, tmp_path / "csrc")
    assert bench.source_digest(str(tmp_path / "csrc")) == bench.source_digest()
    with open(tmp_path / "csrc" / name, "a") as f:
        f.write("// changed\n")
    assert bench.source_digest(str(tmp_path / "csrc")) != bench.source_digest()


@pytest.mark.parametrize("cls,w,tiles", [
    ("flux", grid(64, 256, 64), True), ("flux", grid(64, 257, 64), False), ("mc", grid(64, 257, 64), True),
    ("mc", grid(16, 592, 12), True), ("mc", grid(16, 593, 12), False), ("proj", grid(16, 593, 12), False),
    ("mc", grid(256, 129, 256), True), ("md", grid(256, 213, 256), True), ("flux", grid(256, 213, 256), False),
    ("mc", grid(512, 129, 512), False), ("proj", grid(512, 385, 512), False), ("mc", grid(16, 10, 16), False),
    ("mc", grid(16, 17, 16, order=9), False)])
def test_kernel_symbol_follows_the_rows(cls, w, tiles):
    assert ("_tile" in bench.kernel_symbol(cls, w)) == tiles

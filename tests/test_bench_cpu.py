"""bench.py's own rules: when a committed counter summary is out of date."""
import os
import shutil

import pytest

import bench


@pytest.mark.parametrize("name", ["lmvd.hip", "tile.h", "fft_reg.h", "fft_lds.h", "substep_adjoint.h"])
def test_digest_covers_the_device_code(tmp_path, name):
    src = os.path.join(os.path.dirname(bench.__file__), "paper_2206_09878_amd", "csrc")
    shutil.copytree(src, tmp_path / "csrc")
    assert bench.source_digest(str(tmp_path / "csrc")) == bench.source_digest()
    with open(tmp_path / "csrc" / name, "a") as f:
        f.write("// changed\n")
    assert bench.source_digest(str(tmp_path / "csrc")) != bench.source_digest()

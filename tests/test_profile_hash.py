"""The hash that ties profiled counters to the kernels they were taken on covers
every source of the product's kernels: a change to any of them changes it."""
import os
import shutil

import pytest

import profile_tools
from paper_2501_13512_amd import build

FILES = build.OBJECTS["mvm"] + ["zconv.h", "zpass.h", "fft_core.h", "cx.h", "kernels.h"]


@pytest.mark.parametrize("name", FILES)
def test_any_source_changes_the_hash(tmp_path, monkeypatch, name):
    src = tmp_path / "csrc"
    shutil.copytree(profile_tools.CSRC, src)
    monkeypatch.setattr(profile_tools, "CSRC", str(src))
    before = profile_tools.kernel_hash()
    with open(os.path.join(src, name), "a") as f:
        f.write("// changed\n")
    assert profile_tools.kernel_hash() != before

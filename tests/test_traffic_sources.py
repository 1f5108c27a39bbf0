"""The hash that ties a counter record to the kernel sources covers every file
that the measured kernels are compiled from."""
import os
import re
import shutil

import pytest

import bench
from paper_2201_10132_amd import profile_summary

ROOT, CSRC = bench.ROOT, os.path.join("paper_2201_10132_amd", "csrc")


def _included(name):
    """name and the project's headers that it includes, recursively."""
    text = open(os.path.join(ROOT, CSRC, name)).read()
    out = {name}
    for h in re.findall(r'#include "([^/"]+)"', text):
        out |= _included(h)
    return out


@pytest.mark.parametrize("module", [bench, profile_summary])
def test_every_source_of_the_step_changes_the_hash(module, tmp_path, monkeypatch):
    files = _included("tpl_kernels.hip")
    assert {"tpl_kernels.hip", "tpl_step.h", "tpl_internal.h"} <= files
    before = module.kernel_source_sha()
    for name in files:
        root = tmp_path / name
        shutil.copytree(os.path.join(ROOT, CSRC), root / CSRC)
        monkeypatch.setattr(module, "ROOT", str(root))
        assert module.kernel_source_sha() == before
        with open(root / CSRC / name, "a") as f:
            f.write("// a change")
        assert module.kernel_source_sha() != before, name

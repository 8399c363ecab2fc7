"""The counters that bench.py reports count for the kernels' sources as they were measured."""

import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_14442_amd", "csrc")


@pytest.fixture
def bench(monkeypatch):
    monkeypatch.syspath_prepend(ROOT)
    import bench as module

    yield module
    sys.modules.pop("bench", None)


def test_hash_covers_what_the_kernels_include(bench):
    for name in set(bench.KERNEL_SOURCES) - {"abi.hip"}:  # host code, which launches other kernels too
        with open(os.path.join(CSRC, name), encoding="utf-8") as f:
            local = {i for i in re.findall(r'#include "(\w+\.\w+)"', f.read())}  # ../../include: the C ABI
        assert local <= set(bench.KERNEL_SOURCES), (name, local - set(bench.KERNEL_SOURCES))

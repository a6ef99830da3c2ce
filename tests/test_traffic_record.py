"""Host-only: the sources that each kernel's traffic figures are tied to are all
the sources its code comes from."""

import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_03893_amd", "csrc")
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def includes(name, seen):
    if name not in seen:
        seen.add(name)
        for inc in re.findall(r'#include "(kvx_\w+\.(?:h|hip))"', open(os.path.join(CSRC, name)).read()):
            includes(inc, seen)
    return seen


@pytest.mark.parametrize("kernel", sorted(bench.KERNEL_SOURCES))
def test_hash_covers_every_include(kernel):
    sources = bench.KERNEL_SOURCES[kernel]
    assert set(sources) == includes(sources[0], set())

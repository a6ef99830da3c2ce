"""Host-only: the sources that each kernel's traffic figures are tied to are all
the sources its code comes from."""

import json
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


def test_recorded_counters_are_of_the_current_sources():
    """bench.py drops a record of other sources in silence: such a record says so.
    Every record says which run and form it counted."""
    rec = json.load(open(bench.TRAFFIC_FILE))
    for workload, kernels in rec.items():
        for kernel, ent in kernels.items():
            current = ent["kernel_hash"] == bench.kernel_hash(kernel)
            assert ent["note"] and (current or "earlier source" in ent["note"]), f"{workload}: {kernel}"
            assert kernel in ent["kernel"]

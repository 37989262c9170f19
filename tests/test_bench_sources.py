"""The counter figures that bench.py takes from a committed summary are void once a source of the kernels changes: each
kernel family names every file that it is compiled from."""

import os
import re

import pytest

import bench
from paper_2301_12836_amd import build


def text(name):
    with open(os.path.join(build.CSRC, name)) as f:
        return f.read()


def compiled_from(name, seen=()):
    """A source and the headers under csrc/ that it includes, directly or not."""
    files = {name}
    for inc in re.findall(r'#include "(\w+\.h)"', text(name)):
        if inc not in seen:
            files |= compiled_from(inc, (*seen, name))
    return files


@pytest.mark.parametrize("prefix", sorted(bench.FAMILY_SOURCES))
def test_families_name_all_their_sources(prefix):
    sources = [f for f in os.listdir(build.CSRC) if f.endswith(".hip") and re.search(r'LS_PNAME\(T, "%s' % prefix, text(f))]
    assert sources
    assert set().union(*(compiled_from(f) for f in sources)) <= set(bench.FAMILY_SOURCES[prefix])

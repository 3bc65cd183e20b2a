"""The sources whose hash decides whether a stored byte count of `bench.py` still
describes the kernels: every header of the library that a group's kernels
include has to be among them."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_1905_06700_amd", "csrc")


def includes(name):
    with open(os.path.join(CSRC, name)) as f:
        return set(re.findall(r'^#include "(rt3d_\w+\.h)"', f.read(), re.M))


def test_every_included_header_is_hashed():
    for group, files in bench.GROUP_SOURCES.items():
        have = set(files) | {"rt3d_dev.h"}
        for name in have:
            missing = includes(name) - have
            assert not missing, (group, name, missing)

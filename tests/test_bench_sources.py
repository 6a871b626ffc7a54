"""Committed counters count as current only while every source of the kernel is
the one they were taken on: the hash covers the traversal and the headers beside
it that it includes."""
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = "paper_2210_12859_amd/csrc/"


def test_hash_covers_the_included_headers():
    need, todo = set(), ["kd_traverse.hip"]
    while todo:
        f = todo.pop()
        if f in need:
            continue
        need.add(f)
        src = open(os.path.join(ROOT, CSRC, f)).read()
        todo += re.findall(r'^#include "([^/"]+)"', src, flags=re.M)
    assert need == {os.path.basename(p) for p in bench.TRAVERSE_SOURCES}

"""Committed counter traffic is quoted by bench.py only while the kernels are the
ones it was taken on: an edit to any source that defines a kernel in
KERNEL_KEYS, or to a header it includes, changes the hash that says so.
"""
import os
import re
import shutil

import pytest

import bench

CSRC = os.path.join("paper_1709_01126_amd", "csrc")


def sources():
    folder = os.path.join(bench.ROOT, CSRC)
    names = {f[:-1] for _, frags in bench.KERNEL_KEYS.values() for f in frags if f.endswith("<")}
    names |= {"stencil_march", "stencil_wave"}   # named by their modes alone
    text = {n: open(os.path.join(folder, n)).read() for n in os.listdir(folder)}
    found = {n for n, s in text.items() for k in names if re.search(rf"^{k}\(", s, re.M)}
    assert all(any(re.search(rf"^{k}\(", s, re.M) for s in text.values()) for k in names)
    return sorted(found | {"stencil_ops.hpp", "solver.hpp"})


@pytest.mark.parametrize("name", sources())
def test_hash_follows_every_kernel_source(name, tmp_path, monkeypatch):
    shutil.copytree(os.path.join(bench.ROOT, CSRC), tmp_path / CSRC)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    before = bench.kernel_source_hash()
    with open(tmp_path / CSRC / name, "a") as f:
        f.write("// edited\n")
    assert bench.kernel_source_hash() != before

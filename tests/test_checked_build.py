"""Checked builds (libpot3d_checked.so) name the file and line of an index out
of range.  Each source file keeps its own record; every file whose kernels test
indices has to be asked for it, under its own name.
"""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1709_01126_amd", "csrc")


def test_every_checked_source_is_reported_by_name():
    sources = {n: open(os.path.join(CSRC, n)).read() for n in sorted(os.listdir(CSRC)) if n.endswith(".hip")}
    checked = {n for n, s in sources.items() if re.search(r"\bCHK\(", s)}
    assert {"kernels.hip", "onchip.hip", "line.hip"} <= checked
    asked = dict(re.findall(r'Source\{"(\w+\.hip)", (\w+)\}', sources["kernels.hip"]))
    assert set(asked) == checked
    for name, reader in asked.items():   # defined in the file it stands for (or that file's own read_oob_line)
        assert reader == "read_oob_line" if name == "kernels.hip" else re.search(rf"unsigned {reader}\(\)", sources[name])
    for name, s in sources.items():
        assert not re.search(r'index at \w+\.hip', s), f"{name}: a message that names one file for all"

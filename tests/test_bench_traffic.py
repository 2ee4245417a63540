"""The stamp of the committed traffic summaries: it covers every source that decides what a projection's
launch moves, so a summary of other code is not reported as this code's."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2609_25405_amd", "csrc")
KERNELS = ("gemm.hip", "gemm_big.hip")


def hashed():
    return {os.path.basename(f) for f in bench.KERNEL_SOURCES}


def test_stamp_covers_kernels_and_their_includes():
    todo, need = list(KERNELS), set()
    while todo:
        f = todo.pop()
        if f in need:
            continue
        need.add(f)
        with open(os.path.join(CSRC, f), encoding="utf-8") as fh:
            todo += [i for i in re.findall(r'#include "([^"]+)"', fh.read()) if os.path.exists(os.path.join(CSRC, i))]
    assert need <= hashed(), need - hashed()
    assert "step.hip" in hashed()      # chooses splits, row groups and GemmArgs::wide


def test_changed_copy_policy_changes_the_stamp(tmp_path, monkeypatch):
    before = bench.kernel_source_hash()
    copies = []
    for f in bench.KERNEL_SOURCES:
        with open(f, encoding="utf-8") as fh:
            text = fh.read()
        copies.append(str(tmp_path / os.path.basename(f)))
        with open(copies[-1], "w", encoding="utf-8") as fh:
            fh.write(text.replace("kNonTemporal = 2", "kNonTemporal = 0"))
    monkeypatch.setattr(bench, "KERNEL_SOURCES", copies)
    assert bench.kernel_source_hash() != before


def test_changed_comment_keeps_the_stamp(tmp_path, monkeypatch):
    before = bench.kernel_source_hash()
    copies = []
    for f in bench.KERNEL_SOURCES:
        with open(f, encoding="utf-8") as fh:
            text = fh.read()
        copies.append(str(tmp_path / os.path.basename(f)))
        with open(copies[-1], "w", encoding="utf-8") as fh:
            fh.write("// another comment\n" + text)
    monkeypatch.setattr(bench, "KERNEL_SOURCES", copies)
    assert bench.kernel_source_hash() == before

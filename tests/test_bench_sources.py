"""Counter summaries that bench.py reports count as current only for the sources
their kernels are built from (CPU)."""
import os
import re
import shutil

import pytest

import bench

CSRC = os.path.join("paper_2607_12422_amd", "csrc")


@pytest.mark.parametrize("sources", [bench.FUSED_SOURCES, bench.ATTN_SOURCES, bench.GEMM_SOURCES])
def test_every_included_source_counts(sources, tmp_path, monkeypatch):
    """A summary is dropped when any file changes that the kernel's source
    includes, directly or not."""
    todo, seen = [s for s in sources if s.endswith(".hip")], set()
    while todo:
        name = todo.pop()
        path = os.path.join(bench.ROOT, CSRC, name)
        if name in seen or not os.path.exists(path):
            continue
        seen.add(name)
        todo += re.findall(r'#include "([\w.]+)"', open(path).read())
    assert seen == set(sources)
    shutil.copytree(os.path.join(bench.ROOT, CSRC), tmp_path / CSRC)
    (tmp_path / "profiles").mkdir()
    summary = tmp_path / "profiles" / "s.txt"
    summary.write_text(f"kernel_source_sha256: {bench.source_sha256(sources)}\ntraffic_bytes_per_launch: 7\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    for name in sources:
        assert bench.counter_traffic("s.txt", sources) == 7
        changed = tmp_path / CSRC / name
        text = changed.read_text()
        changed.write_text(text + "\n")
        assert bench.counter_traffic("s.txt", sources) is None, name
        changed.write_text(text)

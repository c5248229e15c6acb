"""Host: the hash that dates the stored counter readings covers every source of the level kernels."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2507_02401_amd", "csrc")


def _closure(name, seen):
    if name not in seen:
        seen.add(name)
        for inc in re.findall(r'#include "(\w+\.h)"', open(os.path.join(CSRC, name)).read()):
            _closure(inc, seen)
    return seen


def test_source_hash_sees_every_included_header(tmp_path, monkeypatch):
    sources = _closure("kernels.hip", set())
    copy = tmp_path / "paper_2507_02401_amd" / "csrc"
    copy.mkdir(parents=True)
    for name in sources:
        (copy / name).write_text(open(os.path.join(CSRC, name)).read())
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    base = bench.source_hash()
    for name in sorted(sources):
        text = (copy / name).read_text()
        (copy / name).write_text(text + "// changed\n")
        assert bench.source_hash() != base, name
        (copy / name).write_text(text)

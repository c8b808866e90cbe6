"""The benchmark's stored traffic count holds for the sources it was taken on."""
import json
import os
import re
import shutil
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_traffic_goes_with_every_source_of_the_kernel(tmp_path, monkeypatch):
    """A change of the kernel's file, of the tile loop that issues its loads, of its
    plans or of the planes' layout makes the count void."""
    import bench
    names = {os.path.basename(p) for p in bench.GEMM_SOURCES}
    with open([p for p in bench.GEMM_SOURCES if p.endswith("residue.hip")][0]) as f:
        included = set(re.findall(r'#include "(\w+\.h)"', f.read()))
    assert {"int8_tile.h", "residue.h"} <= included & names and "layout.h" in names
    copies = [str(tmp_path / os.path.basename(p)) for p in bench.GEMM_SOURCES]
    for src, dst in zip(bench.GEMM_SOURCES, copies):
        shutil.copy(src, dst)
    record = tmp_path / "traffic.json"
    record.write_text(json.dumps({"kernel": "k", "source_sha256_16": bench.source_hash(copies), "bytes_per_launch": 5}))
    monkeypatch.setattr(bench, "GEMM_SOURCES", copies)
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(record))
    assert bench.traffic_for("k") == 5 and bench.traffic_for("other") is None
    for path in copies:
        with open(path) as f:
            text = f.read()
        with open(path, "w") as f:
            f.write(text + "\n")
        assert bench.traffic_for("k") is None, path
        with open(path, "w") as f:
            f.write(text)
    assert bench.traffic_for("k") == 5

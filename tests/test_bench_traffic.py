"""The measured traffic that bench.py reports is dropped when any source of the fibre passes changes."""
import json
import os
import shutil

import bench


def test_every_pass_source_is_guarded(tmp_path, monkeypatch):
    srcs = [shutil.copy(f, tmp_path / os.path.basename(f)) for f in bench.KERNEL_SRCS]
    names = {os.path.basename(f) for f in srcs}
    assert {"lsx_kernels.hip", "lsx_rowsplit.hip", "lsx_pass.h", "lsx_internal.h"} <= names
    monkeypatch.setattr(bench, "KERNEL_SRCS", srcs)
    rec = tmp_path / "traffic.json"
    rec.write_text(json.dumps({"kernel_source_sha256_16": bench.kernel_source_hash(),
                               "layer2_pass": {"fp64": {"hbm_bytes_per_launch": 5.0}}}))
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(rec))
    assert bench.measured_traffic("fp64") == 5.0
    assert bench.measured_traffic("mix_fp32") is None
    for f in srcs:
        text = open(f).read()
        with open(f, "a") as out:
            out.write("\n")
        assert bench.measured_traffic("fp64") is None, f
        with open(f, "w") as out:
            out.write(text)
        assert bench.measured_traffic("fp64") == 5.0

"""bench.py keys its records of the headline kernel's counters by a hash that
changes with every source the kernel is compiled from."""
import os
import shutil

import bench


def test_key_covers_the_included_headers(tmp_path, monkeypatch):
    src = os.path.dirname(bench.KERNEL_SRC)
    for name in os.listdir(src):
        if name.endswith((".hip", ".h", ".cpp")):
            shutil.copy(os.path.join(src, name), tmp_path)
    key = bench.kernel_source_hash()
    monkeypatch.setattr(bench, "KERNEL_SRC", str(tmp_path / os.path.basename(bench.KERNEL_SRC)))
    assert bench.kernel_source_hash() == key
    for name, used in (("fb_kernels.hip", True), ("fb_device.h", True), ("fb_bpl.h", True), ("fb_split.h", True),
                       ("fb_internal.h", True), ("fb_mvs.hip", False)):
        with open(tmp_path / name, "a") as f:
            f.write("\n")
        assert (bench.kernel_source_hash() != key) == used, name
        key = bench.kernel_source_hash()

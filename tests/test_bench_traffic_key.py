"""The counter summary that bench.py quotes holds for the kernel it was taken on (CPU): its key
covers the kernel's source and the table of its tiles."""
import shutil

import bench


def test_key_follows_every_source_of_the_kernel(tmp_path, monkeypatch):
    copies = []
    for path in bench.KERNEL_SOURCES:
        copies.append(str(tmp_path / path.rsplit("/", 1)[1]))
        shutil.copy(path, copies[-1])
    assert {c.rsplit("/", 1)[1] for c in copies} >= {"elb_kernels.h", "stage_kernels.hip"}
    key = bench.kernel_source_hash()
    monkeypatch.setattr(bench, "KERNEL_SOURCES", copies)
    assert bench.kernel_source_hash() == key
    profile = tmp_path / "profile.md"
    profile.write_text(f"kernel source sha256: `{key}`\nHBM bytes per launch (scaled): `1.5e8`\n")
    monkeypatch.setattr(bench, "TRAFFIC_PROFILE", str(profile))
    assert bench.measured_traffic() == 1.5e8
    for c in copies:
        with open(c, "a") as f:
            f.write("// another tile\n")
        assert bench.measured_traffic() is None
        shutil.copy(bench.REPO + "/paper_2211_16933_amd/csrc/" + c.rsplit("/", 1)[1], c)
        assert bench.measured_traffic() == 1.5e8

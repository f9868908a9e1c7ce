"""What bench.py says about the attention kernel (no GPU needed)."""
import os
import re
import shutil

import pytest

import bench
from paper_2509_04377_amd import build, synth


@pytest.mark.parametrize("name", sorted(synth.WORKLOADS))
@pytest.mark.parametrize("splits", [1, 4])
def test_the_report_names_kernels_that_exist(name, splits):
    source = "".join(open(os.path.join(build.CSRC, f)).read() for f in ("paged_decode.hip", "paged_decode_bf16.hip"))
    defined = set(re.findall(r"__global__[^;{]*?\b(\w+_kernel)\(", source))
    wl = synth.WORKLOADS[name]
    kernels = re.findall(r"\w+_kernel", bench.attention_kernels(wl, splits))
    assert kernels and set(kernels) <= defined
    assert kernels[0] == ("paged_decode_kernel" if wl.dtype == "f32" else "paged_decode_bf16_kernel")
    assert ("paged_decode_reduce_kernel" in kernels) == (splits > 1)


def test_the_report_leaves_open_who_merges_splits():
    """Rows in up to twelve splits have a merge launch in the first layer of a step or in none: the report does not add it to every call."""
    for wl in synth.WORKLOADS.values():
        label = bench.attention_kernels(wl, 4)
        assert "+ paged_decode_reduce_kernel" not in label and "in its launch, or" in label


def test_the_source_hash_covers_what_chooses_and_builds_the_kernel(tmp_path, monkeypatch):
    root = tmp_path / "paper_2509_04377_amd"
    shutil.copytree(build.CSRC, root / "csrc")
    before = bench.kernel_source_hash()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_source_hash() == before
    for name in ("pe_api.hip", "paged_decode.hip", "paged_decode_bf16.hip", "pe_device.h", "pe_launch.h"):
        path = root / "csrc" / name
        text = path.read_text()
        path.write_text(text + "//")
        assert bench.kernel_source_hash() != before, name
        path.write_text(text)
    monkeypatch.setattr(build, "FLAGS", build.FLAGS + ["-g"])
    assert bench.kernel_source_hash() != before

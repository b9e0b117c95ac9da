"""The digest that tells whether committed counter figures still belong to the kernels: it has to cover the files that hold
them, wherever they are moved."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_digest_covers_every_bf16_attention_kernel():
    csrc = os.path.join(ROOT, "paper_2509_24014_amd", "csrc")
    holding = set()
    for name in os.listdir(csrc):
        if name.endswith((".hip", ".hpp")):
            with open(os.path.join(csrc, name)) as f:
                if re.search(r"__global__[^;{]*\battn_bf16\w*_kernel\s*\(", f.read()):
                    holding.add(name)
    assert len(holding) >= 2
    covered = {os.path.basename(p) for p in bench._kernel_sources()}
    assert holding <= covered
    assert {"tile_bf16.hpp", "kernels.hpp"} <= covered
    assert re.fullmatch(r"[0-9a-f]{16}", bench._kernel_source_digest())


def test_digest_changes_with_the_kernel_body(monkeypatch, tmp_path):
    import shutil
    copy = tmp_path / "paper_2509_24014_amd" / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_2509_24014_amd", "csrc"), copy, ignore=shutil.ignore_patterns("*.o"))
    before = bench._kernel_source_digest()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench._kernel_source_digest() == before
    for name in ("attn_bf16_kernel.hpp", "attn_bf16_splitk.hip"):
        with open(copy / name, "a") as f:
            f.write("// another kernel\n")
        after = bench._kernel_source_digest()
        assert after != before
        before = after

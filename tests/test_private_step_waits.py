"""Counted waits of the barrier-free loop of the 32-row sparse kernel, read from the assembly hipcc makes of it here.

A counted wait in inline assembly is a promise about what was issued after the copy it waits for. What was issued between
the fence in front of it and the wait itself is certain: one tile copy, D / 16 loads of a wave. A wait that leaves more than
that in flight would rest on where the compiler put some other load (the block-number load may legally move across the copies),
and a load of the tile that is read next could then still be on its way."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_24014_amd import build as lib_build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc here")
    out = str(tmp_path_factory.mktemp("asm") / "splitk.s")
    subprocess.run([HIPCC, *lib_build.FLAGS, "-S", "--cuda-device-only", os.path.join(lib_build.CSRC, "attn_bf16_splitk.hip"), "-o", out],
                   check=True, capture_output=True, timeout=300)
    with open(out) as f:
        text = f.read()
    found = {}
    for m in re.finditer(r"^(_ZN7sparsed\d+attn_bf16_splitk_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb1E\w*):(.*?)^\.Lfunc_end", text, re.M | re.S):
        found[tuple(int(m.group(i)) for i in (2, 3, 4))] = m.group(5)
    return found


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("block_k", [32, 64, 128])
def test_counted_waits_leave_only_the_copy_issued_since_the_fence(kernels, D, block_k):
    body = kernels[(D, 1, block_k)]
    waits = [int(n) for n in re.findall(r"#ASMSTART\s+s_waitcnt vmcnt\((\d+)\)", body)]
    counted = [n for n in waits if n > 0]
    assert len(counted) >= 4, "two counted waits in each of the two steady steps"
    assert max(counted) <= D // 16, f"waits {sorted(set(counted))} leave more in flight than the {D // 16} loads of one tile copy"

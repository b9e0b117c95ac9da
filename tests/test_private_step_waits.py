"""Counted waits of the barrier-free loop of the split-key kernel, read from the assembly hipcc makes of every form of it here.

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
def assembly(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc here")
    out = str(tmp_path_factory.mktemp("asm") / "splitk.s")
    subprocess.run([HIPCC, *lib_build.FLAGS, "-S", "--cuda-device-only", os.path.join(lib_build.CSRC, "attn_bf16_splitk.hip"), "-o", out],
                   check=True, capture_output=True, timeout=300)
    with open(out) as f:
        return f.read()


@pytest.fixture(scope="module")
def kernels(assembly):
    found = {}
    for m in re.finditer(r"^_ZN7sparsed\d+attn_bf16_splitk_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb1ELi(\d+)ELb(\d)E\w*:(.*?)^\.Lfunc_end",
                         assembly, re.M | re.S):
        key = tuple(int(m.group(i)) for i in range(1, 6))   # head dim, row groups, keys a block, tile streams, lists or every tile
        assert key not in found
        found[key] = m.group(6)
    return found


FORMS = [(D, 1, block_k, streams, 1) for D in (64, 128) for block_k in (32, 64, 128) for streams in (1, 2)] + [(D, 1, 64, 2, 0) for D in (64, 128)]


def test_every_barrier_free_form_is_looked_at(kernels):
    assert sorted(kernels) == sorted(FORMS)


@pytest.mark.parametrize("form", FORMS)
def test_counted_waits_leave_only_the_copy_issued_since_the_fence(kernels, form):
    D, body = form[0], kernels[form]
    waits = [int(n) for n in re.findall(r"#ASMSTART\s+s_waitcnt vmcnt\((\d+)\)", body)]
    counted = [n for n in waits if n > 0]
    assert len(counted) >= 4, "two counted waits in each of the two steady steps"
    assert max(counted) <= D // 16, f"waits {sorted(set(counted))} leave more in flight than the {D // 16} loads of one tile copy"


def test_written_out_copies_bring_their_own_wait_states(assembly):
    """The compiler puts no wait states between its own instructions and a load inside an assembly block. A vector instruction that
    writes a scalar register (the restore of a spilled one, say) needs five before a load reads that register, a write of m0 one.
    Each block with copies has them inside; and as the compiler cannot be told that a block writes m0, a kernel with such blocks
    uses it nowhere else."""
    copies = 0
    for body in re.findall(r"^_ZN7sparsed\d+attn_bf16_splitk_kernelI\w*:(.*?)^\.Lfunc_end", assembly, re.M | re.S):
        blocks = [b for b in re.findall(r"#ASMSTART(.*?);;#ASMEND", body, re.S) if "buffer_load" in b]
        if not blocks:
            continue
        assert not re.search(r"\bm0\b", re.sub(r"#ASMSTART.*?;;#ASMEND", "", body, flags=re.S))
        for block in blocks:
            since_start = since_m0 = 0
            for line in (x.strip() for x in block.strip().splitlines()):
                if line.startswith("buffer_load"):
                    assert since_start >= 5 and since_m0 >= 1, block
                    copies += 1
                states = int(line.split()[1], 0) + 1 if line.startswith("s_nop") else 1
                since_start += states
                since_m0 = 0 if re.match(r"s_\w+ m0,", line) else since_m0 + states
    assert copies > 1000

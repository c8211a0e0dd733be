"""The order of the sparse attention's tile loop, read from the compiled kernel's assembly.

How far workgroups that share K/V tiles drift apart, and with it the reads from HBM, depends
on the order of exponentials, V operand reads and MFMAs in the loop, so the source fixes it.
Every copy of the loop (scheduled and fixed grid, even and odd steps, the last step) must have
it, whatever the compiler does with the code around."""
import os
import re
import subprocess

import pytest

from paper_2609_01925_amd import build as B

PRE, AHEAD = 3, 2  # pairs of probabilities ahead of the MFMAs; V operands read this many MFMAs ahead


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    try:
        cc = B.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "attn.s")
    subprocess.run([cc, f"--offload-arch={B.ARCH}", *B.COMMON, *B.DEVICE_FLAGS, *B.EXTRA["attn.hip"], "--cuda-device-only",
                    "-S", os.path.join(B.CSRC, "attn.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read().split("\n")


def _blocks(lines, kernel):
    """Basic blocks of a kernel as lists of mnemonics."""
    start = next(i for i, x in enumerate(lines) if re.match(r"_Z\w*" + kernel + r"\w*:", x))
    blocks = [[]]
    for x in lines[start + 1:]:
        if x.startswith(".Lfunc_end"):
            return blocks
        if re.match(r"\.LBB|; %bb", x):
            blocks.append([])
        t = x.split(";")[0].split()
        if t and not t[0].startswith("."):
            blocks[-1].append(t[0])


@pytest.mark.parametrize("rows,mfmas", [(128, 16), (64, 8)])
def test_sparse_loop_order(assembly, rows, mfmas):
    is_mfma = lambda x: x.startswith("v_mfma")  # noqa: E731
    loops = [b for b in _blocks(assembly, f"attn_kernelILi{rows}ELb0E")
             if sum(map(is_mfma, b)) == mfmas and sum(x.startswith("v_exp") for x in b) == 2 * mfmas]
    assert len(loops) >= 6, "three copies of the step on each of the two paths"
    for b in loops:
        at = [i for i, x in enumerate(b) if is_mfma(x)]
        beside = [b[i:j] for i, j in zip(at, at[1:] + [len(b)])]
        count = lambda name: [sum(x.startswith(name) for x in seg) for seg in beside]  # noqa: E731
        assert count("v_exp") == [2] * (mfmas - PRE) + [0] * PRE
        assert count("ds_read") == [2] * (mfmas - AHEAD) + [0] * AHEAD
        assert count("v_dot2")[:mfmas - PRE] == [0] * (mfmas - PRE)

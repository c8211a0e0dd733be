"""How the list builders of the selection read a VS head's direction masks, from the compiled
kernels' assembly.

A row takes eight mask bytes per lane and 256 key blocks (four chunks of both directions).
sel_mid runs a head in one workgroup, so nothing else covers the latency of those reads: they
are to be in flight together, not each behind a branch and a wait of its own."""
import os
import re
import subprocess

import pytest

from paper_2609_01925_amd import build as B


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    try:
        cc = B.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "select.s")
    subprocess.run([cc, f"--offload-arch={B.ARCH}", *B.COMMON, *B.DEVICE_FLAGS, *B.EXTRA.get("select.hip", []),
                    "--cuda-device-only", "-S", os.path.join(B.CSRC, "select.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read().split("\n")


def _runs_of_reads(lines, kernel, mnemonic):
    """Lengths of the runs of `mnemonic` within one basic block and without a wait between."""
    start = next(i for i, x in enumerate(lines) if re.match(rf"_Z\w*\d{kernel}E\w*:", x))
    runs, n = [], 0
    for x in lines[start + 1:]:
        t = x.split(";")[0].split()
        if x.startswith(".Lfunc_end") or re.match(r"\.LBB|; %bb", x) or (t and t[0] == "s_waitcnt"):
            if n:
                runs.append(n)
            n = 0
        if x.startswith(".Lfunc_end"):
            return runs
        n += bool(t) and t[0] == mnemonic


# sel_mid counts and fills; the other two also read the route, a byte of its own
@pytest.mark.parametrize("kernel,mnemonic,others,rows", [("sel_mid", "ds_read_u8", 0, 2),
                                                         ("sel_csr_count", "global_load_ubyte", 1, 1),
                                                         ("sel_csr_fill", "global_load_ubyte", 1, 1)])
def test_mask_reads_in_flight_together(assembly, kernel, mnemonic, others, rows):
    assert sorted(_runs_of_reads(assembly, kernel, mnemonic)) == [1] * others + [8] * rows

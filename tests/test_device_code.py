"""What the device code built here has to hold for its blocks to exchange sums,
read from the assembly of the sources (CPU; nothing is run)."""
import os
import re
import subprocess

import pytest

from paper_2507_23189_amd import build as B

pytestmark = pytest.mark.slow


def kernel_lines(tmp_path, source, kernel):
    """Instructions of the kernel whose mangled name holds `kernel`."""
    out = str(tmp_path / "device.s")
    subprocess.run([B.hipcc(), "-x", "hip", *B.HIPCC_FLAGS, f"-I{B.INCLUDE}", f"-I{B.CSRC}", "-S", "--cuda-device-only",
                    os.path.join(B.CSRC, source), "-o", out], check=True, capture_output=True)
    body = re.search(rf"^(\S*{kernel}\S*):(.*?)^\.Lfunc_end", open(out).read(), re.S | re.M).group(2)
    return [ln.split(";")[0].strip() for ln in body.splitlines() if ln.split(";")[0].strip()]


def test_annulus_adds_are_waited_for_before_a_block_counts_as_done(tmp_path):
    """A workgroup barrier leaves other waves' memory operations under way: every
    wave waits for its own adds before the barrier that lets one lane count the
    block, and the last block read the totals."""
    code = kernel_lines(tmp_path, "metrics.hip", "metrics_sums")
    adds = [i for i, ln in enumerate(code) if re.match(r"global_atomic_add_x2 v\[\d+:\d+\], v\[\d+:\d+\], ", ln)
            and not ln.endswith("sc0")]
    assert len(adds) == 1                      # the annulus sums, result unused
    count, = (i for i, ln in enumerate(code) if ln.startswith("global_atomic_add_x2") and ln.endswith("sc0"))
    assert adds[0] < count
    barriers = [i for i in range(adds[0], count) if code[i] == "s_barrier"]
    assert barriers
    between = code[adds[0]:barriers[0]]
    wait = [i for i, ln in enumerate(between) if ln == "s_waitcnt vmcnt(0)"]
    assert wait, "no wait for the adds before the barrier"
    # All lanes' waves come through it: past the loop, with the mask restored.
    assert any(ln.startswith("s_or_b64 exec, exec") for ln in between[:wait[0]])

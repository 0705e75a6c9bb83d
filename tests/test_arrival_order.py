"""A workgroup's word is in place before its arrival at the counter is issued.

The last workgroup to arrive decides on the words that the others posted and
clears them; a word still on its way at that moment would be missed, and would
land on the cleared workspace.  Read here from the gfx950 assembly of the
verification kernels (compiled from the sources, no GPU needed): walking back
from every counter increment whose result is used, a wait for all outstanding
memory operations comes before any write to device memory."""
import os
import re
import subprocess

import pytest

from paper_2310_07177_amd import build

# Returning increments (sc0) are arrivals; the writes that may carry a word.
ARRIVAL = re.compile(r"^\s*global_atomic_add(_x2)?\s.*\bsc0\b")
WRITE = re.compile(r"^\s*(global|flat|buffer)_(atomic_(swap|cmpswap)|store)")
WAIT_ALL = re.compile(r"^\s*s_waitcnt\s.*vmcnt\(0\)")


def assembly(src, out):
    cmd = [build.HIPCC] + build.FLAGS + ["-S", "--cuda-device-only", os.path.join(build.CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(out) as f:
        return f.read().splitlines()


@pytest.mark.parametrize("src", ["verify.hip", "verify_greedy.hip", "verify_tree.hip"])
def test_word_before_arrival(src, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("needs hipcc")
    lines = assembly(src, str(tmp_path / "out.s"))
    arrivals = [k for k, l in enumerate(lines) if ARRIVAL.match(l)]
    assert len(arrivals) >= 4
    for k in arrivals:
        for j in range(k - 1, -1, -1):
            if WAIT_ALL.match(lines[j]):
                break
            assert not WRITE.match(lines[j]), f"{src}: no wait between\n{lines[j]}\nand\n{lines[k]}"

"""A kernel that reports its own end to the host waits for the stores of all its waves
first: read from the assembly that the build's compiler gives, no GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2507_11094_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_set_read_waits_for_every_wave(tmp_path):
    out = tmp_path / "set.s"
    subprocess.check_call([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "set.hip"),
                           "-o", str(out)], stderr=subprocess.DEVNULL)
    body = re.search(r"^\S*k_set_unpack_one\S*:.*?s_endpgm", out.read_text(), flags=re.M | re.S).group(0)
    lines = [x.split(";")[0].strip() for x in body.splitlines()]
    lines = [x for x in lines if x]
    barriers = [i for i, x in enumerate(lines) if x.startswith("s_barrier")]
    assert len(barriers) == 1
    # the wait stands in the block of the barrier, after the last store
    at = barriers[0]
    start = max(i for i in range(at) if lines[i].endswith(":"))
    waits = [i for i in range(start, at) if re.match(r"s_waitcnt\b.*vmcnt\(0\)", lines[i])]
    assert waits, lines[start:at + 1]
    assert not any("store" in x for x in lines[waits[-1]:at])

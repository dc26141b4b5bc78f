"""That the compiled update kernels stream what their source streams: a hint on a store is lost without a word when
the compiler joins the store with another one.  Reads the assembly of this library's own kernels; no GPU."""
import os
import re
import subprocess

import pytest

from paper_2509_03110_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_descent_streams_velocities_and_sums(tmp_path):
    out = str(tmp_path / "stream.s")
    subprocess.run([HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "kernels_stream.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    seen = 0
    for m in re.finditer(r"^(_ZN4lsam\S*descent_kernelILi(\d)ELb(\d)ELb(\d)E\S*):\s*; @.*?\n(.*?)\.Lfunc_end", text, re.S | re.M):
        ascent, stream = int(m[2]), int(m[4])
        stores = re.findall(r"^\s+global_store_dwordx4 .*$", m[5], re.M)
        words = 2 if ascent and stream else 1
        # velocities and sums always; the iterates, and the ascent's point, past the caches only
        want = words * (2 + (1 + (ascent > 0)) * stream)
        assert len(stores) == words * (3 + (ascent > 0)) and sum(" nt" in s for s in stores) == want, (m[1], stores)
        seen += 1
    assert seen == 14

"""The batch's mixed kernel calls its small tiles (they are not inlined), so the
compiler takes their arguments for values per lane unless the code makes them
scalar.  A buffer access through a descriptor of such values becomes a loop that
reads one lane's descriptor at a time and compares it with the others'; the
compiled tiles have none of these.  And the kernel itself reads its descriptors
by scalar loads, which it does only while no call could write them (no GPU
needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1408_3526_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="ROCm compilers not available")
def test_called_tiles_use_scalar_descriptors(tmp_path):
    out = str(tmp_path / "rmdf_batch.s")
    r = subprocess.run(["hipcc", *build.HIP_FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, "rmdf_batch.hip"), "-o", out],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    text = open(out).read()
    bodies = {n: b for n, b in re.findall(r"^(_ZN4rmdfL7tile\d+\w*):(.*?)^\.Lfunc_end", text, re.M | re.S)}
    assert len(bodies) == 2, sorted(bodies)
    for name, body in bodies.items():
        assert "buffer_load" in body and "buffer_store" in body, name
        assert "v_cmp_eq_u64" not in body, (name, body.count("v_cmp_eq_u64"))
    kernel, = re.findall(r"^_ZN4rmdf13k_batch_mixed\w*:(.*?)^\.Lfunc_end", text, re.M | re.S)
    # (the frame counter is the one vector load by a global address)
    assert len(re.findall(r"^\tglobal_load", kernel, re.M)) <= 2

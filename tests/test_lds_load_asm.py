"""Loads from memory straight to LDS take their LDS address from m0, and the hardware needs one wait state between the
scalar instruction that writes m0 and the load.  The compiler keeps that distance for its own instructions but not inside
assembly blocks, so it is checked in the code generated for the kernels that use such loads."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source,least", [("fwd.hip", 8), ("short.hip", 48)])  # K and V of a piece: four row groups each, six forms
def test_a_wait_state_follows_every_write_of_m0(tmp_path, source, least):
    from paper_2508_18224_amd.build import FLAGS
    out = tmp_path / "out.s"
    flags = [f for f in FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC, *flags, "--offload-device-only", "-S", "-o", str(out),
                          os.path.join(ROOT, "paper_2508_18224_amd", "csrc", source)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    loads, since = 0, 99                                           # wait states since the last write of m0
    for line in out.read_text().splitlines():
        op = line.split(";")[0].strip()
        if not op or op.startswith(".") or op.endswith(":"):
            continue
        if re.match(r"buffer_load_\w+ .*\blds\b", op):
            loads += 1
            assert since >= 1, line
        if re.match(r"s_\w+ m0\b", op):
            since = 0
        else:
            since += int(op.split()[1], 0) + 1 if op.startswith("s_nop") else 1
    assert loads >= least

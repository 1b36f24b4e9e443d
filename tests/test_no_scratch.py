"""The main kernels use nearly every vector register of their occupancy.  Where a change takes more, the compiler puts values in scratch
memory and says nothing: checked in the code generated for every form of them, also those that no test launches often."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source,kernels", [("fwd.hip", 6), ("short.hip", 6), ("bwd.hip", 12)])
def test_no_kernel_spills_vector_registers(tmp_path, source, kernels):
    from paper_2508_18224_amd.build import FLAGS
    out = tmp_path / "out.s"
    flags = [f for f in FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC, *flags, "--offload-device-only", "-S", "-o", str(out),
                          os.path.join(ROOT, "paper_2508_18224_amd", "csrc", source)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    spills = dict(re.findall(r"\.name:\s+(_ZN3nsa\S+)\n(?:.*\n)*?\s+\.vgpr_spill_count:\s+(\d+)", out.read_text()))
    assert len(spills) >= kernels, sorted(spills)
    scratch = dict(re.findall(r"\.name:\s+(_ZN3nsa\S+)\n\s+\.private_segment_fixed_size:\s+(\d+)", out.read_text()))
    assert scratch.keys() == spills.keys()
    assert {k: (n, scratch[k]) for k, n in spills.items() if n != "0" or scratch[k] != "0"} == {}

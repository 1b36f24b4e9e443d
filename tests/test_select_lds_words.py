"""Block selection keeps its lists in LDS, where lanes of a wavefront read what other lanes wrote.  The compiler may move a read
across a write of another type, so all such accesses are of one type, and every hand-over between lanes has a fence of the
wavefront around it.  Both are checked in the optimised device code as the compiler describes it."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_lds_lists_are_words_of_one_type_between_fences(tmp_path):
    from paper_2508_18224_amd.build import FLAGS
    out = tmp_path / "select.ll"
    flags = [f for f in FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC, *flags, "--offload-device-only", "-S", "-emit-llvm", "-o", str(out),
                          os.path.join(ROOT, "paper_2508_18224_amd", "csrc", "select.hip")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    text = out.read_text()
    meta = dict(re.findall(r"^!(\d+) = !\{(.*)\}$", text, re.M))
    kernels = re.findall(r"^define [^\n]*k_select_blocks.*?^\}", text, re.M | re.S)
    assert kernels
    for body in kernels:
        lds = [l for l in body.splitlines() if re.search(r"\b(load|store)\b", l) and "addrspace(3)" in l]
        assert len(lds) > 20
        types = set()
        for line in lds:
            tag = re.search(r"!tbaa !(\d+)", line)
            if tag:                                               # (an access without a type aliases everything)
                types.add(meta[meta[tag.group(1)].split(", ")[1].lstrip("!")].split(",")[0])
        assert types == {'!"int"'}
        # survivors compacted -> keys in place of scores -> ranking -> the next row's list, and the picks of the rounds
        assert len(re.findall(r'fence syncscope\("wavefront"\) release', body)) >= 4

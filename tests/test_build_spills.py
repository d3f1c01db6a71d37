"""The build's check on the counting search's instances: a kernel that spills
scalar registers is refused, others may."""
import os

import pytest

from paper_2305_14641_amd import build

REMARKS = """\
./qc_count.h:168:1: remark: Function Name: _ZN2qc7k_countILi2ELi1024ELi1ELi0ELi0EEEvPKNS_8GraphDevE [-Rpass-analysis=kernel-resource-usage]
./qc_count.h:168:1: remark:     TotalSGPRs: 78 [-Rpass-analysis=kernel-resource-usage]
./qc_count.h:168:1: remark:     SGPRs Spill: {count} [-Rpass-analysis=kernel-resource-usage]
./qc_count.h:168:1: remark:     VGPRs Spill: 10 [-Rpass-analysis=kernel-resource-usage]
./qc_bfs.h:1:1: remark: Function Name: _ZN2qc5k_bfsEv [-Rpass-analysis=kernel-resource-usage]
./qc_bfs.h:1:1: remark:     SGPRs Spill: 7 [-Rpass-analysis=kernel-resource-usage]
"""


def test_remarks_are_read():
    got = build.scalar_spills(REMARKS.format(count=2))
    assert sorted(got.values()) == [2, 7]


def test_a_spilling_instance_is_refused():
    build.check_spills("x.hip", REMARKS.format(count=0))
    with pytest.raises(RuntimeError, match="k_count"):
        build.check_spills("x.hip", REMARKS.format(count=2))
    build.check_spills("qc_count_512.hip", REMARKS.format(count=0))
    with pytest.raises(RuntimeError, match="no resource remarks"):
        build.check_spills("qc_count_512.hip", "")


def test_the_compiler_still_says_so(tmp_path, monkeypatch):
    """A kernel compiled as the library's are: its remarks are there to read."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    (tmp_path / "one.hip").write_text(
        "#include <hip/hip_runtime.h>\n__global__ void k_count_probe(int *p) { p[threadIdx.x] = 1; }\n")
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    monkeypatch.setattr(build, "OBJDIR", str(tmp_path))
    seen = {}
    monkeypatch.setattr(build, "check_spills", lambda src, text: seen.update(build.scalar_spills(text)))
    build._compile("one.hip")
    assert list(seen.values()) == [0] and "k_count_probe" in next(iter(seen))

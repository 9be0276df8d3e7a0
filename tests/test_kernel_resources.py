"""What the compiler reports of the built kernels' resources (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2604_03957_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_the_popcount_decode_kernels_use_no_scratch():
    """A decode kernel's wavefront keeps all its weight loads in flight; any access to scratch waits for them
    (they complete in order), which cost a fifth of the bandwidth of one token at K > 8192."""
    src = os.path.join(build.CSRC, "kernels_gemv_popc.hip")
    cmd = [HIPCC] + build.HIPCC_FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", src,
                                         "-o", os.devnull]
    report = subprocess.run(cmd, stderr=subprocess.PIPE, text=True, check=True).stderr
    names = re.findall(r"Function Name: (\S+)", report)
    scratch = [int(b) for b in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", report)]
    assert len(names) == len(scratch) > 100
    assert any("k_gemv_popc" in n for n in names) and any("k_linear_one" in n for n in names)
    assert [(n, b) for n, b in zip(names, scratch) if b] == []


def _scratch_of(source):
    """{mangled kernel name: bytes of scratch per lane} as the compiler reports them."""
    cmd = [HIPCC] + build.HIPCC_FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                                         os.path.join(build.CSRC, source), "-o", os.devnull]
    report = subprocess.run(cmd, stderr=subprocess.PIPE, text=True, check=True).stderr
    names = re.findall(r"Function Name: (\S+)", report)
    scratch = [int(b) for b in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", report)]
    assert names and len(names) == len(scratch)
    return dict(zip(names, scratch))


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_the_matrix_core_decode_kernels_use_no_scratch():
    """The ring of weight requests runs on behind everything a workgroup does; an access to scratch would wait for it."""
    scratch = _scratch_of("kernels_gemv_fp4.hip")
    assert any("k_gemv_fp4" in n for n in scratch)
    assert {n: b for n, b in scratch.items() if b} == {}
    # several blocks per workgroup: the instances the launcher can choose (more than 8 wavefronts only with four chunks each)
    several = {tuple(map(int, m.groups())) for m in (re.search(r"k_gemv_fp4ILi(\d+)ELi(\d+)ELi(\d+)ELb[01]ELb1EE", n) for n in scratch) if m}
    assert several == {(2, 2, 8), (2, 4, 8), (3, 2, 8), (4, 2, 8), (4, 2, 16)}


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source,kernel,instances", [("kernels_gemm_fp4_wide.hip", "k_gemm_fp4_wide", 3), ("kernels_gemm_fp4_lds.hip", "k_gemm_fp4_lds", 6)])
def test_kernels_that_count_their_loads_use_no_scratch(source, kernel, instances):
    """These wait for a direct load into LDS by the number of younger memory operations of the wavefront; an access to
    scratch among them would be counted, and the wait end before the data is there."""
    scratch = {n: b for n, b in _scratch_of(source).items() if kernel in n}
    assert len(scratch) == instances and set(scratch.values()) == {0}

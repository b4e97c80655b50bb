"""Vector registers of kernels that lie close below a wavefront's worth (no GPU: compiled here).  16 elements per lane: 80 leave room
for six wavefronts per SIMD; with 81 to 88, five, 2^26 elements took 1 to 3 % longer.  Tables of blocks of 2048 with four wavefronts per
block: 72 leave room for seven; with 74 to 85, five or six, 4000 tensors of a block each took 3 to 6 % longer."""
import os
import re
import subprocess

import pytest

from paper_2505_00347_amd import build as libbuild

FLAT = ["2, 4, 64, false, false, true", "3, 4, 128, true, false, true", "3, 3, 128, false, true, false"]
TABLE = ["3, 2, 128, true, false, true", "4, 2, 128, true, true, true"]


SHORT = ["4, 2, false, true, false", "2, 3, true, false, false", "3, 3, true, true, true"]


def registers(kernels, tmp_path):
    if not os.path.exists(libbuild.HIPCC):
        pytest.skip("needs hipcc")
    jobs = []
    for i, k in enumerate(kernels):
        source = tmp_path / ("%d.hip" % i)
        source.write_text('#include "solo_step_big.h"\nnamespace solo { template __global__ void %s; }\n' % k)
        jobs.append(subprocess.Popen([libbuild.HIPCC, *libbuild.FLAGS, "-I" + libbuild.CSRC, "--cuda-device-only", "-S", str(source), "-o",
                                      str(source) + ".s"]))
    assert [job.wait() for job in jobs] == [0] * len(jobs)
    used = [int(re.search(r"\.vgpr_count:\s+(\d+)", (tmp_path / ("%d.hip.s" % i)).read_text()).group(1)) for i in range(len(kernels))]
    return dict(zip(kernels, used))


def test_six_wavefronts_per_simd(tmp_path):
    used = registers(["chunk16_kernel<%s>(const StepArgs)" % k for k in FLAT] + ["multi_chunk16_kernel<%s>(const MultiArgs)" % k for k in TABLE], tmp_path)
    assert max(used.values()) <= 80, used


def test_seven_wavefronts_per_simd_in_tables_of_short_blocks(tmp_path):
    used = registers(["multi_big_quad_kernel<%s>(const MultiArgs)" % k for k in SHORT], tmp_path)
    assert max(used.values()) <= 72, used

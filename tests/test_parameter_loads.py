"""How the kernels for short buffers load parameters and bf16 gradients (no GPU: the device code of a few instantiations).  With loads that allocate in the caches a
step behind other work, whose lines are still there to be written back, took up to half as long again."""
import os
import re
import subprocess

import pytest

from paper_2505_00347_amd import build as libbuild

# (loads of 16 bytes of a lane's elements: those of a full wavefront's share, and of a ragged one where they all exist)
KERNELS = [("chunk8_kernel<2, 3, 128, true, false, false>(SOLO_FIRST_ARGS, const StepRest)", 6),
           ("chunk8_kernel<4, 4, 128, false, false, true>(SOLO_FIRST_ARGS, const StepRest)", 4),
           ("big_quad_kernel<2, 3, true, false, false>(SOLO_FIRST_ARGS, const StepRest)", 4)]


@pytest.mark.parametrize("kernel,count", KERNELS)
def test_parameters_and_bf16_gradients_are_loaded_past_the_caches(kernel, count, tmp_path):
    if not os.path.exists(libbuild.HIPCC):
        pytest.skip("needs hipcc")
    source = tmp_path / "a.hip"
    source.write_text('#include "solo_step_big.h"\nnamespace solo { template __global__ void %s; }\n' % kernel)
    subprocess.check_call([libbuild.HIPCC, *libbuild.FLAGS, "-I" + libbuild.CSRC, "--cuda-device-only", "-S", str(source), "-o", str(tmp_path / "a.s")])
    loads = re.findall(r"global_load_dwordx4 .*", (tmp_path / "a.s").read_text())
    assert sum(load.split()[-1] == "nt" for load in loads) == count, loads

"""Where the arguments of the kernels for short launches lie, as the compiler places them (no GPU: the device code of a few instantiations)."""
import os
import re
import subprocess

import pytest

from paper_2505_00347_amd import build as libbuild

SOURCE = """#include "solo_step_big.h"
namespace solo {
template __global__ void big_quad_kernel<2, 3, true, false, false>(SOLO_FIRST_ARGS, const StepRest);
template __global__ void chunk8_kernel<2, 3, 128, true, false, false>(SOLO_FIRST_ARGS, const StepRest);
}
"""


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not os.path.exists(libbuild.HIPCC):
        pytest.skip("needs hipcc")
    folder = tmp_path_factory.mktemp("arguments")
    (folder / "a.hip").write_text(SOURCE)
    subprocess.check_call([libbuild.HIPCC, *libbuild.FLAGS, "-I" + libbuild.CSRC, "--cuda-device-only", "-S", str(folder / "a.hip"), "-o",
                           str(folder / "a.s")])
    return (folder / "a.s").read_text()


def first_args_bytes(tmp_path, value):
    """Whether kFirstArgsBytes is `value`."""
    source = tmp_path / "b.hip"
    source.write_text('#include "solo_step.h"\nstatic_assert(solo::kFirstArgsBytes == %d, "");\n' % value)
    return subprocess.run([libbuild.HIPCC, *libbuild.FLAGS, "-I" + libbuild.CSRC, "--cuda-device-only", "-fsyntax-only", str(source)],
                          capture_output=True).returncode == 0


def test_the_rest_of_the_arguments_lies_where_the_kernel_reads_it(listing, tmp_path):
    kernels = re.findall(r"- \.agpr_count.*?\.args:(.*?)\.group_segment_fixed_size", listing, re.S)
    assert len(kernels) == 2
    for args in kernels:
        explicit = [(int(a), int(b)) for a, b in re.findall(r"\.offset:\s+(\d+)\s+\.size:\s+(\d+)\s+\.value_kind:\s+(?:by_value|global_buffer)", args)]
        assert len(explicit) == 9
        assert first_args_bytes(tmp_path, explicit[-1][0]) and not first_args_bytes(tmp_path, explicit[-1][0] + 8)


def test_the_first_arguments_are_in_registers(listing):
    assert re.findall(r"\.amdhsa_user_sgpr_kernarg_preload_length (\d+)", listing) == ["14", "14"]

"""Where one form of a kernel ends and the next begins.  The sizes that other tests place on and behind these lines come from
here; they are compared with the rules of the library's source and of the benchmark."""
import os
import subprocess
from types import SimpleNamespace

import pytest

from paper_2505_00347_amd import build as libbuild

# Flat buffers, 8 elements per lane up to so many elements.
LAST8_FP32 = 20 << 18
LAST8_BF16 = 20 << 18
LAST8_BF16_COPY = 12 << 18
PIECES8 = 16 << 8                   # tables: so many pieces
QUAD_BLOCKS = 1024                  # blocks of 2048, four wavefronts each: so many blocks


def last8(bf16, copy=False, rank=13):
    return LAST8_FP32 if not bf16 else LAST8_BF16_COPY if copy else LAST8_BF16       # (whatever the rank of the quantile)


def pieces(sizes):
    """Pieces of a table: whole chunks of 1024, and 512 elements each behind them up to the end of the last code word."""
    return sum(n // 1024 + -(-(-(-n // 80) * 80 - n // 1024 * 1024) // 512) * (n % 1024 > 0) for n in sizes)


RULES = [(bf16, copy, rank) for bf16 in (False, True) for copy in (False, True) for rank in (1, 13, 16, 17, 24, 39, 64, 65, 128)]


def test_lines_of_the_library(tmp_path):
    if not os.path.exists(libbuild.HIPCC):
        pytest.skip("needs hipcc")
    rules = "".join("static_assert(narrow_buffer(%d, %d, %d) && !narrow_buffer(%d, %d, %d), \"\");\n" % (
        last8(*r), *r[:2], last8(*r) + 1, *r[:2]) for r in RULES)
    source = tmp_path / "lines.hip"
    source.write_text('#include "solo_step_big.h"\nusing namespace solo;\n%sstatic_assert(narrow_table_up_to() == %d, "");\n'
                      'static_assert(kQuadUpTo == %d && quad_table(%d, 1) && !quad_table(%d, 1), "");\n' % (
                          rules, PIECES8, QUAD_BLOCKS, QUAD_BLOCKS, QUAD_BLOCKS + 1))
    subprocess.check_call([libbuild.HIPCC, *libbuild.FLAGS, "-I" + libbuild.CSRC, "--cuda-device-only", "-fsyntax-only", str(source)])


def test_kernel_names_of_the_benchmark():
    import bench

    def name(sizes, launch="flat", B=128, grad="bf16", p=0.1, mp=False):
        w = SimpleNamespace(tensors=[("t", k) for k in sizes], block_size=B, grad_dtype=grad, quantile_p=p)
        return bench.step_kernel_name(w, sum(sizes), mp, launch)

    for bf16, copy, rank in RULES:
        n, how = last8(bf16, copy, rank), dict(grad="bf16" if bf16 else "fp32", mp=copy, p=(rank - 0.5) / 128)
        assert [name([k], **how) for k in (n, n + 1)] == ["solo::chunk8_kernel", "solo::chunk16_kernel"]
    assert [name([1024] * k, "multi") for k in (PIECES8, PIECES8 + 1)] == ["solo::multi_chunk8_kernel", "solo::multi_chunk16_kernel"]
    assert [name([2048 * k], B=2048) for k in (QUAD_BLOCKS, QUAD_BLOCKS + 1)] == ["solo::big_quad_kernel", "solo::big_kernel"]

"""Wait states that MI355X asks for and that the compiler keeps for its own instructions but not around those inside an
asm block: behind a vector instruction that writes a scalar register (a lane read reloads a spilled one), two in front of
a vector instruction that reads it, five in front of an access of memory that does.  Looked for in the device code of the built library, and in small kernels
in which nothing stands between the two."""
import os
import re
import struct
import subprocess

import pytest

from paper_2505_00347_amd import build as libbuild

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
VECTOR_READ, MEMORY_READ = 2, 5
WRITES = re.compile(r"\tv_(?:read(?:first)?lane_b32 (s\d+|vcc_lo|vcc_hi),|cmp_\w+ (s\[\d+:\d+\]),)")
SCALARS = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b|\b(vcc_lo|vcc_hi)\b")


def scalars(operands):
    out = set()
    for first, last, one, vcc in SCALARS.findall(operands):
        out |= {vcc} if vcc else set(range(int(first), int(last) + 1)) if first else {int(one)}
    return out


def too_close(listing):
    """(kernel, write, read, wait states between) of every read that comes too early, straight on in the code."""
    lines = [x.split(";")[0].split("//")[0].rstrip() for x in listing.splitlines()]
    lines = [x for x in lines if x and (x.startswith("\t") and not x.startswith("\t.") or x.endswith(":"))]
    found, kernel = [], ""
    for k, line in enumerate(lines):
        if not line.startswith("\t"):
            kernel = line if "_Z" in line else kernel
            continue
        wrote = WRITES.match(line)
        if not wrote:
            continue
        left, passed = scalars(wrote.group(1) or wrote.group(2)), 0
        for after in lines[k + 1:k + 12]:
            if passed >= MEMORY_READ or not left:
                break
            if not after.startswith("\t"):
                continue
            name, _, operands = after.strip().partition(" ")
            results, _, sources = operands.partition(",")
            if name == "s_nop":
                passed += int(operands, 0) + 1
                continue
            memory = name.startswith(("global_", "flat_", "scratch_", "buffer_"))
            need = MEMORY_READ if memory else VECTOR_READ if name.startswith("v_") else 0
            if passed < need and left & scalars(operands if memory else sources):
                found.append((kernel, line.strip(), after.strip(), passed))
            if not memory and not name.startswith("ds_"):
                left -= scalars(results)
            passed += 1
    return found


def device_code(library):
    """The gfx950 code objects of the offload bundles inside a library."""
    with open(library, "rb") as f:
        data = f.read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", -1
    while (at := data.find(magic, at + 1)) >= 0:
        (count,), pos = struct.unpack_from("<Q", data, at + len(magic)), at + len(magic) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + name].decode()
            pos += 24 + name
            if target.endswith("gfx950") and size:
                yield data[at + offset:at + offset + size]


def test_the_scan_sees_what_it_looks_for():
    write, nop, move = "\tv_readlane_b32 s9, v84, 1\n", "\ts_nop %d\n", "\tv_mov_b32_e32 v52, s9\n"
    assert [x[3] for x in too_close("_Zk:\n" + write + move)] == [0]
    assert [x[3] for x in too_close(write + nop % 0 + move)] == [1]
    assert not too_close(write + nop % 1 + move)
    assert not too_close(write + "\ts_add_u32 s9, s9, s8\n" + move)
    store = "\tglobal_store_dwordx4 v0, v[2:5], s[8:9] offset:1024\n"
    assert [x[3] for x in too_close(write + nop % 3 + store)] == [4]
    assert not too_close(write + nop % 4 + store)
    assert len(too_close("\tv_cmp_gt_u32_e64 s[8:9], v1, v2\n" + move)) == 1


def test_built_library(tmp_path):
    if not os.path.exists(libbuild.LIB) or not os.path.exists(OBJDUMP):
        pytest.skip("needs the built library and llvm-objdump")
    seen, found = 0, []
    for k, code in enumerate(device_code(libbuild.LIB)):
        path = tmp_path / ("%d.co" % k)
        path.write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        seen += len(re.findall(r"\tv_readlane_b32 s", listing))
        found += too_close(listing)
    assert seen > 1000               # (the listings are there)
    assert not found, "%d, the first ones: %s" % (len(found), found[:5])


PROBE = """
#include "solo_step.h"
using namespace solo;
__global__ void constant_in_vector(float *out, const float *in)
{
    const float x = u2f((uint32_t)__builtin_amdgcn_readfirstlane((int)f2u(in[threadIdx.x])));
    out[threadIdx.x] = in_vector(x);
}
__global__ void streamed(float *const *out)
{
    float *const base = (float *)uniform64((uint64_t)out[threadIdx.x]);
    stream_store_f4<0>(base, threadIdx.x * 16u, make_float4(1.0f, 2.0f, 3.0f, 4.0f));
}
"""


def compiled(text, tmp_path):
    if not os.path.exists(libbuild.HIPCC):
        pytest.skip("needs hipcc")
    source, listing = tmp_path / "probe.hip", tmp_path / "probe.s"
    source.write_text(text)
    subprocess.check_call([libbuild.HIPCC, *libbuild.FLAGS, "-I" + libbuild.CSRC, "--cuda-device-only", "-S", str(source), "-o", str(listing)])
    return listing.read_text()


def test_helpers_behind_a_lane_read(tmp_path):
    listing = compiled(PROBE, tmp_path)
    assert listing.count("\tv_readfirstlane_b32") >= 3 and "global_store_dwordx4" in listing
    assert not too_close(listing)

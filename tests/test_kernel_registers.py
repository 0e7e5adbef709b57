"""Registers of the built kernels, from the metadata of the library's own code
objects: the selection of the chunked prefill and the fused passes keep their
working sets in registers (spilled ones go through scratch memory, on paths that
are latency-bound throughout)."""

import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2601_22379_amd import spla

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    at = blob.find(BUNDLE)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(BUNDLE))
        p = at + len(BUNDLE) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + n] and size:
                yield blob[at + off:at + off + size]
            p += 24 + n
        at = blob.find(BUNDLE, p)


def metadata(elf):
    """The AMDGPU metadata note (type 32) of a code object."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    size, num = struct.unpack_from("<HH", elf, 54)
    for i in range(num):
        kind, _, off, _, _, length = struct.unpack_from("<IIQQQQ", elf, phoff + i * size)
        p = off
        while kind == 4 and p < off + length:  # PT_NOTE
            n, d, t = struct.unpack_from("<III", elf, p)
            body = p + 12 + (n + 3) // 4 * 4
            if t == 32:
                return msgpack.unpackb(elf[body:body + d])
            p = body + (d + 3) // 4 * 4
    return {}


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(spla.LIB_PATH):
        pytest.skip("the HIP library has not been built")
    with open(spla.LIB_PATH, "rb") as f:
        blob = f.read()
    found = [k for c in code_objects(blob) for k in metadata(c).get("amdhsa.kernels", [])]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found),
                           capture_output=True, text=True, check=True).stdout.splitlines()
    return {re.sub(r"\(.*", "", n).split("spla::", 1)[1]: k for n, k in zip(names, found)}


@pytest.mark.parametrize("pattern,spills,vgprs", [
    # 256-thread selections: several workgroups per compute unit
    (r"prefill_select_kernel<\d+, false, 256,", 0, 128),
    # 1024 threads leave 128 registers; 32 blocks, or 16 windows, per thread fill them
    (r"prefill_select_kernel<(4|8|16), false, 1024,", 0, 128),
    (r"prefill_select_kernel<32, false, 1024,", 8, 128),
    (r"prefill_select_kernel<\d+, true, 1024,", 24, 128),
    (r"prefill_group_kernel<", 0, 256),
    # up to 2048 blocks: the step and the three-wave decode; the four-wave decode
    (r"decode_kernel<[1-6], \d+, 8, (true|false), 3,", 0, 168),
    (r"decode_kernel<[1-4], \d+, 8, false, 4,", 1, 128),
])
def test_no_working_set_is_spilled(kernels, pattern, spills, vgprs):
    hit = {n: k for n, k in kernels.items() if re.match(pattern, n)}
    assert hit
    for n, k in hit.items():
        assert k[".vgpr_spill_count"] <= spills and k[".vgpr_count"] <= vgprs, (
            n, k[".vgpr_spill_count"], k[".vgpr_count"])

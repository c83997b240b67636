"""What the built kernels ask of a compute unit, read from the metadata that the compiler writes beside them in the library:
no kernel uses private memory (the runtime would have to back it on the device at a first launch), and the pipelined global
kernel keeps the wavefronts per SIMD and the workgroups per unit that its tile shapes are chosen for."""
import os
import re
import struct

import pytest

import paper_2603_12646_amd as fa

msgpack = pytest.importorskip("msgpack")   # the metadata's encoding

UNIT_LDS = 160 * 1024


def code_objects(data):
    """The gfx950 code objects of a library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length].decode()
            pos += 24 + length
            if "gfx950" in name and size:
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + 1)


def kernels_of(code):
    """Metadata of the kernels of a code object: the AMDGPU note (type 32) of its note sections."""
    shoff, shentsize, shnum = struct.unpack_from("<Q", code, 0x28)[0], *struct.unpack_from("<HH", code, 0x3A)
    for i in range(shnum):
        kind, _, _, offset, size = struct.unpack_from("<IQQQQ", code, shoff + i * shentsize + 4)
        if kind != 7:   # SHT_NOTE
            continue
        pos = offset
        while pos < offset + size:
            namesz, descsz, note = struct.unpack_from("<III", code, pos)
            name = code[pos + 12:pos + 12 + namesz].rstrip(b"\0")
            desc = pos + 12 + (namesz + 3) // 4 * 4
            if name == b"AMDGPU" and note == 32:
                yield from msgpack.unpackb(code[desc:desc + descsz])["amdhsa.kernels"]
            pos = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(fa.LIB_PATH):
        from paper_2603_12646_amd.build import build_library
        build_library(verbose=False)
    with open(fa.LIB_PATH, "rb") as f:
        data = f.read()
    found = {k[".name"]: k for code in code_objects(data) for k in kernels_of(code)}
    assert len(found) > 40
    return found


def test_no_private_memory(kernels):
    assert {n: k[".private_segment_fixed_size"] for n, k in kernels.items() if k[".private_segment_fixed_size"]} == {}
    assert not [n for n, k in kernels.items() if k[".uses_dynamic_stack"]]


def test_global_kernels_keep_their_occupancy(kernels):
    """Wavefronts per SIMD from 512 registers in steps of eight; four-wavefront workgroups put one wavefront on each SIMD."""
    seen = set()
    for name, k in kernels.items():
        m = re.search(r"fa_fwd_global_kernelINS_\d+(B?F16)ELi(\d+)ELi(\d)ELi(\d+)ELb(\d)ELb(\d)", name)
        if not m:
            continue
        head_dim, blocks, waves, bias, rope = (int(x) for x in m.groups()[1:])
        registers = k[".vgpr_count"] + k.get(".agpr_count", 0)
        per_simd = 512 // (-(-registers // 8) * 8)
        if waves > 4:
            want = waves // 4
        elif head_dim == 32:
            want = 4 if blocks == 1 else (2 if bias else 3)
        else:
            want = 3 if head_dim == 64 and blocks == 1 else 2
        assert per_simd >= want, (name, registers)
        groups = 1 if waves > 4 else want
        assert groups * k[".group_segment_fixed_size"] <= UNIT_LDS, (name, k[".group_segment_fixed_size"])
        seen.add((m.group(1), head_dim, blocks, waves, bias, rope))
    assert len(seen) >= 36


def test_exchanges_write_no_register_in_an_asm_block_alone():
    """An exchange between lanes takes both registers in with a value: the compiler then waits for a matrix product that still
    writes them.  Only the dot product that starts a sum (its operands are the probabilities, behind all products) has an
    output of its own."""
    src = os.path.join(os.path.dirname(fa.LIB_PATH), "csrc", "fa_kernels.hip")
    with open(src) as f:
        outputs = [line.strip() for line in f if re.search(r'"=&?v"', line)]
    assert all("v_dot2_f32_f16" in line for line in outputs), outputs

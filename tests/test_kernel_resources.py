"""Registers of the built kernels, from the metadata of the code objects in libscd.so: a hot kernel that
needs more than its registers spills to scratch memory, which no numerics test shows."""
import re
import struct

import pytest

import paper_2606_07684_amd as scd

msgpack = pytest.importorskip("msgpack")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        q = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", blob, q)
        q += 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, q)
            name = blob[q + 24:q + 24 + n]
            q += 24 + n
            if b"gfx950" in name:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, q)


def _metadata(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        if kind != 7:  # SHT_NOTE
            continue
        off, n = struct.unpack_from("<QQ", elf, shoff + i * size + 0x18)
        name, desc, note = struct.unpack_from("<III", elf, off)
        if note == 32:  # NT_AMDGPU_METADATA
            start = off + 12 + (name + 3) // 4 * 4
            yield msgpack.unpackb(elf[start:start + desc])


@pytest.fixture(scope="module")
def spills():
    scd.load_library()
    with open(scd.lib_path(), "rb") as f:
        blob = f.read()
    out = {}
    for elf in _code_objects(blob):
        for meta in _metadata(elf):
            for k in meta["amdhsa.kernels"]:
                out[k[".name"]] = k[".vgpr_spill_count"]
    assert len(out) > 100
    return out


# The most registers an instance of each kernel family may spill.
@pytest.mark.parametrize("kernel,most", [
    ("reuse_decode_bf16_kernel", 2), ("patch_align_act_bf16_kernel", 0),
    ("encode_kv_bf16_kernel", 0), ("encode_bf16_kernel", 0),
    ("gemm_nt_kernel", 2), ("gemm_staged_bf16_kernel", 0)])
def test_spilled_registers(spills, kernel, most):
    got = {n: v for n, v in spills.items() if re.search(r"\d%s" % kernel, n)}
    assert got
    assert {n: v for n, v in got.items() if v > most} == {}

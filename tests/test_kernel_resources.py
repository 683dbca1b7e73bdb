"""What the kernels in the built library take of a compute unit, from the metadata the compiler wrote into it: registers
kept in scratch memory and local memory decide how many workgroups run beside each other, and no result shows either."""
import re
import struct

import pytest

import paper_2406_18485_amd as P

msgpack = pytest.importorskip("msgpack")

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        (n,), pos = struct.unpack_from("<Q", blob, at + len(MAGIC)), at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, id_len = struct.unpack_from("<QQQ", blob, pos)
            if b"gfx950" in blob[pos + 24:pos + 24 + id_len]:
                yield blob[at + offset:at + offset + size]
            pos += 24 + id_len
        at = blob.find(MAGIC, at + 1)


def _notes(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, n = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(n):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        if kind != 7:   # SHT_NOTE
            continue
        at, length = struct.unpack_from("<QQ", elf, shoff + i * size + 0x18)
        end = at + length
        while at < end:
            name, desc, what = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if what == 32:   # NT_AMDGPU_METADATA
                yield msgpack.unpackb(elf[at:at + desc], raw=False)
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(P.binding.LIB_PATH, "rb") as f:
        blob = f.read()
    found = {k[".name"]: k for elf in _code_objects(blob) for note in _notes(elf) for k in note["amdhsa.kernels"]}
    assert len(found) > 60
    return found


def _named(kernels, part):
    some = {n: k for n, k in kernels.items() if re.search(part, n)}
    assert some, part
    return some


def test_the_16_bit_kernels_keep_nothing_in_scratch_memory(kernels):
    for name, k in _named(kernels, "10fwd_kernel|bwd_step_kernel|bwd_dkv_kernel|9dq_kernel").items():
        # (head_dim 64, four key splits, two workgroups per unit, a run of steps: one register, loaded once behind the steps)
        most = 8 if "ELi64ELi4ELi2ELi32E" in name else 0
        assert k[".private_segment_fixed_size"] <= most, (name, k[".private_segment_fixed_size"])


def test_the_fp32_forward_leaves_room_for_other_workgroups(kernels):
    """A unit has 160 KB: six workgroups of 16 rows at head_dim 32, four at 64, two at 128.  Only the padded 16-row kernels hold registers
    in scratch memory."""
    for name, k in _named(kernels, "14fwd_f32_kernel").items():
        np, exact = re.search(r"ILi(\d+)ELb(\d)E", name).groups()
        assert k[".group_segment_fixed_size"] * {"32": 6, "64": 4, "128": 2}[np] <= 160 * 1024, name
        assert k[".private_segment_fixed_size"] == 0 or (exact == "0" and k[".private_segment_fixed_size"] <= 132), name

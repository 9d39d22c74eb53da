"""Registers and scratch memory of the built kernels, as the compiler recorded them in the library (no GPU needed)."""
import re
import struct

import pytest

import paper_2603_14224_amd as sik
from paper_2603_14224_amd.build import LIB

msgpack = pytest.importorskip("msgpack")


def _sections(elf):
    """name -> (offset, size) of a 64-bit little-endian ELF image."""
    off, = struct.unpack_from("<Q", elf, 0x28)
    size, count, names = struct.unpack_from("<HHH", elf, 0x3A)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, off + i * size) for i in range(count)]
    at = heads[names][4]
    return {elf[at + h[0]:elf.index(b"\0", at + h[0])].decode(): (h[4], h[5]) for h in heads}


def _kernels():
    """Mangled name -> metadata record of every gfx950 kernel in the library: each source file's code object lies in a
    bundle of its own, and its notes hold the records as one MessagePack map."""
    sik.lib()  # builds the library if there is none
    with open(LIB, "rb") as f:
        image = f.read()
    off, size = _sections(image)[".hip_fatbin"]
    fat, found = image[off:off + size], {}
    at = fat.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entries, = struct.unpack_from("<Q", fat, at + 24)
        p = at + 32
        for _ in range(entries):
            begin, length, name = struct.unpack_from("<QQQ", fat, p)
            target = fat[p + 24:p + 24 + name]
            p += 24 + name
            if b"gfx950" not in target:
                continue
            code = fat[at + begin:at + begin + length]
            note, _ = _sections(code)[".note"]
            owner, desc, _ = struct.unpack_from("<III", code, note)
            start = note + 12 + (owner + 3) // 4 * 4
            for k in msgpack.unpackb(code[start:start + desc], strict_map_key=False)["amdhsa.kernels"]:
                found[k[".name"]] = k
        at = fat.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 1)
    return found


@pytest.mark.parametrize("part", ["select_attend_kernel", "attn_q2_kernel", "compress_kernel", "quantize_kv_kernel",
                                  "encode_kernel"])
def test_no_scratch_memory(part):
    # a spilled register in the last workgroup's exchange puts a wait in front of loads that are meant to go out together
    some = {n: k for n, k in _kernels().items() if part in n}
    assert some
    bad = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in some.items()
           if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not bad


def test_registers_leave_room_for_four_compressing_workgroups():
    # 4 workgroups x 6 wavefronts on 4 SIMDs with 512 registers each, in steps of 8: 80 registers per lane
    some = {n: k for n, k in _kernels().items() if "compress_kernel" in n}
    assert len(some) == 2
    assert all(k[".max_flat_workgroup_size"] == 384 and k[".group_segment_fixed_size"] <= 160 * 1024 // 4
               for k in some.values())
    assert all(k[".vgpr_count"] <= 80 for k in some.values()), {n: k[".vgpr_count"] for n, k in some.items()}


def test_two_head_pair_workgroups_share_a_compute_unit():
    # workgroups of a pair launch wait for each other, two to a compute unit: 2 x 8 wavefronts on 4 SIMDs of 512 registers,
    # and 160 KB of LDS for two times the static part and the 64 KB that the plan may ask for
    some = {n: k for n, k in _kernels().items() if "step_kernel" in n and k[".max_flat_workgroup_size"] == 512}
    assert len(some) == 20
    assert all(k[".vgpr_count"] <= 128 and k[".vgpr_spill_count"] == 0 for k in some.values())
    assert all(k[".group_segment_fixed_size"] + 64 * 1024 <= 80 * 1024 for k in some.values())


def test_long_chunks_of_rows_are_built_for_pairs_only():
    # (tokens per thread in registers, in LDS, 16-bit first pass, records, forced set, heads) of every variant
    built = {tuple(map(int, re.search(r"step_kernelILi\dELi\dELi(\d+)ELi(\d+)ELb(\d)ELb(\d)ELb(\d)ELi(\d)E", n).groups()))
             for n in _kernels() if "step_kernel" in n}
    assert {v[:2] for v in built if v[2:] == (0, 0, 0, 4)} == {(1, 0), (2, 0), (3, 0), (4, 0), (6, 0)}
    assert {v[:2] for v in built if v[5] == 2} == {(16, 0), (24, 0), (24, 8), (28, 8), (32, 8)}

"""Registers that the decode kernels spill to memory, as the compiler states them in the library's code objects."""
import os
import re
import struct

import msgpack
import pytest

from paper_2505_22758_amd import build as lib_build

EM_AMDGPU, NT_AMDGPU_METADATA, SHT_NOTE = 224, 32, 7


def _kernels():
    """{(kind, weights, sequences, head dimension, query heads per KV head): spilled vector registers} of the row-partitioned, wide and one-sequence instances."""
    data = open(lib_build.LIB, "rb").read()
    out = {}
    for m in re.finditer(b"\x7fELF\x02\x01\x01", data):
        elf = data[m.start():]
        if struct.unpack_from("<H", elf, 18)[0] != EM_AMDGPU:
            continue
        shoff, (shentsize, shnum) = struct.unpack_from("<Q", elf, 40)[0], struct.unpack_from("<HH", elf, 58)
        for i in range(shnum):
            kind, off, size = struct.unpack_from("<I", elf, shoff + i * shentsize + 4) + struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
            if kind != SHT_NOTE:
                continue
            namesz, descsz, note = struct.unpack_from("<III", elf, off)
            if note != NT_AMDGPU_METADATA:
                continue
            start = off + 12 + (namesz + 3) // 4 * 4
            for k in msgpack.unpackb(elf[start:start + descsz])["amdhsa.kernels"]:
                f = re.search(r"(wide|solo|fused)_decode_kernelI((?:L[ib]\d+E)+)E", k[".name"])
                if f:
                    out[(f.group(1),) + tuple(int(v) for v in re.findall(r"L[ib](\d+)E", f.group(2)))] = k[".vgpr_spill_count"]
    return out


def test_decode_kernels_spill_nothing_where_it_costs():
    """A reload is a load: the wait for it drains a wave's ring of weights.  The one-sequence kernel spills nothing.  The wide pass neither, but for its instances of one sequence
    with bf16 and int8 weights and head dimension 128: there what is spilled are addresses of a projection's end, and computing them at the end instead is slower."""
    if not os.path.exists(lib_build.LIB):
        pytest.skip("library not built")
    kernels = _kernels()
    assert sum(k[0] == "solo" for k in kernels) == 9 and sum(k[0] == "wide" for k in kernels) >= 27, sorted(kernels)
    for (kind, wd, *rest), spilled in kernels.items():
        allowed = 20 if kind == "wide" and wd in (0, 1) and rest[0] == 1 and rest[1] == 128 else 0
        assert spilled <= allowed, (kind, wd, rest, spilled)

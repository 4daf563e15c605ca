"""Registers that the compiler spills in the dK/dV kernels that take whole groups and all steps, from the metadata of the library as it is built: what
only some launches need (parts of a group and their sums, a walk that leaves steps out) must cost the others none.  (No GPU is needed.)"""
import os
import re
import struct

import pytest

from paper_2412_05496_amd import build

msgpack = pytest.importorskip("msgpack")
# (D, mask_mod, score_mod, waves keep their own rows, canvas walk): bytes a lane; the others have none
SCRATCH = {
    (128, 5, 6, 0, 0): 36, (64, 1, 1, 1, 0): 12, (64, 3, 4, 1, 0): 8, (64, 5, 0, 1, 0): 12, (64, 5, 1, 1, 0): 16,
    (64, 5, 6, 0, 0): 48, (64, 2051, 2, 1, 0): 28, (64, 2051, 2, 0, 0): 8,
    (64, 32, 0, 0, 1): 8, (64, 96, 0, 0, 1): 20, (64, 160, 0, 0, 1): 8, (64, 224, 0, 0, 1): 8,
}


def kernels(library):
    """name -> metadata, of the gfx950 code objects in the library"""
    data, out, magic = open(library, "rb").read(), {}, b"__CLANG_OFFLOAD_BUNDLE__"
    for at in (m.start() for m in re.finditer(magic, data)):
        pos = at + len(magic)
        count, pos = struct.unpack_from("<Q", data, pos)[0], pos + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target, pos = data[pos + 24:pos + 24 + length], pos + 24 + length
            if not target.startswith(b"hip") or not size:
                continue
            elf = data[at + offset:at + offset + size]
            assert elf[:4] == b"\x7fELF"
            sections, entry, n = struct.unpack_from("<Q", elf, 0x28)[0], *struct.unpack_from("<HH", elf, 0x3A)
            for k in range(n):
                kind, = struct.unpack_from("<I", elf, sections + k * entry + 4)
                start, = struct.unpack_from("<Q", elf, sections + k * entry + 0x18)
                if kind != 7:                       # SHT_NOTE
                    continue
                name_len, note_len, note = struct.unpack_from("<III", elf, start)
                if note != 32:                      # NT_AMDGPU_METADATA
                    continue
                body = start + 12 + (name_len + 3) // 4 * 4
                for kernel in msgpack.unpackb(elf[body:body + note_len])["amdhsa.kernels"]:
                    out[kernel[".name"]] = kernel
    return out


@pytest.mark.skipif(not os.path.exists(build.LIB), reason="the library is not built")
def test_the_others_pay_nothing_for_divided_groups_and_steps_left_out():
    seen, leaving = {}, {}
    for name, kernel in kernels(build.LIB).items():
        m = re.match(r"_ZN8flexattn15bwd_dkdv_kernelILi(\d+)ELj(\d+)ELj(\d+)ELb([01])ELb([01])ELNS_6GroupsE0ELb([01])EEEv", name)
        if m:
            (leaving if m.group(6) == "1" else seen)[tuple(int(g) for g in m.groups()[:5])] = kernel[".private_segment_fixed_size"]
    assert len(seen) > 30 and set(SCRATCH) <= set(seen)
    assert {k: v for k, v in seen.items() if v > SCRATCH.get(k, 0)} == {}
    # a relative bias spills where it leaves steps out, which launches with few hidden steps then do not
    assert {k: v for k, v in leaving.items() if v} == {(128, 2051, 2, 0, 0): 24}


@pytest.mark.skipif(not os.path.exists(build.LIB), reason="the library is not built")
def test_no_forward_is_compiled_twice():
    """Canvases in cells have forward kernels of their own at D = 64 only: at D = 128 they would be those of any canvas again."""
    names = list(kernels(build.LIB))
    cells = [n for n in names if re.match(r"_ZN8flexattn10fwd_kernelILi(64|128)ELi\dELj(160|224)E", n)]
    assert any("ILi64E" in n for n in cells) and not [n for n in cells if "ILi128E" in n]
    assert any(re.match(r"_ZN8flexattn10fwd_kernelILi128ELi\dELj32E", n) for n in names)

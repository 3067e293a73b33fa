"""What the library's code objects say: no few-token kernel keeps part of its state in scratch memory, and the static device memory is what the
header names."""
import os
import re
import struct

from paper_2206_15014_amd import binding


def _scratch_bytes():
    """kernel name -> scratch bytes per lane, from the kernel descriptors of the library's gfx950 code objects"""
    data, found = open(binding.library_path(), "rb").read(), {}
    for m in re.finditer(b"\x7fELF", data):
        o = data[m.start():]
        machine, table, size, count = struct.unpack_from("<H20xQ10xHH", o, 18)
        if machine != 224:                    # EM_AMDGPU
            continue
        sections = [struct.unpack_from("<IIQQQQIIQQ", o, table + size * i) for i in range(count)]
        for s in sections:
            if s[1] != 11:                    # SHT_DYNSYM
                continue
            names = sections[s[6]][4]
            for at in range(s[4], s[4] + s[5], 24):
                name, _, _, section, value = struct.unpack_from("<IBBHQ", o, at)
                text = o[names + name:o.index(b"\0", names + name)].decode()
                if text.endswith(".kd"):
                    _, address, offset = sections[section][2:5]
                    found[text[:-3]] = struct.unpack_from("<I", o, offset + value - address + 4)[0]
    return found


def test_few_token_kernels_do_not_spill():
    kernels = {k: v for k, v in _scratch_bytes().items() if "gemm_few_" in k}
    assert len(kernels) == 22 * 8             # patterns and widths; four tiles, for one GEMM and for several
    assert not {k: v for k, v in kernels.items() if v}


def test_device_memory_of_its_own_is_what_the_header_names():
    """The library's static device arrays, from its code objects' zero-initialised sections, against the sizes in include/nm.h."""
    header = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "nm.h")).read()
    named = sorted(int(n) << int(shift) for n, shift in re.findall(r"#define NM_[A-Z_]+_BYTES \((\d+)u << (\d+)\)", header))
    data, held = open(binding.library_path(), "rb").read(), []
    for m in re.finditer(b"\x7fELF", data):
        o = data[m.start():]
        machine, table, size, count = struct.unpack_from("<H20xQ10xHH", o, 18)
        if machine != 224:
            continue
        for i in range(count):
            _, kind, flags, _, _, length = struct.unpack_from("<IIQQQQ", o, table + size * i)
            if kind == 8 and flags & 2 and length > 4096:     # SHT_NOBITS, allocated
                held.append(length >> 12 << 12)
    assert sorted(held) == named

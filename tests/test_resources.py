"""What the compiled kernels keep in scratch memory, read from the metadata of the built library: CPU only."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_07304_amd", "libslimattn.so")


def _kernels(path):
    """name -> metadata of every kernel in the code objects that a library carries (ELF64 notes of type 32, msgpack)."""
    data, found, at = open(path, "rb").read(), {}, 1
    while (at := data.find(b"\x7fELF", at)) >= 0:
        sh_off, sh_size, sh_num = struct.unpack_from("<Q", data, at + 0x28)[0], *struct.unpack_from("<HH", data, at + 0x3a)
        for i in range(sh_num):
            kind, _, _, off, size = struct.unpack_from("<IQQQQ", data, at + sh_off + i * sh_size + 4)
            p, end = at + off, at + off + size
            while kind == 7 and p + 12 <= end:
                name_len, desc_len, note = struct.unpack_from("<III", data, p)
                desc = p + 12 + (name_len + 3) // 4 * 4
                if note == 32 and data[p + 12:p + 18] == b"AMDGPU":
                    found.update((k[".name"], k) for k in msgpack.unpackb(data[desc:desc + desc_len])["amdhsa.kernels"])
                p = desc + (desc_len + 3) // 4 * 4
        at += 4
    return found


def test_scratch_of_the_kernels():
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    kernels = _kernels(LIB)
    assert len(kernels) >= 50
    # two registers of the 128-row INT8 prefill at D = 128, with either result type; nothing else
    spilling = re.compile(r"slim_prefill_kernelILi128ELb1ELb[01]ELi0ELb0E")
    for name, k in kernels.items():
        assert k[".private_segment_fixed_size"] <= (12 if spilling.search(name) else 0), (name, k[".private_segment_fixed_size"])

"""Registers of the two-step kernels, from the metadata of the built code objects.

Registers spilled in these kernels are reloaded behind the populations they have in
flight: variants with 130 to 364 bytes a lane ran up to 2.6 times as long as the two steps
they replace.  The bound is the largest size that measured faster than one step a pass.
"""
import re
import struct

import msgpack

from paper_2506_09242_amd import lbm


def kernels():
    """(name, bytes of scratch a lane) of every kernel of the library."""
    data = open(lbm.LIB_PATH, "rb").read()
    out = []
    for m in re.finditer(b"\x7fELF\x02\x01\x01\x40", data):  # ELF64 of the AMD HSA ABI
        o = m.start()
        shoff, = struct.unpack_from("<Q", data, o + 0x28)
        shentsize, shnum = struct.unpack_from("<HH", data, o + 0x3A)
        for k in range(shnum):
            _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", data, o + shoff + k * shentsize)
            if kind != 7:  # SHT_NOTE
                continue
            p = o + off
            while p < o + off + size:
                namesz, descsz, note = struct.unpack_from("<III", data, p)
                name = data[p + 12:p + 12 + namesz]
                d = p + 12 + (namesz + 3) // 4 * 4
                if note == 32 and name.startswith(b"AMDGPU"):
                    for kern in msgpack.unpackb(data[d:d + descsz])["amdhsa.kernels"]:
                        out.append((kern[".name"], kern[".private_segment_fixed_size"]))
                p = d + (descsz + 3) // 4 * 4
    return out


def test_two_step_kernels_spill_little():
    ks = [(n, s) for n, s in kernels() if "k_two_steps" in n]
    assert len(ks) >= 100
    assert [k for k in ks if k[1] > 128] == []

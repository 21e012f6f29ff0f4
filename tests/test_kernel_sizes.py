"""Code of the kernels with chains.  A loop's rare paths lie at the kernel's end: one further away than a branch reaches (128 KB) costs the loop a jump each time it is
not taken, and who takes it finds them in no instruction cache."""
import os
import struct

import paper_1512_02595_amd


def kernel_sizes():
    built = os.path.join(os.path.dirname(paper_1512_02595_amd.__file__), "libctc_mi355x.so")
    with open(built, "rb") as f:
        data = f.read()
    found = {}
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:                    # EM_AMDGPU
            sections, size, count = struct.unpack_from("<Q", data, at + 40)[0], *struct.unpack_from("<HH", data, at + 58)
            table = [struct.unpack_from("<IIQQQQIIQQ", data, at + sections + i * size) for i in range(count)]
            for kind, offset, length, link in ((s[1], s[4], s[5], s[6]) for s in table):
                if kind != 11:                                                   # SHT_DYNSYM
                    continue
                names = at + table[link][4]
                for i in range(length // 24):
                    name, info, _, _, _, code = struct.unpack_from("<IBBHQQ", data, at + offset + 24 * i)
                    if info & 15 == 2:                                           # STT_FUNC
                        found[data[names + name:data.index(b"\0", names + name)].decode()] = code
        at = data.find(b"\x7fELF", at + 1)
    return found


def test_kernels_with_chains():
    sizes = {name: size for name, size in kernel_sizes().items() if "lattice" in name}
    print(sorted(sizes.values()))
    assert len(sizes) >= 6 and max(sizes.values()) <= 264 << 10

"""What the compiled sweep kernels hold, read from the metadata of the library
built here: the engines that launch a workgroup per chain keep no spilled
registers.  Scratch memory costs every launch of a kernel that uses any (6 to
8 us where every compute unit has work), which short calls notice."""
import re
import struct

from paper_1403_4560_amd import binding


def kernel_metadata(path):
    """(name, private segment bytes) of every kernel: keys of one msgpack map, in
    alphabetical order."""
    data = open(path, "rb").read()
    out = {}
    for m in re.finditer(rb"\.name(?:[\xa0-\xbf]|\xd9.|\xda..)(_ZN2ea\w+)\xbb\.private_segment_fixed_size(.{5})", data, re.S):
        v = m.group(2)
        out[m.group(1).decode()] = (v[0] if v[0] < 0x80 else v[1] if v[0] == 0xCC else
                                    struct.unpack(">H", v[1:3])[0] if v[0] == 0xCD else struct.unpack(">I", v[1:5])[0])
    return out


def test_chain_engines_spill_no_registers():
    binding.load()
    kernels = kernel_metadata(binding.LIB_PATH)
    names = ("row_sweep_kernel", "group_sweep_kernel", "batch_sweep_kernel", "site_sweep_kernel", "tiny_sweep_kernel",
             "hbm_sweep_kernel", "quad_sweep_kernel")
    seen = {n: {k: v for k, v in kernels.items() if n in k} for n in names}
    assert all(seen.values()), {n: len(v) for n, v in seen.items()}
    spilled = {k: v for group in seen.values() for k, v in group.items() if v}
    assert not spilled, spilled

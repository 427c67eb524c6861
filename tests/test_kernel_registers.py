"""The built library's kernel metadata: the grouped GEMMs of a multi-token call keep everything
in registers.  A kernel that spills says so in its code object's note (per kernel: spilled vector
registers, bytes of scratch memory per lane); the slim kernels hold raw weights of three K steps
and two sets of operands beside their accumulators, so a format whose raw step is too large
spills inside the K loop."""
import struct

import msgpack

import paper_2607_09686_amd.moecache as moecache


def kernels(path):
    """Metadata of every kernel in the library's embedded gfx950 code objects."""
    with open(path, "rb") as f:
        data = f.read()
    out, at = {}, data.find(b"AMDGPU\0\0")
    while at >= 0:
        namesz, descsz, kind = struct.unpack_from("<III", data, at - 12)
        if (namesz, kind) == (7, 32):  # NT_AMDGPU_METADATA
            for k in msgpack.unpackb(data[at + 8:at + 8 + descsz])["amdhsa.kernels"]:
                out[k[".name"]] = k
        at = data.find(b"AMDGPU\0\0", at + 8)
    return out


def test_wide_and_slim_kernels_use_no_scratch():
    names = kernels(moecache.LIB_PATH)
    for fmt in (8, 2, 12, 14):
        for kernel in ("gateup_wide", "down_wide", "gateup_slim", "down_slim"):
            found = [v for n, v in names.items() if f"pf_{kernel}_kernelILi{fmt}E" in n]
            assert len(found) == (0 if fmt == 14 and "slim" in kernel else 1)  # Q6_K: wide only
            for k in found:
                assert (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) == (0, 0), k[".name"]

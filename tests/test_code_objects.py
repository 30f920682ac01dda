"""What the compiler made of the kernels, from the metadata of the library built here (no GPU needed)."""
import os
import struct

import msgpack

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _kernels(path):
    """{symbol: metadata} of every device kernel in the library: the AMDGPU metadata notes (type 32) of the code objects in it."""
    blob = open(path, "rb").read()
    out = {}
    at = blob.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:   # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", blob, at + 40)
            entry, count = struct.unpack_from("<HH", blob, at + 58)
            for i in range(count):
                header = at + shoff + i * entry
                if struct.unpack_from("<I", blob, header + 4)[0] != 7:   # SHT_NOTE
                    continue
                offset, size = struct.unpack_from("<QQ", blob, header + 24)
                o, end = at + offset, at + offset + size
                while o < end:
                    name_size, desc_size, kind = struct.unpack_from("<III", blob, o)
                    desc = o + 12 + (name_size + 3) // 4 * 4
                    if kind == 32:
                        for k in msgpack.unpackb(blob[desc:desc + desc_size], strict_map_key=False)["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    o = desc + (desc_size + 3) // 4 * 4
        at = blob.find(b"\x7fELF", at + 4)
    return out


def test_no_row_kernel_keeps_its_loads_in_scratch_memory():
    """A load that is parked in scratch memory has to be waited for first: kernels that ask for everything at once then make
    several trips to memory one after the other."""
    from paper_2605_00789_amd import binding as B
    rows = {k: m for k, m in _kernels(B.lib_path()).items() if "rows_kernel" in k}
    assert len(rows) >= 50
    scratch = {k: m[".private_segment_fixed_size"] for k, m in rows.items() if m[".private_segment_fixed_size"]}
    assert not scratch, scratch


def test_no_finishing_kernel_keeps_its_loads_in_scratch_memory():
    """The same for the kernels that sum the records of a split hidden axis.  One variant (sixteen records, at most four keys a
    thread) keeps three words there."""
    from paper_2605_00789_amd import binding as B
    names = ("fd_tail_select", "fd_epilogue", "colsum_tail", "colsum_edges", "edge_keys", "edge_select")
    kernels = {k: m for k, m in _kernels(B.lib_path()).items() if any(n in k for n in names)}
    assert all(any(n in k for k in kernels) for n in names)
    scratch = {k: m[".private_segment_fixed_size"] for k, m in kernels.items() if m[".private_segment_fixed_size"]}
    assert all("edge_select_kernelILi16ELi4E" in k and size <= 12 for k, size in scratch.items()), scratch

"""No-GPU check: the kernels that count their loads in flight keep everything in registers.  A spilled value is read back with a load, and the wait
behind it takes the requests for the stages ahead with it."""
import struct

import msgpack

import paper_2311_04951_amd as sv

COUNTED = ("gemm_tile_kernel", "gemm_cols_kernel", "gemm_wide_kernel", "attn_blocks_kernel")


def _kernels():
    """Name -> scratch bytes of every kernel in the built library, from the metadata note of its code objects."""
    data, out = open(sv.LIB_PATH, "rb").read(), {}
    at = data.find(b"AMDGPU\0\0")
    while at >= 0:
        name_bytes, bytes_, kind = struct.unpack("<III", data[at - 12:at])
        if name_bytes == 7 and kind == 32:
            for k in msgpack.unpackb(data[at + 8:at + 8 + bytes_])["amdhsa.kernels"]:
                out[k[".name"]] = k[".private_segment_fixed_size"]
        at = data.find(b"AMDGPU\0\0", at + 8)
    return out


def test_kernels_with_counted_waits_use_no_scratch():
    kernels = _kernels()
    counted = {n: b for n, b in kernels.items() if any(c in n for c in COUNTED)}
    assert all(any(c in n for n in counted) for c in COUNTED) and len(counted) > 200
    assert {n: b for n, b in counted.items() if b} == {}

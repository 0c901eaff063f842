"""No-GPU check: the kernels that count their loads in flight keep everything in registers.  A spilled value is read back with a load, and the wait
behind it takes the requests for the stages ahead with it."""
import struct

import msgpack

import paper_2311_04951_amd as sv

COUNTED = ("gemm_tile_kernel", "gemm_cols_kernel", "gemm_wide_kernel", "attn_blocks_kernel")


def _kernels():
    """Name -> (scratch, LDS) bytes of every kernel in the built library, from the metadata note of its code objects."""
    data, out = open(sv.LIB_PATH, "rb").read(), {}
    at = data.find(b"AMDGPU\0\0")
    while at >= 0:
        name_bytes, bytes_, kind = struct.unpack("<III", data[at - 12:at])
        if name_bytes == 7 and kind == 32:
            for k in msgpack.unpackb(data[at + 8:at + 8 + bytes_])["amdhsa.kernels"]:
                out[k[".name"]] = k[".private_segment_fixed_size"], k[".group_segment_fixed_size"]
        at = data.find(b"AMDGPU\0\0", at + 8)
    return out


def test_kernels_with_counted_waits_use_no_scratch():
    kernels = _kernels()
    counted = {n: b for n, b in kernels.items() if any(c in n for c in COUNTED)}
    assert all(any(c in n for n in counted) for c in COUNTED) and len(counted) > 200
    assert {n: b for n, b in counted.items() if b[0]} == {}


def test_two_workgroups_of_a_head_fit_a_compute_unit():
    """Heads (epilogue 0) of up to 32 rows by 128 columns, and of 48 where there are several rounds of workgroups: two rings in 160 KB of LDS."""
    lds = {rows: [b for n, (_, b) in _kernels().items() if "gemm_tile_kernelILi0E" in n and f"ELi{rows}ELi2ELi1ELi4ELi2E" in n] for rows in (2, 3)}
    assert len(lds[2]) == 3 and max(lds[2]) <= 80 * 1024                                     # bf16, int8, int4
    assert len(lds[3]) == 6 and sum(b <= 80 * 1024 for b in lds[3]) == 3

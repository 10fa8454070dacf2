"""What the compiler's metadata in the built library says of every kernel: no private segment (a kernel with one has the
runtime provide scratch memory on its queue, also at the entry point that allocates nothing) and no spilled vector register."""
import struct

import pytest

from paper_2604_04335_amd.build import LIB_PATH

msgpack = pytest.importorskip("msgpack")

NOTE = struct.pack("<I", 32) + b"AMDGPU\0\0"  # an ELF note's type (code object metadata) and name; its sizes stand before


def _kernels():
    blob = open(LIB_PATH, "rb").read()
    at = blob.find(NOTE)
    while at >= 0:
        name_size, size = struct.unpack_from("<II", blob, at - 8)
        if name_size == 7:
            desc = blob[at + len(NOTE):at + len(NOTE) + size]
            yield from msgpack.unpackb(desc, strict_map_key=False)["amdhsa.kernels"]
        at = blob.find(NOTE, at + 1)


def test_no_kernel_uses_scratch():
    kernels = {k[".name"]: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in _kernels()}
    for part in ("attn_fwd_kernel", "attn_fwd_pp_kernel", "AttnListParams", "noalloc_plan_kernel", "merge_kernel", "sp_"):
        assert any(part in n for n in kernels), part
    assert not {n: v for n, v in kernels.items() if v != (0, 0)}

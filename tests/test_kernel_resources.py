"""What the built library says of its kernels.  Its metadata: no private segment (a kernel with one has the runtime provide
scratch memory on its queue, also at the entry point that allocates nothing) and no spilled vector register.  Its
instructions: what a launch may share with others, and how far a matrix instruction is from the first reader of its result."""
import os
import re
import struct
import subprocess

import pytest

from paper_2604_04335_amd.build import LIB_PATH

msgpack = pytest.importorskip("msgpack")

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
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


def _listing(tmp_path):
    """{kernel name: its instructions} of the code object that holds the attention kernels."""
    blob = open(LIB_PATH, "rb").read()
    starts = [m.start() for m in re.finditer(re.escape(b"\x7fELF"), blob)][1:]  # the first is the host library's own
    for i, at in enumerate(starts):
        part = blob[at:starts[i + 1] if i + 1 < len(starts) else len(blob)]
        if b"attn_fwd_pp_kernel" in part and NOTE in part:
            (tmp_path / "code").write_bytes(part)
            break
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp_path / "code")], capture_output=True, text=True, check=True).stdout
    kernels, lines = {}, None
    for line in text.splitlines():
        head = re.match(r"^[0-9a-f]+ <(\w+)>:$", line)
        if head:
            lines = kernels.setdefault(head.group(1), [])
        elif lines is not None and line.strip():
            lines.append(line.split("//")[0].strip())
    return {n: v for n, v in kernels.items() if "attn_fwd" in n}


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_launches_by_formula_share_no_memory(tmp_path):
    """A pack whose items travel with the kernel takes no work counter and leaves no clock sample: nothing that calls on other
    streams could share."""
    for name, lines in _listing(tmp_path).items():
        shares = [x for x in lines if x.startswith(("global_atomic", "s_memtime", "s_memrealtime"))]
        assert (len(shares) == 0) == ("AttnListParams" in name), (name, shares)


def _registers(operand):
    m = re.match(r"^v\[?(\d+)(?::(\d+))?\]?$", operand.strip())
    return set(range(int(m.group(1)), int(m.group(2) or m.group(1)) + 1)) if m else set()


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_maxima_wait_for_their_scores(tmp_path):
    """The row maxima are inline asm, in front of which the compiler inserts no wait states.  12 of them must lie between an MFMA
    of 8 passes and a reader of its result: one per instruction, n + 1 for s_nop n; the next MFMA issues 8 after the last."""
    checked = 0
    for name, lines in _listing(tmp_path).items():
        for i, line in enumerate(lines):
            if not line.startswith("v_mfma"):
                continue
            result = _registers(line.split(None, 1)[1].split(",")[0])
            now, last = 1, 0  # in wait states since the MFMA issued
            for after in lines[i + 1:]:
                op, _, operands = after.partition(" ")
                if now > 12 or op in ("s_branch", "s_endpgm"):
                    break
                if op == "v_max3_f32":
                    checked += 1
                    assert not result & set().union(*(_registers(x) for x in operands.split(",")[1:])), (name, line, after, now - 1)
                if op.startswith("v_mfma"):
                    now = last = max(now, last + 8)
                now += int(operands) + 1 if op == "s_nop" else 1
    assert checked > 0

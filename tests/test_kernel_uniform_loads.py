"""The K loop of the tiled GEMM kernels takes its buffer loads with descriptors
and offsets in scalar registers.  (Where a uniform value has ended up in vector
registers, after a division say, the compiler makes a loop over the lanes of
every load.)  The gfx950 code objects are those built here from this
repository's sources."""

import os
import re
import subprocess

import pytest

from paper_2609_04098_amd import nvfp4 as C
from tests.test_kernel_resources import device_objects, elf_sections

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
INSN = re.compile(r"^\s+(\S+).*// ([0-9A-F]+):")
TARGET = re.compile(r"<\S+\+0x([0-9a-f]+)>\s*$")


def k_loops(asm):
    """Per kernel: for each loop (backward branch) with MFMAs, its number of
    v_readfirstlane instructions."""
    found, kernel, base, code = {}, None, 0, []
    for line in asm.splitlines():
        if line.endswith(">:"):
            kernel, code = line.split("<", 1)[1][:-2], []
            base = int(line.split(None, 1)[0], 16)
            continue
        m = INSN.match(line)
        if not m:
            continue
        op, at = m.group(1), int(m.group(2), 16)
        code.append((at, op))
        t = TARGET.search(line) if op.startswith(("s_cbranch", "s_branch")) else None
        if t and base + int(t.group(1), 16) < at:
            body = [o for a, o in code if a >= base + int(t.group(1), 16)]
            if any(o.startswith("v_mfma") for o in body):
                found.setdefault(kernel, []).append(sum(o.startswith("v_readfirstlane") for o in body))
    return found


def test_no_loop_over_lanes_in_the_k_loop(tmp_path):
    if not os.path.exists(C.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("library not built, or no llvm-objdump")
    fat = elf_sections(open(C.LIB_PATH, "rb").read())[".hip_fatbin"]
    loops = {}
    for i, co in enumerate(device_objects(fat)):
        path = tmp_path / ("%d.co" % i)
        path.write_bytes(co)
        asm = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], check=True, stdout=subprocess.PIPE).stdout
        loops.update((k, v) for k, v in k_loops(asm.decode()).items() if "gemm_lds_kernel" in k)
    assert len(loops) == 14, sorted(loops)       # every configuration, bf16 and FP32 output
    assert not any(any(v) for v in loops.values()), {k: v for k, v in loops.items() if any(v)}

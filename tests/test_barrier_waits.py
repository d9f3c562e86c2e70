"""No wave passes a barrier with LDS reads outstanding where copies into LDS
follow: a slot of a copy ring is released by a barrier, and s_barrier does not
wait for the reads that a wave has issued. Read off the library's own gfx950
code (no GPU): a straight-line count of LDS reads since the last wait."""
import os
import re
import shutil
import struct
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_04164_amd",
                   "libbrownout_moe.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

pytestmark = pytest.mark.skipif(not (os.path.exists(OBJDUMP) and shutil.which("objcopy")), reason="needs llvm-objdump and objcopy")


def device_code(lib, tmp_path):
    """The gfx950 code objects of the library (one per source)."""
    fat = str(tmp_path / "fatbin")
    subprocess.run(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", lib, fat], check=True)
    data = open(fat, "rb").read()
    out = []
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start()
        (n,), pos = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in name and size:
                out.append(str(tmp_path / f"code{len(out)}"))
                open(out[-1], "wb").write(data[at + offset:at + offset + size])
    return out


def unwaited_barriers(code):
    """{kernel: [barriers passed with LDS reads outstanding and copies into LDS before the next barrier]},
    {kernel: barriers that copies follow}."""
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", code], check=True, capture_output=True, text=True).stdout
    bad, seen = {}, {}
    kernel, reads, pending = None, 0, None
    for line in text.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
        if head:
            kernel, reads, pending = head[1], 0, None
            continue
        op = line.split("//")[0].split()
        if not op:
            continue
        if op[0].startswith("ds_read") or op[0].startswith("ds_load"):
            reads += 1
        elif op[0] == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", line)
            if m:
                reads = min(reads, int(m[1]))
        elif op[0] == "s_barrier":
            pending = (line.strip(), reads)
        elif op[0].startswith("global_load_lds") and pending:
            seen[kernel] = seen.get(kernel, 0) + 1
            if pending[1]:
                bad.setdefault(kernel, []).append(pending)
            pending = None
    return bad, seen


def test_no_lds_read_outstanding_at_a_barrier_that_frees_a_slot(tmp_path):
    bad, seen = {}, {}
    for code in device_code(LIB, tmp_path):
        b, s = unwaited_barriers(code)
        bad.update(b)
        seen.update(s)
    for name in ("route_kernel", "skinny_dma_kernel", "grouped_gemm_dma_kernel"):
        assert any(name in k for k in seen), f"no barrier of {name} found"
    assert not bad, {k: v[:2] for k, v in bad.items()}

"""The device code of the built library (this project's own kernels, disassembled): no register is saved where
a masked-off region would lose it.

A branch that only some lanes take is a region between an instruction that narrows the execution mask and one
that widens it again, at the block the lanes that skip the region jump to.  A vector register written at
the start of that block, ahead of the widening, is written for the lanes of the region only -- for none, if
none took it.  The compiler has placed the saves of registers that it ran out of there (a step counter among
them, so that a step loop did not end); kernels are written so that it does not."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2504_21440_amd.build as hipbuild

_OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
_WIDEN = re.compile(r"s_(or_b64 exec, exec|andn2_saveexec_b64|or_saveexec_b64)")
_WRITE = re.compile(r"(v_(?!cmp|cmpx|readlane|readfirstlane|writelane|nop)|scratch_|ds_|global_|flat_|buffer_)")


def _code_objects(lib):
    """The gfx950 code objects of a library's offload bundles."""
    blob = open(lib, "rb").read()
    at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + idlen] and size:
                yield blob[at + off:at + off + size]
            p += 24 + idlen
        at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _lost_writes(lines):
    """(kernel, instruction) of every vector write between the block that a skipped region's lanes jump to (or
    that a loop leaves with no lane on) and the instruction that brings the lanes back."""
    kernel, found, body = None, [], []

    def scan():
        targets = {m.group(1) for t in body for m in [re.match(r"s_cbranch_execz (\S+)", t)] if m}
        for i, t in enumerate(body):
            m = re.match(r"<(L\d+)>:", t)
            if not (m and m.group(1) in targets) and not t.startswith("s_cbranch_execnz"):
                continue
            writes = []
            for u in body[i + 1:]:
                if _WIDEN.match(u):
                    found.extend((kernel, x) for x in writes)
                    break
                if u.startswith(("<", "s_cbranch", "s_branch", "s_endpgm", "s_setpc", "s_and_saveexec",
                                 "s_mov_b64 exec", "s_and_b64 exec", "s_xor_b64 exec", "s_andn2_b64 exec")):
                    break
                if _WRITE.match(u):
                    writes.append(u)

    for line in lines:
        t = line.split("//")[0].strip()
        m = re.match(r"<(_Z\w+|[a-z]\w+)>:", t)
        if m:
            scan()
            kernel, body = m.group(1), []
        elif t:
            body.append(t)
    scan()
    return found


def test_scan_finds_a_lost_write():
    good = ["<_Zk>:", "s_and_saveexec_b64 s[0:1], vcc", "s_cbranch_execz L0", "v_mov_b32_e32 v1, v2", "<L0>:",
            "s_or_b64 exec, exec, s[0:1]", "v_accvgpr_write_b32 a1, v1"]
    bad = good[:5] + ["v_accvgpr_write_b32 a1, v1", "s_andn2_saveexec_b64 s[0:1], s[2:3]"]
    assert _lost_writes(good) == []
    assert _lost_writes(bad) == [("_Zk", "v_accvgpr_write_b32 a1, v1")]


@pytest.mark.skipif(not os.path.exists(_OBJDUMP) and not shutil.which("llvm-objdump"), reason="no disassembler")
def test_no_kernel_writes_registers_where_its_lanes_are_off(tmp_path):
    if not os.path.exists(hipbuild.LIB):
        hipbuild.build()
    tool = _OBJDUMP if os.path.exists(_OBJDUMP) else shutil.which("llvm-objdump")
    kernels, lost = 0, []
    for k, blob in enumerate(_code_objects(hipbuild.LIB)):
        obj = tmp_path / f"{k}.o"
        obj.write_bytes(blob)
        r = subprocess.run([tool, "-d", "--symbolize-operands", "--no-show-raw-insn", "--no-leading-addr", str(obj)],
                           capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-500:]
        lines = r.stdout.split("\n")
        kernels += sum(1 for t in lines if re.match(r"<_Z\w+>:", t))
        lost += _lost_writes(lines)
    assert kernels > 100  # the library was read
    assert not lost, f"{len(lost)} register writes are lost, in {sorted({n for n, _ in lost})}: {lost[:4]}"

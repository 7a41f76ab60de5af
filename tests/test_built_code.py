"""What the compiler makes of a region that some lanes execute (behind a saveexec): the block in which it ends is also
entered past it, with only those lanes active, or none.  A vector instruction placed there in front of the one that
activates all lanes again - a spilled register's reload, a constant formed anew - leaves the others' values
undefined.  Seen in a build of the 256 x 256 kernel, whose records then lost a quarter of their faults without an
error; read here off the library as it is built."""
import os
import re
import struct
import subprocess

import pytest

from paper_2311_05782_amd import fi

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LANE_OPS = ("v_writelane", "v_readlane", "v_readfirstlane", "v_cmp")    # whatever the active lanes; scalar results


def _code_objects():
    data = open(fi.LIB_PATH, "rb").read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, entry)
            if size and b"gfx950" in data[entry + 24:entry + 24 + n]:
                yield data[at + off:at + off + size]
            entry += 24 + n
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _misplaced(text):
    """(kernel, label, instruction) for every vector instruction between the target of a branch past a region and
    the end of that region."""
    found, kernel, label, waiting, skips = [], None, None, [], set()
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]* ?<(\w+)>:", line)
        if m:
            if re.fullmatch(r"L\d+", m.group(1)):
                label, waiting = m.group(1), []
            else:                                          # labels are counted per kernel
                kernel, label, skips = m.group(1), None, set(re.findall(r"s_cbranch_execz (L\d+)\b", _body(text, line)))
            continue
        op = line.split()[:1]
        if not op or label not in skips:
            continue
        op = op[0]
        if op.startswith("s_"):
            if re.match(r"\s*s_or_b64 exec, exec,", line):
                found += [(kernel, label, w) for w in waiting]
            if re.match(r"\s*s_\w+ exec\b", line) or "saveexec" in op or op.startswith(("s_cbranch", "s_branch", "s_setpc", "s_endpgm")):
                label = None
        elif not op.startswith(LANE_OPS):
            waiting.append(line.strip())
    return found


def _body(text, header):
    start = text.index(header) + len(header)
    end = re.compile(r"^[0-9a-f]* ?<(?!L\d+>)\w+>:", re.M).search(text, start)
    return text[start:end.start() if end else len(text)]


SAMPLE = """0000000000002500 <kernel>:
	s_and_saveexec_b64 s[2:3], vcc
	s_cbranch_execz L1
	global_atomic_add v1, v2, s[4:5]
0000000000002510 <L1>:
	v_writelane_b32 v9, s8, 3
	%s
	s_or_b64 exec, exec, s[2:3]
	v_mov_b32_e32 v8, 0x20000
"""


def test_the_reading_finds_what_it_looks_for():
    assert _misplaced(SAMPLE % "v_mov_b32_e32 v7, 0x20000") == [("kernel", "L1", "v_mov_b32_e32 v7, 0x20000")]
    assert _misplaced(SAMPLE % "scratch_load_dword v7, off, off") == [("kernel", "L1", "scratch_load_dword v7, off, off")]
    assert not _misplaced(SAMPLE % "s_nop 0")


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_value_is_formed_where_lanes_are_missing(tmp_path):
    n, kernels = 0, set()
    for code in _code_objects():
        path = tmp_path / ("%d.elf" % n)
        path.write_bytes(code)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(path)], check=True,
                              stdout=subprocess.PIPE, text=True).stdout
        kernels |= set(re.findall(r"<(_Z\w+)>:", text))
        assert not _misplaced(text)
        n += 1
    assert n > 10 and sum("gemm_fi_multi_kernel" in k for k in kernels) == 28

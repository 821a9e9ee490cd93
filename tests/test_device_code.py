"""Properties of the built library's gfx950 code that no run shows reliably,
read from its disassembly (CPU only: nothing is launched)."""

from __future__ import annotations

import re
import struct
import subprocess
from pathlib import Path

import pytest

from paper_2609_20971_amd import build

OBJDUMP = Path(build.HIPCC).resolve().parents[1] / "llvm" / "bin" / "llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    """Lines of every gfx950 code object of the library, one list per object."""
    if not Path(build.OUT).exists():
        build.build()
    data = Path(build.OUT).read_bytes()
    out = []
    for m in re.finditer(re.escape(MAGIC), data):
        # A bundle: magic, entry count, then per entry offset, size, triple.
        at = m.start() + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length].decode()
            at += 24 + length
            if "gfx950" in triple:
                path = tmp_path_factory.mktemp("code") / "k.co"
                path.write_bytes(data[m.start() + off:m.start() + off + size])
                text = subprocess.run([str(OBJDUMP), "-d", "--no-show-raw-insn", str(path)], check=True,
                                      stdout=subprocess.PIPE, text=True).stdout
                out.append([line.split("//")[0].strip() for line in text.splitlines()])
    assert len(out) == len(build.SOURCES)
    return out


def _is_lds_copy(line):
    op = line.split(" ")[0]
    return "load_lds" in op or (op.startswith("buffer_load") and line.endswith(" lds"))


def _sgprs(operand):
    m = re.match(r"s\[(\d+):(\d+)\]$|s(\d+)$", operand)
    if m is None:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def test_lds_copies_keep_their_wait_states(listing):
    """The wait states that the hardware leaves to the program, and the compiler
    does not add inside inline assembly: one instruction between a scalar write
    of m0 and the global -> LDS copy that takes its LDS address from it (without
    it the copy may still see the previous address), and five wait states between
    a vector instruction that writes a scalar register and the copy that reads it
    (its base address)."""
    copies, bad = 0, []
    for lines in listing:
        code = [line for line in lines if line and not line.endswith(":")]
        for k, line in enumerate(code):
            if not _is_lds_copy(line):
                continue
            copies += 1
            if re.match(r"s_\w+ m0, ", code[k - 1]):
                bad.append((code[k - 1], line))
            base = set().union(*(_sgprs(x) for x in re.split(r"[ ,]+", line)))
            states = 0
            for before in reversed(code[max(0, k - 5):k]):
                written = re.match(r"v_\w+ (s\d+|s\[\d+:\d+\]),", before)
                if states < 5 and written and _sgprs(written[1]) & base:
                    bad.append((before, line))
                nop = re.match(r"s_nop (\d+)", before)
                states += int(nop[1]) + 1 if nop else 1
    assert copies > 100  # the tile copies of the attention and selection kernels
    assert not bad, f"{len(bad)} findings in {copies} copies, e.g. {bad[0]}"

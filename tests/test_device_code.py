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
                out.append(text.splitlines())
    assert len(out) == len(build.SOURCES)
    return out


def _functions(lines):
    """(name, [(address, instruction)]) of every function of a listing."""
    out = []
    for line in lines:
        if m := re.match(r"[0-9a-f]+ <(.+)>:", line):
            out.append((m[1], []))
        elif out and (m := re.match(r"\s+(\S.*?)\s*//\s*([0-9A-F]+):", line)):
            out[-1][1].append((int(m[2], 16), m[1]))
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
        code = [text for _, code in _functions(lines) for _, text in code]
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


LDS_WRITE = re.compile(r"ds_(write|add|sub|max|min|or|and|xor|inc|dec|cmpst|wrxchg)")


def _barriers_with_writes_pending(code):
    """Barriers that some path reaches with an LDS write of the wave not waited for."""
    at = {address: k for k, (address, _) in enumerate(code)}
    pending = [None] * len(code)  # at the instruction's start, over all paths to it
    pending[0], work, bad = False, [0], set()
    while work:
        k = work.pop()
        address, text = code[k]
        op, state = text.split()[0], pending[k]
        if op == "s_barrier" and state:
            bad.add(text + f" at {address:#x}")
        if op == "s_waitcnt" and ("lgkmcnt(0)" in text or text.split()[1] == "0"):
            state = False
        elif LDS_WRITE.match(op):
            state = True
        following = [] if op in ("s_endpgm", "s_branch", "s_setpc_b64") else [k + 1]
        if re.match(r"s_c?branch", op):
            offset = int(text.split()[1])
            following.append(at[address + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)])
        for j in following:
            if j < len(code) and (pending[j] is None or state and not pending[j]):
                pending[j] = state or bool(pending[j])
                work.append(j)
    return bad


def test_lds_writes_are_waited_for_before_a_barrier(listing):
    """A barrier publishes a wave's LDS writes only if the wave has waited for
    them.  The compiler does that for __syncthreads, but where a wait of the
    program's own stands directly before it, its wait for LDS was lost on the way
    round a loop: the waves of a shared row read each other's pairs too early, and
    a few lists in a million differed from run to run."""
    barriers, bad = 0, []
    for lines in listing:
        for name, code in _functions(lines):
            barriers += sum(text == "s_barrier" for _, text in code)
            bad += [(name, x) for x in _barriers_with_writes_pending(code)]
    assert barriers > 100
    assert not bad, f"{len(bad)} barriers, e.g. {bad[0]}"

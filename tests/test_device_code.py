"""Properties of the built gfx950 code that the compiler does not see to by
itself, read from the disassembly of libssa.so's own code objects.  No GPU."""
import os
import re
import struct
import subprocess

import pytest

from paper_2606_05933_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{symbol: [(address, instruction text)]} of every function of every code object."""
    if not os.path.exists(build.LIB):
        build.build()
    data = open(build.LIB, "rb").read()
    out, at = {}, data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    tmp = tmp_path_factory.mktemp("code")
    while at >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + n].decode()
            p += 24 + n
            if "gfx950" not in target or not size:
                continue
            co = tmp / f"{at}.co"
            co.write_bytes(data[at + off:at + off + size])
            name = None
            for line in subprocess.run([OBJDUMP, "-d", str(co)], capture_output=True, text=True,
                                       check=True).stdout.splitlines():
                m = re.match(r"[0-9a-f]+ <(.*)>:", line)
                if m:
                    name = (at, m.group(1))
                    out[name] = []
                elif name and "//" in line:
                    text, _, rest = line.partition("//")
                    out[name].append((int(rest.split(":")[0], 16), text.strip()))
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    return out


def test_lds_copies_never_follow_an_m0_write_directly(kernels):
    """A scalar write of M0 and a global -> LDS load need one wait state between
    them, which the compiler does not supply for inline assembly."""
    copies, bad = 0, []
    for name, code in kernels.items():
        text = [ins for _, ins in code]
        for before, ins in zip([""] + text, text):
            if ins.startswith("global_load_lds"):
                copies += 1
                if re.match(r"\S+\s+m0\b", before):
                    bad.append((name[1], before, ins))
    assert copies > 1000
    assert not bad, (len(bad), bad[:3])


def vgprs(text):
    """Vector registers an instruction names."""
    regs = set()
    for lo, hi in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        regs.update(range(int(lo), int(hi) + 1))
    return regs | {int(r) for r in re.findall(r"\bv(\d+)\b", text)}


def first_use_in_flight(code, at_of, start):
    """The first instruction, on any path from the load code[start], that names one
    of its destination registers before a wait that covers the load (its count is
    at most the vector-memory operations issued since); None if there is none."""
    dest = vgprs(code[start][1].split(",")[0])
    seen, todo = set(), [(start + 1, 0)]
    while todo:
        i, younger = todo.pop()
        if (i, younger) in seen or i >= len(code):
            continue
        seen.add((i, younger))
        addr, ins = code[i]
        op = ins.split()[0]
        wait = re.search(r"vmcnt\((\d+)\)", ins)
        if op == "s_endpgm" or (wait and int(wait.group(1)) <= younger):
            continue
        if dest & vgprs(ins):
            return ins
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            younger = min(younger + 1, 63)
        if op.startswith(("s_branch", "s_cbranch")):
            off = int(ins.split()[1])
            todo.append((at_of[addr + 4 + 4 * (off - 65536 if off >= 32768 else off)], younger))
        if op != "s_branch":
            todo.append((i + 1, younger))
    return None


def test_streamed_loads_keep_their_registers_until_they_land(kernels):
    """The decode items' value loads are inline assembly, so the compiler takes
    their destinations as written when they are issued: nothing may read or
    overwrite them before the wait, on no path, and not those of the last loads,
    whose values go unused."""
    loads, bad = 0, []
    for name, code in kernels.items():
        if "attention_kernel" not in name[1]:
            continue
        at_of = {addr: i for i, (addr, _) in enumerate(code)}
        for i, (_, ins) in enumerate(code):
            if re.match(r"global_load_dwordx4 .* off nt$", ins):
                loads += 1
                use = first_use_in_flight(code, at_of, i)
                if use:
                    bad.append((name[1][:60], ins, use))
    assert loads >= 4 * 3 * 4
    assert not bad, (len(bad), bad[:3])

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
    """{symbol: [instruction text]} of every function of every code object."""
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
                elif name and line.startswith("\t"):
                    out[name].append(line.split("//")[0].strip())
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    return out


def test_lds_copies_never_follow_an_m0_write_directly(kernels):
    """A scalar write of M0 and a global -> LDS load need one wait state between
    them, which the compiler does not supply for inline assembly."""
    copies, bad = 0, []
    for name, code in kernels.items():
        for before, ins in zip([""] + code, code):
            if ins.startswith("global_load_lds"):
                copies += 1
                if re.match(r"\S+\s+m0\b", before):
                    bad.append((name[1], before, ins))
    assert copies > 1000
    assert not bad, (len(bad), bad[:3])

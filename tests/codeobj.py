"""What the built library's own device code says of itself: register and scratch use from
the code objects' metadata, and their instructions."""
from __future__ import annotations

import os
import re
import struct
import subprocess
import tempfile

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(lib: str):
    """The gfx950 code objects of a library's fat binaries, as bytes."""
    data = open(lib, "rb").read()
    out, at = [], data.find(MAGIC)
    while at >= 0:
        (n,), p = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + tlen]:
                out.append(data[at + off:at + off + size])
            p += 24 + tlen
        at = data.find(MAGIC, at + 24)
    return out


def _tool(args, code: bytes) -> str:
    with tempfile.NamedTemporaryFile(suffix=".co") as f:
        f.write(code)
        f.flush()
        return subprocess.run([os.path.join(LLVM, args[0])] + args[1:] + [f.name], stdout=subprocess.PIPE,
                              text=True, check=True).stdout


def _demangle(names):
    out = subprocess.run(["c++filt"], input="\n".join(names), stdout=subprocess.PIPE, text=True, check=True).stdout
    # "void ct::kernel<1, true>(float const*, ...)" -> "kernel<1, true>"
    return [re.sub(r"^(?:void )?ct::", "", n).split("(")[0] for n in out.splitlines()]


def kernel_resources(lib: str) -> dict:
    """{kernel: {metadata key: value}} of every kernel in the library."""
    keys = ("private_segment_fixed_size", "vgpr_count", "sgpr_count", "vgpr_spill_count", "sgpr_spill_count")
    out = {}
    for code in code_objects(lib):
        notes = _tool(["llvm-readelf", "--notes"], code).split("  - .agpr_count:")[1:]
        names = _demangle([re.search(r"\.name:\s+(\S+)", k).group(1) for k in notes])
        for name, k in zip(names, notes):
            out[name] = {key: int(re.search(r"\.%s:\s+(\d+)" % key, k).group(1)) for key in keys}
    return out


def instructions(lib: str, family: str):
    """(kernel symbol, [(address, opcode, operands, branch target or None)]) of every
    kernel whose symbol holds `family`."""
    for code in code_objects(lib):
        if family.encode() not in code:
            continue
        for part in re.split(r"\n(?=[0-9a-f]{16} <)", _tool(["llvm-objdump", "-d"], code))[1:]:
            head, body = part.split("\n", 1)
            start, sym = int(head[:16], 16), head[18:-2]
            if family not in sym:
                continue
            rows = []
            for line in body.splitlines():
                m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):.*?(?:<.*\+0x([0-9a-f]+)>)?$", line)
                if m:
                    op, args, addr, to = m.groups()
                    rows.append((int(addr, 16), op, args, start + int(to, 16) if to else None))
            yield sym, rows

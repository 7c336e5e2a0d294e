"""The device code inside the built library: its kernels' resources and instructions, as the compiler left them."""
import os
import re
import struct
import subprocess
import tempfile

from paper_2507_22424_amd import build as b

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _images():
    """The gfx950 ELF images of the library, one per source file that has kernels."""
    with open(b.LIB_PATH, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        n, p = struct.unpack_from("<Q", data, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                yield data[at + offset:at + offset + size]
            p += 24 + length
        at = data.find(MAGIC, at + 1)


def _tool(name, *args):
    """Output of an LLVM tool for each image."""
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "image")
        for image in _images():
            with open(path, "wb") as f:
                f.write(image)
            yield subprocess.run([os.path.join(LLVM, name), *args, path], check=True, capture_output=True, text=True).stdout


def short_name(symbol):
    """_ZN2sv8gemm_midILi3ELi1ELi3ELi0EEEv... -> gemm_mid<3,1,3,0>"""
    m = re.match(r"_ZN2sv(\d+)(\w+)", symbol)
    if not m:
        return symbol
    name, rest = m[2][:int(m[1])], m[2][int(m[1]):]
    args = re.match(r"I((?:Li\d+E)+)E", rest)
    return name + ("<" + ",".join(re.findall(r"Li(\d+)E", args[1])) + ">" if args else "")


def instructions():
    """Of every kernel: (name, [(address, mnemonic and operands, address a branch goes to or None)])."""
    for text in _tool("llvm-objdump", "-d"):
        for part in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            symbol, body = part.split(">:", 1)
            lines = re.findall(r"^\t(\S.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(?:<\S+?(?:\+0x([0-9a-f]+))?>)?\s*$", body, re.M)
            start = int(lines[0][1], 16) if lines else 0
            yield short_name(symbol), [(int(a, 16), op, start + int(t or "0", 16) if "branch" in op else None) for op, a, t in lines]


def scratch_bytes():
    """Of every kernel: (name, bytes of scratch memory a lane needs)."""
    for text in _tool("llvm-readelf", "--notes"):
        for part in re.split(r"^  - ", text, flags=re.M):
            symbol = re.search(r"^\s+\.symbol:\s+(\S+)\.kd$", part, re.M)
            if symbol:
                yield short_name(symbol[1]), int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", part)[1])

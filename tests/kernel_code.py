"""The device code of the built library: its kernels' instructions and the registers they were given."""
import os
import re
import struct
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

from paper_2207_04604_amd import build

LLVM = "/opt/rocm/llvm/bin/"


def _objects():
    """The gfx950 code objects in the library's offload bundles."""
    if not os.path.exists(build.OUT):
        build.build_library()
    data = open(build.OUT, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        count, = struct.unpack_from("<Q", data, m.end())
        at = m.end() + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            if size and b"gfx950" in data[at + 24:at + 24 + length]:
                yield data[m.start() + offset:m.start() + offset + size]
            at += 24 + length


def _tool(args, code):
    with tempfile.NamedTemporaryFile(suffix=".o") as f:
        f.write(code)
        f.flush()
        return subprocess.run([LLVM + args[0], *args[1:], f.name], check=True, capture_output=True, text=True).stdout


def _names(mangled):
    """Readable names without their arguments: k_share<Engine<ArithS, 13, 3, 13, false> >."""
    out = subprocess.run(["c++filt"], input="\n".join(mangled), check=True, capture_output=True, text=True).stdout
    return [n.split("(")[0].replace("void d2::", "").replace("d2::", "") for n in out.split("\n")]


def _each_object(read):
    found = {}
    with ThreadPoolExecutor(max_workers=4) as pool:
        for part in pool.map(read, _objects()):
            found.update(part)
    return dict(zip(_names(found), found.values()))


def instructions(select):
    """{kernel: select(its disassembly)}"""
    def read(code):
        text = _tool(["llvm-objdump", "-d", "--no-show-raw-insn"], code)
        parts = re.split(r"^[0-9a-f]+ <(\S+)>:\n", text, flags=re.M)
        return {name: select(body) for name, body in zip(parts[1::2], parts[2::2])}
    return _each_object(read)


def registers():
    """{kernel: (vector registers, of them spilled)}"""
    def read(code):
        found = {}
        for entry in _tool(["llvm-readelf", "--notes"], code).split("- .agpr_count")[1:]:
            number = lambda key: int(re.search(r"\.%s:\s+(\d+)" % key, entry).group(1))
            found[re.search(r"\.symbol:\s+(\S+)\.kd", entry).group(1)] = (number("vgpr_count"), number("vgpr_spill_count"))
        return found
    return _each_object(read)

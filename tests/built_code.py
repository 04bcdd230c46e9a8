"""What the tests read of the library built here: its bundled code objects and
the registers of its kernels (holds no test of its own)."""
import re
import shutil
import struct
import subprocess


def llvm_tool(name):
    return shutil.which(name) or f"/opt/rocm/llvm/bin/{name}"


def code_objects(lib):
    """The gfx950 code objects bundled in the library."""
    data = open(lib, "rb").read()
    at, out = 0, []
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        (n,), p = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length] and size:
                out.append(data[at + off:at + off + size])
            p += 24 + length
        at += 24
    return out


def kernel_registers(lib, tmp):
    """{mangled kernel name: (vector registers, spilled ones)} from the notes."""
    out = {}
    for i, obj in enumerate(code_objects(lib)):
        path = tmp / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([llvm_tool("llvm-readelf"), "--notes", str(path)], capture_output=True, text=True,
                               check=True).stdout
        for k in notes.split(".agpr_count:")[1:]:
            def field(f):
                return re.search(rf"\.{f}:\s+(\S+)", k)[1]
            out[field("name")] = (int(field("vgpr_count")), int(field("vgpr_spill_count")))
    return out

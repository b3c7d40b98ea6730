"""The gfx950 code inside the built library, for tests of what the compiler made."""
import os
import re
import shutil
import struct
import subprocess

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def tool(name):
    return shutil.which(name) or os.path.join("/opt/rocm/llvm/bin", name)


def library():
    import paper_2201_03611_amd as rise

    return os.path.join(os.path.dirname(rise.__file__), "librise.so")


def code_objects(path):
    """The gfx950 code objects of a library of offload bundles."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            ident = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in ident and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + len(MAGIC))


def kernels(path, tmp_path):
    """{mangled name: {field: number}} of the kernels' metadata (registers, LDS, scratch)."""
    out = {}
    for i, code in enumerate(code_objects(path)):
        obj = tmp_path / f"{i}.co"
        obj.write_bytes(code)
        notes = subprocess.run([tool("llvm-readelf"), "--notes", str(obj)], capture_output=True,
                               text=True, check=True).stdout
        for entry in re.split(r"\n  - (?=\.)", notes)[1:]:
            fields = dict(re.findall(r"^\s*\.(\w+):\s+(\S+)$", entry, flags=re.M))
            # a kernel's own fields follow those of its arguments
            name = re.search(r"^    \.name:\s+(\S+)$", entry, flags=re.M)
            if name and "vgpr_count" in fields:
                out[name[1]] = {k: int(v) for k, v in fields.items() if v.isdigit()}
    return out

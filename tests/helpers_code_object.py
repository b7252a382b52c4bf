"""Resource notes of the kernels in the built library (CPU only)."""
import functools
import re
import struct
import subprocess
import tempfile

import paper_2602_02071_amd as baps

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects(data):
    """The gfx950 code objects of a library linked by hipcc (one bundle per source)."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + tl]:
                yield data[at + off:at + off + size]
            p += 24 + tl
        at = data.find(magic, p)


@functools.lru_cache(maxsize=None)
def kernel_resources():
    """{demangled kernel name: dict(vgpr, spill, scratch, lds)} of the library."""
    out = {}
    for co in _code_objects(open(baps.LIB_PATH, "rb").read()):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(co)
            f.flush()
            txt = subprocess.run([READELF, "--notes", "--demangle", f.name], capture_output=True, text=True, check=True).stdout
        for part in txt.split("  - .agpr_count:")[1:]:
            def val(key):
                return re.search(r"^\s+\.%s:\s+'?([^'\n]+?)'?\s*$" % key, part, re.M).group(1)
            out[val("name")] = dict(vgpr=int(val("vgpr_count")), spill=int(val("vgpr_spill_count")),
                                    scratch=int(val("private_segment_fixed_size")),
                                    lds=int(val("group_segment_fixed_size")))
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True, check=True).stdout.split("\n")
    return {n.replace("baps::(anonymous namespace)::", ""): v for n, v in zip(names, out.values())}

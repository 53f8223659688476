"""What the built library's own device code (gfx950) has to look like where the sources rely on it: register spills of the
tiled kernels."""
import os
import re
import struct
import subprocess

import pytest

from paper_2508_19373_amd import binding as B

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    """The gfx950 code object of expert_ffn.hip, taken out of the library's offload bundles."""
    for tool in ("llvm-objdump", "llvm-readelf"):
        if not os.path.exists(os.path.join(LLVM, tool)):
            pytest.skip("no " + tool)
    if not os.path.exists(B._LIB_PATH):
        import __graft_entry__ as g
        g.build()
    data, magic, at = open(B._LIB_PATH, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, id_len = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + id_len]
            p += 24 + id_len
            blob = data[at + off:at + off + size]
            if b"gfx950" in target and b"grouped_gemm_tall_kernel" in blob:
                path = tmp_path_factory.mktemp("co") / "expert_ffn.elf"
                path.write_bytes(blob)
                return str(path)
        at += len(magic)
    pytest.fail("no device code with the tiled kernels in " + B._LIB_PATH)


def _tool(name, *args):
    return subprocess.run([os.path.join(LLVM, name), *args], capture_output=True, text=True, check=True).stdout


def test_tiled_kernels_do_not_spill(code_object):
    """At 256 + 256 registers a little more address arithmetic spills; the plain gate/up projection has had one spilled
    register, outside its k-loop, from the start, the others none."""
    notes = _tool("llvm-readelf", "--notes", code_object)
    spills = {}
    for kernel in re.split(r"- \.agpr_count:", notes)[1:]:
        name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
        spills[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    plain = {n: s for n, s in spills.items() if "grouped_gemm_dlds_kernel" in n or "grouped_gemm_even_kernel" in n}
    assert len(plain) == 7
    for name, n in plain.items():
        assert n <= (1 if "grouped_gemm_dlds_kernelILi256ELb1E" in name else 0), (name, n)
    tall = {n: s for n, s in spills.items() if "grouped_gemm_tall_kernel" in n}
    assert len(tall) == 4 and all(s <= 2 for s in tall.values()), tall

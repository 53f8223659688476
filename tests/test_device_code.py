"""What the built library's own device code (gfx950) has to look like where the sources rely on it: register spills of the
tiled kernels, and the waits around matrix instructions that the compiler does not know to be any."""
import os
import re
import struct
import subprocess

import pytest

from paper_2508_19373_amd import binding as B

LLVM = "/opt/rocm/llvm/bin"


def _code_object(tmp_path_factory, kernel):
    """The gfx950 code object with this kernel, taken out of the library's offload bundles."""
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
            if b"gfx950" in target and kernel in blob:
                path = tmp_path_factory.mktemp("co") / "expert_ffn.elf"
                path.write_bytes(blob)
                return str(path)
        at += len(magic)
    pytest.fail("no device code with %s in %s" % (kernel.decode(), B._LIB_PATH))


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    """That of expert_ffn.hip."""
    return _code_object(tmp_path_factory, b"grouped_gemm_tall_kernel")


@pytest.fixture(scope="module")
def flow_code_object(tmp_path_factory):
    """That of expert_flow.hip."""
    return _code_object(tmp_path_factory, b"grouped_flow_kernel")


def _tool(name, *args):
    return subprocess.run([os.path.join(LLVM, name), *args], capture_output=True, text=True, check=True).stdout


def _spills(code_object):
    notes = _tool("llvm-readelf", "--notes", code_object)
    spills = {}
    for kernel in re.split(r"- \.agpr_count:", notes)[1:]:
        name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
        spills[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    return spills


def test_tiled_kernels_do_not_spill(code_object):
    """At 256 + 256 registers a little more address arithmetic spills; the plain gate/up projection has had one spilled
    register, outside its k-loop, from the start, the others none."""
    spills = _spills(code_object)
    plain = {n: s for n, s in spills.items() if "grouped_gemm_dlds_kernel" in n or "grouped_gemm_even_kernel" in n}
    assert len(plain) == 7
    for name, n in plain.items():
        assert n <= (1 if "grouped_gemm_dlds_kernelILi256ELb1E" in name else 0), (name, n)
    tall = {n: s for n, s in spills.items() if "grouped_gemm_tall_kernel" in n}
    assert len(tall) == 4 and all(s <= 2 for s in tall.values()), tall
    # the gate/up projections whose walks over K begin apart: as those that they stand in for
    spread = {n: s for n, s in spills.items() if "grouped_gemm_spread_kernel" in n}
    assert len(spread) == 1 and all(s <= 1 for s in spread.values()), spread
    spread = {n: s for n, s in spills.items() if "grouped_gemm_spread_tall_kernel" in n}
    assert len(spread) == 1 and all(s <= 2 for s in spread.values()), spread


def test_streaming_tiles_do_not_spill(flow_code_object):
    """A spilled register of theirs would be read and written in every k-tile."""
    flow = {n: s for n, s in _spills(flow_code_object).items() if "grouped_flow_kernel" in n}
    assert len(flow) == 10 and not any(flow.values()), flow


def _regs(operand):
    """Vector registers an operand names."""
    m = re.fullmatch(r"-?\|?v(?:\[(\d+):(\d+)\]|(\d+))\|?", operand)
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


class _Instr:
    def __init__(self, line, start):
        text, _, comment = line.strip().partition("//")
        self.addr = int(comment.split(":")[0], 16) - start
        self.op, _, rest = text.strip().partition(" ")
        self.operands = [o.strip() for o in rest.split(",")] if rest else []
        target = re.search(r"<[^>+]+(?:\+0x([0-9a-fA-F]+))?>", comment)
        self.target = int(target.group(1) or "0", 16) if target and self.op.startswith(("s_branch", "s_cbranch")) else None
        self.mfma = self.op.startswith("v_mfma")
        self.states = int(self.operands[0]) + 1 if self.op == "s_nop" else 1


def _tall_kernels(code_object):
    kernels, cur = {}, None
    for line in _tool("llvm-objdump", "-d", code_object).splitlines():
        head = re.match(r"([0-9a-f]+) <(\S+)>:", line)
        if head:
            cur = None
            if re.search("grouped_gemm_(spread_)?tall_kernel", head.group(2)):
                start = int(head.group(1), 16)
                cur = kernels.setdefault(head.group(2), [])
        elif cur is not None and line.startswith("\t") and "//" in line:
            cur.append(_Instr(line, start))
    return kernels


def test_matrix_instructions_in_inline_assembly_keep_their_distance(code_object):
    """The extra rows of a tall tile accumulate in vector registers through inline assembly, and the compiler inserts no
    waits for it.  Nobody may touch such a result within the instruction's latency (8 passes of 4 cycles, 11 wait states
    before an access by anything but the next MFMA on the same accumulator; asked for here: 16 instructions), and no
    vector instruction may write an operand within the 2 wait states before it."""
    kernels = _tall_kernels(code_object)
    assert len(kernels) == 5
    for name, code in kernels.items():
        index = {ins.addr: i for i, ins in enumerate(code)}
        own = [i for i, ins in enumerate(code) if ins.mfma and ins.operands[0].startswith("v")]
        assert len(own) > 100, name
        for i in own:
            dst = _regs(code[i].operands[0])
            assert code[i].operands[3] == code[i].operands[0]
            todo, seen = [(i + 1, 16)], set()
            while todo:
                at, left = todo.pop()
                if left <= 0 or at >= len(code) or (at, left) in seen:
                    continue
                seen.add((at, left))
                ins = code[at]
                touched = [o for o in ins.operands if _regs(o) & dst]
                if ins.mfma and ins.operands[0] == code[i].operands[0]:
                    assert not any(_regs(o) & dst for o in ins.operands[1:3]), (name, hex(ins.addr))
                else:
                    assert not touched, (name, hex(code[i].addr), ins.op, ins.operands)
                if ins.op == "s_endpgm":
                    continue
                if ins.target is not None:
                    todo.append((index[ins.target], left - 1))
                if ins.op != "s_branch":
                    todo.append((at + 1, left - ins.states))
            sources, at, left = _regs(code[i].operands[1]) | _regs(code[i].operands[2]) | dst, i - 1, 2
            while left > 0:
                ins = code[at]
                if ins.op.startswith("v_") and not ins.mfma and not ins.op.startswith("v_cmp"):
                    assert not _regs(ins.operands[0]) & sources, (name, hex(code[i].addr), ins.op, ins.operands)
                left, at = left - ins.states, at - 1

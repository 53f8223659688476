"""The C-ABI library loads without a GPU, exports every symbol the header declares, and
rejects invalid arguments on the host before any device call."""
import ctypes
import os
import re

import pytest

from paper_2508_19373_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B._LIB_PATH):
        import __graft_entry__ as g
        g.build()
    return B.lib()


def _declared_functions(header="moe_shard.h"):
    src = open(os.path.join(ROOT, "include", header)).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(moe_[a-z0-9_]+)\s*\(", src)))


def test_every_declared_symbol_is_exported(lib):
    names = _declared_functions()
    assert set(names) == set(B.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_every_declared_debug_symbol_is_exported(lib):
    names = _declared_functions("moe_shard_debug.h")
    assert set(names) == set(B.DEBUG_EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None
    src = open(os.path.join(ROOT, "include", "moe_shard_debug.h")).read()
    assert int(re.search(r"MOE_DEBUG_UNIT_INTS\s+(\d+)", src).group(1)) == B.DEBUG_UNIT_INTS


def test_every_declared_int4_symbol_is_exported_and_validates(lib):
    names = _declared_functions("moe_int4.h")
    assert set(names) == set(B.INT4_EXPORTS)
    src = open(os.path.join(ROOT, "include", "moe_int4.h")).read()
    assert int(re.search(r"MOE_INT4_GROUP\s+(\d+)", src).group(1)) == B.INT4_GROUP
    P = 0x1000
    dq, q = lib.moe_int4_dequantize, lib.moe_int4_quantize
    assert dq(P, P, 100, P, None) == B.MOE_ERR_INVALID_ARG      # not a multiple of the group size
    assert dq(P, P, -64, P, None) == B.MOE_ERR_INVALID_ARG
    assert dq(None, P, 64, P, None) == B.MOE_ERR_INVALID_ARG
    assert dq(P, P, 64, P + 8, None) == B.MOE_ERR_INVALID_ARG   # misaligned
    assert dq(P, P, 0, P, None) == B.MOE_OK                     # empty: nothing launched
    assert q(P, 96, P, P, None) == B.MOE_ERR_INVALID_ARG
    assert q(P, 64, None, P, None) == B.MOE_ERR_INVALID_ARG
    assert q(P, 0, P, P, None) == B.MOE_OK


def test_header_constants_match_binding():
    src = open(os.path.join(ROOT, "include", "moe_shard.h")).read()
    for name in ("MOE_ERR_INVALID_ARG", "MOE_ERR_UNSUPPORTED_SHAPE", "MOE_ERR_WORKSPACE", "MOE_ERR_HIP"):
        m = re.search(name + r"\s*=\s*(-?\d+)", src)
        assert int(m.group(1)) == getattr(B, name)
    for name in ("MOE_RENORM_TOPK", "MOE_LOGITS_GIVEN", "MOE_Y_PERM_BF16", "MOE_OUT_F32", "MOE_FFN_SKIP_GATEUP",
                 "MOE_FFN_SKIP_DOWN", "MOE_FFN_TILED", "MOE_FFN_LEAVE_ROOM", "MOE_NO_COMBINE"):
        m = re.search(name + r"\s*=\s*1u\s*<<\s*(\d+)", src)
        assert 1 << int(m.group(1)) == getattr(B, name)
    assert ctypes.sizeof(B.MoeShard) == 24


def test_status_strings(lib):
    assert B.status_string(0) == "ok"
    for s in (-1, -2, -3, -4):
        assert B.status_string(s) not in ("ok", "unknown status")
    assert B.status_string(-99) == "unknown status"


P = 0x1000  # a fake, aligned, non-null "device pointer": validation must fail before it is touched


def test_route_topk_validation(lib):
    f = lib.moe_route_topk
    assert f(P, P, P, 4, 64, 8, 0, 0, P, P, None) == B.MOE_ERR_INVALID_ARG       # k < 1
    assert f(P, P, P, 4, 64, 8, 9, 0, P, P, None) == B.MOE_ERR_INVALID_ARG       # k > E
    assert f(P, P, P, 4, 64, 300, 2, 0, P, P, None) == B.MOE_ERR_INVALID_ARG     # E too large
    assert f(P, P, P, -1, 64, 8, 2, 0, P, P, None) == B.MOE_ERR_INVALID_ARG      # T < 0
    assert f(None, P, P, 4, 64, 8, 2, 0, P, P, None) == B.MOE_ERR_INVALID_ARG    # x missing
    assert f(P, P, None, 4, 64, 8, 2, 0, P, P, None) == B.MOE_ERR_INVALID_ARG    # logits missing
    assert f(P, P, P, 4, 60, 8, 2, 0, P, P, None) == B.MOE_ERR_UNSUPPORTED_SHAPE  # H % 8
    assert f(P, P, P, 4, 64, 8, 2, 1 << 7, P, P, None) == B.MOE_ERR_INVALID_ARG  # unknown flag
    assert f(P + 2, P, P, 4, 64, 8, 2, 0, P, P, None) == B.MOE_ERR_INVALID_ARG   # misaligned x


def _shard(**kw):
    d = dict(n_experts=8, n_local_experts=8, expert_offset=0, hidden=512, inter_full=1024, inter_slice=1024)
    d.update(kw)
    return B.MoeShard(**d)


@pytest.mark.parametrize("bad", [
    dict(n_local_experts=0), dict(n_local_experts=3), dict(expert_offset=-1),
    dict(n_local_experts=4, expert_offset=6), dict(inter_slice=300), dict(inter_slice=2048),
    dict(n_experts=0), dict(n_experts=512, n_local_experts=512), dict(hidden=0),
])
def test_shard_descriptor_validation(lib, bad):
    s = _shard(**bad)
    assert B.moe_workspace_bytes(4, 2, s) == 0
    assert lib.moe_permute(P, P, 4, 2, ctypes.byref(s), P, P, P, P, P, 1024, None) == B.MOE_ERR_INVALID_ARG
    assert lib.moe_expert_ffn(P, P, 8, ctypes.byref(s), P, P, P, P, P, P, 1 << 30, 0, None) == B.MOE_ERR_INVALID_ARG


def test_permute_validation(lib):
    s = _shard()
    need = B.moe_workspace_bytes(4, 2, s)
    assert need > 0
    f = lib.moe_permute
    assert f(P, P, 4, 2, None, P, P, P, P, P, need, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, 4, 2, ctypes.byref(s), P, P, P, P, P, need - 1, None) == B.MOE_ERR_WORKSPACE
    assert f(P, P, 4, 2, ctypes.byref(s), P, P, P, P, None, need, None) == B.MOE_ERR_WORKSPACE
    assert f(P, None, 4, 2, ctypes.byref(s), P, P, P, P, P, need, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, 4, 17, ctypes.byref(s), P, P, P, P, P, need, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, 1 << 23, 2, ctypes.byref(s), P, P, P, P, P, need, None) == B.MOE_ERR_INVALID_ARG
    s2 = _shard(hidden=12)
    assert f(P, P, 4, 2, ctypes.byref(s2), P, P, P, P, P, need, None) == B.MOE_ERR_UNSUPPORTED_SHAPE
    # a permuted copy needs x; without one (index arrays only) x may be missing too
    assert f(None, P, 4, 2, ctypes.byref(s), P, P, P, P, P, need, None) == B.MOE_ERR_INVALID_ARG
    assert f(None, P, 4, 2, ctypes.byref(s), None, P, None, P, P, need, None) == B.MOE_ERR_INVALID_ARG   # row_src missing


def test_expert_ffn_validation(lib):
    f = lib.moe_expert_ffn
    s = _shard()
    W = 1 << 30
    assert f(P, P, -1, ctypes.byref(s), P, P, P, P, P, P, W, 0, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, 8, ctypes.byref(s), P, None, P, P, P, P, W, 0, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, 8, ctypes.byref(s), P, P, P, P, P, P, W, B.MOE_OUT_F32, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, 8, ctypes.byref(_shard(hidden=520)), P, P, P, P, P, P, W, 0, None) == B.MOE_ERR_UNSUPPORTED_SHAPE
    assert f(P, P, 8, ctypes.byref(_shard(inter_full=1000, inter_slice=500)), P, P, P, P, P, P, W, 0, None) \
        == B.MOE_ERR_UNSUPPORTED_SHAPE
    assert f(P, P, 8, ctypes.byref(s), P, P, P + 8, P, P, P, W, 0, None) == B.MOE_ERR_INVALID_ARG
    # the scheduling hints are accepted (an empty call: nothing is launched), unknown bits are not
    hints = B.MOE_FFN_TILED | B.MOE_FFN_LEAVE_ROOM
    assert f(P, P, 0, ctypes.byref(s), P, P, P, P, P, P, W, hints, None) == B.MOE_OK
    assert f(P, P, 0, ctypes.byref(s), P, P, P, P, P, P, W, 1 << 8, None) == B.MOE_ERR_INVALID_ARG
    # decode-sized call on a Mixtral-shaped shard needs split-K scratch; a prefill-sized one room for the
    # partial sums of tiles cut along K (65536 / 16 column blocks rows, whatever the capacity)
    mix = _shard(hidden=4096, inter_full=14336, inter_slice=14336)
    need = B.moe_ffn_workspace_bytes(32, mix)
    # streaming kernel: 16 wavefronts x 14 k-steps x 2 K slices of 32 rows; the tiled kernels, which
    # MOE_FFN_TILED may ask for, up to 15 further slices of the 32 rows: the larger of the two
    assert need == max(2 * 32 * 4096 * 4, 15 * 32 * 4096 * 4)
    assert B.moe_ffn_workspace_bytes(8192, mix) == 4096 * 4096 * 4
    assert B.moe_ffn_workspace_bytes(8192, _shard(hidden=4096, inter_full=512, inter_slice=512)) == 0   # K too short to cut
    # a single expert with a few hundred rows: the tiled down projection is cut along K
    one = _shard(n_experts=1, n_local_experts=1, hidden=3584, inter_full=20480, inter_slice=20480)
    assert B.moe_ffn_workspace_bytes(1024, one) == (65536 // 14) * 3584 * 4   # up to 16 slices, all but the first in scratch
    assert f(P, P, 32, ctypes.byref(mix), P, P, P, P, P, None, 0, 0, None) == B.MOE_ERR_WORKSPACE
    assert f(P, P, 32, ctypes.byref(mix), P, P, P, P, P, P, need - 1, 0, None) == B.MOE_ERR_WORKSPACE


def test_expert_ffn_gather_validation(lib):
    f = lib.moe_expert_ffn_gather
    s = _shard()
    W = 1 << 30
    assert f(P, None, 2, P, 8, ctypes.byref(s), P, P, P, P, P, P, W, 0, None) == B.MOE_ERR_INVALID_ARG    # no row map
    assert f(P, P, 0, P, 8, ctypes.byref(s), P, P, P, P, P, P, W, 0, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, 17, P, 8, ctypes.byref(s), P, P, P, P, P, P, W, 0, None) == B.MOE_ERR_INVALID_ARG
    assert f(None, P, 2, P, 8, ctypes.byref(s), P, P, P, P, P, P, W, 0, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, 2, P, -1, ctypes.byref(s), P, P, P, P, P, P, W, 0, None) == B.MOE_ERR_INVALID_ARG
    mix = _shard(hidden=4096, inter_full=14336, inter_slice=14336)
    assert f(P, P, 2, P, 32, ctypes.byref(mix), P, P, P, P, P, None, 0, 0, None) == B.MOE_ERR_WORKSPACE


def test_combine_validation(lib):
    f = lib.moe_combine
    assert f(P, P, P, 4, 2, 512, None, None, None, None, 0, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, P, 4, 2, 512, P, P, None, P, 0, None) == B.MOE_ERR_INVALID_ARG   # x without w_s
    assert f(P, P, P, 4, 2, 512, None, P, P, P, 0, None) == B.MOE_ERR_INVALID_ARG   # gate without y_shared
    assert f(P, P, P, 4, 2, 510, None, None, None, P, 0, None) == B.MOE_ERR_UNSUPPORTED_SHAPE
    assert f(P, P, P, 4, 0, 512, None, None, None, P, 0, None) == B.MOE_ERR_INVALID_ARG
    assert f(P, P, P, 4, 2, 512, None, None, None, P, B.MOE_RENORM_TOPK, None) == B.MOE_ERR_INVALID_ARG


def test_binding_refuses_host_tensors(lib):
    import torch
    t = torch.zeros(4, 8)
    with pytest.raises(ValueError):
        B.moe_route_topk(t, t, t, 4, 8, 8, 2, 0, t, t, stream=0)


def test_public_headers_are_plain_c(tmp_path):
    """The boundary is a C ABI: every header under include/ compiles as C99 on its own."""
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no C compiler")
    inc = os.path.join(ROOT, "include")
    for name in sorted(os.listdir(inc)):
        if not name.endswith(".h"):
            continue
        src = tmp_path / (name + ".c")
        src.write_text('#include "%s"\nint main(void) { return 0; }\n' % name)
        r = subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-I", inc, "-c", str(src),
                            "-o", str(tmp_path / (name + ".o"))], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr


def test_forward_returns_the_first_error_of_its_steps():
    """Every check of the separate calls holds for the whole-forward call (host checks only, nothing is launched)."""
    import ctypes
    L, shard = B.lib(), B.make_shard(8, 8, 0, 512, 1024, 1024)
    sp = ctypes.byref(shard)
    assert L.moe_forward(None, sp, sp, None) == B.MOE_ERR_INVALID_ARG
    args = B.MoeForwardArgs(T=4, k=2)
    assert L.moe_forward(ctypes.byref(args), None, sp, None) == B.MOE_ERR_INVALID_ARG
    assert L.moe_forward(ctypes.byref(args), sp, sp, None) == B.MOE_ERR_INVALID_ARG      # no logits
    args = B.MoeForwardArgs(T=4, k=9)
    assert L.moe_forward(ctypes.byref(args), sp, sp, None) == B.MOE_ERR_INVALID_ARG      # k above the expert count


def _forward_args(shard, T=4, k=2, **kw):
    """Arguments no check objects to (fake addresses: nothing may be launched with them)."""
    ws, fws = B.moe_workspace_bytes(T, k, shard), B.moe_ffn_workspace_bytes(T * k, shard)
    names = [n for n, t in B.MoeForwardArgs._fields_ if t is ctypes.c_void_p and n not in
             ("y_shared", "shared_gate_x", "w_shared_gate")]
    d = dict({n: P for n in names}, workspace_bytes=ws, ffn_workspace_bytes=fws, T=T, k=k)
    d.update(kw)
    return B.MoeForwardArgs(**d)


@pytest.mark.parametrize("other", [dict(n_local_experts=4), dict(n_local_experts=4, expert_offset=4), dict(hidden=1024),
                                   dict(n_experts=16, n_local_experts=16)])
def test_forward_refuses_shards_that_disagree(lib, other):
    """expert_offsets has n_local_experts + 1 entries and the combine reads rows of `hidden` values: with two
    descriptions that differ the experts would read past the one or walk the other with another length."""
    a, b = _shard(n_experts=16) if "n_experts" in other else _shard(), _shard(**other)
    for one, two in ((a, b), (b, a)):
        args = _forward_args(a, combine_flags=1 << 30)      # (the last step's check would end the call in any case)
        args.workspace_bytes = args.ffn_workspace_bytes = 1 << 40
        assert lib.moe_forward(ctypes.byref(args), ctypes.byref(one), ctypes.byref(two), None) == B.MOE_ERR_INVALID_ARG


@pytest.mark.parametrize("bad,status", [
    (dict(route_flags=1 << 7), B.MOE_ERR_INVALID_ARG), (dict(w_router=None), B.MOE_ERR_INVALID_ARG),
    (dict(slot_row=None), B.MOE_ERR_INVALID_ARG), (dict(x_perm=P + 8), B.MOE_ERR_INVALID_ARG),
    (dict(workspace_bytes=0), B.MOE_ERR_WORKSPACE),
    (dict(w_up=P + 8), B.MOE_ERR_INVALID_ARG), (dict(x_perm=None, w_down=None), B.MOE_ERR_INVALID_ARG),
    (dict(ffn_workspace=None), B.MOE_ERR_WORKSPACE), (dict(ffn_workspace_bytes=16), B.MOE_ERR_WORKSPACE),
    (dict(ffn_flags=B.MOE_OUT_F32), B.MOE_ERR_INVALID_ARG),
    (dict(combine_flags=B.MOE_RENORM_TOPK), B.MOE_ERR_INVALID_ARG), (dict(y_out=P + 8), B.MOE_ERR_INVALID_ARG),
    (dict(w_shared_gate=P), B.MOE_ERR_INVALID_ARG), (dict(w_shared_gate=P, shared_gate_x=P), B.MOE_ERR_INVALID_ARG),
])
def test_forward_checks_every_step_before_it_enqueues_any(lib, bad, status):
    """One bad argument of any step, all others good: the error of that step's own call, and no step has been launched
    (here, without a GPU, a launch would come back as a HIP error instead)."""
    shard = _shard(hidden=4096, inter_full=14336, inter_slice=14336)
    args = _forward_args(shard, **bad)
    assert lib.moe_forward(ctypes.byref(args), ctypes.byref(shard), ctypes.byref(shard), None) == status


@pytest.mark.parametrize("bad,name", [
    (dict(route_flags=1 << 7), "moe_route_topk"), (dict(slot_row=None), "moe_permute"),
    (dict(w_up=None), "moe_expert_ffn"), (dict(x_perm=None, w_up=None), "moe_expert_ffn_gather"),
    (dict(combine_flags=1 << 30), "moe_combine"),
])
def test_forward_error_names_the_step(lib, bad, name):
    shard = _shard()
    with pytest.raises(B.MoeError, match="^%s failed" % name):
        B.moe_forward(_forward_args(shard, **bad), shard, shard, stream=0)
    with pytest.raises(B.MoeError, match="^moe_forward failed"):
        B.moe_forward(_forward_args(shard), shard, _shard(hidden=1024), stream=0)


def test_forward_without_an_output_is_an_error_unless_asked_for(lib):
    """A missing y_out is the error it is for moe_combine; ending before the combine is a flag."""
    shard = _shard()
    args = _forward_args(shard, y_out=None)
    assert lib.moe_forward(ctypes.byref(args), ctypes.byref(shard), ctypes.byref(shard), None) == B.MOE_ERR_INVALID_ARG
    assert args.step == 4
    # with the flag the combine's arguments do not matter, the other steps' do (nothing is launched here either)
    args = _forward_args(shard, y_out=None, combine_flags=B.MOE_NO_COMBINE | 1, w_up=None)
    assert lib.moe_forward(ctypes.byref(args), ctypes.byref(shard), ctypes.byref(shard), None) == B.MOE_ERR_INVALID_ARG
    assert args.step == 3
    assert lib.moe_combine(P, P, P, 4, 2, 512, None, None, None, P, B.MOE_NO_COMBINE, None) == B.MOE_ERR_INVALID_ARG


def test_int4_sizes_beyond_the_grid_are_refused_on_the_host(lib):
    """The smallest refused sizes: 2^31 - 1 blocks, of 2048 weights when quantising, of 8192 when dequantising."""
    p = 64  # any aligned address: the call ends before it is used
    assert lib.moe_int4_quantize(p, 2048 * 0x7FFFFFFE + 64, p, p, None) == B.MOE_ERR_UNSUPPORTED_SHAPE
    assert lib.moe_int4_quantize(p, 2048 * 0x7FFFFFFF, p, p, None) == B.MOE_ERR_UNSUPPORTED_SHAPE
    assert lib.moe_int4_dequantize(p, p, 8192 * 0x7FFFFFFF, p, None) == B.MOE_ERR_UNSUPPORTED_SHAPE

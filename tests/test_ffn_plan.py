"""Host logic of moe_expert_ffn's kernel choice (CPU only, through moe_debug_ffn_plan): the
decoding regime streams weights, the prefill regime runs the tiled MFMA kernel, and launches with
too few tiles are cut along K.  The expectations below are the measured crossovers."""
import pytest

from paper_2508_19373_amd import binding as B

MIXTRAL = dict(hidden=4096, inter_full=14336, inter_slice=14336)


def _shard(E, E_loc, **kw):
    return B.make_shard(E, E_loc, 0, kw["hidden"], kw["inter_full"], kw["inter_slice"])


def test_routed_experts_switch_regime_near_twenty_rows_per_expert():
    s = _shard(8, 8, **MIXTRAL)
    # both GEMMs stream weights while the fullest expert is planned within 16 rows (one pass of the
    # 16-row streaming kernel, 6.0-6.2 TB/s); from there on the tiled kernels, which stream every
    # panel once whatever the rows (measured at 64 tokens: gate/up 318 us tiled, 333 us streaming
    # with 32 rows per pass; down projection 178 us either way)
    for T, walk1, walk2 in ((16, True, True), (32, True, True), (48, False, False), (64, False, False),
                            (96, False, False), (128, False, False), (4096, False, False)):
        w1, w2, mt, slices = B.moe_debug_ffn_plan(T * 2, s)
        assert (w1, w2) == (walk1, walk2), T
    # up to 16 rows expected in the fullest expert: 16 rows per pass, 16 wavefronts, K = 14336 in 2 slices
    assert B.moe_debug_ffn_plan(32, s) == (True, True, 1, 2)
    assert B.moe_debug_ffn_plan(128, s)[2] == 2
    # the headline prefill shape: tiled kernels; K slices for the remainder tiles only (see below)
    assert B.moe_debug_ffn_plan(8192, s) == (False, False, 2, 16)
    assert B.moe_ffn_workspace_bytes(8192, s) == 4096 * 4096 * 4


def test_single_shared_expert_never_runs_its_down_projection_on_a_handful_of_tiles():
    s = _shard(1, 1, hidden=3584, inter_full=20480, inter_slice=20480)   # H / 256 = 14 column blocks
    assert B.moe_debug_ffn_plan(16, s)[:2] == (True, True)               # decode: stream both
    # 32 rows: the gate/up projection has 160 tiles, which stream at the HBM rate (measured 103.5 us
    # for the shared expert's two GEMMs against 110.4 with the 32-row streaming kernel); the down
    # projection's 14 tiles still lose to streaming
    assert B.moe_debug_ffn_plan(32, s)[:2] == (False, True)
    for rows in (64, 128, 256, 512, 1024):
        w1, w2, mt, slices = B.moe_debug_ffn_plan(rows, s)
        assert not w1 and not w2 and slices >= 2, rows
    assert B.moe_debug_ffn_plan(256, s) == (False, False, 2, 16)
    assert B.moe_debug_down_slices([0, 256], 256, s)[:2] == (0, 16)       # 14 tiles, each in 16 slices of 20 k-tiles
    assert B.moe_debug_down_slices([0, 1024], 1024, s)[:2] == (0, 4)      # 56 tiles
    assert B.moe_debug_down_slices([0, 4096], 4096, s)[:2] == (16, 1)     # 224 tiles: enough on their own
    assert B.moe_ffn_workspace_bytes(256, s) == 15 * 256 * 3584 * 4
    assert B.moe_ffn_workspace_bytes(4096, s) == (65536 // 14) * 3584 * 4


def test_expert_parallel_shard_is_planned_on_its_expected_rows():
    full = _shard(8, 8, **MIXTRAL)
    ep8 = _shard(8, 1, **MIXTRAL)
    # T = 1024, k = 2: capacity 2048 rows, of which one expert of eight expects 256: tiled kernels
    assert B.moe_debug_ffn_plan(2048, ep8)[:2] == (False, False)
    assert B.moe_debug_ffn_plan(2048, full)[:2] == (False, False)
    # decode: 16 rows expected on the one local expert, but up to 128 possible: 32 rows per pass
    assert B.moe_debug_ffn_plan(128, ep8)[2] == 2
    assert B.moe_debug_ffn_plan(16, ep8)[2] == 1            # capacity itself is 16 rows


def test_expert_parallel_shard_is_planned_for_more_than_its_balanced_share():
    # two of eight experts (EP = 4).  The shard that sets the step's latency is the one that received
    # more than a quarter of the rows, so rows per pass and kernel family are chosen for twice the
    # balanced share: 32 tokens x top-2 = 64 assignments, 16 expected here, planned for 32
    ep4 = _shard(8, 2, **MIXTRAL)
    full = _shard(8, 8, **MIXTRAL)
    assert B.moe_debug_ffn_plan(32, ep4)[:3] == (True, True, 1)     # 16 tokens: 8 rows expected, 16 planned
    assert B.moe_debug_ffn_plan(64, ep4)[:3] == (False, False, 2)   # 32 tokens: 32 rows planned, tiled kernels
    assert B.moe_debug_ffn_plan(128, ep4)[:2] == (False, False)
    # the unsharded layer at the same rows per expert keeps 16 rows per pass and the streaming kernel
    assert B.moe_debug_ffn_plan(64, full)[:3] == (True, True, 1)


def _offsets(counts):
    import numpy as np
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)


def test_down_projection_slices_follow_the_routing():
    ep4 = _shard(8, 2, **MIXTRAL)        # 16 column blocks, 224 k-tiles
    cap = 32768
    def used(*counts):
        return B.moe_debug_down_slices(_offsets(counts), cap, ep4)[:2]    # (row blocks run whole, slices of the rest)
    assert used(0, 0) == (0, 1)
    assert used(200, 100) == (0, 8)      # 2 row blocks x 16 = 32 tiles: every tile in 8 slices
    assert used(300, 100) == (0, 5)      # 3 row blocks (256 + 64, 128): 48 tiles
    assert used(700, 0) == (0, 5)        # 512 + 188 padded to 256: 48 tiles
    assert used(700, 700) == (0, 2)      # 96 tiles
    assert used(1100, 1000) == (8, 16)   # 8 whole row blocks (128 tiles), the 128-row remainder in 16 slices
    assert used(1024, 512) == (0, 2) and used(10240, 5120) == (60, 1)    # no remainder tiles; 960 tiles = 3.75 rounds
    # the hot shard: 78 + 50 row blocks = 2048 tiles = 8 rounds exactly; the remainder tiles in 16 slices
    assert used(20000, 12768) == (128, 16)
    # 35 row blocks (two of them padded) = 560 tiles = 2.2 rounds: the 48 tiles of the last three in 5 slices
    assert used(5000, 3770) == (32, 5)
    assert used(5120, 3584) == (32, 8)   # 34 row blocks, no remainders: the last two in 8 slices
    # the scratch is sized for any routing: 65536 / 16 rows, or 15 slices of the capacity
    assert B.moe_ffn_workspace_bytes(cap, ep4) == 4096 * 4096 * 4
    # the unsharded layer: 32 row blocks = 512 tiles = 2 rounds; the 3 x 16 remainder tiles in 5 slices
    full = _shard(8, 8, **MIXTRAL)
    counts = (1030, 1000, 1100, 1024, 960, 1090, 1020, 968)
    info = B.moe_debug_down_slices(_offsets(counts), 8192, full)
    assert info[:2] == (32, 5)
    assert info[2] == sum(c % 256 for c in counts if c % 256 <= 128) and info[3] == 4096
    with pytest.raises(B.MoeError):
        B.moe_debug_down_slices([0, 5, 3], cap, ep4)
    with pytest.raises(B.MoeError):
        B.moe_debug_down_slices([0, 5, cap + 1], cap, ep4)


@pytest.mark.parametrize("E_loc,hidden,inter,cap,max_rows", [
    (2, 4096, 14336, 32768, 3000), (2, 4096, 14336, 32768, 30000), (8, 4096, 14336, 8192, 8192),
    (1, 3584, 20480, 4096, 4096), (4, 512, 1024, 3000, 3000), (60, 2048, 1408, 16384, 16384),
    (16, 3584, 2560, 6000, 2000), (3, 256, 640, 900, 900), (5, 2048, 2048, 9000, 9000),
])
def test_sliced_work_list_covers_every_tile_and_slice_once(E_loc, hidden, inter, cap, max_rows):
    import numpy as np
    rng = np.random.default_rng(E_loc * 1000 + hidden)
    shard = _shard(E_loc, E_loc, hidden=hidden, inter_full=inter, inter_slice=inter)
    ncb, nk = (hidden + 255) // 256, inter // 64
    n_sliced_cases = 0
    for trial in range(40):
        R = int(rng.integers(0, max_rows + 1))
        cuts = np.sort(rng.integers(0, R + 1, size=E_loc - 1))
        counts = np.diff(np.concatenate([[0], cuts, [R]]))
        if trial % 5 == 0:
            counts = (counts // 256) * 256          # no remainder tiles
        offs = _offsets(counts)
        (keep_rb, slices, rows, scratch), units = B.moe_debug_down_slices(offs, cap, shard, with_units=True)
        if nk < 16:
            assert slices == 1
        n_sliced_cases += slices > 1
        # ordinal of every 256-row block, experts in order
        def blocks(c, pad_low):
            pad = 128 if (c >= 256 or pad_low) else 192
            r = c % 256
            return c // 256 + (r > pad), int(64 < r <= pad) + int(0 < r <= 64 or 128 < r <= pad)
        # a down projection that may be cut along K pads a remainder above 128 rows to a 256-row
        # block from 128 tiles on if K is at least 48 k-tiles; otherwise only when the launch fills the chip
        pad_low = sum(sum(blocks(c, False)) for c in counts) * ncb >= (128 if nk >= 48 else 256)
        first_rb = np.concatenate([[0], np.cumsum([blocks(c, pad_low)[0] for c in counts])])
        # the tiles that have to exist, from the row-block rule written out
        tiles = set()
        for e, c in enumerate(counts):
            c, r, pad = int(c), int(c) % 256, 128 if (c >= 256 or pad_low) else 192
            heights = [256] * (c // 256 + (r > pad))
            if r <= pad:
                heights += [128] * int(r > 64) + [64] * int(0 < r <= 64 or r > 128)
            r0 = int(offs[e])
            for h in heights:
                tiles |= {(h, e, r0, nb) for nb in range(ncb)}
                r0 += h
        if not pad_low or nk < 16:
            plain = B.moe_debug_gemm_units(offs, cap, ncb)
            if (sum(sum(blocks(c, False)) for c in counts) * ncb >= 256) == pad_low:
                assert tiles == {(int(h), int(e), int(r0), int(nb)) for h, e, r0, _, nb in plain if h}
        seen = {}
        scratch_cells = set()
        for h, e, r0, nb, z, kt0, n, srow in units:
            if h == 0:
                continue
            key = (int(h), int(e), int(r0), int(nb))
            assert key in tiles
            seen.setdefault(key, []).append((int(z), int(kt0), int(n)))
            height = min(int(h), int(offs[e + 1]) - int(r0))
            if z == 0:
                assert srow == -1
            else:
                assert 0 <= srow and srow + height <= scratch
                cells = {(int(srow) + i, int(nb)) for i in range(height)}
                assert not (cells & scratch_cells)      # no two workgroups write the same partial sums
                scratch_cells |= cells
        assert set(seen) == tiles
        n_units = 0
        for key, parts in seen.items():
            parts.sort()
            h, e, r0, nb = key
            whole = h == 256 and first_rb[e] + (r0 - offs[e]) // 256 < keep_rb
            want = 1 if whole else slices
            n_units += 0 if whole else want
            assert [z for z, _, _ in parts] == list(range(want))
            assert parts[0][1] == 0 and sum(n for _, _, n in parts) == nk
            assert all(a[1] + a[2] == b[1] for a, b in zip(parts, parts[1:]))
            assert all(n >= 8 for _, _, n in parts) or want == 1
        assert slices == 1 or n_units <= 256            # what is cut fits one round of workgroups
        assert keep_rb <= first_rb[-1]
        if slices > 1:
            assert (slices - 1) * rows <= scratch
            # partial sums of one slice tile the compact rows without gaps: cells = rows x column blocks
            assert len(scratch_cells) == (slices - 1) * rows * ncb
    assert n_sliced_cases > 0 or nk < 16


def test_k_extents_without_a_fast_streaming_kernel_go_to_the_tiled_kernel_early():
    # Qwen1.5-MoE under TP 4: the padded slice is 384 wide, a K extent only the generic streaming kernel covers
    s = B.make_shard(60, 60, 0, 2048, 1536, 384)
    w1, w2, mt, slices = B.moe_debug_ffn_plan(64 * 4, s)
    assert w1 and not w2


def test_invalid_arguments():
    L = B.lib()
    import ctypes
    plan = (ctypes.c_int32 * 4)()
    s = _shard(8, 8, **MIXTRAL)
    assert L.moe_debug_ffn_plan(-1, ctypes.byref(s), plan) == B.MOE_ERR_INVALID_ARG
    assert L.moe_debug_ffn_plan(8, None, plan) == B.MOE_ERR_INVALID_ARG
    assert L.moe_debug_ffn_plan(8, ctypes.byref(s), None) == B.MOE_ERR_INVALID_ARG


def test_hint_for_routed_experts_beside_an_overlapped_shared_expert():
    from paper_2508_19373_amd.layer import routed_hint_beside_shared as hint
    shared = _shard(1, 1, hidden=2048, inter_full=5632, inter_slice=5632)       # Qwen1.5-MoE's shared expert
    full = _shard(60, 60, hidden=2048, inter_full=1408, inter_slice=1408)      # 60 x 11 = 660 gate/up tiles
    ep2 = _shard(60, 30, hidden=2048, inter_full=1408, inter_slice=1408)       # 330
    tp2ep4 = _shard(60, 15, hidden=2048, inter_full=1408, inter_slice=704)     # 90
    for T in (16, 32):                                                           # the shared expert streams: no hint
        assert hint(full, shared, T) == 0 and hint(ep2, shared, T) == 0
    for T in (64, 96, 256, 4096):                                                # the shared expert has a tiled GEMM
        assert hint(full, shared, T) == B.MOE_FFN_TILED
        assert hint(ep2, shared, T) == B.MOE_FFN_LEAVE_ROOM
        assert hint(tp2ep4, shared, T) == B.MOE_FFN_LEAVE_ROOM


def test_the_shortest_k_extent_streams_on_its_own_split_with_32_rows_per_pass_only():
    # K = 512: 16 rows per pass on the generic kernel (the tiny layer's gate/up projection at 4 tokens 4.4 us, 7.5 on the
    # split), 32 on eight wavefronts of two steps (64 tokens 7.6 us, 8.6 on the generic kernel)
    for down in (False, True):
        assert B.moe_debug_walk_split(512, 1, down)[0] == 0
        assert B.moe_debug_walk_split(512, 2, down) == (8, 2, 1)
    assert B.moe_debug_walk_split(2048, 1) == (16, 4, 1) and B.moe_debug_walk_split(1024, 2)[2] == 1


def test_no_hint_beside_a_shared_expert_on_the_streaming_tiles():
    """The hint follows the kernel that runs, not the plan for calls without it: a shared expert whose gate/up projection holds
    every compute unit (moe_debug_flow) needs none, unless its bf16 down projection has to start early."""
    import torch
    from paper_2508_19373_amd.layer import ExpertShardLayer, shared_on_streaming_tiles
    layer = ExpertShardLayer.__new__(ExpertShardLayer)
    layer.E, layer.k, layer.H, layer.overlap_shared, layer.gather_in_ffn, layer._gather_auto = 60, 4, 2048, True, True, True
    layer.ffn_shard = _shard(60, 60, hidden=2048, inter_full=1408, inter_slice=1408)
    layer.shared_shard = _shard(1, 1, hidden=2048, inter_full=5632, inter_slice=5632)
    layer.w_gate = torch.empty((60, 1408, 2048), device="meta")
    layer.shared = [torch.empty((1, 5632, 2048), device="meta")]
    for bf16 in (False, True):
        layer.y_perm_bf16, layer._plans = bf16, {}
        for T, flow in ((64, True), (128, True), (300, True), (256, False), (333, False)):
            assert bool(B.moe_debug_flow(T, layer.shared_shard) & B.DEBUG_FLOW_GATEUP) == flow
            assert not all(B.moe_debug_ffn_plan(T, layer.shared_shard)[:2])     # "tiled", says the other plan
            assert shared_on_streaming_tiles(layer.shared_shard, T, bf16) == (flow and not bf16)
            assert (layer._plan(T).hint == 0) == (flow and not bf16), T


def _planning_layer(shard, shared_shard, E, k, bf16):
    """A layer that only plans."""
    import torch
    from paper_2508_19373_amd.layer import ExpertShardLayer
    layer = ExpertShardLayer.__new__(ExpertShardLayer)
    layer.E, layer.k, layer.H, layer.overlap_shared, layer.gather_in_ffn, layer._gather_auto = E, k, shard.hidden, True, True, True
    layer.ffn_shard, layer.shared_shard, layer.y_perm_bf16, layer._plans = shard, shared_shard, bf16, {}
    layer.w_gate = torch.empty((shard.n_local_experts, shard.inter_slice, shard.hidden), device="meta")
    layer.shared = [torch.empty((1, shared_shard.inter_slice, shared_shard.hidden), device="meta")]
    return layer


@pytest.mark.parametrize("n,inter,inter_shared,T,rows", [
    (32, 640, 5120, 1024, 160),     # Qwen2-57B TP=4 EP=2: 255 us with the tiles interleaved, 256 without a hint, 277 with room
    (32, 1280, 10240, 768, 160),    # TP=2 EP=2
    (32, 640, 5120, 384, 128),
    (64, 2560, 20480, 512, 128),    # unsharded
])
def test_no_room_is_left_by_streaming_tiles_of_more_than_64_rows(n, inter, inter_shared, T, rows):
    """Room left beside a tiled shared expert made these layers up to a tenth slower than the tiled kernels: no hint, or
    tiled where a bf16 down projection has to start early."""
    shard = _shard(64, n, hidden=3584, inter_full=2560, inter_slice=inter)
    shared = _shard(1, 1, hidden=3584, inter_full=20480, inter_slice=inter_shared)
    assert B.moe_debug_flow_rows(T * 8, shard) == rows
    assert not B.moe_debug_flow(T, shared) & B.DEBUG_FLOW_GATEUP and not all(B.moe_debug_ffn_plan(T, shared)[:2])
    assert _planning_layer(shard, shared, 64, 8, False)._plan(T).hint == 0
    assert _planning_layer(shard, shared, 64, 8, True)._plan(T).hint == B.MOE_FFN_TILED


@pytest.mark.parametrize("tp", [1, 2, 4])
def test_a_long_bf16_down_projection_beside_streaming_tiles_starts_early(tp):
    """Qwen2-57B with bf16 between the experts and the combine, 384 tokens: 835 us tiled, 946 with room (TP=2 456 / 491); a
    quarter of the shared expert is short enough."""
    shard = _shard(64, 64, hidden=3584, inter_full=2560, inter_slice=2560 // tp)
    shared = _shard(1, 1, hidden=3584, inter_full=20480, inter_slice=20480 // tp)
    assert B.moe_debug_flow_rows(384 * 8, shard) == 64
    assert _planning_layer(shard, shared, 64, 8, True)._plan(384).hint == (B.MOE_FFN_TILED if tp < 4 else B.MOE_FFN_LEAVE_ROOM)
    assert _planning_layer(shard, shared, 64, 8, False)._plan(384).hint == B.MOE_FFN_LEAVE_ROOM

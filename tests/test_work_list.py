"""Host logic of the prefill grouped GEMM: the per-workgroup tile list, run on the CPU through
moe_debug_gemm_units.  For any routing, the tiles of all workgroups must cover every routed row of
every column block exactly once, never reach into another expert's rows, and the grid bound the
launcher uses must hold."""
import ctypes

import numpy as np
import pytest

from paper_2508_19373_amd import binding as B


def _offsets(rows):
    return np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)


def _check_cover(rows, cap_rows, ncb):
    offs = _offsets(rows)
    units = B.moe_debug_gemm_units(offs, cap_rows, ncb)
    cover = np.zeros((max(int(offs[-1]), 1), ncb), dtype=np.int32)
    n_tiles = 0
    for h, e, row0, row_end, nb in units.tolist():
        if h == 0:
            continue
        assert h in (256, 128, 64)
        assert 0 <= e < len(rows) and 0 <= nb < ncb
        assert offs[e] <= row0 < row_end == offs[e + 1]
        cover[row0:min(row0 + h, row_end), nb] += 1
        n_tiles += 1
    assert (cover[:int(offs[-1])] == 1).all()
    return units, n_tiles


def test_tiles_cover_every_row_once_random_routings():
    rng = np.random.default_rng(1234)
    for trial in range(120):
        n_local = int(rng.integers(1, 17))
        ncb = int(rng.integers(1, 9))
        kind = trial % 4
        if kind == 0:    # anything, including empty experts
            rows = rng.integers(0, 700, n_local) * (rng.random(n_local) < 0.8)
        elif kind == 1:  # just around the block heights
            rows = rng.choice([63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 320, 449, 512], n_local)
        elif kind == 2:  # multinomial as routing gives
            rows = rng.multinomial(int(rng.integers(1, 6000)), rng.dirichlet(np.ones(n_local)))
        else:            # a few rows per expert only
            rows = rng.integers(0, 40, n_local)
        rows = rows.astype(np.int64)
        cap = int(rows.sum()) + int(rng.integers(0, 300))
        _check_cover(rows, cap, ncb)


def test_empty_routing_and_single_row():
    units, n = _check_cover(np.zeros(8, dtype=np.int64), 0, 4)
    assert n == 0 and (units[:, 0] == 0).all()
    units, n = _check_cover(np.array([0, 0, 1, 0]), 1, 3)
    assert n == 3 and sorted(int(r[0]) for r in units if r[0]) == [64, 64, 64]


def test_remainder_tiles_and_padding():
    # a remainder of up to 64 / up to 128 rows is a 64- / 128-row tile; a larger one is padded to a
    # 256-row tile when the expert has a 256-row block to share the weights with (a second
    # remainder tile would stream them a second time), and is 128 + 64 rows up to 192 otherwise
    for rows in range(1, 1200):
        units, _ = _check_cover(np.array([rows]), rows, 1)
        h = units[:, 0][units[:, 0] > 0]
        r = rows % 256
        pad = 128 if rows >= 256 else 192
        assert (h == 64).sum() == (0 < r <= 64 or 128 < r <= pad)
        assert (h == 128).sum() == (64 < r <= pad)
        assert (h == 256).sum() == rows // 256 + (r > pad)
        assert h.sum() - rows < (64 if r <= pad else 128)


def test_experts_below_256_rows_are_padded_only_in_launches_that_fill_the_chip():
    rows = np.array([150, 190, 130, 100, 60, 193, 170, 129])
    few, _ = _check_cover(rows, int(rows.sum()), 2)       # 2 column blocks: 26 tiles in all
    many, _ = _check_cover(rows, int(rows.sum()), 112)    # 112 column blocks: 1456 tiles
    def heights(units, expert):
        return sorted(int(h) for h, e, _, _, nb in units if h and e == expert and nb == 0)
    for e, r in enumerate(rows):
        want_few = [256] if r > 192 else ([64, 128] if r > 128 else ([128] if r > 64 else [64]))
        want_many = [256] if r > 128 else ([128] if r > 64 else [64])
        assert heights(few, e) == want_few and heights(many, e) == want_many, (e, r)
    # the switch is at 256 tiles counted before any such padding
    rows = np.array([150] * 8)                            # 16 row blocks
    assert (np.asarray(_check_cover(rows, 1200, 15)[0])[:, 0] == 256).sum() == 0      # 240 tiles
    assert (np.asarray(_check_cover(rows, 1200, 16)[0])[:, 0] == 256).sum() == 8 * 16  # 256 tiles


def test_full_tiles_first_and_balanced_over_xcds():
    # 8 experts of about 1024 rows, 112 column blocks (the GEMM1 shape of an 8 x 14336 layer)
    rows = np.array([1040, 1030, 1050, 1024, 1000, 1047, 1033, 1025])
    units, _ = _check_cover(rows, int(rows.sum()), 112)
    per_xcd = []
    for x in range(8):   # workgroup b runs on XCD b % 8, in the order of b
        h = units[x::8, 0]
        h = h[h > 0]
        assert (np.diff(h) <= 0).all()          # 256-row tiles first, remainder tiles last
        per_xcd.append(((h == 256).sum(), (h == 64).sum()))
    full, small = zip(*per_xcd)
    assert max(full) - min(full) <= 1 and max(small) - min(small) <= 1
    # neighbours on one XCD share the weight panel: row blocks of one (expert, column block) are adjacent
    x0 = units[0::8]
    x0 = x0[x0[:, 0] == 256]
    same = (x0[1:, 1] == x0[:-1, 1]) & (x0[1:, 4] == x0[:-1, 4])
    assert same.mean() > 0.7


def test_invalid_arguments():
    L = B.lib()
    offs = np.array([0, 5, 3], dtype=np.int32)   # decreasing
    out = np.zeros((64, B.DEBUG_UNIT_INTS), dtype=np.int32)
    assert L.moe_debug_gemm_units(offs.ctypes.data, 2, 8, 1, out.ctypes.data, 64) == B.MOE_ERR_INVALID_ARG
    offs = np.array([0, 5, 9], dtype=np.int32)
    assert L.moe_debug_gemm_units(offs.ctypes.data, 2, 8, 1, out.ctypes.data, 64) == B.MOE_ERR_INVALID_ARG  # last > cap
    assert L.moe_debug_gemm_units(offs.ctypes.data, 2, 16, 1, out.ctypes.data, 2) == B.MOE_ERR_WORKSPACE


def _check_even_cover(rows, cap_rows, ncb):
    offs = _offsets(rows)
    units = B.moe_debug_even_units(offs, cap_rows, ncb)
    cover = np.zeros((max(int(offs[-1]), 1), ncb), dtype=np.int32)
    for h, e, row0, row_end, nb in units.tolist():
        if h == 0:
            continue
        assert h == 160 and 0 <= e < len(rows) and 0 <= nb < ncb
        assert offs[e] <= row0 < row_end == offs[e + 1] and (row0 - offs[e]) % 160 == 0
        cover[row0:min(row0 + h, row_end), nb] += 1
    assert (cover[:int(offs[-1])] == 1).all()
    return units


def test_even_row_blocks_cover_every_row_once():
    rng = np.random.default_rng(99)
    for trial in range(80):
        n_local = int(rng.integers(1, 70))
        ncb = int(rng.integers(1, 9))
        if trial % 3 == 0:
            rows = rng.integers(0, 700, n_local) * (rng.random(n_local) < 0.8)
        elif trial % 3 == 1:
            rows = rng.choice([1, 159, 160, 161, 319, 320, 321, 480, 481], n_local)
        else:
            rows = rng.multinomial(int(rng.integers(1, 20000)), rng.dirichlet(np.ones(n_local)))
        rows = rows.astype(np.int64)
        _check_even_cover(rows, int(rows.sum()) + int(rng.integers(0, 300)), ncb)
    units = _check_even_cover(np.zeros(5, dtype=np.int64), 0, 3)
    assert (units[:, 0] == 0).all()


def test_even_row_blocks_of_one_column_block_are_neighbours_on_one_xcd():
    # 60 experts of 250 to 300 rows, 11 column blocks (the gate/up projection of a 60 x 1408 layer at
    # 4096 tokens): the two row blocks of an (expert, column block) run side by side on one XCD, so
    # the second reader of the weight panel finds it in that XCD's L2
    rng = np.random.default_rng(3)
    rows = rng.integers(250, 301, 60)
    units = _check_even_cover(rows, int(rows.sum()), 11)
    assert (units[:, 0] == 160).sum() == 60 * 11 * 2
    pairs = same = 0
    for x in range(8):
        u = units[x::8]
        u = u[u[:, 0] > 0]
        for a, b in zip(u[:-1], u[1:]):
            if a[2] != b[2] and a[1] == b[1] and a[4] == b[4]:
                same += 1
        pairs += len(u) // 2
    assert same >= 0.95 * pairs


def test_tile_rows_rule():
    qwen = B.make_shard(60, 60, 0, 2048, 1408, 1408)
    # rows per expert just below one or two blocks of 160 rows
    assert B.moe_debug_tile_rows(4096 * 4, qwen) == 160      # 273 rows per expert
    assert B.moe_debug_tile_rows(2048 * 4, qwen) == 160      # 137
    assert B.moe_debug_tile_rows(3072 * 4, qwen) == 256      # 205: a second block for most experts, nothing saved
    assert B.moe_debug_tile_rows(1536 * 4, qwen) == 256      # 102
    assert B.moe_debug_tile_rows(8192 * 4, qwen) == 256      # 546
    assert B.moe_debug_tile_rows(4096 * 4, B.make_shard(60, 30, 0, 2048, 1408, 1408)) == 256   # 30 local experts
    assert B.moe_debug_tile_rows(4096 * 2, B.make_shard(8, 8, 0, 4096, 14336, 14336)) == 256   # 1024 rows per expert
    assert B.lib().moe_debug_tile_rows(-1, ctypes.byref(qwen)) == B.MOE_ERR_INVALID_ARG
    assert B.lib().moe_debug_tile_rows(-1, None) == B.MOE_ERR_INVALID_ARG


def test_calls_just_below_320_rows_per_expert_keep_the_160_row_tiling():
    """One tall block holds 304 rows: with 306 to 330 rows on average most experts would have a remainder tile behind it,
    two blocks of 160 rows hold them all."""
    for shard in (B.make_shard(60, 60, 0, 2048, 1408, 1408), B.make_shard(64, 64, 0, 3584, 2560, 1280),
                  B.make_shard(64, 32, 32, 3584, 2560, 2560)):
        for avg, tall in ((256, True), (304, True), (306, False), (315, False), (330, False), (331, True)):
            cap = avg * shard.n_experts
            assert B.moe_debug_tall(cap, shard) == tall, avg
            assert (B.moe_debug_tile_rows(cap, shard) == 160) == (avg <= 330)


def test_tall_row_blocks_only_where_their_offsets_fit_32_bits():
    """A tall block reaches 304 rows of K bf16 values with 32-bit byte offsets from its first row."""
    fits = 0xFFFFFFFF // (2 * 304) // 64 * 64
    for K, ok in ((fits, True), (fits + 64, False), (1 << 24, False)):
        assert B.moe_debug_tall(4 * 300, B.make_shard(4, 4, 0, 1024, K, K)) == ok
        assert B.moe_debug_tall(4 * 300, B.make_shard(4, 4, 0, K, 1024, 1024)) == ok


def _routings_for_tall_blocks(rng, n_local):
    kind = rng.integers(0, 4)
    if kind == 0:
        return rng.integers(0, 1500, n_local) * (rng.random(n_local) < 0.8)
    if kind == 1:    # around the heights where a block more, or a remainder tile, becomes necessary
        return rng.choice([1, 64, 129, 193, 255, 256, 257, 272, 273, 288, 304, 305, 320, 512, 513, 544, 608, 609, 767, 768,
                           1024, 1053, 1216, 1217, 4096 + 255, 8192 + 17], n_local)
    if kind == 2:    # as a balanced router spreads a batch
        return rng.multinomial(n_local * int(rng.integers(150, 1200)), np.ones(n_local) / n_local)
    return rng.integers(0, 260, n_local)


@pytest.mark.parametrize("n_local,ncb,nk,max_slices", [(8, 112, 64, 0), (8, 16, 224, 16), (2, 16, 224, 16), (60, 11, 32, 0),
                                                       (60, 8, 22, 2), (5, 3, 40, 5), (4, 14, 320, 16), (1, 1, 16, 2)])
def test_tall_row_blocks_cover_every_row_and_k_tile_once(n_local, ncb, nk, max_slices):
    rng = np.random.default_rng(n_local * 100 + ncb)
    n_tall = 0
    for _ in range(60):
        rows = np.asarray(_routings_for_tall_blocks(rng, n_local), dtype=np.int64)
        offs = _offsets(rows)
        R = int(offs[-1])
        cap = R + int(rng.integers(0, 300))
        units = B.moe_debug_tall_units(offs, cap, ncb, nk, max_slices)
        cover = np.zeros((max(R, 1), ncb), dtype=np.int64)      # k-tiles summed for each row and column block
        scratch_rows = min(65536 // ncb, (max(max_slices, 1) - 1) * cap)
        cells = {}
        for h, e, row0, row_end, nb, z, kt0, n, srow in units[units[:, 0] > 0].tolist():
            assert h in (304, 288, 272, 256, 128, 64)
            assert 0 <= nb < ncb and offs[e] <= row0 < row_end == offs[e + 1]
            assert 0 <= kt0 and n >= 1 and kt0 + n <= nk
            end = min(row0 + h, row_end)
            cover[row0:end, nb] += n
            n_tall += h > 256
            assert (srow == -1) == (z == 0)
            if z > 0:
                assert 0 <= srow and srow + end - row0 <= scratch_rows
                for r in range(end - row0):
                    assert cells.setdefault((srow + r, nb), (z, row0 + r)) == (z, row0 + r)
                    # the partial sums of one row and slice: one place, whatever the column block
                    assert cells.setdefault((srow + r, "row"), (z, row0 + r)) == (z, row0 + r)
        assert (cover[:R] == nk).all(), rows
    assert n_tall > 0 or ncb < 8


def test_tall_row_blocks_are_the_fewest_that_hold_the_remainder():
    for rows in list(range(1, 1300)) + [4096 + 200, 4096 + 255, 16 * 256 + 1, 20 * 256 + 255]:
        units = B.moe_debug_tall_units(_offsets([rows]), rows, 256, 64, 0)
        h = units[(units[:, 0] > 0) & (units[:, 4] == 0), 0]
        q, r = divmod(rows, 256)
        if q and 0 < r <= (48 if q == 1 else min(16 * q, 144)):   # a larger one is a tile of its own, as in the plain list
            nx = -(-r // (16 * q))
            assert sorted(h) == sorted([256 + 16 * nx] * -(-r // (16 * nx)) + [256] * (q - -(-r // (16 * nx))))
        else:
            plain = B.moe_debug_gemm_units(_offsets([rows]), rows, 256)
            assert sorted(h) == sorted(plain[(plain[:, 0] > 0) & (plain[:, 4] == 0), 0])
    # a launch that leaves compute units idle has none: a remainder tile of its own costs nothing there
    units = B.moe_debug_tall_units(_offsets([1040, 1050]), 2090, 20, 64, 0)
    assert set(units[:, 0].tolist()) == {0, 256, 64}


@pytest.mark.parametrize("rows,ncb,nk,max_slices,tall", [
    # as many rounds of 256 tiles either way: the remainder tiles run on units that would idle beside tall ones
    ([302, 333, 332, 368, 303, 320, 325, 333], 16, 56, 7, False),
    ([349, 329, 312, 171, 173, 301, 729, 236], 16, 224, 16, False),
    ([315, 292, 295, 321], 16, 224, 16, False),
    ([126, 1394, 588, 267, 148, 421, 126, 303], 14, 64, 0, False),
    ([2304, 2305, 2320, 2337], 8, 32, 0, False),
    # a round fewer, or many rounds
    ([306, 281, 282, 295, 273, 300, 269, 317], 56, 64, 0, True),
    ([255, 281, 265, 253, 238, 241, 279, 231], 28, 64, 0, True),
    ([1053] * 8, 112, 64, 0, True),
    ([1053] * 8, 16, 224, 16, True),
    # a down projection that is cut into more slices
    ([2066], 16, 224, 16, True),
    ([283, 290, 271, 281, 265, 289, 294, 279], 16, 112, 14, True),
])
def test_remainders_are_dealt_out_only_where_the_launch_ends_sooner(rows, ncb, nk, max_slices, tall):
    """Routings measured both ways: dealing the remainders to the full blocks where that saves no round of tiles made the
    launch up to a third longer (half the chip idle beside tiles of 304 rows)."""
    units = B.moe_debug_tall_units(_offsets(rows), sum(rows), ncb, nk, max_slices)
    assert bool((units[:, 0] > 256).any()) == tall


def test_debug_tall_names_the_gemms_that_run_the_kernel_with_tall_blocks():
    """Decided per GEMM, by the function the launcher asks."""
    up, down, down16 = B.DEBUG_TALL_GATEUP, B.DEBUG_TALL_DOWN, B.DEBUG_TALL_DOWN_BF16
    full, tp4 = B.make_shard(8, 8, 0, 4096, 14336, 14336), B.make_shard(8, 8, 0, 4096, 14336, 3584)
    shared = B.make_shard(1, 1, 0, 2048, 5632, 5632)
    assert B.moe_debug_tall_gemms(2 * 4096, full) == up | down | down16
    assert B.moe_debug_tall_gemms(8 * 300, full) == up          # down: 128 tall tiles on 256 compute units
    assert B.moe_debug_tall_gemms(8 * 300, tp4) == 0            # nor does a round of the gate/up projection go away
    assert B.moe_debug_tall_gemms(8 * 160, full) == 0           # no expert with a full block
    assert B.moe_debug_tall_gemms(8 * 160, B.make_shard(8, 4, 0, 4096, 14336, 14336)) & down == 0
    assert B.moe_debug_tall_gemms(333, shared) == 0             # 88 tiles
    assert B.moe_debug_tall_gemms(4096, shared) == 0            # no remainder (one expert that takes every row)
    assert B.moe_debug_tall_gemms(4100, shared) == 0            # 128 tiles in two slices each would be no faster than 136
    assert B.moe_debug_tall_gemms(300, B.make_shard(1, 1, 0, 1024, 1024, 1024)) == 0


def test_a_sample_of_edge_rows_comes_from_the_lists_that_run():
    """Rows in tiles cut along K: of the list with tall blocks where the call runs that, whatever the other lists say."""
    import sampling
    rng = np.random.default_rng(0)
    qwen, n_cut = B.make_shard(60, 60, 0, 2048, 1408, 1408), 0
    for _ in range(8):
        offs = _offsets(rng.multinomial(4096 * 4, np.ones(60) / 60))
        units = B.moe_debug_tall_units(offs, 4096 * 4, 8, 22, B.moe_debug_ffn_plan(4096 * 4, qwen)[3])
        cut = units[(units[:, 0] > 0) & (units[:, 5] >= 1)]
        rows, n = sampling.edge_rows(offs, 4096 * 4, qwen)
        assert n == len(cut)
        for h, e, row0, row_end in cut[:, :4]:
            assert ((rows >= row0) & (rows < min(row0 + h, row_end))).any()
        tall = units[(units[:, 0] > 256) & (units[:, 4] == 0)]
        for h, e, row0, row_end in tall[:, :4]:                 # the first of a tall tile's extra rows, and its last row
            assert {min(int(row0) + 256, int(row_end) - 1), int(min(row0 + h, row_end)) - 1} <= set(rows.tolist())
        n_cut += len(cut)
    assert n_cut > 0
    # one 160-row and one plain call
    assert sampling.edge_rows(_offsets([320] * 60), 320 * 60, qwen)[1] == 0
    mix = B.make_shard(8, 8, 0, 4096, 14336, 14336)
    offs = _offsets([180, 190, 150, 160, 130, 170, 141, 200])
    assert sampling.edge_rows(offs, int(offs[-1]), mix)[1] == sum(
        1 for u in B.moe_debug_down_slices(offs, int(offs[-1]), mix, with_units=True)[1] if u[0] > 0 and u[4] >= 1)

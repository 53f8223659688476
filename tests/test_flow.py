"""The streaming tiles, the grouped GEMM for experts of up to about 160 rows (csrc/grouped_flow.hpp): when it runs (host) and what it
computes at the edges of its tiles (device, against the CPU oracle)."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2508_19373_amd import binding as B
from paper_2508_19373_amd import inputs as I
from paper_2508_19373_amd.layer import ExpertShardLayer, bf16_tensor

BOTH = B.DEBUG_FLOW_GATEUP | B.DEBUG_FLOW_DOWN


def test_when_it_runs():
    mixtral = B.make_shard(8, 8, 0, 4096, 14336, 14336)
    assert B.moe_debug_flow(16, mixtral) == B.DEBUG_FLOW_DOWN        # one 16-row pass over long rows streams as fast
    assert B.moe_debug_flow(64, mixtral) == B.DEBUG_FLOW_DOWN        # 8 rows per expert, 14 planned
    assert B.moe_debug_flow(128, mixtral) == BOTH
    assert B.moe_debug_flow(848, mixtral) == BOTH                    # 106 rows per expert, 127 planned
    assert B.moe_debug_flow_rows(848, mixtral) == 128 and B.moe_debug_flow_rows(860, mixtral) == 160
    assert B.moe_debug_flow(1120, mixtral) == BOTH                   # 140, 164 planned
    assert B.moe_debug_flow(1140, mixtral) == 0
    assert B.moe_debug_flow(2160, mixtral) == B.DEBUG_FLOW_DOWN      # 270: two passes of 160, for the down projection
    tp8 = B.make_shard(8, 8, 0, 4096, 14336, 1792)
    assert B.moe_debug_flow(2160, tp8) == BOTH                       # and where 112 tall tiles would fill less than half a round
    assert B.moe_debug_flow(2800, tp8) == 0
    one = B.make_shard(8, 1, 0, 4096, 14336, 14336)
    assert B.moe_debug_flow(256, one) == B.DEBUG_FLOW_GATEUP         # 256 output strips of the down projection: one each
    assert B.moe_debug_flow(0, one) == 0
    tiny = B.make_shard(8, 8, 0, 512, 1024, 1024)
    assert B.moe_debug_flow(128, tiny) == 0                          # 17 MB of weights
    qwen_tp8 = B.make_shard(60, 60, 0, 2048, 1536, 192)
    assert B.moe_debug_flow(1024, qwen_tp8) == BOTH                  # K = 192, three k-tiles: the shortest it takes
    assert B.moe_debug_flow(1024, B.make_shard(60, 60, 0, 2048, 1024, 128)) == B.DEBUG_FLOW_GATEUP
    assert B.moe_debug_flow(4, qwen_tp8) == 0                        # four experts at most: 48 gate/up strips


@pytest.mark.parametrize("rows", [2, 22, 60])
def test_the_tiles_fill_the_rounds_of_the_launch_that_runs(rows):
    """60 experts' GEMMs in rounds of 240 workgroups where 16 compute units stay free, of 256 where none do: the last round
    is not nearly empty."""
    qwen = B.make_shard(60, 60, 0, 2048, 1408, 1408)
    offs = np.arange(61) * rows
    for which in (B.DEBUG_FLOW_GATEUP, B.DEBUG_FLOW_DOWN):
        for flags, wgs in ((0, 256), (B.MOE_FFN_LEAVE_ROOM, 240)):
            tiles = B.moe_debug_flow_tiles(offs, 60 * rows, qwen, which, flags)
            assert tiles % 60 == 0 and tiles / wgs >= 0.9 * -(-tiles // wgs), (tiles, wgs)


def _counts(n, avg, special, rng):
    c = rng.integers(0, 2 * avg, n)
    c[:len(special)] = special
    c[len(special):] = c[len(special):] * max(avg * n - sum(special), 0) // max(int(c[len(special):].sum()), 1)
    return c


CASES = [
    # n, H, I_s, average rows, first experts' rows: tiles of 64 x 256 and 64 x 128, two and three row passes
    (24, 1024, 704, 40, [64, 65, 0, 1, 130, 63]),
    # 64 x 128 for both, strips that do not divide by the tile
    (15, 2048, 704, 20, [16, 17, 0, 64, 65]),
    # 128-row tiles
    (28, 1024, 704, 90, [128, 129, 0, 1, 257, 127]),
    # 160-row tiles: one pass and a few rows more, and two passes
    (28, 1024, 704, 130, [160, 161, 0, 1, 320, 159]),
    (28, 1024, 704, 265, [320, 321, 0, 480, 1, 290]),
    # three k-tiles: the loaders are more than a tile ahead
    (64, 1536, 192, 10, [0, 0, 33, 64, 65, 1]),
    (64, 1536, 192, 80, [0, 128, 129, 1]),
    # five, and one row per expert or none
    (64, 1024, 320, 2, [0, 1, 9]),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,H,I_s,avg,special", CASES)
@pytest.mark.parametrize("gather", [False, True])
def test_against_oracle(n, H, I_s, avg, special, gather):
    """fp32 and bf16 y_perm, rows permuted or read in place.  Tolerance: h and (bf16) y are rounded to bf16 once, 1.6e-3
    and 2.3e-3 rel-L2; sums in another order differ by 1e-6."""
    rng = np.random.default_rng(n + avg)
    counts = _counts(n, avg, special, rng)
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offs[-1])
    cap = R + 5
    shard = B.make_shard(n, n, 0, H, I_s, I_s)
    assert B.moe_debug_flow(cap, shard) & B.DEBUG_FLOW_DOWN
    wg, wu, wd = I.make_expert_weights(4, I.MoEShape("f", H, n, 1, I_s, True))
    k = 2
    T = (cap + k - 1) // k
    x = I.make_x(5, T, H)
    row_src = rng.permutation(T * k)[:cap].astype(np.int32)
    xp = x[row_src // k]
    ref = O.expert_ffn(xp[:R], offs, wg, wu, wd)
    W = [bf16_tensor(w) for w in (wg, wu, wd)]
    h = torch.empty((cap, I_s), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(max(B.moe_ffn_workspace_bytes(cap, shard), 256), dtype=torch.uint8, device="cuda")
    d_offs, d_src = torch.from_numpy(offs).cuda(), torch.from_numpy(row_src).cuda()
    rows = bf16_tensor(x if gather else xp)
    outs = []
    for flags in (0, B.MOE_FFN_LEAVE_ROOM, B.MOE_Y_PERM_BF16):
        y = torch.full((cap, H), float("nan"), dtype=torch.bfloat16 if flags & B.MOE_Y_PERM_BF16 else torch.float32,
                       device="cuda")
        if gather:
            B.moe_expert_ffn_gather(rows, d_src, k, d_offs, cap, shard, *W, h, y, ws, flags)
        else:
            B.moe_expert_ffn(rows, d_offs, cap, shard, *W, h, y, ws, flags)
        y = y.float().cpu().numpy().astype(np.float64)
        assert np.all(np.isnan(y[R:])), "rows past R must not be written"
        rel = np.linalg.norm(y[:R] - ref) / np.linalg.norm(ref)
        assert rel < 5e-3, (flags, rel)
        outs.append(y[:R])
    assert np.array_equal(outs[0], outs[1])          # fewer workgroups, the same tiles


@pytest.mark.parametrize("total", [*range(0, 70), 1019, 1020, 1026, 4095])
def test_every_take_below_the_total_is_a_tile(total):
    """The ids with a tile are those below the total, whatever its remainder by the XCDs, and they are all tiles once; each
    XCD's are neighbours."""
    places = [B.moe_debug_flow_place(i, total) for i in range(total + 80)]
    assert sorted(places[:total]) == list(range(total)) and set(places[total:]) == {-1}
    for xcd in range(8):
        mine = places[xcd:total:8]
        assert mine == list(range(mine[0], mine[0] + len(mine))) if mine else True


def _taken(total, workgroups, ahead, counter, rng):
    """Places computed by workgroups that take `ahead` tiles before their first and one more during each, and end at the
    first that is none, in an order of progress drawn at random."""
    done, n = [], [0]
    slots, ended, dealt = [[] for _ in range(workgroups)], [False] * workgroups, [0] * workgroups

    def take(w):
        i = n[0] if counter else w + dealt[w] * workgroups
        n[0] += 1
        dealt[w] += 1
        slots[w].append(B.moe_debug_flow_place(i, total))

    running = list(range(workgroups))
    late = rng.random() < 0.5       # the others start when the first are well on
    while running:
        some = running[:max(1, len(running) // 8)] if late and len(done) < total // 2 else running
        w = some[rng.integers(len(some))]
        if not slots[w] and not dealt[w]:
            for _ in range(ahead):
                take(w)
            continue
        place = slots[w].pop(0)
        if place < 0:
            running.remove(w)
            continue
        take(w)
        done.append(place)
    return done


@pytest.mark.parametrize("workgroups", [1, 7, 16, 30, 240])
@pytest.mark.parametrize("ahead", [1, 2, 3])
@pytest.mark.parametrize("counter", [False, True])
def test_no_tile_is_lost_between_the_look_ahead_and_the_end(workgroups, ahead, counter):
    rng = np.random.default_rng(workgroups * 8 + ahead)
    for total in (1, 8, 61, 95, 240, 241, 486, 1026, 1031):
        assert sorted(_taken(total, workgroups, ahead, counter, rng)) == list(range(total))


@pytest.mark.gpu
@pytest.mark.parametrize("n,H,I_s", [
    (23, 1024, 704),     # a tile looked up ahead
    (61, 2048, 192),     # three k-tiles of the down projection, three tiles ahead; and the shapes between
    (57, 3584, 320),
    (59, 2048, 384),
])
@pytest.mark.parametrize("beside", [False, True])
def test_tiles_from_the_counter_give_the_same_bits(n, H, I_s, beside):
    """Beside another stream the tiles come from a counter that the permutation clears; every forward starts it anew, and
    every tile is taken, also where few workgroups run at first because another call's tiles hold the compute units."""
    k = 4
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")
    W = dict(w_gate=(r(n, I_s, H) * 0.02).bfloat16(), w_up=(r(n, I_s, H) * 0.02).bfloat16(),
             w_down=(r(n, H, I_s) * 0.02).bfloat16(), w_router=r(H, n) * 0.02)
    layer = ExpertShardLayer(n_experts=n, top_k=k, hidden=H, inter_full=I_s, inter_slice=I_s, max_tokens=600, **W)
    side = torch.cuda.Stream()
    one, rows = B.make_shard(1, 1, 0, 1024, 2048, 2048), 8192
    sx, sh, sy = r(rows, 1024).bfloat16(), r(rows, 2048).bfloat16(), r(rows, 1024)
    sw = [(r(*s) * 0.02).bfloat16() for s in ((1, 2048, 1024), (1, 2048, 1024), (1, 1024, 2048))]
    so = torch.tensor([0, rows], dtype=torch.int32, device="cuda")
    sws = torch.empty(max(B.moe_ffn_workspace_bytes(rows, one), 256), dtype=torch.uint8, device="cuda")
    ragged = False
    for tokens in (300, 600, 37, 100, 183):   # permuted by one workgroup and (more than 2048 assignments) by several
        x = r(tokens, H).bfloat16()
        which = B.moe_debug_flow(tokens * k, layer.ffn_shard)
        assert which
        want = layer.forward(x).clone()
        offs = layer.expert_offsets.cpu().numpy()
        ragged |= any(which & b and B.moe_debug_flow_tiles(offs, tokens * k, layer.ffn_shard, b) % 8 for b in (1, 2))
        plan = layer._plan(tokens)
        layer._plan = lambda _, p=plan: p._replace(hint=B.MOE_FFN_LEAVE_ROOM)
        for _ in range(3):
            layer.y_perm.fill_(float("nan"))
            layer.h_ws.fill_(float("nan"))
            torch.cuda.synchronize()
            if beside:
                B.moe_expert_ffn(sx, so, rows, one, *sw, sh, sy, sws, B.MOE_FFN_TILED, side)
            assert torch.equal(layer.forward(x), want)
            torch.cuda.synchronize()
        del layer._plan
    assert ragged, "no launch whose tiles do not divide by the XCDs"


@pytest.mark.gpu
@pytest.mark.parametrize("H,I_s,counts", [
    (2048, 192, [300, 129, 64, 1, 0, 255]),            # tiles of all heights
    (4096, 128, [257, 40, 511]),
    (2048, 1024, [260] * 40 + [300, 1, 256, 0, 401]),  # with tall row blocks
])
def test_walks_over_k_that_begin_apart(H, I_s, counts):
    """Tiled gate/up projections on rows of a multiple of 4 KB start K at an eighth that depends on the expert and the output
    column; tolerance as above."""
    n = len(counts)
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offs[-1])
    shard = B.make_shard(n, n, 0, H, I_s, I_s)
    wg, wu, wd = I.make_expert_weights(6, I.MoEShape("f", H, n, 1, I_s, True))
    x = I.make_x(7, R, H)
    ref = O.expert_ffn(x, offs, wg, wu, wd)
    h = torch.empty((R, I_s), dtype=torch.bfloat16, device="cuda")
    y = torch.empty((R, H), device="cuda")
    ws = torch.empty(max(B.moe_ffn_workspace_bytes(R, shard), 256), dtype=torch.uint8, device="cuda")
    B.moe_expert_ffn(bf16_tensor(x), torch.from_numpy(offs).cuda(), R, shard, bf16_tensor(wg), bf16_tensor(wu),
                     bf16_tensor(wd), h, y, ws, B.MOE_FFN_TILED)
    got = y.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < 5e-3


@pytest.mark.gpu
@pytest.mark.parametrize("tokens", [16, 200])   # route and permutation in one kernel or two
def test_a_small_batch_uses_the_workspace_for_the_counters_only(tokens):
    """Without the hint that takes tiles from the counters a batch of up to 2048 assignments leaves the workspace as it is;
    with it, all but the last 256 bytes."""
    n, H, I_s, k = 24, 1024, 704, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")
    layer = ExpertShardLayer(n_experts=n, top_k=k, hidden=H, inter_full=I_s, inter_slice=I_s, max_tokens=tokens,
                             w_router=r(H, n) * 0.02, w_gate=r(n, I_s, H).bfloat16(), w_up=r(n, I_s, H).bfloat16(),
                             w_down=r(n, H, I_s).bfloat16())
    x = r(tokens, H).bfloat16()
    plan = layer._plan(tokens)
    layer.workspace = torch.empty(B.moe_workspace_bytes(tokens, k, layer.shard), dtype=torch.uint8, device="cuda")
    for hint in (0, B.MOE_FFN_TILED, B.MOE_FFN_LEAVE_ROOM):
        layer.workspace.fill_(0xAB)
        layer._plan = lambda _, h=hint: plan._replace(hint=h)
        layer.forward(x)
        used = (layer.workspace != 0xAB).cpu()
        assert bool(used.any()) == (hint == B.MOE_FFN_LEAVE_ROOM) and not used[:-256].any()


@pytest.mark.gpu
@pytest.mark.parametrize("H,I_s,avg,n,mine,flow_rows", [
    (2048, 704, 20, 30, [0, 13, 29], 64),     # tiles of 64 rows, one region of K per expert
    (4096, 1792, 20, 4, [1], 64),             # four regions each
    (4096, 5632, 40, 1, None, 64),            # 16
    (2048, 704, 90, 30, [0, 13, 29], 128),
    (4096, 1792, 130, 6, [2, 5], 160),
    (2048, 704, 270, 30, [0, 13, 29], 0),     # tiled gate/up with its walks spread
    (2048, 512, 400, 3, [1], 0),
])
def test_a_rows_bits_do_not_depend_on_the_other_rows(H, I_s, avg, n, mine, flow_rows):
    """The experts `mine` get the same rows of x in two batches of one size in which all the others differ (with one expert:
    their first 17 rows): the same kernels add the same products in the same order."""
    rng = np.random.default_rng(H + avg)
    cap = n * avg
    if n == 1:
        mine, counts = [0], [np.array([cap]), np.array([cap // 2])]
        keep = {0: 17}
    else:
        keep = {e: int(rng.integers(1, 2 * avg)) for e in mine}
        counts = []
        for i in range(2):
            w = rng.random(n) ** (1 if i else 4) + 1e-3
            w[mine] = 0
            c = np.floor((cap - sum(keep.values())) * w / w.sum()).astype(np.int64)
            for e in mine:
                c[e] = keep[e]
            counts.append(c)
    shard = B.make_shard(n, n, 0, H, I_s, I_s)
    flow = B.moe_debug_flow(cap, shard)
    assert (flow & B.DEBUG_FLOW_GATEUP != 0) == (flow_rows != 0)
    if flow_rows:
        assert B.moe_debug_flow_rows(cap, shard) == flow_rows
    else:
        assert not B.moe_debug_ffn_plan(cap, shard)[0]
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")
    W = [(r(*s) * 0.02).bfloat16() for s in ((n, I_s, H), (n, I_s, H), (n, H, I_s))]
    own = {e: r(keep[e], H).bfloat16() for e in mine}
    ws = torch.empty(max(B.moe_ffn_workspace_bytes(cap, shard), 256), dtype=torch.uint8, device="cuda")
    got = []
    for c in counts:
        offs = np.concatenate([[0], np.cumsum(c)]).astype(np.int32)
        x = r(cap, H).bfloat16()
        for e in mine:
            x[offs[e]:offs[e] + keep[e]] = own[e]
        for flags in (0, B.MOE_FFN_LEAVE_ROOM):
            h = torch.zeros((cap, I_s), dtype=torch.bfloat16, device="cuda")
            y = torch.zeros((cap, H), device="cuda")
            B.moe_expert_ffn(x, torch.from_numpy(offs).cuda(), cap, shard, *W, h, y, ws, flags)
            out = [torch.cat([t[offs[e]:offs[e] + keep[e]].float() for e in mine]) for t in (h, y)]
            got.append(out if flow & B.DEBUG_FLOW_DOWN else out[:1])    # (a tiled down projection may be cut along K)
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)


@pytest.mark.parametrize("blocks", [11, 12, 13, 16, 17, 23, 32, 40])
def test_row_blocks_of_a_large_expert_in_groups(blocks):
    """Every tile once; from 12 row blocks on, 32 neighbouring tiles on an XCD touch few row and column blocks together."""
    ncb = 56
    offs = np.array([0, 256 * blocks, 256 * blocks + 300], dtype=np.int32)
    units = B.moe_debug_gemm_units(offs, int(offs[-1]), ncb)
    full = [(b, u) for b, u in enumerate(units.tolist()) if u[0] == 256 and u[1] == 0]
    seen = {(u[2] // 256, u[4]) for _, u in full}
    assert len(full) == len(seen) == blocks * ncb and seen == {(r, c) for r in range(blocks) for c in range(ncb)}
    windows = within = 0
    for xcd in range(8):
        mine = [(u[2] // 256, u[4]) for b, u in full if b % 8 == xcd]
        for i in range(0, len(mine) - 32, 32):
            rows, cols = ({t[j] for t in mine[i:i + 32]} for j in (0, 1))
            windows += 1
            # s row blocks and the column blocks that 32 tiles of them touch, s <= 8 in a group (11 alone: 11 + 4)
            within += len(rows) <= (8 if blocks >= 12 else 11) and len(rows) + len(cols) <= (14 if blocks >= 12 else 15)
    assert within >= 0.75 * windows          # the others lie across a change of groups

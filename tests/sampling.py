"""Token samples for parity checks at sizes where the oracle cannot evaluate every token.

Each output row of the layer depends on its own token only, so a sample of tokens is a valid
check; what a uniform sample can miss is the few rows that sit at the edges of the kernels' work
units (the last rows of an expert, the short tiles behind its full row blocks, tiles whose K range
is cut into slices).  `stratified_tokens` therefore starts from those rows, as the library's own
host-side work-list introspection reports them for the routing at hand, and fills up with random
tokens."""
import numpy as np

from paper_2508_19373_amd import binding as B


def _units(offs, cap_rows, ffn_shard, gateup, y_bf16):
    """The work list one GEMM of the tiled kernels runs for this routing, records of moe_debug_tall_units."""
    H, I_s = ffn_shard.hidden, ffn_shard.inter_slice
    ncb, nk = ((I_s + 127) // 128, H // 64) if gateup else ((H + 255) // 256, I_s // 64)
    tall = B.moe_debug_tall_gemms(cap_rows, ffn_shard)
    if tall == 0 and B.moe_debug_tile_rows(cap_rows, ffn_shard) == 160:
        plain = B.moe_debug_even_units(offs, cap_rows, ncb)
    elif tall & (B.DEBUG_TALL_GATEUP if gateup else B.DEBUG_TALL_DOWN_BF16 if y_bf16 else B.DEBUG_TALL_DOWN):
        slices = 0 if gateup or y_bf16 or I_s // 64 < 16 else min(I_s // 64 // 8, 16)
        return B.moe_debug_tall_units(offs, cap_rows, ncb, nk, slices)
    elif not gateup and not y_bf16:
        _, units = B.moe_debug_down_slices(offs, cap_rows, ffn_shard, with_units=True)
        row_end = np.asarray(offs)[np.minimum(units[:, 1], len(offs) - 2) + 1]
        return np.column_stack([units[:, :3], row_end, units[:, 3:]])
    else:
        plain = B.moe_debug_gemm_units(offs, cap_rows, ncb)
    out = np.zeros((len(plain), B.DEBUG_DEVICE_INTS), dtype=np.int32)
    out[:, :5], out[:, 7], out[:, 8] = plain, nk, -1
    return out


def edge_rows(offs, cap_rows, ffn_shard, y_bf16=False):
    """Permuted rows at the boundaries of every tile of both grouped GEMMs, the first and last
    row of every local expert, both sides of a tall tile's 256 rows, and a row inside every tile of the down projection
    that runs as K slices (one per tile and slice)."""
    offs = np.asarray(offs, dtype=np.int32)
    rows = set()
    for e in range(offs.size - 1):
        if offs[e + 1] > offs[e]:
            rows.update((int(offs[e]), int(offs[e + 1]) - 1))
    n_sliced = 0
    for gateup in (True, False):
        units = _units(offs, cap_rows, ffn_shard, gateup, y_bf16)
        units = units[units[:, 0] > 0]
        edge = units[(units[:, 4] == 0) | (units[:, 4] == units[:, 4].max(initial=0))]
        for h, e, row0, row_end in edge[:, :4].tolist():
            end = min(row0 + h, row_end)
            rows.update((row0, end - 1))
            if 256 < h < 512:
                rows.update((row0 + 255, min(row0 + 256, end - 1)))
        for h, e, row0, row_end, nb, z in units[units[:, 5] >= 1, :6].tolist():
            rows.add(row0 + ((7 * z + 3 * nb) % max(min(row0 + h, row_end) - row0, 1)))
            n_sliced += 1
    return np.array(sorted(rows), dtype=np.int64), n_sliced


def stratified_tokens(T, k, offs, row_src, ffn_shard, n_random, seed=1):
    """Sorted unique token ids: the tokens that own the edge rows, plus `n_random` random ones
    (all tokens if T is no larger than that).  Returns (tokens, number of edge rows, rows in sliced tiles)."""
    if T <= n_random:
        return np.arange(T), 0, 0
    rows, n_sliced = edge_rows(offs, T * k, ffn_shard)
    edge_tokens = np.unique(np.asarray(row_src)[rows] // k) if rows.size else np.array([], dtype=np.int64)
    rng = np.random.default_rng(seed)
    rnd = rng.choice(T, size=n_random, replace=False)
    return np.unique(np.concatenate([edge_tokens, rnd])), rows.size, n_sliced

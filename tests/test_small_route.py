"""Selection and permutation of small batches in one kernel (moe_forward), and the permutation's paths, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2508_19373_amd import binding as B
from paper_2508_19373_amd.layer import ExpertShardLayer

pytestmark = pytest.mark.gpu


def _layer(E, k, H, E_loc, off, T, renorm, g):
    r = lambda *s: torch.randn(s, generator=g, device="cuda")
    return ExpertShardLayer(n_experts=E, top_k=k, hidden=H, inter_full=64, inter_slice=64, n_local_experts=E_loc,
                            expert_offset=off, renorm=renorm, w_router=r(H, E) * 0.02, w_gate=r(E_loc, 64, H).bfloat16(),
                            w_up=r(E_loc, 64, H).bfloat16(), w_down=r(E_loc, H, 64).bfloat16(), max_tokens=max(T, 1))


@pytest.mark.parametrize("E,k,E_loc,off", [(60, 4, 60, 0), (64, 8, 32, 32), (17, 1, 17, 0), (128, 16, 64, 0), (256, 3, 256, 0),
                                           (8, 2, 2, 6)])
@pytest.mark.parametrize("T", [1, 16, 17, 32, 33, 128])   # one kernel up to 32 tokens
@pytest.mark.parametrize("given", [False, True])
def test_route_and_permute_in_a_forward(E, k, E_loc, off, T, given):
    """Top-k ids and the permutation equal the oracle's for the logits the GPU used, ties and signed zeros included."""
    g = torch.Generator(device="cuda")
    g.manual_seed(E + T)
    layer = _layer(E, k, 128, E_loc, off, T, E == 64, g)
    x = torch.randn((T, 128), generator=g, device="cuda").bfloat16()
    logits = None
    if given:
        logits = (torch.randn((T, E), generator=g, device="cuda") * 2).round() / 2   # many ties
        logits[0, ::2] = -0.0
        logits[0, 1::2] = 0.0
    layer.forward(x, logits)
    torch.cuda.synchronize()
    L = layer.logits[:T].cpu().numpy()
    idx, w32, _ = O.route_topk(L, k, layer.renorm)
    assert np.array_equal(layer.topk_idx[:T].cpu().numpy(), idx)
    assert np.allclose(layer.topk_w[:T].cpu().numpy(), w32, rtol=2e-6, atol=1e-9)
    offs, row_src, slot_row, _ = O.permute(np.zeros((T, 8), np.uint16), idx, E_loc, off)
    R = int(offs[-1])
    assert np.array_equal(layer.expert_offsets.cpu().numpy(), offs)
    assert np.array_equal(layer.row_src[:R].cpu().numpy(), row_src[:R])
    assert np.array_equal(layer.slot_row[:T * k].cpu().numpy(), slot_row)


@pytest.mark.parametrize("T,k,E,E_loc,off", [(512, 2, 8, 8, 0), (513, 2, 8, 4, 4), (1024, 2, 8, 8, 0), (1025, 2, 256, 256, 0),
                                             (16384, 4, 60, 60, 0), (16385, 4, 60, 15, 45)])
def test_permutation_at_the_edges_of_its_kernels(T, k, E, E_loc, off):
    """One workgroup up to 2048 assignments; two kernels up to 64 workgroups of 1024, three beyond."""
    rng = np.random.default_rng(T)
    idx = np.stack([rng.permutation(E)[:k] for _ in range(T)]).astype(np.int32)
    shard = B.make_shard(E, E_loc, off, 64, 64, 64)
    i32 = lambda n: torch.full((n,), -5, dtype=torch.int32, device="cuda")
    eo, rs, sr = i32(E_loc + 1), i32(T * k), i32(T * k)
    ws = torch.empty(B.moe_workspace_bytes(T, k, shard), dtype=torch.uint8, device="cuda")
    B.moe_permute(None, torch.from_numpy(idx).cuda(), T, k, shard, None, eo, rs, sr, ws)
    offs, row_src, slot_row, _ = O.permute(np.zeros((T, 8), np.uint16), idx, E_loc, off)
    R = int(offs[-1])
    assert np.array_equal(eo.cpu().numpy(), offs) and np.array_equal(sr.cpu().numpy(), slot_row)
    assert np.array_equal(rs.cpu().numpy()[:R], row_src[:R]) and np.all(rs.cpu().numpy()[R:] == -5)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("H", [8, 1000, 1024, 2056, 4096])
@pytest.mark.parametrize("shared", [False, True])
def test_combine_row_groups_and_column_passes(k, H, shared):
    """Every number of slots, columns in passes of 2048: missing slots, remainders, a shared expert or none."""
    rng = np.random.default_rng(k * H)
    T, R = 37, 37 * k
    y = rng.standard_normal((R, H)).astype(np.float32)
    slot = rng.permutation(R).astype(np.int32).reshape(T, k)
    slot[rng.random((T, k)) < 0.2] = -1
    w = rng.random((T, k)).astype(np.float32)
    x = torch.from_numpy(rng.standard_normal((T, H)).astype(np.float32)).bfloat16()
    ys = rng.standard_normal((T, H)).astype(np.float32)
    wg = (rng.standard_normal(H) * 0.05).astype(np.float32)
    ref = np.zeros((T, H))
    for j in range(k):
        ok = slot[:, j] >= 0
        ref[ok] += w[ok, j, None].astype(np.float64) * y[slot[ok, j]]
    if shared:
        ref += 1.0 / (1.0 + np.exp(-(x.double().numpy() @ wg.astype(np.float64))))[:, None] * ys
    dev = lambda a: torch.from_numpy(a).cuda()
    out = torch.full((T, H), float("nan"), device="cuda")
    B.moe_combine(dev(y), dev(slot.reshape(-1)), dev(w), T, k, H, dev(ys) if shared else None, x.cuda() if shared else None,
                  dev(wg) if shared else None, out, B.MOE_OUT_F32)
    # fp32 sums of up to 17 products of size one
    assert np.abs(out.cpu().numpy() - ref).max() < 17 * 2.0 ** -23 * 16

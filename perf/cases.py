"""The work a user of this package has it do, as measurable cases: the Expert module of one MoE layer on one
device's shard (ExpertShardLayer.forward, eager or replayed as the HIP graph its capture() returns), and the INT4
backup of expert weights (moe_int4_quantize / moe_int4_dequantize).

The model shapes, shards and token counts are those of `paper_2508_19373_amd.inputs`, the benchmark and the latency
table; token counts between them are free, odd ones included, as batches and prompt chunks come.  Inputs have the
distributions of `inputs.py` (x ~ N(0,1), weights ~ N(0,0.02), the models' router weights, or Zipf(1.2)-popular
experts given as logits) but are drawn on the GPU.
"""
import math
from functools import lru_cache

import numpy as np
import torch

from paper_2508_19373_amd import binding as B
from paper_2508_19373_amd import inputs as I
from paper_2508_19373_amd.latency_table import legal_shards
from paper_2508_19373_amd.layer import ExpertShardLayer

MODELS = {"tiny": I.TINY, "mixtral": I.MIXTRAL, "qwen": I.QWEN, "qwen2_57b": I.QWEN2_57B}


def _layer(name, model, tokens, *, tp=1, ep=1, ep_rank=0, routing="balanced", graph=False, y_perm_bf16=False,
           out_f32=False):
    case = dict(op="layer", model=model, tokens=tokens, tp=tp, ep=ep, ep_rank=ep_rank, routing=routing, graph=graph,
                y_perm_bf16=y_perm_bf16, out_f32=out_f32)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest layer: a handful of short kernels issued one by one, bound by launches and latency
        _layer("tiny_64", "tiny", 64),
        # a decoding step of a small batch on the whole layer: every weight is read once for two rows each
        _layer("mixtral_decode_16", "mixtral", 16, graph=True),
        # a prompt batch on the whole layer: about a thousand rows per expert
        _layer("mixtral_prefill_4096", "mixtral", 4096),
        # a tensor-parallel device's decoding step (a quarter of every expert)
        _layer("mixtral_tp4_decode_64", "mixtral", 64, tp=4, graph=True),
        # the same device in prefill
        _layer("mixtral_tp4_prefill_8192", "mixtral", 8192, tp=4),
        # the expert-parallel device that holds the two most popular experts of a skewed routing
        _layer("mixtral_ep4_hot_8192", "mixtral", 8192, ep=4, routing="zipf"),
        # many small experts and a shared one: decoding, ...
        _layer("qwen_decode_32", "qwen", 32, graph=True),
        # ... the ragged tail of a chunked prompt (bf16 between the experts and the combine, as a memory-tight user
        # sets it), ...
        _layer("qwen_chunk_333", "qwen", 333, y_perm_bf16=True),
        # ... and a full prompt batch
        _layer("qwen_prefill_4096", "qwen", 4096),
        # a hybrid TP x EP device of the largest model, mixed batch, fp32 partial sums for the reduction that follows
        _layer("qwen2_57b_tp2_ep2_1000", "qwen2_57b", 1000, tp=2, ep=2, routing="zipf", out_f32=True),
        # switching strategies: one device's share (two Mixtral-sized experts) of the INT4 backup back to bf16
        dict(name="int4_dequantize_352m", op="dequantize", n=2 * 3 * 4096 * 14336),
        # building that backup
        dict(name="int4_quantize_352m", op="quantize", n=2 * 3 * 4096 * 14336),
    ]


def draw(rng):
    limit = max(_cost(c) for c in listed())
    if rng.random() < 0.2:
        n = 64 * int(2.0 ** rng.uniform(12.0, 24.0))
        return dict(op=rng.choice(["dequantize", "quantize"]), n=n)
    while True:
        model = rng.choice(["tiny", "mixtral", "mixtral", "qwen", "qwen", "qwen2_57b"])
        tokens = int(2.0 ** rng.uniform(0.0, 13.0))
        tp, ep = rng.choice(legal_shards(MODELS[model]))
        if model == "tiny":
            tp, ep = 1, 1
        skewed = ep > 1 and rng.random() < 0.5
        case = _layer(None, model, tokens, tp=tp, ep=ep, ep_rank=rng.choice([0, ep - 1]),
                      routing="zipf" if skewed else "balanced", graph=tokens <= 256 and rng.random() < 0.6,
                      y_perm_bf16=rng.random() < 0.15, out_f32=rng.random() < (0.4 if tp > 1 else 0.1))
        if _cost(case) <= limit:
            return case


def _shape(case):
    return MODELS[case["model"]].shard(tp_degree=case["tp"], ep_degree=case["ep"], ep_rank=case["ep_rank"])


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal_bf16(g, shape, std=1.0):
    """N(0, std) in bf16, drawn in fp32 a slice of the first dimension at a time."""
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    for part in out if len(shape) > 2 else [out]:
        part.copy_(torch.randn(part.shape, generator=g, device="cuda").mul_(std))
    return out


def _prepare_layer(case, seed):
    s, T, g = _shape(case), case["tokens"], _generator(seed)
    H, E, n = s.hidden, s.n_experts, s.n_local_experts
    x = _normal_bf16(g, (T, H))
    w_router, logits = None, None
    if case["routing"] == "zipf":
        gumbel = -torch.empty((T, E), device="cuda").exponential_(generator=g).log_()
        logits = gumbel + torch.from_numpy(np.log(I.zipf_popularity(E)).astype(np.float32)).cuda()
    elif s.router == "uniform":
        a = 0.02 * math.sqrt(3.0)
        w_router = torch.empty((H, E), device="cuda").uniform_(-a, a, generator=g)
    else:
        w_router = torch.randn((H, E), generator=g, device="cuda").mul_(0.02)

    def ffn(experts, inter):
        return (_normal_bf16(g, (experts, inter, H), 0.02), _normal_bf16(g, (experts, inter, H), 0.02),
                _normal_bf16(g, (experts, H, inter), 0.02))

    gate, up, down = ffn(n, s.inter_slice)
    shared = ffn(1, s.inter_shared_slice) if s.inter_shared else None
    w_shared_gate = _normal_bf16(g, (H,), 0.02).float() if s.inter_shared else None
    layer = ExpertShardLayer(
        n_experts=E, top_k=s.top_k, hidden=H, inter_full=s.inter, inter_slice=s.inter_slice, n_local_experts=n,
        expert_offset=s.expert_offset, renorm=s.renorm, w_router=w_router, w_gate=gate, w_up=up, w_down=down,
        shared=shared, w_shared_gate=w_shared_gate, inter_shared_full=s.inter_shared,
        inter_shared_slice=s.inter_shared_slice, max_tokens=T, y_perm_bf16=case["y_perm_bf16"],
        out_f32=case["out_f32"])
    state = dict(op="layer", layer=layer, x=x, logits=logits, graph=None)
    if case["graph"]:
        state["graph"], state["y"] = layer.capture(x, logits)
    return state


def prepare(case, seed):
    if case["op"] == "layer":
        return _prepare_layer(case, seed)
    n, g = case["n"], _generator(seed)
    codes = torch.empty(n // 2, dtype=torch.uint8, device="cuda")
    qparams = torch.empty((n // B.INT4_GROUP, 2), dtype=torch.bfloat16, device="cuda")
    if case["op"] == "dequantize":
        # what quantising N(0, 0.02) weights leaves: 4.7 standard deviations between a group's extremes
        codes.random_(0, 256, generator=g)
        spread = torch.randn((n // B.INT4_GROUP, 2), generator=g, device="cuda").mul_(0.1).add_(1.0)
        qparams.copy_(spread * torch.tensor([0.0063, -0.047], device="cuda"))
        weights = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    else:
        weights = torch.empty(n, dtype=torch.bfloat16, device="cuda")
        for part in weights.split(1 << 26):
            part.copy_(torch.randn(part.shape, generator=g, device="cuda").mul_(0.02))
    return dict(op=case["op"], n=n, codes=codes, qparams=qparams, weights=weights)


def run(state):
    if state["op"] == "layer":
        if state["graph"] is not None:
            state["graph"].replay()
            return state["y"]
        return state["layer"].forward(state["x"], state["logits"])
    if state["op"] == "dequantize":
        B.moe_int4_dequantize(state["codes"], state["qparams"], state["n"], state["weights"])
        return state["weights"]
    B.moe_int4_quantize(state["weights"], state["n"], state["codes"], state["qparams"])
    return state["codes"], state["qparams"]


@lru_cache(maxsize=None)
def _pick_probabilities(model, routing):
    """Probability of each expert to be among a token's top k."""
    s = MODELS[model]
    if routing != "zipf":
        return np.full(s.n_experts, s.top_k / s.n_experts)
    order = np.argsort(-I.make_zipf_logits(0, 4096, s.n_experts), axis=1)[:, :s.top_k]
    return np.bincount(order.ravel(), minlength=s.n_experts) / 4096.0


def work(case):
    if case["op"] != "layer":
        return {"bytes": case["n"] * (2.0 + 0.5 + 4.0 / B.INT4_GROUP), "flops": 2.0 * case["n"]}
    s, T = _shape(case), case["tokens"]
    H, E, off, n = s.hidden, s.n_experts, s.expert_offset, s.n_local_experts
    p = _pick_probabilities(case["model"], case["routing"])[off:off + n]
    rows, active = T * float(p.sum()), float((1.0 - (1.0 - p) ** T).sum())  # expected
    flops = 6.0 * rows * H * s.inter_slice + 6.0 * T * H * s.inter_shared_slice
    nbytes = 2.0 * 3.0 * H * (active * s.inter_slice + s.inter_shared_slice)
    nbytes += 2.0 * T * H + (4.0 if case["out_f32"] else 2.0) * T * H
    if case["routing"] == "zipf":
        nbytes += 4.0 * T * E
    else:
        flops += 2.0 * T * H * E
        nbytes += 4.0 * H * E
    return {"bytes": nbytes, "flops": flops}


def _cost(case):
    w = work(case)
    return w["bytes"] / 6e12 + w["flops"] / 1.5e15


def tolerance(case):
    if case["op"] != "layer":
        return "exact"
    # against the same layer in 64 bits: rel 2.35e-3 with bf16 out (2.9e-3 with bf16 before the combine too, 1.66e-3 with
    # fp32 out), largest difference 0.8e-2 to 1.45e-2; two implementations with sums in another order are closer
    return {"rel": 5e-3, "max": 0.06}

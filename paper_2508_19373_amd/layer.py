"""One Expert-module call on one shard: owns the device buffers (allocated once through torch)
and issues the C-ABI calls in order.  No arithmetic happens here."""
from __future__ import annotations

from typing import NamedTuple

import numpy as np
import torch

from . import binding as B


def bf16_tensor(bits: np.ndarray, device="cuda") -> torch.Tensor:
    """uint16 bf16 bit patterns (numpy) -> torch.bfloat16 tensor on the device, same bits."""
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(device).view(torch.bfloat16)


def bf16_bits(t: torch.Tensor) -> np.ndarray:
    return t.detach().contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


FFN_ALIGN = 64  # moe_expert_ffn needs I_s % 64 == 0


def _pad_inter(w_gate, w_up, w_down, inter_slice):
    """Zero-pad an intermediate slice to the next multiple of FFN_ALIGN: extra gate/up rows and
    down columns of zeros add silu(0) * 0 = 0 times 0 to every output, so results are unchanged
    (memory plumbing for tensor-parallel slices such as 1408 / 4 = 352; no arithmetic here)."""
    pad = -inter_slice % FFN_ALIGN
    if pad == 0:
        return w_gate, w_up, w_down, inter_slice
    E, _, H = w_gate.shape
    g = torch.zeros((E, inter_slice + pad, H), dtype=w_gate.dtype, device=w_gate.device)
    u = torch.zeros_like(g)
    d = torch.zeros((E, H, inter_slice + pad), dtype=w_down.dtype, device=w_down.device)
    g[:, :inter_slice].copy_(w_gate)
    u[:, :inter_slice].copy_(w_up)
    d[:, :, :inter_slice].copy_(w_down)
    return g, u, d, inter_slice + pad


_SIDE_STREAMS = {}


def _side_stream(device):
    """One second stream per device for every layer of the process (layers run one after the other)."""
    key = str(torch.device(device))
    if key not in _SIDE_STREAMS:
        _SIDE_STREAMS[key] = torch.cuda.Stream(device=device)
    return _SIDE_STREAMS[key]


def routed_hint_beside_shared(ffn_shard, shared_shard, T) -> int:
    """Scheduling hint (a moe_expert_ffn flag, or 0) for the routed experts' call when the shared
    expert of T tokens runs beside it on a second stream.

    A tiled shared expert cannot start beside resident weight-streaming workgroups (each tiled
    workgroup needs a compute unit's whole LDS): the routed experts are kept tiled too, so that the
    two streams interleave tile by tile.  Measured: -8 to -20 % at 64 to 256 tokens on shards with
    60 or 64 local experts (two or more rounds of tiles even with a few rows per expert, so the
    tiled kernels stream as fast as the streaming kernel); +5 to +16 % on shards with 15 or 30
    experts, hence the tile count.  Those leave 16 compute units to the shared expert instead (30
    experts, 96 / 128 tokens: 177 / 179 -> 170 / 173 us).  A streaming shared expert needs neither.  (For a shared expert
    both of whose GEMMs run as moe_debug_ffn_plan says; shared_on_streaming_tiles comes first.)"""
    if all(B.moe_debug_ffn_plan(T, shared_shard)[:2]):
        return 0
    gateup_tiles = ffn_shard.n_local_experts * ((ffn_shard.inter_slice + 127) // 128)
    return B.MOE_FFN_TILED if gateup_tiles >= 512 else B.MOE_FFN_LEAVE_ROOM


def shared_on_streaming_tiles(shared_shard, T, y_perm_bf16) -> bool:
    """Whether the shared expert of T tokens holds every compute unit by itself: its gate/up projection runs the streaming
    tiles (moe_debug_flow; a workgroup of a whole LDS stays on each unit for the launch), whatever moe_debug_ffn_plan says
    of it, and its down projection, cut along K or streaming, is over soon.  Then room left by the routed experts' call
    serves nobody and tiles of theirs interleave with nothing, so the call needs no hint.  Hint as for tiled / none, us:
    Qwen1.5-MoE 64 tokens 232 / 230, EP=2 48: 150 / 137, EP=4 150: 114 / 111, Qwen2-57B 48: 705 / 697, EP=4 100: 293 / 275,
    EP=8 150: 229 / 210, TP=2 48: 393 / 376, TP=2 EP=2 300: 297 / 288, TP=4 EP=2 48: 158 / 141.  Not with a bf16 down projection:
    uncut, its H / 256 tiles walk all of K and have to start early (Qwen1.5-MoE 160 tokens 239 / 264, Qwen2-57B TP=2 EP=2 48:
    251 / 293)."""
    return not y_perm_bf16 and bool(B.moe_debug_flow(T, shared_shard) & B.DEBUG_FLOW_GATEUP)


class _Plan(NamedTuple):
    ffn_ws: int
    ffn_ws_sh: int
    hint: int
    gather: bool
    routed_first: bool


class ExpertShardLayer:
    """route -> permute -> expert FFN (-> shared expert FFN) -> combine, on the current stream.

    Weights are torch.bfloat16 CUDA tensors in the layouts of include/moe_shard.h.  A slice of
    the intermediate dimension that is not a multiple of 64 is zero-padded once, here, and the
    FFN calls then describe the padded matrices.
    ``y_perm_bf16`` / ``out_f32`` select the element types of the intermediate and the output.
    """

    def __init__(self, *, n_experts, top_k, hidden, inter_full, inter_slice, n_local_experts=None, expert_offset=0,
                 renorm=True, w_router=None, w_gate=None, w_up=None, w_down=None, shared=None, w_shared_gate=None,
                 inter_shared_full=0, inter_shared_slice=0, max_tokens=0, y_perm_bf16=False, out_f32=False,
                 overlap_shared=True, gather_in_ffn=None, device="cuda"):
        n_local_experts = n_experts if n_local_experts is None else n_local_experts
        self.E, self.k, self.H = n_experts, top_k, hidden
        self.shard = B.make_shard(n_experts, n_local_experts, expert_offset, hidden, inter_full, inter_slice)
        self.renorm = renorm
        w_gate, w_up, w_down, padded = _pad_inter(w_gate, w_up, w_down, inter_slice)
        self.ffn_shard = B.make_shard(n_experts, n_local_experts, expert_offset, hidden,
                                      padded * (inter_full // inter_slice), padded)
        self.w_router, self.w_gate, self.w_up, self.w_down = w_router, w_gate, w_up, w_down
        self.w_shared_gate = w_shared_gate
        self.shared, self.shared_shard = None, None
        if shared is not None:
            *self.shared, padded = _pad_inter(*shared, inter_shared_slice)
            self.shared_shard = B.make_shard(1, 1, 0, hidden, padded * (inter_shared_full // inter_shared_slice),
                                             padded)
        self.y_perm_bf16, self.out_f32 = y_perm_bf16, out_f32
        self.device = device
        # the shared expert depends on x only: it may run on a second stream (default priority) beside
        # routing, permutation and the routed experts, and joins before the combine
        # the routed experts can read their rows of x in place through row_src (no permuted copy of
        # x).  That saves about half of moe_permute's time and costs about 1 % of GEMM1's (scattered
        # rows), so by default it is used unless the slice is wide: measured break-even near
        # I_s = 12000 (Mixtral unsharded, I_s = 14336: permute -14 us, GEMM1 +16 us).  The weight-streaming
        # kernel loads its rows once per workgroup either way, so calls that it serves always gather
        # (gathers(T) below).
        self.gather_in_ffn = (inter_slice < 12288) if gather_in_ffn is None else bool(gather_in_ffn)
        self._gather_auto = gather_in_ffn is None
        self.overlap_shared = bool(overlap_shared) and shared is not None
        self._side = _side_stream(device) if self.overlap_shared else None
        self.Tmax = -1
        # {0, T} for the shared expert's call, one immutable device tensor per token count: a
        # captured graph keeps reading the tensor it was captured with
        self._sh_offsets = {}
        # buffers a captured graph still points at are kept alive when a larger batch makes the
        # layer allocate anew, so replaying an older graph stays valid (it works on its own buffers)
        self._captured, self._retired = False, []
        self._plans = {}
        if max_tokens:
            self._alloc(max_tokens)

    _BUFFERS = ("logits", "topk_idx", "topk_w", "x_perm", "expert_offsets", "row_src", "slot_row", "h_ws", "y_perm",
                "workspace", "ffn_ws", "y_out", "h_sh", "y_shared", "ffn_ws_sh")

    def _retire(self, names):
        if self._captured:
            self._retired.extend(getattr(self, n) for n in names if getattr(self, n, None) is not None)

    def _alloc(self, T):
        d, k, H, E = self.device, self.k, self.H, self.E
        self._retire(self._BUFFERS)
        cap = max(T * k, 1)
        Tn = max(T, 1)
        ydt = torch.bfloat16 if self.y_perm_bf16 else torch.float32
        self.logits = torch.empty((Tn, E), dtype=torch.float32, device=d)
        self.topk_idx = torch.empty((Tn, k), dtype=torch.int32, device=d)
        self.topk_w = torch.empty((Tn, k), dtype=torch.float32, device=d)
        self.x_perm = None if self.gather_in_ffn else torch.empty((cap, H), dtype=torch.bfloat16, device=d)
        self.expert_offsets = torch.empty(self.shard.n_local_experts + 1, dtype=torch.int32, device=d)
        self.row_src = torch.empty(cap, dtype=torch.int32, device=d)
        self.slot_row = torch.empty(cap, dtype=torch.int32, device=d)
        self.h_ws = torch.empty((cap, self.ffn_shard.inter_slice), dtype=torch.bfloat16, device=d)
        self.y_perm = torch.empty((cap, H), dtype=ydt, device=d)
        self.workspace = torch.empty(max(B.moe_workspace_bytes(T, k, self.shard), 256), dtype=torch.uint8, device=d)
        self.ffn_ws = torch.empty(max(B.moe_ffn_workspace_bytes(cap, self.ffn_shard), 256), dtype=torch.uint8, device=d)
        self.y_out = torch.empty((Tn, H), dtype=torch.float32 if self.out_f32 else torch.bfloat16, device=d)
        if self.shared is not None:
            self.h_sh = torch.empty((Tn, self.shared_shard.inter_slice), dtype=torch.bfloat16, device=d)
            self.y_shared = torch.empty((Tn, H), dtype=ydt, device=d)
            self.ffn_ws_sh = torch.empty(max(B.moe_ffn_workspace_bytes(Tn, self.shared_shard), 256),
                                         dtype=torch.uint8, device=d)
        self.Tmax = T

    def _shared_offsets(self, T):
        """Device tensor {0, T}: written once, on first use of this token count, and complete
        before this returns (whatever stream the kernels then run on)."""
        t = self._sh_offsets.get(T)
        if t is None:
            if torch.cuda.is_current_stream_capturing():
                raise RuntimeError("run one eager forward with this token count before capturing a graph")
            t = torch.tensor([0, T], dtype=torch.int32).to(self.device)
            torch.cuda.current_stream().synchronize()
            self._sh_offsets[T] = t
        return t

    @property
    def sh_offsets(self):
        """The shared expert's offsets for the most recent token count."""
        return self._sh_offsets[self._last_T]

    def gathers(self, T) -> bool:
        """Whether a forward of T tokens reads the routed experts' rows of x in place (no permuted copy)."""
        if self.gather_in_ffn or not self._gather_auto:
            return self.gather_in_ffn
        # GEMM1 on a kernel that streams the weights: the rows are few
        return bool(B.moe_debug_ffn_plan(T * self.k, self.ffn_shard)[0] or
                    B.moe_debug_flow(T * self.k, self.ffn_shard) & B.DEBUG_FLOW_GATEUP)

    def _weight_bytes(self):
        """Bytes of the routed and of the shared experts' matrices on this device."""
        return 6 * self.w_gate.numel(), 6 * self.shared[0].numel()

    def _shared_tiled(self, T):
        return not all(B.moe_debug_ffn_plan(T, self.shared_shard)[:2])

    def _routed_first(self, T) -> bool:
        """Whether a graph holds the routed experts' branch first (see forward).  Not before a shared expert of several
        hundred MB, which fills the time of the router and the permutation, nor before a tiled one that ends last (the
        routed experts few, or the tokens many).  Routed / shared first, us: Qwen1.5-MoE 128 tokens 245 / 256, TP=4 16 tokens 85 / 87,
        TP=8 100 tokens 85 / 94, Qwen2-57B TP=2 EP=2 48 tokens 246 / 257; unsharded (440 MB) 16 tokens 644 / 628; Qwen1.5
        TP=2 EP=4 (130 MB routed) 16 tokens 60 / 62, 128: 93 / 84, TP=4 200: 121 / 111.  Nor, from 33 tokens on, before one on the
        streaming tiles, which holds the units the longer the more of the weights are its own (Qwen2-57B TP=2 EP=4, half as
        much shared as routed, 100 tokens 193 / 166, Qwen1.5 EP=4, a quarter, 48: 107 / 96; EP=2, an eighth, 100: 143 / 150)."""
        routed, shared = self._weight_bytes()
        # with a token or two the routed experts that have rows are as few bytes as the shared one (Qwen1.5 EP=2, 2 tokens: 59 / 53)
        active = routed * min(1.0, T * self.k / self.E)
        tiled = self._shared_tiled(T)
        ratio = 7.0 if tiled and shared_on_streaming_tiles(self.shared_shard, T, self.y_perm_bf16) else 1.25
        return shared <= 256e6 and active >= ratio * shared and (not tiled or (routed >= 135e6 and T <= 160))

    def _plan(self, T) -> "_Plan":
        """What a forward of T tokens needs to know about itself: a function of T, the shards and the switches,
        kept per token count (at most 256 of them)."""
        key = (T, self.gather_in_ffn, self.overlap_shared)
        plan = self._plans.get(key)
        if plan is None:
            sh = self.shared is not None
            hint = 0
            if sh and self.overlap_shared and not shared_on_streaming_tiles(self.shared_shard, T, self.y_perm_bf16):
                hint = routed_hint_beside_shared(self.ffn_shard, self.shared_shard, T)
                # Planned for up to 64 rows per expert the kernel whose weight stream never stops is the faster one also beside the
                # shared expert's tiles, with room left for them (tiled / with room, us: Qwen1.5-MoE 333 tokens 270 / 260, 600:
                # 302 / 292).
                rows = B.moe_debug_flow_rows(T * self.k, self.ffn_shard)
                routed, shared = self._weight_bytes()
                if hint == B.MOE_FFN_TILED and 0 < rows <= (128 if self.H >= 3072 else 64):
                    hint = B.MOE_FFN_LEAVE_ROOM
                # not in two row passes (Qwen2-57B TP=4 2107 tokens 630 / 671) or with more rows than 64 on short slices (TP=8 482
                # tokens 202 / 209) or 160 for few experts (Qwen1.5 EP=4 1497: 208 / 212)
                elif hint == B.MOE_FFN_LEAVE_ROOM and ((rows == 160 and T * self.k > 165 * self.E) or
                                                       (rows > 64 and self.ffn_shard.inter_slice < 512) or
                                                       (rows == 160 and self.ffn_shard.n_local_experts < 24)):
                    hint = B.MOE_FFN_TILED
                # nor beside as much shared weight as there is routed: those tiles are half of the work, and the two calls
                # interleave tile by tile (Qwen2-57B EP=8, 48 / 128 / 256 tokens 192 / 216 / 240 tiled, 214 / 226 / 270)
                # (or, from 160 tokens on, beside as few: Qwen1.5 TP=2 EP=4 256 tokens 92 / 96)
                if hint != 0 and rows > 0 and (2 * shared >= routed or (routed < 135e6 and T > 160)):
                    hint = B.MOE_FFN_TILED
                # With more rows than 64 room left costs more than it gives: the shared expert's tiles start on 16 units and the
                # rest of them wait for the routed call's end all the same.  Without, its stream is over sooner (with room / no
                # hint, and tiled, us: Qwen2-57B TP=4 EP=2 384 tokens 203 / 193, 192, 1024: 277 / 256, 255, TP=2 EP=2 under Zipf(1.2)
                # 768: 499 / 440, 462, Qwen1.5 TP=2 EP=2 768: 143 / 127, 134, 2048: 210 / 187, 197; 92 shards and token counts, none
                # to room 0.977 eager, 0.962 in a graph).  A bf16 shared down projection, uncut, walks all of K and has to start
                # early: tiled there (38 of them: 0.988, 0.978; no hint 1.005, 1.014), and with up to 64 rows where that walk is long
                # and the gate/up projection before it tiled as well (Qwen2-57B 192 / 384 tokens 825 / 946 with room, 768 / 835 tiled,
                # TP=2 448 / 491, 416 / 456; 256 tokens, one row block, 2 % slower; Qwen1.5, 5632, 256 to 512 tokens 4 % slower).
                if hint == B.MOE_FFN_LEAVE_ROOM and rows > 64:
                    hint = B.MOE_FFN_TILED if self.y_perm_bf16 else 0
                elif (hint == B.MOE_FFN_LEAVE_ROOM and rows > 0 and self.y_perm_bf16 and
                      self.shared_shard.inter_slice >= 8192 and
                      not B.moe_debug_flow(T, self.shared_shard) & B.DEBUG_FLOW_GATEUP):
                    hint = B.MOE_FFN_TILED
            plan = _Plan(B.moe_ffn_workspace_bytes(T * self.k, self.ffn_shard),
                         B.moe_ffn_workspace_bytes(T, self.shared_shard) if sh else 0, hint, self.gathers(T),
                         sh and self._routed_first(T))
            if len(self._plans) >= 256:
                self._plans.clear()
            self._plans[key] = plan
        return plan

    def forward(self, x: torch.Tensor, logits: torch.Tensor | None = None, stream=None) -> torch.Tensor:
        T = x.shape[0]
        if T > self.Tmax:
            if torch.cuda.is_current_stream_capturing():
                raise RuntimeError("run one eager forward with this token count before capturing a graph")
            self._alloc(T)
        self._last_T = T
        k, H = self.k, self.H
        plan = self._plan(T)
        # the FFN scratch depends on the regime (decode-sized calls need split-K partials)
        if plan.ffn_ws > self.ffn_ws.numel():
            self._retire(("ffn_ws",))
            self.ffn_ws = torch.empty(plan.ffn_ws, dtype=torch.uint8, device=self.device)
        if self.shared is not None and plan.ffn_ws_sh > self.ffn_ws_sh.numel():
            self._retire(("ffn_ws_sh",))
            self.ffn_ws_sh = torch.empty(plan.ffn_ws_sh, dtype=torch.uint8, device=self.device)
        flags = B.MOE_RENORM_TOPK if self.renorm else 0
        if logits is not None:
            self.logits[:T].copy_(logits)
            flags |= B.MOE_LOGITS_GIVEN
        yflag = B.MOE_Y_PERM_BF16 if self.y_perm_bf16 else 0
        cflags = yflag | (B.MOE_OUT_F32 if self.out_f32 else 0)
        ptr = B._ptr
        gate_x = x if self.w_shared_gate is not None else None
        # one call for the whole chain: a decoding batch's kernels take less time than the marshalling of four
        # calls.  The addresses are taken anew each time, nothing is kept from one forward to the next.
        args = B.MoeForwardArgs(
            ptr(x), ptr(self.w_router), ptr(self.logits), ptr(self.topk_idx), ptr(self.topk_w),
            None if plan.gather else ptr(self.x_perm), ptr(self.expert_offsets), ptr(self.row_src), ptr(self.slot_row),
            ptr(self.workspace), self.workspace.numel(), ptr(self.w_gate), ptr(self.w_up), ptr(self.w_down),
            ptr(self.h_ws), ptr(self.y_perm), ptr(self.ffn_ws), self.ffn_ws.numel(),
            None, ptr(gate_x), ptr(self.w_shared_gate), ptr(self.y_out), T, k, flags, yflag | plan.hint, cflags)
        if self.shared is None:
            B.moe_forward(args, self.shard, self.ffn_shard, stream)
            return self.y_out[:T]
        args.combine_flags = B.MOE_NO_COMBINE     # the combine waits for the shared expert
        sh_offsets = self._shared_offsets(T)
        if self.overlap_shared:
            if stream is not None:
                raise ValueError("overlap_shared works on torch's current stream only")
            main = torch.cuda.current_stream()
            self._side.wait_stream(main)          # x (and sh_offsets) are ready where main stands now
            def shared():
                # a streaming shared expert leaves 16 compute units free, so that the router and the
                # permutation on the main stream, each a workgroup or two on the critical path, start
                # at once instead of waiting for a resident workgroup to finish (-2 to -3.5 % at 16 to 64 tokens)
                B.moe_expert_ffn(x, sh_offsets, T, self.shared_shard, self.shared[0], self.shared[1], self.shared[2],
                                 self.h_sh, self.y_shared, self.ffn_ws_sh, yflag | B.MOE_FFN_LEAVE_ROOM, self._side)

            # Eager, the shared expert first: it starts while the host enqueues the others.  A graph runs its branches in the
            # order of their first kernels and the combine on the first one's queue, so there the routed experts, where they
            # end last, come first: a queue waits 10 us for another one's kernel.
            if torch.cuda.is_current_stream_capturing() and plan.routed_first:
                B.moe_forward(args, self.shard, self.ffn_shard, main)
                shared()
            else:
                shared()
                B.moe_forward(args, self.shard, self.ffn_shard, main)
            main.wait_stream(self._side)
        else:
            B.moe_forward(args, self.shard, self.ffn_shard, stream)
            B.moe_expert_ffn(x, sh_offsets, T, self.shared_shard, self.shared[0], self.shared[1], self.shared[2],
                             self.h_sh, self.y_shared, self.ffn_ws_sh, yflag, stream)
        B.moe_combine(self.y_perm, self.slot_row, self.topk_w, T, k, H, self.y_shared, gate_x, self.w_shared_gate,
                      self.y_out, cflags, stream)
        return self.y_out[:T]

    def capture(self, x: torch.Tensor, logits: torch.Tensor | None = None):
        """Capture one forward on (x, logits) into a HIP graph; returns (graph, output view).
        Decode-sized layers are a chain of short kernels, so replaying a graph removes most of
        the launch gaps.  The library enqueues kernels only (no memset nodes, no allocation),
        which is what makes the capture legal; x / logits are read in place at every replay."""
        self.forward(x, logits)  # eager warm-up: sizes the buffers, sets the shared-expert offsets
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        self._captured = True
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                out = self.forward(x, logits)
        torch.cuda.current_stream().wait_stream(side)
        return graph, out

    @classmethod
    def from_inputs(cls, li, **kw) -> "ExpertShardLayer":
        """Build from paper_2508_19373_amd.inputs.LayerInputs (uploads the weights)."""
        s = li.shape
        kw.setdefault("max_tokens", li.T)
        shared = None
        if li.ws_gate is not None:
            shared = tuple(bf16_tensor(w) for w in (li.ws_gate, li.ws_up, li.ws_down))
        return cls(n_experts=s.n_experts, top_k=s.top_k, hidden=s.hidden, inter_full=s.inter,
                   inter_slice=s.inter_slice, n_local_experts=s.n_local_experts, expert_offset=s.expert_offset,
                   renorm=s.renorm,
                   w_router=None if li.w_router is None else torch.from_numpy(li.w_router).cuda(),
                   w_gate=bf16_tensor(li.w_gate), w_up=bf16_tensor(li.w_up), w_down=bf16_tensor(li.w_down),
                   shared=shared,
                   w_shared_gate=None if (li.w_shared_gate is None or shared is None) else torch.from_numpy(li.w_shared_gate).cuda(),
                   inter_shared_full=s.inter_shared, inter_shared_slice=s.inter_shared_slice,
                   **kw)

"""Buffers of one MoE verify layer plus the library call of its five steps.  No arithmetic here:
the class only owns the output / scratch tensors (allocated once) and marshals arguments."""
from __future__ import annotations

import torch

from . import binding as B


class MoEVerifyLayer:
    """route -> permute -> grouped SwiGLU -> combine on preallocated buffers.

    T tokens = B sequences x (gamma+1) positions (the tokens one verification pass scores).
    """

    def __init__(self, T, d_model, d_ff, E, k, dtype, device="cuda", renorm=True,
                 fuse_gather=True):
        """fuse_gather: moe_permute writes indices only and the gate/up GEMM gathers token rows
        itself (moe_expert_up_swiglu_gather); False materialises x_perm first."""
        self.T, self.d, self.f, self.E, self.k = T, d_model, d_ff, E, k
        self.dtype, self.renorm = dtype, renorm
        self.fuse_gather = fuse_gather and T * d_model * (4 if dtype == torch.float32 else 2) < 2 ** 32
        P = T * k
        dev = torch.device(device)
        i32 = dict(dtype=torch.int32, device=dev)
        self.topk_idx = torch.empty((T, k), **i32)
        self.topk_w = torch.empty((T, k), dtype=torch.float32, device=dev)
        self.expert_offsets = torch.empty((E + 1,), **i32)
        self.row_src = torch.empty((P,), **i32)
        self.row_of = torch.empty((P,), **i32)
        self.x_perm = torch.empty((P, d_model), dtype=dtype, device=dev)
        self.y_perm = torch.empty((P, d_model), dtype=dtype, device=dev)
        self.out = torch.empty((T, d_model), dtype=dtype, device=dev)
        self.h = torch.empty((P, d_ff), dtype=dtype, device=dev)
        # Of a small batch's router workgroups (moe_layer_forward_counted), 0 between calls once _own_counter() has
        # cleared it.
        self.counter = torch.empty((1,), **i32) if T <= 64 and E <= 64 and dev.type == "cuda" else None
        self._counter_is_clear = False
        self.h_packed = None                     # allocated on first use of packed weights
        self.x_packed = None

    # Which projections run on tile-packed operands (measured crossovers, average rows per
    # expert r = T*k/E).  Gate/up, with the gather of its rows: from r >= 48, and at any r for
    # d_model < 4096 (layers of 64 experts x 2048 x 1408, packed / row-major, us: 64 tokens 140 / 151, even 192 / 205, 320 210 / 215,
    # even 205 / 214, 640 273 / 271, even 224 / 244, 1285 324 / 339, even 255 / 254, 2040 379 / 387; 16 x 2048 x 3072, 200 115 / 122, 640
    # 136 / 148; 8 x 3072 x 1024, 100 52 / 54).  Down:
    # from r >= 96, or with d_ff < 4096, or from r >= 56 where its narrow tiles fill the chip (at most
    # 128 tiles of 256 outputs: 8 experts x 4096 outputs, 65 rows each 156 us against 173 row-major;
    # 16 x 5120, 75 rows 287 against 264).
    # Only the device knows how many experts a batch meets: at least k, however many rows there are.  Below 48 rows gate/up
    # goes packed where it is ahead for few of them as well: at least 8192 outputs and 256 tiles of 128, and from 20 rows, or from
    # 4 where k experts have 192 tiles (layer, us, row-major / packed gate/up, by active experts: 8 x 4096 x 14336, 4 rows all 453 /
    # 450, 7 437 / 444, 6 377 / 356, 5 318 / 325, 4 254 / 242, 3 205 / 215, 2 137 / 136, 20 rows all 470 / 458, 40 rows 488 / 476, but one row, 5
    # active 296 / 313; 16 x 5120 x 8192, 20 rows all 673 / 662, 2 186 / 181, 1 160 / 155, but 14 rows, 2 153 / 171, 1 112 / 137;
    # 16 x 4096 x 4096, 24 rows all 290 / 302, 2 79 / 109).  The packed down projection has no form for few experts (row-major /
    # packed, gate/up packed: 8 x 4096 x 14336, 8 rows all 454 / 449, 4 251 / 287, 2 143 / 206; 16 x 2048 x 8192, 8 rows all 292 / 271, 8
    # 156 / 182, 2 69 / 112), so its lines stay above.
    PACKED_UP_MIN_ROWS = 48
    PACKED_UP_MIN_ROWS_WIDE = 20
    PACKED_UP_MIN_ROWS_ACTIVE = 4
    PACKED_UP_WIDE = 8192
    PACKED_UP_MIN_TILES = 256
    PACKED_UP_MIN_TILES_ACTIVE = 192
    PACKED_DOWN_MIN_ROWS = 96
    PACKED_DOWN_MIN_ROWS_FEW_TILES = 56

    @classmethod
    def packed_plan(cls, n_pairs, E, d_model, d_ff, few_experts=False, k=1):
        """(gate/up on packed operands?, down on packed operands?) for a batch of n_pairs (token, expert)
        pairs that meets at least k experts; few_experts: a draft model's, which may meet a single one."""
        up = n_pairs >= cls.PACKED_UP_MIN_ROWS * E or d_model < 4096
        min_rows = (cls.PACKED_DOWN_MIN_ROWS_FEW_TILES if E * -(-d_model // 256) <= 128 else
                    cls.PACKED_DOWN_MIN_ROWS)
        down = up and (n_pairs >= min_rows * E or d_ff < 4096)
        tiles = -(-d_ff // 128)                  # of 128 gate/up outputs, per expert
        if not few_experts and d_ff >= cls.PACKED_UP_WIDE and E * tiles >= cls.PACKED_UP_MIN_TILES:
            up = up or n_pairs >= cls.PACKED_UP_MIN_ROWS_WIDE * E or (
                n_pairs >= cls.PACKED_UP_MIN_ROWS_ACTIVE * E and k * tiles >= cls.PACKED_UP_MIN_TILES_ACTIVE)
        return up, down

    # Packed gate/up: rows gathered by the GEMM itself (64-byte requests, once per 128 outputs), or written
    # tile-packed first ((T + n_pairs) rows and a launch).  Gathering is ahead up to 2048 outputs at any batch
    # size (us, packed first / gathered, 64 experts x 2048 x 1408, top-6: 64 tokens 74.5 / 70.7, 320 118 / 110,
    # 1285 167 / 158; 32 x 512 x 2048, 1600 tokens 62.3 / 60.5) and up to 4096 with few rows per expert (16 x 2048 x
    # 4096, 50 rows 89.5 / 87.6; 150 rows 130 / 134); wider ones read the rows too often (8 x 4096 x 14336, 256
    # rows 473 / 493; 16 x 5120 x 8192, 32 rows 451 / 459).
    GATHER_MAX_FF = 2048
    GATHER_MAX_FF_FEW_ROWS = 4096
    GATHER_FEW_ROWS = 64

    @classmethod
    def gathers_packed(cls, n_pairs, E, d_ff):
        """Whether the packed gate/up GEMM reads the token rows in place (row-major)."""
        return d_ff <= cls.GATHER_MAX_FF or (
            d_ff <= cls.GATHER_MAX_FF_FEW_ROWS and n_pairs <= cls.GATHER_FEW_ROWS * E)

    @staticmethod
    def pack_weights(w_gate, w_up, w_down, stream=None):
        """One-time re-layout of the expert weights for the tile-packed kernels (bf16 only):
        returns the dict to pass as `packed=` to forward().  The row-major tensors stay valid and
        are still used whenever packed_plan() sends a projection to the row-major kernels."""
        out = {}
        for name, w in (("w_gate", w_gate), ("w_up", w_up), ("w_down", w_down)):
            wp = torch.empty_like(w)
            B.moe_pack_weights(w, wp, stream)
            out[name] = wp
        return out

    def _own_counter(self, stream):
        """The counter, cleared on the stream of the first call that runs at once: whatever stream the layer was made
        on owes it nothing.  None while a capture comes before that call: its clearing would only be recorded."""
        if self.counter is not None and not self._counter_is_clear:
            with torch.cuda.stream(stream if stream is not None else torch.cuda.current_stream(self.out.device)):
                if torch.cuda.is_current_stream_capturing():
                    return None
                self.counter.zero_()
            self._counter_is_clear = True
        return self.counter

    def forward(self, x, w_router, w_gate, w_up, w_down, bias=None, residual=None, out=None,
                stream=None, marks=None, draft_remap=None, packed=None):
        """Enqueues the layer.  `marks`, if given, is a sequence of six torch events recorded on
        `stream` before the router and after each of the five steps (route, permute, gate/up,
        down, combine): the benchmark's per-kernel times.  On the tile-packed path the permute
        step includes the gather of the token rows into tile-packed form, unless the gate/up
        kernel gathers them (gathers_packed()).  Without marks a small batch routes and permutes in one launch.
        `draft_remap` ([E] int32 from moe_nearest_draft_expert) switches to the draft model's
        routing: selected experts that are not resident are replaced by their nearest draft
        expert, so only draft experts compute.
        `packed` (from pack_weights) lets the expert GEMMs run on tile-packed operands where
        packed_plan() says they are the faster ones (bf16 only)."""
        out = self.out if out is None else out
        up_packed = down_packed = False
        if packed is not None and self.dtype == torch.bfloat16 and self.fuse_gather:
            # the packed kernels take 16-byte aligned rows only: any other x keeps the shorter plan as well
            up_packed, down_packed = self.packed_plan(
                self.T * self.k, self.E, self.d, self.f,
                few_experts=draft_remap is not None or x.data_ptr() % 16 != 0, k=self.k)
        gathered = (down_packed and self.gathers_packed(self.T * self.k, self.E, self.f)
                    and x.data_ptr() % 16 == 0)
        # x_packed also where this call gathers: x may be another tensor next time, and a captured call must not
        # allocate once such a call has run
        if self.x_packed is None and up_packed:
            self.x_packed = torch.empty(
                (B.moe_packed_h_bytes(self.T * self.k, self.d, self.E),), dtype=torch.uint8,
                device=self.h.device)
        if self.h_packed is None and down_packed:
            self.h_packed = torch.empty(
                (B.moe_packed_h_bytes(self.T * self.k, self.f, self.E),), dtype=torch.uint8,
                device=self.h.device)
        gate = packed["w_gate"] if up_packed else w_gate
        if (marks is None and self.fuse_gather and x.dtype == self.dtype
                and x.shape == (self.T, self.d) and gate.shape == (self.E, self.f, self.d)
                and w_router.shape[0] == self.E):
            layout = (B.ROW_MAJOR if not up_packed else B.PACKED_GATHER if gathered else
                      B.PACKED if down_packed else B.PACKED_UP)
            B.moe_layer_forward(
                x, w_router, bias, draft_remap, gate, packed["w_up"] if up_packed else w_up,
                packed["w_down"] if down_packed else w_down,
                residual, self.k, self.renorm, layout, self.topk_idx, self.topk_w, self.expert_offsets,
                self.row_src, self.row_of, self.x_packed, self.h_packed if down_packed else self.h,
                self.y_perm, out, stream, self._own_counter(stream))
            return out
        # with marks, or x_perm written first: the same steps and layouts as calls of their own
        if marks is not None:
            marks[0].record(stream)
        if draft_remap is None:
            B.moe_route_topk(x, w_router, bias, self.k, self.renorm, self.topk_idx, self.topk_w,
                             stream)
        else:
            B.moe_route_topk_draft(x, w_router, bias, self.k, self.renorm, draft_remap,
                                   self.topk_idx, self.topk_w, stream)
        if marks is not None:
            marks[1].record(stream)
        B.moe_permute(x, self.topk_idx, self.E, None if self.fuse_gather else self.x_perm,
                      self.expert_offsets, self.row_src, self.row_of, stream)
        if up_packed and not gathered:
            # the data movement of the permute step, written once in the GEMM's own layout
            B.moe_permute_rows_packed(x, self.row_src, self.k, self.expert_offsets,
                                      self.T * self.k, self.x_packed, stream)
        if marks is not None:
            marks[2].record(stream)
        if gathered:
            B.moe_expert_up_swiglu_gather_packed(x, self.row_src, self.k, self.expert_offsets,
                                                 packed["w_gate"], packed["w_up"],
                                                 self.T * self.k, self.h_packed, None, stream)
        elif up_packed:
            B.moe_expert_up_swiglu_packed(self.x_packed, self.expert_offsets, packed["w_gate"],
                                          packed["w_up"], self.T * self.k,
                                          self.h_packed if down_packed else self.h,
                                          not down_packed, stream)
        elif self.fuse_gather:
            B.moe_expert_up_swiglu_gather(x, self.row_src, self.k, self.expert_offsets, w_gate,
                                          w_up, self.h, stream)
        else:
            B.moe_expert_up_swiglu(self.x_perm, self.expert_offsets, w_gate, w_up, self.h, stream)
        if marks is not None:
            marks[3].record(stream)
        if down_packed:
            B.moe_expert_down_packed(self.h_packed, self.expert_offsets, packed["w_down"],
                                     self.y_perm, stream)
        else:
            B.moe_expert_down(self.h, self.expert_offsets, w_down, self.y_perm, stream)
        if marks is not None:
            marks[4].record(stream)
        B.moe_combine(self.y_perm, self.row_of, self.topk_w, residual, out, stream)
        if marks is not None:
            marks[5].record(stream)
        return out


class MoEVerifyStack:
    """n_layers x [RMSNorm -> MoE verify layer -> residual add] on one set of shared buffers.

    h_0 = x;  h_{l+1} = h_l + MoE_l(RMSNorm_l(h_l)).  The residual add is fused into
    moe_combine.  Layer weights stay resident in HBM (lists of per-layer tensors).
    """

    def __init__(self, T, d_model, d_ff, E, k, dtype, device="cuda", renorm=True, eps=1e-5):
        self.layer = MoEVerifyLayer(T, d_model, d_ff, E, k, dtype, device, renorm)
        self.eps = eps
        dev = torch.device(device)
        self.normed = torch.empty((T, d_model), dtype=dtype, device=dev)
        self.h = [torch.empty((T, d_model), dtype=dtype, device=dev) for _ in range(2)]

    def forward(self, x, layers, keep_hidden=False, stream=None, marks=None):
        """`layers`: list of dicts with gain, w_router, bias, w_gate, w_up, w_down.
        Returns the final hidden state (and, if keep_hidden, clones of every h_l).
        `marks`: six events recorded around the calls of the first layer (benchmark only)."""
        hidden = [x.clone()] if keep_hidden else None
        cur = x
        for li, L in enumerate(layers):
            nxt = self.h[li % 2]
            B.moe_rmsnorm(cur, L["gain"], self.eps, self.normed, stream)
            self.layer.forward(self.normed, L["w_router"], L["w_gate"], L["w_up"], L["w_down"],
                               L.get("bias"), residual=cur, out=nxt, stream=stream,
                               marks=marks if li == 0 else None)
            cur = nxt
            if keep_hidden:
                hidden.append(cur.clone())
        return (cur, hidden) if keep_hidden else cur


class GraphedStep:
    """One invocation of `fn(stream)` captured in a HIP graph and replayed with a single launch.

    `fn` must only enqueue library calls on preallocated buffers (MoEVerifyLayer.forward,
    MoEVerifyStack.forward without keep_hidden, spec_accept, ...): the library allocates nothing
    and records no memset nodes, so the captured graph is kernels only.  Inputs are read from the
    same tensors on every replay; refresh them in place (`x.copy_(...)`) between replays.
    Pays off where launch gaps matter: few-token configurations and the multi-layer stack
    (about 190 launches per step).
    """

    def __init__(self, fn, warmup=2):
        self.stream = torch.cuda.Stream()          # default priority
        self.stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(self.stream):
            for _ in range(warmup):                # one-time kernel attribute set-up happens here
                fn(self.stream)
        self.stream.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph, stream=self.stream):
            fn(self.stream)

    def replay(self):
        self.graph.replay()

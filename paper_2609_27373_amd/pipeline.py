"""Host driver of one WISE trajectory over the libwise C ABI.

Section 5 of the paper in three phases, all on the device:
  discovery  steps 1..t_d: full causal attention; steps in the window also
             pool their attention mass
  selection  once after step t_d: per-row support + CSR + row order
  reuse      steps t_d+1..T: attention restricted to the fixed support, with
             this step's Q/K/V

Two selection rules (mode):
  "accumulate"  the window steps' block masses are summed into one fp32
                accumulator and selected once
  "union"       the paper's eq. (block_working_set): each window step's
                masses are selected on their own (B_q^(t, eta)) into a
                bitmask, and the support is the union of those sets

Two late-step kernels compute the same outputs (late_kernel):
  "rows"     wise_sparse_attn, one work-group per support row
  "grouped"  wise_sparse_attn_grouped, work-groups of consecutive rows over
             the union of their supports (faster where supports are dense)
  "auto"     grouped where the library offers it and the selected support's
             density (nnz over the causal block pairs) is at least
             group_density (by default the measured break-even of the
             library's group shape and head_dim, GROUP_DENSITY; some shapes
             and grids too small to fill the chip, GROUP_QUERIES, never),
             rows otherwise.  The
             first select() reads nnz back (one synchronisation); later ones
             copy it to pinned host memory asynchronously, and the choice
             follows when the copy has landed (checked without waiting at
             each select() and late step), so the host never waits on the
             device again.  Both kernels give the same outputs, so when the
             switch happens does not change any result.  A select() under
             graph capture keeps the current choice.

Buffers are allocated once per trajectory (torch device memory); every call
enqueues on the current stream and returns (except the first select() in
"auto" mode, which waits for the selection to read its size).
"""

from __future__ import annotations

import torch

from . import wise


class WisePipeline:
    MODES = ("accumulate", "union")
    LATE_KERNELS = ("auto", "rows", "grouped")
    # Density from which "auto" picks the grouped kernel, by (block, rows per
    # group, head_dim); None: never (slower at every density measured).  The
    # union of consecutive rows' supports grows as the density falls, and the
    # break-even is where it costs what the shared staging saves.  Late step,
    # grouped over one-row time on the same supports:
    #   block 64, 4 rows, d 128: 1.35 at density 0.43, 1.14 at 0.67, 1.03 at
    #     0.79; 0.95 at 0.90 and 0.93 at 0.95 (8192 and 16384 tokens), 0.98 to
    #     1.01 at 0.91 (4096), 1.03 at 0.89 (2048)
    #   block 64, 2 rows, d 128 (lengths 256 does not divide): 1.18 at 0.54,
    #     0.98 at 1.00
    #   block 64, 2 rows, d 96: 1.14 at 0.52, 1.03 at 0.79, 1.02 at 0.91, 0.99
    #     at 0.96, 0.98 at 1.00
    #   block 64, 2 rows, d 64: 1.09 at 0.23, 1.06 at 0.56, 1.02 at 0.72, 0.99
    #     at 0.80, 0.92 to 0.96 at 0.92 and 0.96
    #   block 128, 2 rows, d 128: 1.16 at 0.65, 1.05 at 0.80, 1.03 at 0.91,
    #     1.02 at 0.96, 1.00 at 1.00
    GROUP_DENSITY = {(64, 4, 128): 0.86, (64, 2, 128): None, (64, 2, 96): 0.95,
                     (64, 2, 64): 0.77, (128, 2, 128): None}
    # Queries (over batch and heads) up to which "auto" stays with one row per
    # work-group: groups of rows then leave CUs idle and the longest decides.
    # Full supports of 64-key blocks, grouped / one-row us by queries / 256:
    # d 128: 16 (1024 x 4 heads) 34.7 / 25.1, 128 (16384 x 2) 420 / 323, 256
    # (4096 x 16) 116.9 / 103.6, 384 (4096 x 24) 127.3 / 129.5; d 96: 128 (4096
    # x 8) 76.0 / 74.1, 256 (4096 x 16) 85.0 / 84.3, 384 102.4 / 108.1; d 64: 128
    # 64.6 / 63.7, 256 70.4 / 68.3, 384 79.9 / 83.8
    GROUP_QUERIES = 320 * 256

    def __init__(self, batch, heads, seq_len, head_dim, block, tau, flags=wise.WISE_DEFAULT_FLAGS,
                 scale=0.0, device="cuda", mode="accumulate", window=4, kv_heads=0,
                 late_kernel="auto", group_density=None):
        if mode not in self.MODES:
            raise ValueError(f"mode must be one of {self.MODES}")
        if late_kernel not in self.LATE_KERNELS:
            raise ValueError(f"late_kernel must be one of {self.LATE_KERNELS}")
        self.shape = wise.make_shape(batch, heads, seq_len, head_dim, block, scale, kv_heads)
        self.tau = float(tau)
        self.flags = int(flags)
        self.mode = mode
        nb = seq_len // block
        # accumulate mode: the running sum; union mode: one step's masses
        self.acc = torch.zeros((batch, heads, nb, nb), dtype=torch.float32, device=device)
        self.lse = torch.empty((batch, heads, seq_len), dtype=torch.float32, device=device)
        self.schedule = wise.Schedule(self.shape, device)
        self.mass_ws = wise.mass_workspace(self.shape, device)
        self.window = int(window)
        self.masks = None
        if mode == "union":
            words = wise.wise_mask_words(self.shape)
            self.masks = torch.zeros((self.window, batch * heads * nb, words), dtype=torch.int64,
                                     device=device)
        self.filled = 0
        self.late_kernel = late_kernel
        group_rows = wise.wise_sparse_group_rows(self.shape)
        if group_density is None:
            group_density = (self.GROUP_DENSITY.get((block, group_rows, head_dim))
                             if batch * heads * seq_len > self.GROUP_QUERIES else None)
        self.group_density = None if group_density is None else float(group_density)
        self.grouped = late_kernel == "grouped"
        self._auto = late_kernel == "auto" and group_rows > 0 and self.group_density is not None
        self._decided = False
        self._nnz_host = torch.empty(1, dtype=torch.int32, pin_memory=True) if self._auto else None
        self._nnz_event = None

    @classmethod
    def for_config(cls, cfg, tau=None, **kw):
        return cls(cfg.batch, cfg.heads, cfg.seq_len, cfg.head_dim, cfg.block,
                   cfg.tau if tau is None else tau, kv_heads=cfg.kv_heads, **kw)

    def reset(self):
        self.acc.zero_()
        self.filled = 0

    def discovery_step(self, q, k, v, out, accumulate: bool):
        """One discovery step; `accumulate` marks a step of the window."""
        if accumulate and self.mode == "union":
            if self.filled >= self.window:
                raise RuntimeError("more window steps than the union window holds")
            self.acc.zero_()
            wise.wise_dense_attn_accum(self.shape, q, k, v, out, self.lse, self.acc, self.mass_ws)
            wise.wise_select_step(self.shape, self.acc, self.tau, self.masks[self.filled])
            self.filled += 1
        else:
            wise.wise_dense_attn_accum(self.shape, q, k, v, out, self.lse,
                                       self.acc if accumulate else None,
                                       self.mass_ws if accumulate else None)
        return out

    def dense_step(self, q, k, v, out, lse=None):
        wise.wise_dense_attn_accum(self.shape, q, k, v, out, lse, None)
        return out

    def select(self):
        if self.mode == "union":
            if self.filled == 0:
                raise RuntimeError("union mode: no window step was run before select()")
            self.schedule.from_masks(self.masks, self.filled, self.flags)
        else:
            self.schedule.select(self.acc, self.tau, self.flags)
        if self._auto and not torch.cuda.is_current_stream_capturing():
            if not self._decided:
                self._decide(self.schedule.nnz())
                self._decided = True
            else:
                self._poll()
                self._nnz_host.copy_(self.schedule.row_ptr[-1:], non_blocking=True)
                self._nnz_event = torch.cuda.Event()
                self._nnz_event.record()
        return self.schedule

    def _decide(self, nnz: int):
        self.grouped = nnz / wise.wise_support_capacity(self.shape) >= self.group_density

    def _poll(self):
        """Take up the last asynchronously copied support size if it has landed."""
        if self._nnz_event is not None and self._nnz_event.query():
            self._decide(int(self._nnz_host[0]))
            self._nnz_event = None

    def late_step(self, q, k, v, out, lse=None, ordered=True):
        s = self.schedule
        if self._nnz_event is not None and not torch.cuda.is_current_stream_capturing():
            self._poll()
        if self.grouped:
            wise.wise_sparse_attn_grouped(self.shape, q, k, v, s.row_ptr, s.col_idx, out, lse)
        else:
            wise.wise_sparse_attn(self.shape, q, k, v, s.row_ptr, s.col_idx,
                                  s.row_order if ordered else None, out, lse)
        return out

    def capture_late_step(self, q, k, v, out, lse=None) -> "LateStepGraph":
        """The late step on these fixed buffers as a HIP graph (see LateStepGraph)."""
        return LateStepGraph(self, q, k, v, out, lse)


class LateStepGraph:
    """One late step captured in a HIP graph over fixed q/k/v/out (and lse)
    buffers.  A serving loop writes each step's Q/K/V into those buffers and
    calls replay(): one launch of the recorded sparse kernel, which reads the
    support held in the pipeline's schedule buffers at replay time (so a new
    select() needs no re-capture; the kernel chosen at capture stays, and
    both late-step kernels give the same outputs).  The library allocates and clears nothing,
    so the graph holds only the kernel node."""

    def __init__(self, pipe: WisePipeline, q, k, v, out, lse=None):
        self.buffers = (q, k, v, out, lse)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):              # warm-up launch outside the capture
            pipe.late_step(q, k, v, out, lse)
        torch.cuda.current_stream().wait_stream(side)
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            pipe.late_step(q, k, v, out, lse)

    def replay(self):
        self.graph.replay()
        return self.buffers[3]


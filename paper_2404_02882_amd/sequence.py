"""Outer loop over sub-sequences: the paper's ring of ranks on one GPU.

A sequence of N tokens is held as T shards of N/T tokens, each a contiguous
[B,H,N/T,D] tensor (what one rank of the paper holds). Forward hands kv_out of
one to the next as kv_in (Alg. 2: Recv KV from rank i-1, Send KV to rank i+1);
backward hands dkv_in of one to the previous as dkv_out (Alg. 3). On one GPU
nothing has to wait for that: the library takes several shards through a launch
where that fills the device (lasp_seq_fwd). Every shard keeps the state cache its
forward pass filled until its backward pass has used it.
All buffers are allocated once, up front; the calls only enqueue kernels.
"""
from __future__ import annotations

from typing import List, Optional

import torch

from . import lasp


class LaspSequence:
    def __init__(self, B, H, N, D, chunk, dtype: torch.dtype, T=1, segments=0, device="cuda", need_backward=True,
                 token_decay=False, norm_eps: Optional[float] = None, kv_heads=0, Dv=0, recompute=False):
        if N % T != 0:
            raise ValueError("N must be a multiple of T")
        self.B, self.H, self.N, self.D, self.T = B, H, N, D, T
        self.n_sub = N // T
        self.dtype = dtype
        # kv_heads: k, v, dk, dv shards are [B,kv_heads,N/T,D]; groups of H/kv_heads query heads share them
        # Dv: value dimension when it differs from the key dimension D (v, out, dout, dv shards are [..,Dv],
        # states [B,H,D,Dv])
        self.shape = lasp.make_shape(B, H, self.n_sub, D, chunk, dtype, segments, kv_heads, Dv)
        rc = lasp.check_shape(self.shape)
        if rc != 0:
            raise lasp.LaspError(rc, "LaspSequence")
        # token_decay: `decay` of forward / backward is a list of T log-decay shards [B,H,N/T] (float32)
        # instead of the [H] vector of lambdas, and backward also fills dlog_g shards.
        # norm_eps: outputs are normalised (lasp_fwd_norm / lasp_bwd_norm); forward fills `rstd` shards
        # [B,H,N/T], backward takes them and the forward outputs. Both may be set together.
        self.norm_eps = norm_eps
        self.token_decay = token_decay
        # recompute: no state cache is kept between the passes (Sec. 3.4's alternative to caching); every
        # backward call rebuilds the states of its shard from k, v and the state the shard started from,
        # into the tail of the (then larger) scratch buffer, which all shards share
        self.recompute = bool(recompute)
        cache_bytes = lasp.gated_state_cache_bytes if token_decay else lasp.state_cache_bytes
        self.scratch = torch.empty(lasp.seq_scratch_bytes(self.shape, T, token_decay, self.recompute and need_backward),
                                   dtype=torch.uint8, device=device)
        self.caches = [torch.empty(cache_bytes(self.shape), dtype=torch.uint8, device=device)
                       for _ in range(T)] if need_backward and not self.recompute else [None] * T
        st = dict(dtype=torch.float32, device=device)
        # kv[t] = state entering shard t (kv[T] = final); dkv[t] = gradient w.r.t. kv[t]
        self.kv = [torch.zeros(B, H, D, Dv or D, **st) for _ in range(T + 1)]
        self.dkv = [torch.zeros(B, H, D, Dv or D, **st) for _ in range(T + 1)] if need_backward else None
        self.has_kv_in = False
        self.has_dkv_out = False

    def cache_bytes(self) -> int:
        return sum(c.numel() for c in self.caches if c is not None)

    def workspace_bytes(self) -> int:
        return int(self.scratch.numel())

    def _entering(self, given: torch.Tensor, own: torch.Tensor) -> torch.Tensor:
        """`given` as the library can take it (it copies it into `own` on the way), or copied into `own` here."""
        if given.dtype == own.dtype and given.device == own.device and given.shape == own.shape and given.is_contiguous():
            return given
        own.copy_(given)
        return own

    def forward(self, q: List[torch.Tensor], k, v, decay, out: List[torch.Tensor],
                kv_in: Optional[torch.Tensor] = None, rstd: Optional[List[torch.Tensor]] = None) -> torch.Tensor:
        self.has_kv_in = kv_in is not None
        if kv_in is not None:
            kv_in = self._entering(kv_in, self.kv[0])
        norm = self.norm_eps is not None
        if norm and rstd is None:
            raise TypeError("normalised outputs need rstd")
        if self.T == 1 and kv_in is None and not (norm and self.token_decay):
            # one sub-sequence from a zero state: a plain call, whose arguments take the host less time (7 us, 8 us)
            args = (q[0], k[0], v[0])
            if norm:
                lasp.lasp_fwd_norm(self.shape, *args, None, decay, self.norm_eps, out[0], rstd[0], self.kv[1], self.caches[0], self.scratch)
            elif self.token_decay:
                lasp.lasp_gated_fwd(self.shape, *args, decay[0], None, out[0], self.kv[1], self.caches[0], self.scratch)
            else:
                lasp.lasp_fwd(self.shape, *args, None, decay, out[0], self.kv[1], self.caches[0], self.scratch)
            return self.kv[1]
        lasp.lasp_seq_fwd(self.shape, self.T, q, k, v, kv_in, decay, bool(self.token_decay), self.norm_eps if norm else 0.0, out,
                          rstd if norm else None, self.kv, self.caches, self.scratch)
        return self.kv[self.T]

    def backward(self, q, k, v, dout, decay, dq, dk, dv, dkv_out: Optional[torch.Tensor] = None,
                 dlog_g: Optional[List[torch.Tensor]] = None, out: Optional[List[torch.Tensor]] = None,
                 rstd: Optional[List[torch.Tensor]] = None) -> torch.Tensor:
        self.has_dkv_out = dkv_out is not None
        if dkv_out is not None:
            dkv_out = self._entering(dkv_out, self.dkv[self.T])
        norm, token = self.norm_eps is not None, bool(self.token_decay)
        if (norm and (rstd is None or out is None)) or (token and dlog_g is None):
            raise TypeError("normalised outputs need out and rstd, a decay per token dlog_g")
        first = self.kv[0] if self.has_kv_in else None
        if self.T == 1 and dkv_out is None and not (norm and token):   # as in forward
            args, grads = (q[0], k[0], v[0]), (dq[0], dk[0], dv[0])
            if norm:
                lasp.lasp_bwd_norm(self.shape, *args, out[0], rstd[0], dout[0], first, None, decay, self.caches[0], *grads, self.dkv[0],
                                   self.scratch)
            elif token:
                lasp.lasp_gated_bwd(self.shape, *args, dout[0], decay[0], first, self.kv[1], None, self.caches[0], *grads, dlog_g[0],
                                    self.dkv[0], self.scratch)
            else:
                lasp.lasp_bwd(self.shape, *args, dout[0], first, None, decay, self.caches[0], *grads, self.dkv[0], self.scratch)
            return self.dkv[0]
        kv = [first] + self.kv[1:]
        lasp.lasp_seq_bwd(self.shape, self.T, q, k, v, out if norm else None, rstd if norm else None, dout, kv, dkv_out, decay, token,
                          self.caches, dq, dk, dv, dlog_g if token else None, self.dkv, self.scratch)
        return self.dkv[0]


class GraphedStep:
    """One forward + backward pass of a LaspSequence captured in a HIP graph and replayed.

    Short sequences are bound by launches: a pass is up to three kernels for every four sub-sequences
    (one for a short sequence alone; with a decay per token, or sub-sequences that fill the device, for each),
    and the calls that enqueue them; a graph replays all with one submission. The library allocates nothing and never
    synchronises, so its calls can be captured as they are. The graph reads and writes the very
    tensors given here: refresh their contents in place between replays. Per-kernel timing
    (lasp_profile_begin) must be off while capturing.
    """

    def __init__(self, seq: LaspSequence, fwd_kwargs: Optional[dict], bwd_kwargs: Optional[dict] = None, warmup: int = 2):
        """fwd_kwargs None: the graph holds the backward pass alone (the state caches must already hold what a
        forward pass over the same inputs wrote); bwd_kwargs None: the forward pass alone."""
        self.seq = seq
        if fwd_kwargs is None and bwd_kwargs is None:
            raise ValueError("nothing to capture")

        def run():
            if fwd_kwargs is not None:
                seq.forward(**fwd_kwargs)
            if bwd_kwargs is not None:
                seq.backward(**bwd_kwargs)

        # eager passes first, on a side stream as graph capture requires: they set the kernels'
        # LDS attributes (a host-side call that must not fall inside the capture)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for _ in range(max(1, warmup)):
                run()
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            run()

    def replay(self) -> None:
        self.graph.replay()


class BidirSequence:
    """Bidirectional (unmasked) attention O = Q (K^T V) over sub-sequences of any lengths.

    The state is a sum over every token, so nothing is handed from shard to shard: every shard's K^T V is
    added into `kv` (on several devices: their partial states summed across them), then each shard's output
    is computed from the complete state. Backward likewise with dKV = Q^T dO. The library takes several
    shards through a launch (lasp_bidir_seq_*). All buffers are allocated up front; the calls only enqueue
    kernels.
    """

    def __init__(self, B, H, lengths, D, chunk, dtype: torch.dtype, segments=0, device="cuda"):
        self.lengths = [int(n) for n in lengths]
        self.T = len(self.lengths)
        self.shapes = [lasp.make_shape(B, H, n, D, chunk, dtype, segments) for n in self.lengths]
        for shp in self.shapes:
            if lasp.bidir_scratch_bytes(shp) == 0:
                raise lasp.LaspError(lasp.check_shape(shp) or 2, "BidirSequence")
        self._shapes = (lasp.Shape * self.T)(*self.shapes)
        need = lasp.bidir_seq_scratch_bytes(self._shapes, self.T) if self.T else 0
        self.scratch = torch.empty(need, dtype=torch.uint8, device=device)
        st = dict(dtype=torch.float32, device=device)
        self.kv = torch.empty(B, H, D, D, **st)
        self.dkv = torch.empty(B, H, D, D, **st)

    def forward(self, q: List[torch.Tensor], k, v, out: List[torch.Tensor]) -> torch.Tensor:
        if self.T:
            lasp.lasp_bidir_seq_fwd(self._shapes, self.T, q, k, v, self.kv, out, self.scratch)
        return self.kv

    def backward(self, q, k, v, dout, dq, dk, dv) -> torch.Tensor:
        """Needs the state `kv` of the forward pass."""
        if self.T:
            lasp.lasp_bidir_seq_bwd(self._shapes, self.T, q, k, v, dout, self.kv, self.dkv, dq, dk, dv, self.scratch)
        return self.dkv

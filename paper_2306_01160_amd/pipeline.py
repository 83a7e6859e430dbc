"""The two variants' forward / backward passes, one C-ABI call each.

A forward is sort or compaction -> gather, schedule -> attention.  Inputs and
outputs are ``[B,H,T,d]`` CUDA tensors in ORIGINAL order (paper Sec. 3, notations);
labels are ``[B,H,T]`` int32 bucket ids (hash) or uint8 keep flags (QK-dropping).
"""
from __future__ import annotations

from dataclasses import dataclass
from typing import Optional

import torch

from . import binding as sc

_LATE = ("q_p", "k_p", "v_p", "q_idx", "k_idx", "n_q", "n_k", "fwd_work", "bwd_work", "counters", "o_f16",
         "q_off", "k_off", "q_sort_key", "k_sort_key")


@dataclass
class Context:
    """What a forward pass leaves for the backward.  Besides the fields below, as views of the workspace (None where
    the pass has no such thing):

    q_p, k_p, v_p            [S,T,d] permuted rows in the compute format (fp32: rows are read in place; q_p not for bf16
                             without a backward: the kernel fetches its own queries)
    q_idx, k_idx             [S,T] original positions of the permuted rows
    q_sort_key, k_sort_key   [S,T] sort keys, q_off, k_off [S,nb+1] bucket offsets (hash)
    n_q, n_k                 [S] kept counts (QK-dropping)
    fwd_work, bwd_work       work lists; counters [S,4]
    o_f16                    fp16 copy of O (bf16 inputs, backward wanted)
    """
    variant: int
    B: int
    H: int
    nb: int
    sm_scale: float
    flags: int
    dtype: int                   # code of the inputs
    need_bwd: bool
    ws: torch.Tensor
    o: torch.Tensor
    lse: torch.Tensor
    q_bucket_sorted: Optional[torch.Tensor] = None
    k_bucket_sorted: Optional[torch.Tensor] = None

    def _view(self, field, dtype, shape):
        S, T, d = self.B * self.H, self.o.shape[2], self.o.shape[3]
        at = sc.scfa_forward_workspace(self.variant, S, T, d, self.nb, self.dtype, self.need_bwd)[1].get(field)
        if at is None:
            return None
        shape = tuple({"S": S, "T": T, "d": d}.get(n, n) for n in shape)
        n = torch.Size(shape).numel() * dtype.itemsize
        return self.ws[at:at + n].view(dtype).view(shape)

    def __getattr__(self, name):         # only reached for what is not there yet
        if name not in _LATE:
            raise AttributeError(name)
        hash_ = self.variant == sc.SCFA_HASH
        T = self.o.shape[2]
        if name in ("q_p", "k_p", "v_p"):
            value = self._view(name[0] + "_perm", torch.float16, ("S", "T", "d"))
        elif name in ("q_idx", "k_idx"):
            value = self._view(name[0] + "_key", torch.int32, ("S", "T"))
            if hash_:
                value = value & 0xffffff
        elif name in ("q_sort_key", "k_sort_key"):
            value = self._view(name[0] + "_key", torch.int32, ("S", "T")) if hash_ else None
        elif name in ("q_off", "k_off"):
            value = self._view(name, torch.int32, ("S", self.nb + 1)) if hash_ else None
        elif name in ("n_q", "n_k"):
            value = None if hash_ else self._view(name[2] + "_off", torch.int32, ("S",))
        elif name in ("fwd_work", "bwd_work"):
            tiles = sc.scfa_tile_config(self.o.shape[3], sc.SCFA_F32 if self.dtype == sc.SCFA_F32 else sc.SCFA_BF16)
            n = sc.scfa_num_work_items(T, self.nb, tiles[0] if name == "fwd_work" else tiles[2])
            value = self._view("work" if name == "fwd_work" else name, torch.int32, ("S", n, sc.SCFA_WORK_STRIDE))
        elif name == "counters":
            value = self._view(name, torch.int64, ("S", 4))
        else:
            value = self._view(name, torch.float16, tuple(self.o.shape))
        setattr(self, name, value)
        return value


def _rows(x):
    return x if x.is_contiguous() else x.contiguous()


def _forward(variant, q, k, v, label_q, label_k, nb, sm_scale, need_bwd, strict):
    flags = sc.SCFA_FLAG_STRICT_CAUSAL if strict else 0
    need_bwd, sm_scale = bool(need_bwd), float(sm_scale)
    o, lse, ws = sc.scfa_forward(variant, _rows(q), _rows(k), _rows(v), _rows(label_q), _rows(label_k), nb, sm_scale, flags,
                                 need_bwd)
    return o, lse, Context(variant, q.shape[0], q.shape[1], nb, sm_scale, flags, sc.input_code(q), need_bwd, ws, o, lse)


def _backward(ctx, d_o, ws, outs):
    if not ctx.need_bwd:
        raise sc.ScfaError("the forward pass was run with need_bwd=False")
    return sc.scfa_backward(ctx.variant, ctx.ws, ctx.o, ctx.lse, d_o, ctx.nb, ctx.dtype, ctx.sm_scale, ctx.flags, ws=ws, outs=outs)


def hash_forward(q, k, v, bucket_q, bucket_k, nb, sm_scale, need_bwd=True, strict=False):
    """Hash-sparse attention forward (Sec. 3.2).  Returns (O, LSE, ctx)."""
    return _forward(sc.SCFA_HASH, q, k, v, bucket_q, bucket_k, nb, sm_scale, need_bwd, strict)


def hash_backward(ctx: Context, d_o, ws=None, outs=None):
    """dQ, dK, dV (fp32, original order) of hash-sparse attention."""
    return _backward(ctx, d_o, ws, outs)


def qkdrop_forward(q, k, v, keep_q, keep_k, sm_scale, need_bwd=True, strict=False):
    """QK-sparse attention forward (Sec. 3.1).  Returns (O, LSE, ctx)."""
    return _forward(sc.SCFA_QKDROP, q, k, v, keep_q, keep_k, 1, sm_scale, need_bwd, strict)


def qkdrop_backward(ctx: Context, d_o, ws=None, outs=None):
    """dQ, dK, dV (fp32, original order) of QK-sparse attention."""
    return _backward(ctx, d_o, ws, outs)

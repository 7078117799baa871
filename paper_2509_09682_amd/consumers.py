"""Other consumers of the indexed log-sum-exp kernels (marshalling only: every score, softmax and gradient comes from the
C-ABI calls).

bucketed_step: losses whose candidate sets are chosen per BUCKET of positions rather than per batch or per position.
The paper's Sec. 5 ("Comparison Sampling Strategies") names the Scalable Cross-Entropy loss as a case in point: it
groups positions into buckets, picks for each bucket the catalogue items with the largest scores under a cheap proxy,
and takes the cross-entropy of every position over its bucket's items plus its own correct item; the paper notes that
such a loss could run on kernels that need nothing but the indices of the correct and the selected items.  That is the
shared-negatives mode of this library with a list per bucket: every bucket in the same launches, positions read and
results written where they are (cce_neg_bucketed_step).  Buckets so large that each fills the chip by itself go one by
one through the bf16 matrix tiles instead: the positions are brought into bucket order once, each bucket is one forward
and one backward call on its slice, and the results are put back in batch order.  How the buckets and their candidates
are chosen is the caller's business.
"""
from __future__ import annotations

from typing import Optional, Sequence

import torch

from . import binding as B


# bf16 inputs and a hidden size with bf16 tiles: flops of an average bucket (8 positions candidates d) up to which all
# buckets in one launch were the faster form wherever measured (2, 8 and 32 buckets; us for one launch / a launch pair per
# bucket: d = 64, 32 buckets of 0.13 GFLOP 81 / 1294; d = 64, 8 of 17 GFLOP 584 / 696; d = 128, 2 of 34 GFLOP 267 / 295;
# d = 256, 2 of 34 GFLOP 319 / 423).  Beyond, a bucket fills the chip and the cheaper bf16 weights of the tiles count.
_TILE_SIZES = (64, 128, 256)
_BUCKET_FLOPS_FOR_TILES = 3e10


def _one_launch(dt: int, d: int, M: int, n_buckets: int, Kb: int) -> bool:
    if Kb < 1 or M < 1:
        return False
    return dt == B.CCE_F32 or d not in _TILE_SIZES or 8.0 * M * Kb * d < _BUCKET_FLOPS_FOR_TILES * n_buckets


def bucketed_step(H: torch.Tensor, E: torch.Tensor, tgt: torch.Tensor, order: torch.Tensor, bucket_ptr: Sequence[int],
                  bucket_neg: torch.Tensor, grad_loss: Optional[torch.Tensor], dE: torch.Tensor, *,
                  mask_target_collisions: bool = True):
    """Forward + backward of the loss with one candidate list per bucket of positions.

    H [N,d], E [V,d] (both float32 or both bfloat16), tgt [N] int32.
    order      [M] int64: the positions that take part, sorted by bucket (positions left out, e.g. padding, get
               loss = lse = 0 and a zero dH row);
    bucket_ptr B + 1 offsets into `order` (host integers): bucket b owns order[bucket_ptr[b]:bucket_ptr[b+1]];
    bucket_neg [B, Kb] int32: the candidate items of every bucket (a position's own correct item is scored besides);
    grad_loss  [N] float32 upstream gradient of the per-position loss, or None for 1;
    dE         [V,d] float32, ACCUMULATED INTO.
    Returns (loss [N], lse [N], dH [N,d]) in batch order, dH in H's dtype.
    """
    N, d = H.shape
    V = E.shape[0]
    n_buckets, Kb = bucket_neg.shape
    if len(bucket_ptr) != n_buckets + 1 or bucket_ptr[0] != 0 or bucket_ptr[-1] != order.numel():
        raise ValueError("bucket_ptr must hold B + 1 offsets covering `order`")
    dt = B.CCE_F32 if H.dtype == torch.float32 else B.CCE_BF16
    ts = tgt.index_select(0, order).contiguous()
    if _one_launch(dt, d, order.numel(), n_buckets, Kb):
        if any(bucket_ptr[b + 1] < bucket_ptr[b] for b in range(n_buckets)):
            raise ValueError("bucket_ptr must ascend")
        loss = torch.zeros(N, device=H.device, dtype=torch.float32)
        lse = torch.zeros(N, device=H.device, dtype=torch.float32)
        dH = torch.zeros((N, d), device=H.device, dtype=H.dtype)
        desc = B.make_desc(N, V, d, Kb, dt, B.CCE_NEG_SHARED, dH_dtype=dt, mask_target_collisions=int(mask_target_collisions))
        g = grad_loss
        if g is not None and g.numel() != N:   # only the entries of `order` are read
            g = g.new_zeros(N).index_copy_(0, order, g.index_select(0, order).reshape(-1))
        B.cce_neg_bucketed_step(desc, H.contiguous(), E, ts, order.contiguous(), bucket_ptr, bucket_neg.contiguous(),
                                None if g is None else g.contiguous(), loss, lse, dH, dE)
        return loss, lse, dH
    Hs = H.index_select(0, order).contiguous()          # positions in bucket order: slices are contiguous
    gs = None if grad_loss is None else grad_loss.index_select(0, order).contiguous()
    M = order.numel()
    loss_s = torch.empty(M, device=H.device, dtype=torch.float32)
    lse_s = torch.empty(M, device=H.device, dtype=torch.float32)
    dH_s = torch.empty((M, d), device=H.device, dtype=H.dtype)
    kw = dict(dH_dtype=dt, mask_target_collisions=int(mask_target_collisions), fuse_dH=1)
    sizes = {int(bucket_ptr[b + 1]) - int(bucket_ptr[b]) for b in range(n_buckets)} - {0}
    ws = None
    if sizes:   # one workspace for all buckets; the largest bucket is not always the one that needs the most
        ws = B.new_workspace(max((B.make_desc(n, V, d, Kb, dt, B.CCE_NEG_SHARED, **kw) for n in sizes), key=B.cce_neg_workspace_bytes),
                             device=H.device)
    for b in range(n_buckets):
        b0, b1 = int(bucket_ptr[b]), int(bucket_ptr[b + 1])
        if b1 == b0:
            continue
        desc = B.make_desc(b1 - b0, V, d, Kb, dt, B.CCE_NEG_SHARED, **kw)
        desc_b = B.make_desc(b1 - b0, V, d, Kb, dt, B.CCE_NEG_SHARED, reuse_forward_prep=1, **kw)
        neg = bucket_neg[b]
        B.cce_neg_forward(desc, Hs[b0:b1], E, ts[b0:b1], neg, None, loss_s[b0:b1], lse_s[b0:b1], ws)
        B.cce_neg_backward(desc_b, Hs[b0:b1], E, ts[b0:b1], neg, None, lse_s[b0:b1], None if gs is None else gs[b0:b1],
                           dH_s[b0:b1], dE, ws)
    loss = torch.zeros(N, device=H.device, dtype=torch.float32)
    lse = torch.zeros(N, device=H.device, dtype=torch.float32)
    dH = torch.zeros((N, d), device=H.device, dtype=H.dtype)
    loss.index_copy_(0, order, loss_s)
    lse.index_copy_(0, order, lse_s)
    dH.index_copy_(0, order, dH_s)
    return loss, lse, dH

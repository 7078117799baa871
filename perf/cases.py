"""The work that users of this framework have it do, as cases that can be timed and compared.

A case is a dict of plain values.  `prepare` makes, on the GPU and from a seed, what a training or evaluation program
holds before the call (inputs, the workspace it keeps, its gradient buffers); `run` makes one pass through the public
entry points; `work` says what that pass cannot do without; `tolerance` how far another correct implementation at the
same precision may be off.  Shapes are those of the benchmark workloads, the final-layer comparison and the consumer
tests; values are synthetic: hidden states N(0, 1), item rows N(0, 0.02), Zipf targets, padded sequences.

Paths (`path` of a case):
  step      cce_neg_forward + cce_neg_backward of a training step through the C ABI binding; the forward call also forms
            the hidden-state gradient and the backward call reuses what it left, dE is added into a caller-held buffer
  autograd  cce_neg_loss (mean over the valid positions) and loss.backward(), with autograd's dense gradient of the item
            table or with the caller's fp32 buffer
  sampled   a training step whose negatives are drawn inside the kernels (no index matrix)
  filtered  a full-catalogue step late in training with gradient filtering in the backward pass
  forward   scoring without gradients on the library's own scratch memory (evaluation, serving)
  bucketed  one candidate list per bucket of positions (bucketed_step)
"""
from __future__ import annotations

import math

import torch

import paper_2509_09682_amd as P

_MODES = {"shared": P.CCE_NEG_SHARED, "per_position": P.CCE_NEG_PER_POSITION, "full": P.CCE_NEG_FULL}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
_MATRIX_SIZES = (64, 128, 256)


def _case(path, mode, dtype, batch, seq, d, V, K, **more):
    case = dict(path=path, mode=mode, dtype=dtype, batch=batch, seq=seq, d=d, V=V, K=K, pad="right", pad_lo=0.5,
                targets="zipf", zipf=1.1, negatives="uniform")
    case.update(more)
    return case


def listed():
    return [
        # the smallest step: a toy model or a unit test in fp32, where launches and the host decide
        _case("step", "shared", "f32", 16, 32, 64, 4096, 128, name="tiny_f32", pad="bernoulli", pad_lo=0.9,
              targets="uniform", negatives="distinct"),
        # an ordinary step of a mid-sized catalogue: shared uniform negatives, short hidden size
        _case("step", "shared", "bf16", 256, 200, 64, 50_000, 1024, name="mid_shared_d64", pad_lo=0.6),
        # negatives of their own for every position: bound by row gathers and by the scatter into the table gradient
        _case("step", "per_position", "bf16", 128, 200, 128, 1_000_000, 256, name="per_position_d128", pad="none"),
        # no sampling: every item of the catalogue is a candidate
        _case("step", "full", "bf16", 64, 200, 64, 100_000, 0, name="full_catalogue_d64", pad="none"),
        # the largest step: big batch, big catalogue, popularity negatives (the benchmark's headline workload)
        _case("step", "shared", "bf16", 1024, 200, 256, 5_000_000, 4096, name="large_shared_d256", zipf=1.2,
              negatives="popularity"),
        # the loss layer of a PyTorch model: autograd, mean loss, dense table gradient in the table's dtype
        _case("autograd", "shared", "bf16", 1024, 32, 256, 12_000, 511, name="autograd_d256", grads="dense"),
        # negatives drawn in the kernels by popularity: a few items collect most of the pairs
        _case("sampled", "per_position", "bf16", 128, 200, 128, 1_000_000, 256, name="sampled_popularity_d128",
              pad="none", law="popularity"),
        # full catalogue late in training (a peaked softmax), gradients below the threshold dropped
        _case("filtered", "full", "bf16", 64, 200, 64, 100_000, 0, name="filtered_peaked_d64", pad="none", eps=1e-3),
        # training in fp32 from end to end
        _case("step", "shared", "f32", 64, 200, 64, 50_000, 1024, name="shared_f32_d64", pad_lo=0.6),
        # a hidden size of the published timing table that is not a power of two
        _case("step", "shared", "bf16", 256, 200, 320, 100_000, 1024, name="shared_d320", pad_lo=0.6),
        # candidate lists per bucket of positions, buckets of unequal size
        _case("bucketed", "shared", "bf16", 64, 200, 64, 20_000, 256, name="bucketed_d64", pad="bernoulli", pad_lo=0.85,
              buckets=32),
        # evaluation of a small ragged batch against the whole catalogue, forward only
        _case("forward", "full", "bf16", 17, 59, 128, 49_999, 0, name="score_full_d128", pad_lo=0.3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes log-uniform over the range of the listed ones, most of them odd or ragged."""
    while True:
        path = rng.choice(["step"] * 5 + ["autograd"] * 2 + ["sampled", "forward", "bucketed", "filtered"])
        mode = rng.choice({"step": ["shared", "shared", "per_position", "full"], "autograd": ["shared", "full", "per_position"],
                           "sampled": ["per_position", "shared"], "forward": ["shared", "full", "per_position"],
                           "bucketed": ["shared"], "filtered": ["full"]}[path])
        dtype = "bf16" if path == "filtered" or rng.random() < 0.75 else "f32"
        d = rng.choice(_MATRIX_SIZES) if path == "filtered" or rng.random() < 0.7 else rng.choice((32, 48, 96, 192, 320, 512))
        batch, seq = _log_int(rng, 4, 1024), rng.randint(16, 256)
        V = _log_int(rng, 2_000, 1_000_000) if mode != "full" else _log_int(rng, 2_000, 100_000)
        K = 0 if mode == "full" else _log_int(rng, 32, 4096 if mode == "shared" else 512)
        if mode == "shared":
            K = min(K, V // 4)
        more = {"pad": rng.choice(["right", "right", "bernoulli", "none"]), "pad_lo": round(rng.uniform(0.2, 0.9), 2),
                "zipf": rng.choice([1.1, 1.2]), "negatives": rng.choice(["uniform", "popularity"]) if mode == "shared" else "uniform"}
        if path == "autograd":
            more["grads"] = rng.choice(["dense", "buffer"])
        if path == "sampled":
            more["law"] = rng.choice(["uniform", "popularity"])
        if path == "filtered":
            more["eps"] = rng.choice([1e-4, 1e-3])
        if path == "bucketed":
            more["buckets"] = rng.randint(4, 64)
        case = _case(path, mode, dtype, batch, seq, d, V, K, **more)
        # bounds that keep a drawn case below the largest listed one of its kind, in work and in memory
        flops, tiles = 8.0 * batch * seq * (K + 1 if mode != "full" else V) * d, dtype == "bf16" and d in _MATRIX_SIZES
        most = 7e9 if mode == "per_position" else (6e11 if tiles else (1e11 if dtype == "bf16" else 4e10))
        if path == "bucketed":
            most = min(most, 2e10)
        if 1e7 <= flops <= most and V * d <= 1.28e8 and (path != "bucketed" or batch * seq >= 8 * more["buckets"]):
            return case


# ---------------------------------------------------------------------------------------------------------- inputs
def _normal(shape, sigma, dtype, g):
    out = torch.empty(shape, dtype=dtype, device="cuda")
    step = max(1, (1 << 28) // shape[1])
    for r in range(0, shape[0], step):
        rows = min(step, shape[0] - r)
        out[r:r + rows] = sigma * torch.randn((rows, shape[1]), device="cuda", generator=g)
    return out


def _weights(V, power):
    return torch.arange(1, V + 1, dtype=torch.float64, device="cuda").pow(-power)


def _alias_table(weights):
    """Alias table of a law (columns of equal mass, at most two ids each), by prefix sums over the columns below and above
    the mean: light columns are filled from the heavy ones in order, a heavy column that runs short from the next one."""
    V = weights.numel()
    q = weights * (V / weights.sum())
    ids = torch.arange(V, device="cuda")
    light, heavy = ids[q < 1], ids[q >= 1]
    need, spare = torch.cumsum(1 - q[light], 0), torch.cumsum(q[heavy] - 1, 0)
    keep, alias = torch.ones_like(q), ids.clone()
    at = torch.searchsorted(spare, need - (1 - q[light]), right=True).clamp_max(heavy.numel() - 1)
    keep[light], alias[light] = q[light], heavy[at]
    first = torch.searchsorted(need, spare, right=True)            # first light column that takes more than is spare
    short = first < light.numel()
    short[-1] = False
    left = 1 + spare - need[first.clamp_max(max(light.numel() - 1, 0))]
    keep[heavy[short]] = left[short].clamp(0, 1)
    alias[heavy[short]] = heavy[1:][short[:-1]]
    thresh = (keep * 2.0 ** 32).floor().clamp(0, 2.0 ** 32 - 1).to(torch.int64)
    thresh = torch.where(thresh >= 1 << 31, thresh - (1 << 32), thresh).to(torch.int32)     # the same 32-bit words
    return thresh.contiguous(), alias.to(torch.int32).contiguous()


def _mask(case, g):
    batch, seq = case["batch"], case["seq"]
    if case["pad"] == "none":
        return None
    if case["pad"] == "bernoulli":
        return (torch.rand(batch * seq, device="cuda", generator=g) < case["pad_lo"]).to(torch.uint8)
    lengths = torch.randint(max(1, int(case["pad_lo"] * seq)), seq + 1, (batch, 1), device="cuda", generator=g)
    return (torch.arange(seq, device="cuda")[None, :] < lengths).reshape(-1).to(torch.uint8)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    dt = _TORCH[case["dtype"]]
    N, d, V, K, mode = case["batch"] * case["seq"], case["d"], case["V"], case["K"], _MODES[case["mode"]]
    s = {"case": dict(case), "mode": mode, "N": N}
    E = _normal((V, d), 0.02, dt, g)
    rank_to_id = torch.randperm(V, device="cuda", generator=g)
    if case["targets"] == "uniform":
        tgt = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    else:
        cdf = torch.cumsum(_weights(V, case["zipf"]), 0)
        u = torch.rand(N, device="cuda", generator=g, dtype=torch.float64) * cdf[-1]
        tgt = rank_to_id[torch.searchsorted(cdf, u, right=True).clamp_max(V - 1)].to(torch.int32)
    if case["path"] == "filtered":     # hidden states that point at their target's row: correct-item score about 9 above the rest
        rows = E[tgt.long()].float()
        H = (rows * (9.0 / E.float().square().sum(1).mean()) + 0.5 * torch.randn((N, d), device="cuda", generator=g)).to(dt)
    else:
        H = _normal((N, d), 1.0, dt, g)
    mask = _mask(case, g)
    s.update(H=H, E=E, tgt=tgt, mask=mask)

    neg = None
    if case["path"] == "bucketed":
        # positions dealt into buckets of unequal size; the caller knows the bucket boundaries on the host
        B = case["buckets"]
        valid = torch.arange(N, device="cuda") if mask is None else mask.nonzero().reshape(-1)
        share = 0.25 + torch.rand(B, device="cuda", generator=g, dtype=torch.float64)
        cum = torch.cumsum(share / share.sum(), 0)
        of = torch.searchsorted(cum, torch.rand(valid.numel(), device="cuda", generator=g, dtype=torch.float64)).clamp_max(B - 1)
        s["order"] = valid[torch.argsort(of, stable=True)].contiguous()
        s["ptr"] = [0] + torch.cumsum(torch.bincount(of, minlength=B), 0).tolist()
        s["neg"] = torch.randint(0, V, (B, K), device="cuda", generator=g, dtype=torch.int32)
        s["g"] = torch.full((N,), 1.0 / max(valid.numel(), 1), device="cuda")
        s["dE"] = torch.zeros((V, d), device="cuda")
        return s
    if case["path"] == "sampled":
        table = (None, None)
        if case["law"] == "popularity":
            w = torch.empty(V, dtype=torch.float64, device="cuda")
            w[rank_to_id] = _weights(V, 1.2 * 0.75)
            table = _alias_table(w)
        s["table"] = table
        s["smp"] = P.make_sampler(P.CCE_SAMPLER_ALIAS if case["law"] == "popularity" else P.CCE_SAMPLER_UNIFORM, int(seed), 1, *table)
    elif case["mode"] == "shared" and case["negatives"] == "popularity":    # K distinct ids, probability ~ count^0.75
        keys = torch.empty(V, dtype=torch.float64, device="cuda").exponential_(generator=g) / _weights(V, case["zipf"] * 0.75)
        neg = rank_to_id[torch.topk(keys, K, largest=False).indices].to(torch.int32)
    elif case["mode"] == "shared" and case["negatives"] == "distinct":
        neg = torch.randperm(V, device="cuda", generator=g)[:K].to(torch.int32)
    elif mode != P.CCE_NEG_FULL:
        neg = torch.randint(0, V, (K,) if case["mode"] == "shared" else (N, K), device="cuda", generator=g, dtype=torch.int32)
    s["neg"] = neg

    if case["path"] == "autograd":
        s["H"].requires_grad_(True)
        if case["grads"] == "dense":
            s["E"].requires_grad_(True)
        else:
            s["grad_E"] = torch.zeros((V, d), device="cuda")
        return s
    in_dt = P.CCE_F32 if case["dtype"] == "f32" else P.CCE_BF16
    s["loss"], s["lse"] = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
    if case["path"] == "forward":
        s["desc"] = P.make_desc(N, V, d, K, in_dt, mode)
        return s
    fuse = 0 if case["path"] == "filtered" else 1
    s["desc"] = P.make_desc(N, V, d, K, in_dt, mode, fuse_dH=fuse)
    s["desc_bwd"] = P.make_desc(N, V, d, K, in_dt, mode, fuse_dH=fuse, reuse_forward_prep=1, filter_eps=case.get("eps", 0.0))
    s["ws"] = P.new_workspace(s["desc"])
    s["g"] = torch.full((N,), 1.0, device="cuda") / (N if mask is None else mask.sum().clamp_min(1))
    s["dH"], s["dE"] = torch.empty((N, d), device="cuda"), torch.zeros((V, d), device="cuda")
    return s


# ------------------------------------------------------------------------------------------------------------ a pass
def run(s):
    path = s["case"]["path"]
    H, E, tgt, neg, mask = s["H"], s["E"], s["tgt"], s["neg"] if "neg" in s else None, s["mask"]
    if path == "bucketed":
        loss, lse, dH = P.bucketed_step(H, E, tgt, s["order"], s["ptr"], neg, s["g"], s["dE"])
        return loss, lse, dH, s["dE"]
    if path == "autograd":
        H.grad = None
        E.grad = None
        loss = P.cce_neg_loss(H, E, tgt, neg, mask, neg_mode=s["mode"], grad_E_out=s.get("grad_E"))
        loss.backward()
        return loss.detach(), H.grad, s["grad_E"] if "grad_E" in s else E.grad
    if path == "forward":
        P.cce_neg_forward_noalloc(s["desc"], H, E, tgt, neg, mask, s["loss"], s["lse"])
        return s["loss"], s["lse"]
    if path == "sampled":
        P.cce_neg_forward_sampled(s["desc"], s["smp"], H, E, tgt, mask, s["loss"], s["lse"], s["ws"])
        P.cce_neg_backward_sampled(s["desc_bwd"], s["smp"], H, E, tgt, mask, s["lse"], s["g"], s["dH"], s["dE"], s["ws"])
    else:
        P.cce_neg_forward(s["desc"], H, E, tgt, neg, mask, s["loss"], s["lse"], s["ws"])
        P.cce_neg_backward(s["desc_bwd"], H, E, tgt, neg, mask, s["lse"], s["g"], s["dH"], s["dE"], s["ws"])
    return s["loss"], s["lse"], s["dH"], s["dE"]


def work(case):
    """Four products of the size of the score matrix per step (scores, scores again, dH, dE), one in a forward pass, on the
    valid positions; every input and output once, table rows as far as the pass touches them."""
    b = 4 if case["dtype"] == "f32" else 2
    N, d, V, K = case["batch"] * case["seq"], case["d"], case["V"], case["K"]
    share = {"none": 1.0, "bernoulli": case["pad_lo"], "right": (case["pad_lo"] + 1) / 2}[case["pad"]]
    nv = N * share
    n_cand = V if case["mode"] == "full" else K + 1
    if case["mode"] == "full":
        rows = float(V)
    else:   # distinct rows: uniform ids fill the table like balls thrown into V bins, targets count at most once each
        lists = nv if case["mode"] == "per_position" else (case["buckets"] if case["path"] == "bucketed" else 1)
        rows = V * -math.expm1(-float(lists) * K / V)
        rows = min(float(V), rows + (V - rows) * -math.expm1(-nv / V))
    ids = {"full": 0.0, "shared": 4.0 * K * case.get("buckets", 1), "per_position": 4.0 * nv * K}[case["mode"]]
    if case["path"] == "sampled":
        ids = 8.0 * min(V, nv * K) if case["law"] == "popularity" else 0.0
    vectors = N * (4 + 1) + 8.0 * N                        # targets and mask in, loss and lse out
    if case["path"] == "forward":
        return {"bytes": nv * d * b + rows * d * b + ids + vectors, "flops": 2.0 * nv * n_cand * d}
    dH = N * d * (b if case["path"] in ("autograd", "bucketed") else 4)
    dE = V * d * b if case.get("grads") == "dense" else 8.0 * rows * d      # written whole, or rows read and written
    return {"bytes": nv * d * b + rows * d * b + ids + vectors + 4.0 * N + dH + dE, "flops": 8.0 * nv * n_cand * d}


def tolerance(case):
    """About four times the error of this path against the same sums in 64 bits, over the listed and thirty drawn cases.

    Arithmetic in fp32 (fp32 inputs, per-position negatives, hidden sizes without a bf16 matrix kernel, every loss and
    lse): 7e-7.  bf16 matrix kernels: the softmax weights enter the gradients rounded to bf16 (2^-9 a term, averaged over
    the candidates), 2.2e-4, and single elements of rarely touched table rows are off by 0.07 of the root mean square.
    Gradients handed back in bf16 (autograd, bucketed_step): 1.7e-3, the rounding of the result."""
    if case["dtype"] == "f32" or case["path"] == "forward":
        return {"rel": 3e-6, "max": 5e-4}
    if case["path"] in ("autograd", "bucketed"):
        return {"rel": 6.6e-3, "max": 0.3}
    if case["mode"] != "per_position" and case["d"] in _MATRIX_SIZES:
        return {"rel": 1e-3, "max": 0.3}
    return {"rel": 3e-6, "max": 5e-4}

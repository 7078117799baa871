"""Host-side checks of the C ABI that need no GPU: the library loads, exports every declared symbol, and rejects bad
arguments before launching anything."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def binding():
    from paper_2509_09682_amd import binding as B
    from paper_2509_09682_amd import build

    if not os.path.exists(B.LIB_PATH):
        build.build()
    return B


def test_library_exports_every_declared_symbol(binding):
    header = open(os.path.join(ROOT, "include", "cce_neg.h")).read()
    declared = set(re.findall(r"\b(cce_neg_\w+|cce_status_string)\s*\(", header))
    assert declared == set(binding.EXPORTS)
    L = binding.lib()
    for name in declared:
        assert getattr(L, name) is not None


def test_status_strings(binding):
    seen = {binding.status_string(s) for s in range(8)}
    assert len(seen) == 8 and "ok" in seen
    assert binding.status_string(99) == "unknown status"


def test_workspace_bytes_rejects_bad_descriptors(binding):
    B = binding
    good = B.make_desc(512, 4096, 64, 128, B.CCE_F32, B.CCE_NEG_SHARED)
    assert B.cce_neg_workspace_bytes(good) >= 256
    for kw in (dict(N=-1), dict(V=0), dict(d=0), dict(d=12), dict(d=520), dict(K=-1), dict(in_dtype=5),
               dict(neg_mode=3), dict(dH_dtype=B.CCE_BF16), dict(algo=9), dict(V=1 << 31)):
        f = dict(N=512, V=4096, d=64, K=128, in_dtype=B.CCE_F32, neg_mode=B.CCE_NEG_SHARED, dH_dtype=B.CCE_F32, algo=0)
        f.update(kw)
        desc = B.make_desc(f["N"], f["V"], f["d"], f["K"], f["in_dtype"], f["neg_mode"], dH_dtype=f["dH_dtype"], algo=f["algo"])
        assert B.cce_neg_workspace_bytes(desc) == 0, kw
    # workspace stays O(N + K d): growing K or N by 10x must not grow it by the product
    a = B.cce_neg_workspace_bytes(B.make_desc(51200, 50000, 64, 1024, B.CCE_BF16, B.CCE_NEG_SHARED))
    b = B.cce_neg_workspace_bytes(B.make_desc(51200, 50000, 64, 10240, B.CCE_BF16, B.CCE_NEG_SHARED))
    c = B.cce_neg_workspace_bytes(B.make_desc(512000, 50000, 64, 10240, B.CCE_BF16, B.CCE_NEG_SHARED))
    assert b <= a + 10240 * 64 * 16 and c <= b + 512000 * 64 * 8
    # per-position mode: the inverted index is built in slices of a fixed pair budget, so ten times the negatives must
    # not cost ten times the workspace, and the index never outgrows 3/8 of the id matrix (4 N K bytes) plus O(N + V)
    def pp(N, V, K, d=128):
        return B.cce_neg_workspace_bytes(B.make_desc(N, V, d, K, B.CCE_BF16, B.CCE_NEG_PER_POSITION))
    c3 = pp(25600, 1_000_000, 256)
    assert c3 <= 6.125 * 25600 * 256 + 4 * 1_000_000 + 4 * 25600 + (2 << 20)    # one slice of narrow pairs, not 12 N K = 79 MB
    for V in (40, 3000, 1_000_000, 1 << 22):
        for K in (1, 16, 63, 64, 65, 127, 128, 129, 256, 1024, 4096):
            need = [pp(N, V, K) for N in (65_535, 65_536, 65_537, 65_600)]
            assert need[0] > 256 and need == sorted(need), (V, K)               # does not fall where pairs get wide
    assert pp(25600, 1_000_000, 2560) <= 2.1 * c3
    big = pp(204800, 1_000_000, 2560)                                           # 524 M pairs
    assert big <= 0.375 * 4 * 204800 * 2560 * 1.05 + 4 * 1_000_000 + 4 * 204800 + (34 << 20)
    assert pp(1024, 5_000_000, 16) > 4 * 5_000_000                             # huge catalogue, few pairs: indexed (cursor per item)
    assert pp(204800, 5_000_000, 256) == 256                                    # huge catalogue, many pairs: atomics, header only


def test_forward_backward_reject_null_and_small_workspace_before_launch(binding):
    B = binding
    L = B.lib()
    desc = B.make_desc(16, 100, 64, 8, B.CCE_F32, B.CCE_NEG_SHARED)
    fake = ctypes.c_void_p(0x1000)  # never dereferenced: every call below must fail on the host
    st = L.cce_neg_forward(ctypes.byref(desc), None, fake, fake, fake, None, fake, fake, fake, 4096, None)
    assert st == B.CCE_ERR_NULL
    st = L.cce_neg_forward(ctypes.byref(desc), fake, fake, fake, None, None, fake, fake, fake, 4096, None)
    assert st == B.CCE_ERR_NULL  # K > 0 needs neg
    st = L.cce_neg_forward(ctypes.byref(desc), fake, fake, fake, fake, None, fake, fake, None, 4096, None)
    assert st == B.CCE_ERR_WORKSPACE
    st = L.cce_neg_forward(ctypes.byref(desc), fake, fake, fake, fake, None, fake, fake, fake, 8, None)
    assert st == B.CCE_ERR_WORKSPACE
    st = L.cce_neg_forward(ctypes.byref(desc), fake, fake, fake, fake, None, fake, fake, ctypes.c_void_p(0x1004), 4096, None)
    assert st == B.CCE_ERR_WORKSPACE  # misaligned
    st = L.cce_neg_forward(ctypes.byref(desc), fake, fake, fake, fake, None, None, fake, fake, 4096, None)
    assert st == B.CCE_ERR_NULL
    st = L.cce_neg_backward(ctypes.byref(desc), fake, fake, fake, fake, None, None, None, fake, fake, fake, 4096, None)
    assert st == B.CCE_ERR_NULL  # lse missing
    st = L.cce_neg_backward(ctypes.byref(desc), fake, fake, fake, fake, None, fake, None, fake, None, fake, 4096, None)
    assert st == B.CCE_ERR_NULL  # dE missing
    bad = B.make_desc(16, 100, 60, 8, B.CCE_F32, B.CCE_NEG_SHARED)
    st = L.cce_neg_forward(ctypes.byref(bad), fake, fake, fake, fake, None, fake, fake, fake, 4096, None)
    assert st == B.CCE_ERR_SHAPE
    bad = B.make_desc(16, 100, 64, 8, B.CCE_F32, B.CCE_NEG_SHARED, dH_dtype=B.CCE_BF16)
    st = L.cce_neg_backward(ctypes.byref(bad), fake, fake, fake, fake, None, fake, None, fake, fake, fake, 4096, None)
    assert st == B.CCE_ERR_DTYPE
    assert L.cce_neg_workspace_init(None, 4096, None) == B.CCE_ERR_NULL
    assert L.cce_neg_index_status(None, 4096, None) == B.CCE_ERR_NULL


def test_gradient_filtering_is_accepted_only_where_it_is_defined(binding):
    B = binding
    ok = B.make_desc(256, 1000, 64, 0, B.CCE_BF16, B.CCE_NEG_FULL, filter_eps=1e-4)
    assert B.cce_neg_workspace_bytes(ok) > 0
    for kw in (dict(neg_mode=B.CCE_NEG_SHARED, K=64, in_dtype=B.CCE_BF16, d=64),   # sampled modes do not filter (Sec. 3.3)
               dict(neg_mode=B.CCE_NEG_FULL, K=0, in_dtype=B.CCE_F32, d=64),       # fp32 has no bf16 tile
               dict(neg_mode=B.CCE_NEG_FULL, K=0, in_dtype=B.CCE_BF16, d=96)):     # no matrix-core kernel for this d
        desc = B.make_desc(256, 1000, kw["d"], kw["K"], kw["in_dtype"], kw["neg_mode"], filter_eps=1e-4)
        assert B.cce_neg_workspace_bytes(desc) == 0
    for bad in (-1.0, float("nan")):
        assert B.cce_neg_workspace_bytes(B.make_desc(256, 1000, 64, 0, B.CCE_BF16, B.CCE_NEG_FULL, filter_eps=bad)) == 0


def test_sampled_calls_reject_bad_samplers_before_launch(binding):
    B = binding
    L = B.lib()
    fake = ctypes.c_void_p(0x1000)  # never dereferenced
    desc = B.make_desc(16, 100, 64, 8, B.CCE_F32, B.CCE_NEG_PER_POSITION)
    ok = B.make_sampler(B.CCE_SAMPLER_UNIFORM, 1, 0)
    assert L.cce_neg_sample(ctypes.byref(desc), None, fake, None) == B.CCE_ERR_NULL
    assert L.cce_neg_sample(ctypes.byref(desc), ctypes.byref(ok), None, None) == B.CCE_ERR_NULL
    assert L.cce_neg_sample(ctypes.byref(desc), ctypes.byref(B.make_sampler(7, 1, 0)), fake, None) == B.CCE_ERR_SHAPE
    alias_without_table = B.make_sampler(B.CCE_SAMPLER_ALIAS, 1, 0)
    assert L.cce_neg_sample(ctypes.byref(desc), ctypes.byref(alias_without_table), fake, None) == B.CCE_ERR_NULL
    full = B.make_desc(16, 100, 64, 0, B.CCE_F32, B.CCE_NEG_FULL)
    assert L.cce_neg_sample(ctypes.byref(full), ctypes.byref(ok), fake, None) == B.CCE_ERR_UNSUPPORTED
    big = 1 << 30
    st = L.cce_neg_forward_sampled(ctypes.byref(full), ctypes.byref(ok), fake, fake, fake, None, fake, fake, fake, big, None)
    assert st == B.CCE_ERR_UNSUPPORTED
    st = L.cce_neg_forward_sampled(ctypes.byref(desc), ctypes.byref(ok), fake, fake, None, None, fake, fake, fake, big, None)
    assert st == B.CCE_ERR_NULL   # tgt missing
    st = L.cce_neg_forward_sampled(ctypes.byref(desc), ctypes.byref(ok), fake, fake, fake, None, fake, fake, fake, 8, None)
    assert st == B.CCE_ERR_WORKSPACE
    st = L.cce_neg_backward_sampled(ctypes.byref(desc), ctypes.byref(ok), fake, fake, fake, None, None, None, fake, fake,
                                    fake, big, None)
    assert st == B.CCE_ERR_NULL   # lse missing
    st = L.cce_neg_backward_sampled(ctypes.byref(desc), ctypes.byref(alias_without_table), fake, fake, fake, None, fake,
                                    None, fake, fake, fake, big, None)
    assert st == B.CCE_ERR_NULL
    # the shared list the sampled calls draw has its corner of the workspace
    a = B.cce_neg_workspace_bytes(B.make_desc(512, 4096, 64, 128, B.CCE_F32, B.CCE_NEG_SHARED))
    b = B.cce_neg_workspace_bytes(B.make_desc(512, 4096, 64, 1024, B.CCE_F32, B.CCE_NEG_SHARED))
    assert b - a >= (1024 - 128) * 4


def test_binding_refuses_wrong_dtypes_and_shapes_before_any_launch(binding):
    """The C ABI reads raw bytes: a torch.long index tensor, a short mask or a mis-shaped per-position `neg` must be
    refused by the binding (and so by cce_neg_loss) before a pointer is formed.  CPU tensors suffice: a call that got
    past the checks would stop at the CUDA-tensor requirement, with another message."""
    import torch

    B = binding
    N, V, d, K = 6, 50, 16, 4
    desc = B.make_desc(N, V, d, K, B.CCE_F32, B.CCE_NEG_PER_POSITION)
    H, E = torch.zeros(N, d), torch.zeros(V, d)
    tgt = torch.zeros(N, dtype=torch.int32)
    neg = torch.zeros(N, K, dtype=torch.int32)
    mask = torch.ones(N, dtype=torch.uint8)
    loss, lse = torch.zeros(N), torch.zeros(N)
    ws = torch.zeros(1 << 16, dtype=torch.uint8)

    def fwd(**kw):
        a = dict(H=H, E=E, tgt=tgt, neg=neg, mask=mask, loss=loss, lse=lse)
        a.update(kw)
        return B.cce_neg_forward(desc, a["H"], a["E"], a["tgt"], a["neg"], a["mask"], a["loss"], a["lse"], ws)

    with pytest.raises(TypeError, match="tgt"):
        fwd(tgt=tgt.long())
    with pytest.raises(TypeError, match="neg"):
        fwd(neg=neg.long())
    with pytest.raises(TypeError, match="mask"):
        fwd(mask=mask.float())
    with pytest.raises(TypeError, match="H"):
        fwd(H=H.double())
    with pytest.raises(ValueError, match="tgt"):
        fwd(tgt=tgt[:-1])
    with pytest.raises(ValueError, match="mask"):
        fwd(mask=mask[:-1])
    with pytest.raises(ValueError, match="neg"):
        fwd(neg=neg[:, :-1])
    with pytest.raises(ValueError, match="neg"):
        fwd(neg=neg.t().contiguous())          # [K, N]: right size, wrong shape
    with pytest.raises(ValueError, match="neg"):
        fwd(neg=None)
    with pytest.raises(ValueError, match="E"):
        fwd(E=E[:-1])
    with pytest.raises(ValueError, match="CUDA"):   # well-formed arguments get as far as the device-pointer requirement
        fwd()
    g, dH, dE = torch.zeros(N), torch.zeros(N, d), torch.zeros(V, d)
    with pytest.raises(TypeError, match="dE"):
        B.cce_neg_backward(desc, H, E, tgt, neg, mask, lse, g, dH, dE.double(), ws)
    with pytest.raises(TypeError, match="dH"):
        B.cce_neg_backward(desc, H, E, tgt, neg, mask, lse, g, dH.bfloat16(), dE, ws)
    with pytest.raises(ValueError, match="grad_loss"):
        B.cce_neg_backward(desc, H, E, tgt, neg, mask, lse, g[:-1], dH, dE, ws)
    bad_mode = B.make_desc(N, V, d, K, B.CCE_F32, 7)
    with pytest.raises(ValueError, match="neg_mode"):
        B.cce_neg_forward(bad_mode, H, E, tgt, neg, mask, loss, lse, ws)
    # the autograd front end goes through the same checks
    from paper_2509_09682_amd import cce_neg_loss

    with pytest.raises(TypeError, match="tgt"):
        cce_neg_loss(H, E, tgt.long(), neg, mask, neg_mode=B.CCE_NEG_PER_POSITION)


@pytest.mark.parametrize("dtype,limit", [("bf16", 40960), ("f32", 1 << 20)])
def test_workspace_serves_smaller_batches(binding, dtype, limit):
    """Shared and full mode: the bytes asked for do not fall as N grows (one workspace for a batch and a smaller last one;
    bf16 tiles: up to 40,960 positions), and what 4096 positions reserve stays at 16 shares of partial rows."""
    B = binding
    dt = B.CCE_BF16 if dtype == "bf16" else B.CCE_F32
    sizes = sorted(set(list(range(1, 3000, 97)) + list(range(3000, 45000, 331)) + [n + o for n in (1024, 2048, 4096, 16384, 40960, 65536)
                                                                                   for o in (-128, -1, 0, 1, 128)] + [90000, 204800, 600000]))
    for d in (64, 128, 256):
        for mode, cols in ((B.CCE_NEG_SHARED, (1, 100, 600, 4096, 60000)), (B.CCE_NEG_FULL, (700, 30011))):
            for n_cols in cols:
                for fuse in (0, 1):
                    V, K = (70000, n_cols) if mode == B.CCE_NEG_SHARED else (n_cols, 0)
                    need = [B.cce_neg_workspace_bytes(B.make_desc(N, V, d, K, dt, mode, fuse_dH=fuse)) for N in sizes if N <= limit]
                    assert need[0] > 0 and all(a <= b for a, b in zip(need, need[1:])), (d, mode, n_cols, fuse)
    if dtype == "bf16":
        n = B.cce_neg_workspace_bytes(B.make_desc(4096, 5_000_000, 256, 4096, dt, B.CCE_NEG_SHARED, fuse_dH=1))
        assert n <= 4096 * (16 * 1024 + 1024 + 20 + 64 * 8) + (1 << 16)


def test_bucketed_step_refuses_a_grid_that_does_not_fit_before_launch(binding):
    """Candidate blocks beyond what one launch holds, by buckets behind the first table launch (256 entries).  Nothing may be
    launched first: without a GPU that would be a HIP error."""
    B = binding
    n_empty, n = 300, 200
    desc = B.make_desc(n, 1000, 8, 1 << 30, B.CCE_F32, B.CCE_NEG_SHARED)
    ptr = (ctypes.c_int64 * (n_empty + n + 1))(*([0] * n_empty + list(range(n + 1))))
    fake = ctypes.c_void_p(0x1000)  # never dereferenced
    need = int(B.lib().cce_neg_bucketed_workspace_bytes(ctypes.byref(desc), n, n_empty + n))
    assert need > 0
    st = B.lib().cce_neg_bucketed_step(ctypes.byref(desc), fake, fake, fake, fake, n, ptr, n_empty + n, fake, None, fake, fake, fake,
                                       fake, fake, need, None)
    assert st == B.CCE_ERR_SHAPE

"""The dense kernels in fp32 precision (shared lists and the full catalogue, fp32 inputs or hidden sizes without a
bf16-weight matrix kernel) against the fp64 oracle, at the sizes where their tiles, splits and column shares change."""
import numpy as np
import pytest

from test_gpu_parity import check_against_oracle
from workloads import NEG_FULL, NEG_SHARED, make_workload

pytestmark = pytest.mark.gpu

TOL = 1e-5   # the contract of the fp32 path; no 16-bit weight enters here whatever the input type


def _run(w, **kw):
    from hip_harness import run_hip

    return run_hip(w, **kw)


# hidden sizes: the smallest, one short of and one past a block of 32 columns, every width class, the largest
WIDTHS = [("f32", d) for d in (8, 40, 64, 72, 128, 192, 256, 320, 512)] + [("bf16", d) for d in (8, 32, 40, 96, 104, 192, 216, 320, 392, 512)]


@pytest.mark.parametrize("mode", [NEG_SHARED, NEG_FULL])
@pytest.mark.parametrize("dtype,d", WIDTHS)
def test_widths_and_passes(mode, dtype, d):
    import paper_2509_09682_amd as P

    V = 203 if mode == NEG_FULL else 157     # not a multiple of a tile; shared: repeats and collisions in the list
    w = make_workload(f"dense_m{mode}_{dtype}_d{d}", 7, 61, d, V, 0 if mode == NEG_FULL else 77, dtype, mode, 300 + d + mode,
                      pad="bernoulli", pad_p=0.3, g_kind="random", e_sigma=0.1, tgt_dist="zipf")
    check_against_oracle(w, _run(w, fuse_dH=True, reuse_prep=True), TOL)
    check_against_oracle(w, _run(w), TOL)
    check_against_oracle(w, _run(w, fuse_dH=True, validate=1), TOL)            # compacted, dH pass of its own
    if mode == NEG_SHARED:
        w.mask_collisions = 0
        check_against_oracle(w, _run(w, fuse_dH=True, reuse_prep=True, validate=1), TOL)
    w.mask[:] = 1
    out = _run(w, fuse_dH=True, reuse_prep=True, use_mask=False, g=None, repeat_backward=2,
               dH_dtype=P.CCE_BF16 if dtype == "bf16" else P.CCE_F32)
    out["dE"] = out["dE"] * 0.5
    check_against_oracle(w, out, TOL, g=None, dH_tol=4e-3 if dtype == "bf16" else None)   # half an ulp of bf16: 2^-9


@pytest.mark.parametrize("batch,seq,V,K", [(1, 1, 50, 1), (1, 3, 5000, 1500), (1, 33, 3000, 33), (2, 64, 90, 31), (9, 1000, 3000, 200),
                                           (30, 1000, 2000, 40)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 48), ("bf16", 320)])
def test_shapes_from_one_position_to_unsplit_grids(batch, seq, V, K, dtype, d):
    """One position, few positions against many candidates (shares of the list), around a block of positions, and
    enough positions for compaction and for whole lists per block."""
    w = make_workload(f"dense_{batch}x{seq}_K{K}_{dtype}_d{d}", batch, seq, d, V, K, dtype, NEG_SHARED, 77 + seq, g_kind="random",
                      pad="none" if batch * seq < 100 else "right", pad_len_lo=seq // 3, e_sigma=0.1, tgt_dist="zipf")
    for fuse in (True, False):
        check_against_oracle(w, _run(w, fuse_dH=fuse, reuse_prep=fuse), TOL)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 96)])
def test_scores_far_above_the_correct_item(dtype, d):
    """The correct item's score is the first reference; here some candidates score up to 150 nats more, some positions
    have every candidate far below."""
    K = 300
    w = make_workload(f"dense_climb_{dtype}", 3, 40, d, 2000, K, "f32", NEG_SHARED, 77, pad="bernoulli", pad_p=0.1, g_kind="random",
                      e_sigma=0.05)
    H = w.H.reshape(w.N, d).copy()
    E = w.E.reshape(w.V, d).copy()
    for i, up in ((5, 150.0), (17, 60.0), (41, 21.0), (90, 25.0)):   # <h_i, e_v> = up, late in the list
        v = int(w.neg[K // 2 + i])
        E[v] = up * H[i] / float(H[i].astype(np.float64) @ H[i].astype(np.float64))
    for i in (60, 61):                                                # the correct item towers over the rest
        E[w.tgt[i]] = 120.0 * H[i] / float(H[i].astype(np.float64) @ H[i].astype(np.float64))
    w.H, w.E = H.reshape(w.H.shape), E.reshape(w.E.shape)
    if dtype == "bf16":
        from workloads import bf16_bits_from_f32
        import dataclasses

        w = dataclasses.replace(w, H=bf16_bits_from_f32(w.H), E=bf16_bits_from_f32(w.E), in_dtype="bf16")
    # a score of 150 carries 2^-24 * 150 of absolute error into its exponent, hence 9e-6 relative into the gradients
    check_against_oracle(w, _run(w, fuse_dH=True, reuse_prep=True), 4e-5)
    check_against_oracle(w, _run(w), 4e-5)


def test_bad_ids_are_skipped():
    import paper_2509_09682_amd as P

    w = make_workload("dense_bad_ids", 3, 50, 40, 400, 60, "f32", NEG_SHARED, 5, g_kind="random", pad="bernoulli", pad_p=0.2)
    ok = w.neg.copy()
    ref = _run(w, algo=P.CCE_ALGO_GATHER, validate=1)
    assert ref["status"] == P.CCE_OK
    w.neg = ok.copy()
    w.neg[[3, 59]] = (-5, w.V)
    w.tgt = w.tgt.copy()
    w.tgt[7] = w.V + 3
    for fuse in (False, True):
        a = _run(w, algo=P.CCE_ALGO_GATHER, validate=1, fuse_dH=fuse, reuse_prep=fuse)
        b = _run(w, validate=1, fuse_dH=fuse, reuse_prep=fuse)
        assert a["status"] == b["status"] == P.CCE_ERR_INDEX
        for name in ("loss", "lse", "dH", "dE"):
            assert np.max(np.abs(a[name] - b[name])) <= 1e-5 * np.max(np.abs(a[name])), name


@pytest.mark.parametrize("sizes,K", [((1,), 1), ((0, 70, 0, 1, 33, 0), 31), ((5,) * 300 + (0, 900), 64), ((2000, 3), 700)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("bf16", 320)])
def test_buckets_of_any_size_in_one_launch(sizes, K, dtype, d):
    """Empty, tiny and uneven buckets, more buckets than one table launch carries, lists that are split."""
    import dataclasses

    import torch

    import paper_2509_09682_amd as P
    from paper_2509_09682_amd.consumers import _one_launch
    from paper_2509_09682_amd.runner import to_device
    from workloads import NEG_PER_POSITION

    M, n = sum(sizes), len(sizes)
    N = M + 7
    w = make_workload(f"dense_buckets_{n}_{dtype}_d{d}", 1, N, d, 1500, K, dtype, NEG_PER_POSITION, 31 + d, g_kind="random",
                      e_sigma=0.1, tgt_dist="zipf")
    assert _one_launch(P.CCE_F32 if dtype == "f32" else P.CCE_BF16, d, M, n, K)
    rng = np.random.default_rng(3)
    order = rng.permutation(N)[:M]
    bucket_neg = rng.integers(0, w.V, size=(n, K)).astype(np.int32)
    bucket_neg[:, 0] = w.tgt[rng.integers(0, N, size=n)]
    ptr = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    rows = np.zeros((N, K), np.int32)
    w.mask[:] = 0
    for b in range(n):
        rows[order[ptr[b]:ptr[b + 1]]] = bucket_neg[b]
    w.mask[order] = 1
    w = dataclasses.replace(w, neg=rows)
    H, E, tgt, _, _ = to_device(w)
    if dtype == "bf16":
        H, E = H.view(torch.bfloat16), E.view(torch.bfloat16)
    dE = torch.zeros((w.V, d), device="cuda")
    loss, lse, dH = P.bucketed_step(H, E, tgt, torch.from_numpy(order).cuda(), ptr, torch.from_numpy(bucket_neg).cuda(),
                                    torch.from_numpy(w.g).cuda(), dE)
    out = dict(loss=loss.cpu().numpy(), lse=lse.cpu().numpy(), dH=dH.float().cpu().numpy(), dE=dE.cpu().numpy())
    check_against_oracle(w, out, TOL, dH_tol=4e-3 if dtype == "bf16" else None)   # dH in bf16: half an ulp, 2^-9


@pytest.mark.parametrize("dtype,d,batch,validate", [("f32", 40, 60, 0), ("bf16", 320, 60, 0), ("bf16", 64, 60, 0), ("f32", 40, 60, 1), ("f32", 40, 5, 0)])
def test_mask_at_any_address_and_a_copy_of_it_in_the_backward_call(dtype, d, batch, validate):
    """The forward and the backward call get the same mask contents at addresses of different alignment, either way round;
    the backward call reuses the preparation.  5940 positions are compacted, 495 are not."""
    import torch

    import paper_2509_09682_amd as P
    from paper_2509_09682_amd.runner import to_device

    w = make_workload(f"mask_at_{dtype}_d{d}_{batch}", batch, 99, d, 700, 45, dtype, NEG_SHARED, 41 + d, pad="bernoulli",
                      pad_p=0.35, g_kind="random", e_sigma=0.1, tgt_dist="zipf")
    tol = 2e-2 if (dtype, d) == ("bf16", 64) else TOL
    H, E, tgt, neg, mask = to_device(w)
    dt = P.CCE_F32 if dtype == "f32" else P.CCE_BF16
    masks = []
    for shift in (0, 1, 15):
        store = torch.full((w.N + 64,), 1, dtype=torch.uint8, device="cuda")
        store[shift:shift + w.N] = mask
        masks.append(store[shift:shift + w.N])
        assert masks[-1].data_ptr() % 16 == shift
    for fwd, bwd in ((1, 0), (0, 1), (2, 1), (1, 2)):
        desc = P.make_desc(w.N, w.V, d, w.K, dt, NEG_SHARED, validate_indices=validate, fuse_dH=1)
        again = P.make_desc(w.N, w.V, d, w.K, dt, NEG_SHARED, validate_indices=validate, fuse_dH=1, reuse_forward_prep=1)
        ws = P.new_workspace(desc)
        out = {k: torch.full(shape, float("nan"), device="cuda") for k, shape in (("loss", (w.N,)), ("lse", (w.N,)), ("dH", (w.N, d)))}
        out["dE"] = torch.zeros((w.V, d), device="cuda")
        P.cce_neg_forward(desc, H, E, tgt, neg, masks[fwd], out["loss"], out["lse"], ws)
        P.cce_neg_backward(again, H, E, tgt, neg, masks[bwd], out["lse"], torch.from_numpy(w.g).cuda(), out["dH"], out["dE"], ws)
        check_against_oracle(w, {k: v.cpu().numpy() for k, v in out.items()}, tol)


@pytest.mark.parametrize("K", [256, 288, 320])
@pytest.mark.parametrize("batch", [3, 100])
def test_forward_calls_around_the_shortest_list_that_is_split(K, batch):
    """d = 64 in fp32: up to 256 candidates a forward call walks the list whole, from 257 on in shares and a merge launch.  The
    call without a workspace goes first over a larger batch: its scratch memory is used again without being cleared."""
    import torch

    import paper_2509_09682_amd as P
    from paper_2509_09682_amd.runner import to_device

    w = make_workload(f"dense_fwd_{K}_{batch}", batch, 60, 64, 900, K, "f32", NEG_SHARED, K + batch, pad="bernoulli", pad_p=0.3,
                      g_kind="random", e_sigma=0.1, tgt_dist="zipf")
    out = _run(w)
    check_against_oracle(w, out, TOL)
    big = make_workload("dense_fwd_big", 100, 60, 64, 900, 33, "f32", NEG_SHARED, 7, pad="none", g_kind="random")
    for v in (big, w):
        desc = P.make_desc(v.N, v.V, v.d, v.K, P.CCE_F32, NEG_SHARED)
        loss, lse = (torch.full((v.N,), float("nan"), device="cuda") for _ in range(2))
        P.cce_neg_forward_noalloc(desc, *to_device(v), loss, lse)
    for name, t in (("loss", loss), ("lse", lse)):
        assert np.array_equal(t.cpu().numpy().view(np.uint32), out[name].view(np.uint32)), name    # the same kernels, no atomics


@pytest.mark.parametrize("N", [32, 33, 64, 97, 224, 225])
@pytest.mark.parametrize("dtype,d", [("f32", 256), ("f32", 512), ("bf16", 96)])
def test_tiny_steps_in_shares_of_one_tile(N, dtype, d):
    """One to eight tiles of positions: up to seven are walked by a block each, more in shares of two."""
    w = make_workload(f"dense_tiny_{N}_{dtype}_d{d}", 1, N, d, 300, 40, dtype, NEG_SHARED, N + d, pad="none" if N % 2 else "right",
                      pad_len_lo=N - 9, g_kind="random", e_sigma=0.1, tgt_dist="zipf")
    check_against_oracle(w, _run(w, fuse_dH=True, reuse_prep=True), TOL)


@pytest.mark.parametrize("K", [300, 33, 16])
@pytest.mark.parametrize("d", [216, 320, 392])
def test_long_rows_share_scores_and_their_references(d, K):
    """Above 192 columns several wavefronts form parts of a score block and exchange the weights; a score far above its
    reference, in either half of a tile, in the first, a later or the short last one, moves the references of the whole block."""
    import dataclasses

    from workloads import bf16_bits_from_f32

    w = make_workload(f"dense_exchange_{d}_{K}", 3, 45, d, 2000, K, "f32", NEG_SHARED, d + K, pad="bernoulli", pad_p=0.1,
                      g_kind="random", e_sigma=0.05)
    H, E = w.H.reshape(w.N, d).copy(), w.E.reshape(w.V, d).copy()
    for i, at, up in ((5, 3, 150.0), (17, 20, 60.0), (70, 40, 21.0), (90, 170, 25.0), (33, K - 1, 110.0)):   # <h_i, e> = up
        if at < K:
            E[int(w.neg[at])] = up * H[i] / float(H[i].astype(np.float64) @ H[i].astype(np.float64))
    w = dataclasses.replace(w, H=bf16_bits_from_f32(H.reshape(w.H.shape)), E=bf16_bits_from_f32(E.reshape(w.E.shape)), in_dtype="bf16")
    # a score of 150 carries 2^-24 * 150 of absolute error into its exponent, hence 9e-6 relative into the gradients
    check_against_oracle(w, _run(w, fuse_dH=True, reuse_prep=True), 4e-5)
    check_against_oracle(w, _run(w), 4e-5)

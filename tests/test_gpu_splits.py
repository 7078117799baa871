"""Matrix-core tiles where the candidate range is cut into shares: the number of shares changes with the number of
positions (64 up to 1024, 32 up to 2048, 16 above) and is bounded by the length of the list."""
import pytest

from test_gpu_parity import TOL_BF16, check_against_oracle
from workloads import NEG_FULL, make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [40, 1024, 1025, 2048, 2049])
@pytest.mark.parametrize("d,V", [(64, 8199), (128, 8199), (256, 2100), (256, 4103)])
def test_shares_of_the_catalogue(d, V, N):
    from hip_harness import run_hip

    w = make_workload(f"shares_{N}_d{d}_{V}", 1, N, d, V, 0, "bf16", NEG_FULL, 11 + N, g_kind="random", pad="none" if N % 2 else "right",
                      pad_len_lo=N - 20, e_sigma=0.1, tgt_dist="zipf")
    for fuse in (True, False):
        check_against_oracle(w, run_hip(w, fuse_dH=fuse, reuse_prep=fuse), TOL_BF16)


@pytest.mark.parametrize("sizes,d,K", [((5000, 4096), 256, 4096), ((9000, 8192), 128, 4096), ((16512, 16384), 64, 4096), ((41100, 40960), 64, 512)])
def test_one_workspace_for_buckets_of_unequal_size(sizes, d, K, monkeypatch):
    """The loop of bucketed_step over large buckets makes one workspace for the largest.  Against the one-launch form,
    which the oracle covers elsewhere; bf16 softmax weights differ by 2^-9 a term, 2^-9 of the norm at most."""
    import torch

    import paper_2509_09682_amd as P
    from paper_2509_09682_amd import consumers

    g = torch.Generator(device="cuda").manual_seed(5)
    M, V = sum(sizes), 20000
    N = M + 3
    H = torch.randn((N, d), device="cuda", generator=g).to(torch.bfloat16)
    E = (0.05 * torch.randn((V, d), device="cuda", generator=g)).to(torch.bfloat16)
    tgt = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    neg = torch.randint(0, V, (len(sizes), K), device="cuda", generator=g, dtype=torch.int32)
    order = torch.randperm(N, device="cuda", generator=g)[:M]
    up = torch.rand(N, device="cuda", generator=g)
    out = []
    for bound in (0.0, float("inf")):     # a launch pair per bucket, all buckets in one launch
        monkeypatch.setattr(consumers, "_BUCKET_FLOPS_FOR_TILES", bound)
        dE = torch.zeros((V, d), device="cuda")
        loss, lse, dH = P.bucketed_step(H, E, tgt, order, [0, sizes[0], M], neg, up, dE)
        out.append((loss, lse, dH.float(), dE))
    for name, a, b in zip(("loss", "lse", "dH", "dE"), *out):
        err = float((a - b).norm() / b.norm())
        assert err <= (4e-6 if name in ("loss", "lse") else 2.0 ** -7 if name == "dH" else 2.0 ** -9), (name, err)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_both_forms_of_bucketed_step_take_the_same_arguments(dtype, monkeypatch):
    """Columns of a wider candidate matrix, strided hidden states, order and gradient, a gradient vector longer or shorter than
    the batch (its entries at the positions that take part count)."""
    import torch

    import paper_2509_09682_amd as P
    from paper_2509_09682_amd import consumers

    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(6)
    N, V, d, K, M = 70, 300, 64, 21, 50
    H = torch.randn((N, 2, d), device="cuda", generator=g).to(dt)[:, 1]
    E = (0.1 * torch.randn((V, d), device="cuda", generator=g)).to(dt)
    tgt = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    neg = torch.randint(0, V, (3, K + 9), device="cuda", generator=g, dtype=torch.int32)[:, :K]
    order = torch.randperm(N - 5, device="cuda", generator=g)[:M].repeat_interleave(2)[::2]
    up = torch.rand(2 * N, device="cuda", generator=g)
    for bound in ((0.0, float("inf")) if dtype == "bf16" else (0.0,)):
        monkeypatch.setattr(consumers, "_BUCKET_FLOPS_FOR_TILES", bound)
        want = None
        for w in (up[:N], up, up[:N - 5], up[:N, None].expand(N, 2)[:, 0]):
            dE = torch.zeros((V, d), device="cuda")
            out = [*P.bucketed_step(H, E, tgt, order, [0, 20, 20, M], neg, w, dE), dE]
            plain = torch.zeros((V, d), device="cuda")
            ref = [*P.bucketed_step(H.contiguous(), E, tgt, order.contiguous(), [0, 20, 20, M], neg.contiguous(), up[:N], plain), plain]
            want = ref if want is None else want
            for a, b in zip(out[:3] + ref[:3], want[:3] + want[:3]):
                assert torch.equal(a, b)
            # dE is a sum by atomics: up to 50 positions' terms in any order, 50 * 2^-24 of the magnitudes
            assert float((dE - want[3]).abs().max()) <= 1e-5 * float(want[3].abs().max())


def test_scatter_blocks_that_would_cost_another_round():
    """505 candidate blocks on 512 block slots: two chunks of positions go whole, where four blocks each would not fit."""
    from hip_harness import run_hip

    w = make_workload("scatter_round", 1, 300, 128, 505 * 128, 0, "bf16", NEG_FULL, 5, g_kind="random", pad="none", e_sigma=0.1,
                      tgt_dist="zipf")
    check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), TOL_BF16)


@pytest.mark.parametrize("N,K", [(127, 33), (129, 32), (300, 511), (8001, 70), (20000, 41), (33000, 64)])
def test_blocks_of_either_width_at_d256(N, K):
    """d = 256: blocks of 128 positions with and without shares, blocks of 256 (the last case); candidates late in the list whose
    scores outgrow the reference by 90 nats send a block of either kind into the exact form."""
    import dataclasses

    import numpy as np
    from hip_harness import run_hip
    from workloads import NEG_SHARED, bf16_bits_from_f32

    w = make_workload(f"width_{N}_{K}", 1, N, 256, 3000, K, "f32", NEG_SHARED, N + K, g_kind="random", pad="bernoulli", pad_p=0.2,
                      e_sigma=0.05, tgt_dist="zipf")
    H, E = w.H.reshape(w.N, 256).copy(), w.E.reshape(w.V, 256).copy()
    for i in (N // 3, N - 2):
        E[int(w.neg[K - 1 if i > N // 2 else K - 2])] = 90.0 * H[i] / float(H[i].astype(np.float64) @ H[i].astype(np.float64))
    w = dataclasses.replace(w, H=bf16_bits_from_f32(H.reshape(w.H.shape)), E=bf16_bits_from_f32(E.reshape(w.E.shape)), in_dtype="bf16")
    check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), TOL_BF16)


@pytest.mark.parametrize("fuse", [False, True])
@pytest.mark.parametrize("tiles,rest", [(3, 0), (4, 1), (5, 17), (8, 0), (11, 31)])
@pytest.mark.parametrize("d,N,mode", [(64, 25_000, "shared"), (64, 77_000, "full"), (128, 25_000, "full"), (128, 77_000, "shared")])
def test_blocks_that_start_over_part_way_through_a_long_range(d, N, mode, tiles, rest, fuse):
    """Ranges of three tiles (8192 / d candidates each) and more, so that the ring of tile buffers goes round in the form a block
    falls back to when a score outgrows the largest of its first 32 candidates by 90 nats: in the third tile, in the last full one
    and in the last candidate.  196 blocks of 128 positions and 300 of 256 (two row groups) take the candidates in one piece; few of
    the positions are valid, which the launcher does not look at."""
    import dataclasses

    import numpy as np
    from hip_harness import run_hip
    from workloads import NEG_SHARED, bf16_bits_from_f32

    by = 8192 // d
    n = tiles * by + rest
    full = mode == "full"
    w = make_workload(f"over_{d}_{N}_{n}_{mode}", 1, N, d, n if full else 3000, 0 if full else n, "f32", NEG_FULL if full else NEG_SHARED,
                      N + n, g_kind="random", neg_dist="uniform" if full else "uniform_distinct", pad="bernoulli", pad_p=1 - 300 / N,
                      e_sigma=0.05, tgt_dist="zipf")
    H, E = w.H.reshape(w.N, d).copy(), w.E.reshape(w.V, d).copy()
    valid = np.flatnonzero(w.mask)
    tgt = w.tgt.copy()
    for i, k in zip(valid[[7, 150, -3]], (2 * by + 5, (tiles - 1) * by + 40, n - 1)):
        item = k if full else int(w.neg[k])
        E[item] = 90.0 * H[i] / float(H[i].astype(np.float64) @ H[i].astype(np.float64))
        # nobody's target: with p next to 1 there, p - 1 is rounding (2^-9 of p in bf16) against a row of the same size, and the bar
        # of a row against its own largest entry says nothing
        tgt[tgt == item] = 0
    w = dataclasses.replace(w, tgt=tgt, H=bf16_bits_from_f32(H.reshape(w.H.shape)), E=bf16_bits_from_f32(E.reshape(w.E.shape)), in_dtype="bf16")
    check_against_oracle(w, run_hip(w, fuse_dH=fuse, reuse_prep=True), TOL_BF16)


@pytest.mark.parametrize("N,K", [(300, 70), (20_000, 65), (70_000, 96)])
def test_every_block_starts_over_at_d256(N, K):
    """d = 256, blocks of 128 positions with and without shares and blocks of 256 in whole and split rounds: every position has its
    last candidate 90 nats up, so the wavefronts of every block that sees it agree on a second attempt."""
    import dataclasses

    import numpy as np
    from hip_harness import run_hip
    from workloads import NEG_SHARED, bf16_bits_from_f32

    w = make_workload(f"all_over_{N}_{K}", 1, N, 256, 3000, K, "f32", NEG_SHARED, N + K, g_kind="random", neg_dist="uniform_distinct",
                      e_sigma=0.05, h_sigma=0.3, tgt_dist="zipf")
    u = np.random.default_rng(N).standard_normal(256).astype(np.float32)
    u /= np.linalg.norm(u)
    H, E, tgt = w.H.reshape(w.N, 256) + 3.0 * u, w.E.reshape(w.V, 256).copy(), w.tgt.copy()
    E[int(w.neg[-1])] = 30.0 * u
    tgt[tgt == w.neg[-1]] = int(w.neg[0])  # p - 1 with p next to 1 is rounding: see the test above
    w = dataclasses.replace(w, tgt=tgt, H=bf16_bits_from_f32(H.reshape(w.H.shape)), E=bf16_bits_from_f32(E.reshape(w.E.shape)), in_dtype="bf16")
    check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), TOL_BF16)


@pytest.mark.parametrize("d,N,fuse", [(64, 41_000, False), (64, 77_000, False), (64, 41_000, True), (64, 77_000, True), (128, 41_000, False),
                                      (128, 77_000, False), (128, 41_000, True), (256, 32_700, True), (256, 41_000, True)])
def test_sum_of_exponentials_over_a_long_range(d, N, fuse):
    """A peaked softmax over 4096 candidates taken in one piece: the first scores 0, the others all the same, some 2^-12 of it each.
    Every sum they are added to lies between 1 and 2, so an addition loses up to 2^-24, the same at each one where the addends
    are equal.  A lane has 128 sub-tiles of 32 candidates to add up (16 each, joined first, which loses next to nothing); its
    exponentials are off by 2e-6 of themselves (|o| log2 e rounded at 16, the constant, the instruction)."""
    import numpy as np
    from hip_harness import run_hip
    from workloads import bf16_bits_from_f32, f32_from_bf16_bits

    V = 4096
    w = make_workload(f"long_sum_{d}_{N}", 1, N, d, V, 0, "bf16", NEG_FULL, N, pad="bernoulli", pad_p=1 - 400 / N)
    rng = np.random.default_rng(d)
    H, E = np.zeros((N, d), np.float32), np.zeros((V, d), np.float32)
    H[:, 0], H[:, 1] = rng.uniform(8.5, 10, N), rng.uniform(0, 1, N)
    E[1:, 0], E[1:, 1] = -1.0, -(2.0 ** -6)
    w.H, w.E = bf16_bits_from_f32(H), bf16_bits_from_f32(E)
    H = f32_from_bf16_bits(w.H).astype(np.float64)
    out = run_hip(w, fuse_dH=fuse, reuse_prep=True)
    valid = w.mask != 0
    tot = 1.0 + (V - 1) * np.exp(-(H[valid, 0] + H[valid, 1] * 2.0 ** -6))
    err = np.abs(out["lse"][valid].astype(np.float64) - np.log(tot))
    print(f"d {d} N {N} fuse {fuse}: error {err.max():.2e}, bound {np.min(128 * 2.0 ** -24 / tot + 2e-6):.2e}")
    assert np.all(err <= 128 * 2.0 ** -24 / tot + 2e-6)


def _four_late_candidates(d, N, K):
    """300 valid positions in four groups, each of which has one of four candidates 90 nats above the others: in the first tile or
    the fourth, behind the first look at the sums or the second, in the middle and at the end."""
    import dataclasses

    import numpy as np
    from workloads import NEG_SHARED, bf16_bits_from_f32

    w = make_workload(f"four_late_{d}_{N}", 1, N, d, 3000, K, "f32", NEG_SHARED, N + d, g_kind="random", neg_dist="uniform_distinct",
                      pad="bernoulli", pad_p=1 - 300 / N, e_sigma=0.05, h_sigma=0.3, tgt_dist="zipf")
    u = np.linalg.qr(np.random.default_rng(N).standard_normal((d, 4)))[0].T.astype(np.float32)
    H, E, tgt = w.H.reshape(w.N, d) + 3.0 * u[np.arange(w.N) % 4], w.E.reshape(w.V, d).copy(), w.tgt.copy()
    for j, k in enumerate((100, 300, K // 2 - 50, K - 1)):
        E[int(w.neg[k])] = 30.0 * u[j]
        tgt[tgt == w.neg[k]] = int(w.neg[0])  # p - 1 with p next to 1 is rounding: see the tests above
    return dataclasses.replace(w, tgt=tgt, H=bf16_bits_from_f32(H.reshape(w.H.shape)), E=bf16_bits_from_f32(E.reshape(w.E.shape)), in_dtype="bf16")


_LONG_RANGES = [(64, 25_000), (64, 77_000), (128, 25_000), (256, 20_000), (256, 70_000)]  # one and two row groups; blocks of 128 and 256


@pytest.mark.parametrize("d,N", _LONG_RANGES)
def test_blocks_that_start_over_early_in_a_long_range(d, N):
    """A block leaves its range at the next look behind a score that outgrows the reference; at d = 256 its second attempt, which knows
    the tiles seen by then, meets a further one, and the third knows all of them."""
    from hip_harness import run_hip

    w = _four_late_candidates(d, N, 2600)
    check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), TOL_BF16)


@pytest.mark.parametrize("d,N", _LONG_RANGES)
def test_a_position_that_is_no_number_among_blocks_that_start_over(d, N):
    """NaN in one hidden state: no attempt mends that sum, and the others of its block are as without it."""
    import dataclasses

    import numpy as np
    from hip_harness import run_hip
    from oracle import cce_oracle as O
    from oracle.compare import per_position_rel, tensor_rel

    w = _four_late_candidates(d, N, 2600)
    ref = O.run_workload(w, g=w.g.astype(np.float64))
    at = int(np.flatnonzero(w.mask)[5])
    H = w.H.reshape(w.N, d).copy()
    H[at, 3] = 0x7FC0
    out = run_hip(dataclasses.replace(w, H=H.reshape(w.H.shape)), fuse_dH=True, reuse_prep=True)
    v = (w.mask != 0) & (np.arange(w.N) != at)
    assert np.isnan(out["loss"][at]) and np.isnan(out["lse"][at]) and np.isnan(out["dH"][at]).any()
    assert per_position_rel(out["lse"][v], ref.loss[v], ref.lse[v], ref.lse[v]) <= TOL_BF16
    assert tensor_rel(out["dH"][v], ref.dH[v]) <= TOL_BF16

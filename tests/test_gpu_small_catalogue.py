"""Per-position negatives of small catalogues: the index is built in buckets of one id up to 2048, its pairs in more than
one slice, segments from empty to thousands of pairs (one lane group, a block per chunk)."""
import numpy as np
import pytest

from test_gpu_parity import check_against_oracle, pair_budget
from workloads import NEG_PER_POSITION, make_workload

pytestmark = pytest.mark.gpu


# catalogues at the edges of the bucket widths (512 items: one id each; 1023 / 1024; 300,000: 1024 ids each); the last
# two file more pairs than a slice holds
@pytest.mark.parametrize("V,batch,K", [(40, 3, 37), (511, 4, 64), (512, 4, 64), (1023, 4, 300), (1024, 4, 300), (300_000, 4, 64),
                                       (700, 30, 720), (2500, 30, 720), (700, 30, 1400), (2500, 30, 1400)])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 40)])
def test_small_catalogues(V, batch, K, dtype, d):
    from hip_harness import run_hip

    w = make_workload(f"small_V{V}_{dtype}", batch, 200, d, V, K, dtype, NEG_PER_POSITION, 5 + V, g_kind="random", e_sigma=0.05,
                      tgt_dist="zipf", pad="right", pad_len_lo=190)
    # dE rows sum up to thousands of pairs in fp32, whatever the order: 2e-5, twice the contract of single rows
    check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), 2e-5)


def test_one_item_that_collects_a_quarter_of_all_pairs():
    """A bucket beyond an eighth of the pair budget stays out of the index; its pairs are added one by one."""
    from hip_harness import run_hip

    w = make_workload("one_hot_item", 60, 200, 64, 60_000, 720, "bf16", NEG_PER_POSITION, 99, g_kind="random", e_sigma=0.05)
    rng = np.random.default_rng(1)
    neg = w.neg.reshape(w.N, w.K)
    neg[rng.random(neg.shape) < 0.25] = 31_234
    assert w.N * w.K > pair_budget(w.N, w.K) and (neg == 31_234).sum() > pair_budget(w.N, w.K) // 8
    # Every position adds its term about 180 times in a row to one fp32 sum; equal adds round alike, so the row is off by
    # up to 180 sqrt(12000) 2^-25 = 6e-4 of the running sum, which may be twice the final one.  Everything else is exact
    # to the usual figure, which loss, lse and dH show.
    errs = check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), 1.2e-3, row_tol=1.2e-3)
    assert max(errs[k] for k in ("loss", "lse", "dH")) <= 1e-5, errs


@pytest.mark.parametrize("N,K,V,d,dtype,hot", [
    (65536, 65, 3000, 8, "bf16", 0.0), (65537, 65, 3000, 8, "bf16", 0.0), (65537, 65, 3000, 8, "bf16", 0.15),
    (16384, 640, 3000, 8, "bf16", 0.0), (16384, 640, 3000, 8, "bf16", 0.2),
    (65537, 66, 3000, 64, "bf16", 0.0), (65537, 66, 3000, 128, "bf16", 0.0), (65537, 66, 3000, 256, "bf16", 0.0),
    (65537, 66, 3000, 40, "f32", 0.0), (65537, 66, 3000, 128, "f32", 0.15),
    (16384, 520, 3000, 64, "bf16", 0.0), (16384, 520, 3000, 64, "f32", 0.15)])
def test_slices_of_narrow_and_wide_pairs(N, K, V, d, dtype, hot):
    """Up to 65,536 positions a slice holds 2^23 pairs of half the width, above 2^22: one slice of 4.3 M pairs and two; 8.5 M and
    10.5 M narrow pairs in two.  d = 64 / 128 / 256: the correct items ride in the first filing launch.  hot: a bucket beyond an
    eighth of the budget, which stays out of the index in either width."""
    from hip_harness import run_hip

    w = make_workload(f"pairs_{N}_{K}", N, 1, d, V, K, dtype, NEG_PER_POSITION, 3, g_kind="random", e_sigma=0.05, tgt_dist="zipf")
    assert (w.N * w.K > pair_budget(N, K)) == (N != 65536)
    if hot:
        neg = w.neg.reshape(w.N, w.K)
        neg[np.random.default_rng(2).random(neg.shape) < hot] = V - 3
        assert (neg == V - 3).sum() > pair_budget(N, K) // 8
    # as above: 2e-5 for sums of thousands of pairs; the hot row is off by hot K sqrt(N) 2^-25 <= 5e-4 of its running sum, and
    # that row alone: loss, lse and dH show the usual figure
    tol = 1e-3 if hot else 2e-5
    errs = check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), tol, row_tol=tol)
    assert max(errs[k] for k in ("loss", "lse", "dH")) <= 1e-5, errs


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,K,V,d", [(1, 1, 5, 24), (64, 32, 600, 264), (683, 3, 2000, 24), (8192, 64, 900, 8), (4095, 128, 70_000, 40),
                                     (8191, 256, 70_000, 16), (8192, 257, 1_100_000, 8)])
def test_chunks_of_the_index(N, K, V, d, dtype):
    """A chunk of the index is 2048 pairs and doubles up to 8192 with 256 chunks of it: a pair, 2048 and one more, each side of
    2^19 and 2^21 pairs; one to 538 buckets, rows that leave lanes of their group idle; masks that leave a block nothing to file."""
    from hip_harness import run_hip

    w = make_workload(f"chunks_{N}_{K}_{dtype}", N, 1, d, V, K, dtype, NEG_PER_POSITION, 11, g_kind="random", e_sigma=0.05, tgt_dist="zipf",
                      pad="bernoulli" if N > 1 else "none", pad_p=0.4)
    if N > 4000:
        w.mask[100:3000] = 0
    check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), 2e-5)


def test_more_chunks_than_blocks():
    """33.6 M pairs: a block takes several chunks and files its pairs one by one."""
    from hip_harness import run_hip

    w = make_workload("chunks_many", 65536, 1, 8, 30_000, 513, "bf16", NEG_PER_POSITION, 12, g_kind="random", e_sigma=0.05)
    check_against_oracle(w, run_hip(w, fuse_dH=True, reuse_prep=True), 2e-5)

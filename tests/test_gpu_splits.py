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

"""The partial sums of a plan's stage 2 stay within the workspace budget (and
1 GiB) for every precision, also over many chunks, and the sigma is that of
uncut lists.

FP64 and Ozaki (exact digit products, added in FP64) against a plan with the
default budget: another order of the same sums, the bar of test_gpu_split_sums.
BF16x3 against uncut lists in the same chunks (which products share an FP32 sum
depends on the chunks): the same FP32 sums, added in FP64 in another order, the
same bar.
"""
import re

import numpy as np
import pytest

from tests.helpers import case, lib_load, lib_sigma_flat
from tests.test_gpu_split_sums import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mb", [0, 1, 4, 16])
@pytest.mark.parametrize("K,N,tsz,D,i", [(12, 14, 2, 150, 7), (12, 12, 0, 1500, 5)])
def test_partial_sums_stay_within_the_budget(ctx, monkeypatch, capfd, K, N, tsz, D, i, mb):
    from paper_2603_28648_amd import Context
    print(f"partial sums bound: K={K} N={N} 2Sz={tsz} D={D} window={i} budget={mb} MiB", flush=True)
    h, eri, m = case(K, N, tsz, D, i)
    monkeypatch.setenv("DMRG_BF16_CONFIG", "1,529")  # 64 x 64 tiles, stage 2 in pieces
    n = lib_load(ctx, h, eri, m)
    x = np.random.default_rng(27).normal(size=n)
    ref = {p: lib_sigma_flat(ctx, x, p) for p in ("fp64", "ozaki")}
    monkeypatch.setenv("DMRG_WS_BUDGET_MB", str(mb))
    monkeypatch.setenv("DMRG_VERBOSE", "1")
    capfd.readouterr()
    small = Context(0)
    try:
        assert lib_load(small, h, eri, m) == n
        assert mb >= 16 or small.sigma_info("fp64")["n_chunks"] > 1
        got = {p: lib_sigma_flat(small, x, p) for p in ("fp64", "ozaki", "bf16x3")}
        log = capfd.readouterr().err
        monkeypatch.setenv("DMRG_BF16_CONFIG", "1,1")
        lib_load(small, h, eri, m)
        ref["bf16x3"] = lib_sigma_flat(small, x, "bf16x3")
    finally:
        small.close()
    size = {w: int(b) for w, b in re.findall(r"\[dmrg\] (\w+) stage 2: (\d+) bytes of partial sums", log)}
    assert set(size) == {"FP64", "BF16", "Ozaki"}
    vector = 8 * 8 * n  # one padded vector, for the pinned pairs (a row of one entry takes eight)
    assert size["BF16"] <= mb << 20 and size["Ozaki"] <= mb << 20
    assert size["FP64"] <= max(mb << 20, vector)
    for p in ref:
        check(got[p], ref[p])

"""The BF16 autotuner takes the fastest of the configurations that it timed,
with the lists whole or in pieces."""
import re

import numpy as np
import pytest

from tests.helpers import case, lib_load, lib_sigma_flat

pytestmark = pytest.mark.gpu


# budget 0: no partial sums, so that pieces gain nothing over whole lists
@pytest.mark.parametrize("mb", [None, "0"])
@pytest.mark.parametrize("K,N,tsz,D,i", [(8, 8, 0, 64, 3), (12, 14, 2, 150, 7), (12, 12, 0, 1500, 5), (14, 14, 0, 400, 6)])
def test_autotuner_takes_the_fastest_trial(ctx, monkeypatch, capfd, K, N, tsz, D, i, mb):
    from paper_2603_28648_amd import Context
    print(f"autotuner: K={K} N={N} 2Sz={tsz} D={D} window={i} budget={mb}", flush=True)
    h, eri, m = case(K, N, tsz, D, i)
    for name, val in (("DMRG_AUTOTUNE", "1"), ("DMRG_VERBOSE", "1"), ("DMRG_WS_BUDGET_MB", mb)):
        if val is not None:
            monkeypatch.setenv(name, val)
    c = Context(0)
    try:
        n = lib_load(c, h, eri, m)
        capfd.readouterr()
        lib_sigma_flat(c, np.random.default_rng(28).normal(size=n), "bf16x3")
        info = c.sigma_info("bf16x3")
    finally:
        c.close()
    log = re.findall(r"autotune stage (\d) shape (\d+) order (\d) sort (\d) split (\d): ([\d.]+) ms", capfd.readouterr().err)
    for stage in (1, 2):
        t = {int(s) + 16 * int(o) + 256 * int(q) + 512 * int(p): float(ms) for st, s, o, q, p, ms in log if int(st) == stage}
        assert len(t) >= 8
        assert t[info[f"bf_config_stage{stage}"]] == min(t.values())

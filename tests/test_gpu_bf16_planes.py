"""The BF16 hi/lo output of sigma stage 1 (split-BF16x3: two planes, plain
BF16: the hi plane) on every tile shape.

A stage-1 product is one FP32 sum over k in slabs of 32, the same on every
tile shape, so the sigma does not depend on the stage-1 shape at all.
"""
import numpy as np
import pytest

from tests.helpers import case, lib_load, lib_sigma_flat

pytestmark = pytest.mark.gpu

# sectors of at most 29 (one tile), 100 (remainders of 64- and 128-row tiles)
# and about 330 (whole 128-tiles and remainders) a side
SIZES = [(8, 8, 0, 64, 3), (12, 14, 2, 150, 7), (12, 12, 0, 1500, 5)]


# stage-1 shapes 128x64, 64x128, 128x128 (two and three LDS stages), by problem, by part
@pytest.mark.parametrize("shape", [0, 2, 3, 4, 6, 7])
@pytest.mark.parametrize("K,N,tsz,D,i", SIZES)
def test_stage1_planes_are_those_of_64x64_tiles(ctx, monkeypatch, K, N, tsz, D, i, shape):
    print(f"BF16 planes: K={K} N={N} 2Sz={tsz} D={D} window={i} stage-1 shape={shape}", flush=True)
    h, eri, m = case(K, N, tsz, D, i)
    out = {}
    for s in (1, shape):
        monkeypatch.setenv("DMRG_BF16_CONFIG", f"{s},1")
        n = lib_load(ctx, h, eri, m)
        x = np.random.default_rng(25).normal(size=n)
        # BF16 first and between: it leaves the lo plane of the products as it is
        out[s] = [lib_sigma_flat(ctx, y, p) for y, p in ((x, "bf16"), (x, "bf16x3"), (-3.0 * x, "bf16"), (x, "bf16x3"))]
    for a, b in zip(out[1], out[shape]):
        assert np.array_equal(a, b)
    assert np.array_equal(out[shape][1], out[shape][3])

"""Sigma on the direct-to-register FP64 kernels and with stage-2 segment lists
cut into pieces, against the same plan on one workgroup per list.

Both sides add the same products in another order.  A sum of n products with
rounding errors of 1.1e-16 moves by about sqrt(n) of them, times the ratio of
the terms' norm to that of the sum: with n up to 1e6 and a ratio of 10 that is
1.1e-12; the bar is three times that, on the norm and on the largest element.
"""
import numpy as np
import pytest

from tests.helpers import case, lib_load, lib_sigma_flat

pytestmark = pytest.mark.gpu

TOL = 3e-12

# blocks of 1 x 1 to 1 x 4; at most 9 (one 32 x 32 tile), 29 (remainder of a
# tile), 100 (two 64-row tiles) and about 330 (two 256-column tiles) a side
SIZES = [(6, 5, 1, 10, 0), (8, 8, 0, 64, 3), (12, 12, 0, 256, 5), (12, 14, 2, 150, 7), (12, 12, 0, 1500, 5),
         (14, 14, 0, 5000, 6)]


def check(a, b):
    assert np.linalg.norm(a - b) <= TOL * np.linalg.norm(b)
    assert np.max(np.abs(a - b)) <= TOL * np.max(np.abs(b))


@pytest.mark.parametrize("K,N,tsz,D,i", SIZES)
def test_fp64_pieces_match_whole_lists(ctx, monkeypatch, K, N, tsz, D, i):
    print(f"FP64 pieces vs whole lists: K={K} N={N} 2Sz={tsz} D={D} window={i}", flush=True)
    h, eri, m = case(K, N, tsz, D, i)
    n = lib_load(ctx, h, eri, m)
    x = np.random.default_rng(21).normal(size=n)
    got = lib_sigma_flat(ctx, x)
    assert np.array_equal(got, lib_sigma_flat(ctx, x))  # parts are added in a fixed order
    monkeypatch.setenv("DMRG_F64_LDS", "0")
    lib_load(ctx, h, eri, m)
    check(got, lib_sigma_flat(ctx, x))


# shapes with an FP64 accumulator: 128x64, 64x64, 64x128; +16: tiles grouped by
# operand, +512: in pieces
@pytest.mark.parametrize("shape", [0, 1, 2])
@pytest.mark.parametrize("K,N,tsz,D,i", SIZES[:5])
def test_bf16_pieces_match_whole_lists(ctx, monkeypatch, K, N, tsz, D, i, shape):
    print(f"BF16 pieces vs whole lists: K={K} N={N} 2Sz={tsz} D={D} window={i} shape={shape}", flush=True)
    h, eri, m = case(K, N, tsz, D, i)
    x = None
    for prec in ("bf16", "bf16x3"):
        out = {}
        for code in (shape, shape + 512, shape + 16 + 512):
            monkeypatch.setenv("DMRG_BF16_CONFIG", f"{shape},{code}")
            n = lib_load(ctx, h, eri, m)
            if x is None:
                x = np.random.default_rng(22).normal(size=n)
            out[code] = lib_sigma_flat(ctx, x, prec)
            assert ctx.sigma_info(prec)["bf_config_stage2"] == code
        check(out[shape + 512], out[shape])
        check(out[shape + 16 + 512], out[shape])

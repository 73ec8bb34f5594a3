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


# rows and k entries around the slicer's 64-row tasks and its 8, 16, 32 and 64
# lanes a row; k of one slab, its edges and several
@pytest.mark.parametrize("m,n", [(1, 64), (63, 33), (65, 31), (16, 130)])
@pytest.mark.parametrize("k", [16, 17, 32, 33, 64, 65, 128, 129, 256, 300])
@pytest.mark.parametrize("kappa", [3, 6, 7])
def test_ozaki_slices_and_products_at_edges(ctx, monkeypatch, kappa, m, n, k):
    """Element-wise bound of the scheme (rounding of X and dropped digit
    products, plus the FP64 rounding of the reference): test_gpu_ozaki.py."""
    from tests.test_gpu_ozaki import _check, _run
    monkeypatch.setenv("DMRG_OZAKI_SLICES", str(kappa))
    rng = np.random.default_rng(m + 3 * n + 7 * k)
    A, Bt = rng.normal(size=(m, k)), rng.normal(size=(n, k))
    for ta, tb in ((False, True), (True, False)):
        assert _check(A, Bt, _run(ctx, A, Bt, trans_a=ta, trans_b=tb), kappa) <= 1.0


@pytest.mark.parametrize("K,N,tsz,D,i", SIZES[:5])
def test_ozaki_pieces_match_fp64(ctx, K, N, tsz, D, i):
    """47-bit digits: 2^-47 a product and 5 dropped digit products of 2^-48,
    averaged over the terms; the bar is that of the other ozaki sigma tests."""
    print(f"ozaki pieces vs FP64: K={K} N={N} 2Sz={tsz} D={D} window={i}", flush=True)
    h, eri, m = case(K, N, tsz, D, i)
    x = np.random.default_rng(23).normal(size=lib_load(ctx, h, eri, m))
    s64, soz = lib_sigma_flat(ctx, x), lib_sigma_flat(ctx, x, "ozaki")
    assert np.linalg.norm(soz - s64) < 1e-12 * np.linalg.norm(s64)


# largest sector: one-column operator blocks and short rows; one tile; two
# tiles a side; wider than a 256-column tile
@pytest.mark.parametrize("dmax", [1, 2, 3, 9, 17, 33, 64, 130])
@pytest.mark.parametrize("n,tS", [(8, 0), (9, 1)])
def test_su2_direct_kernels_match_the_tiled_ones(ctx, monkeypatch, n, tS, dmax):
    """Operator blocks of any row length and 8-byte alignment, read in place."""
    from tests.test_gpu_su2 import case_ops, device_ops, dev
    import torch
    print(f"su2 direct vs tiled kernels: n={n} 2S={tS} dmax={dmax}", flush=True)
    lsec, rsec, lops, rops, pairs, size, rng = case_ops(n, tS, dmax, 40 + dmax)
    L, R, psi = device_ops(lops), device_ops(rops), dev(rng.normal(size=size))
    out = []
    for tile in ("", "128x64,64"):
        if tile:
            monkeypatch.setenv("DMRG_SU2_TILE", tile)
        got = torch.full_like(psi, float("nan"))
        with ctx.su2_plan(lsec, rsec, n, tS, L, R, pairs) as plan:
            plan.sigma(psi, got)
            torch.cuda.synchronize()
        out.append(got.cpu().numpy())
    check(out[0], out[1])


# the smallest subspace restarts at every step; 24 holds the whole space of
# the smallest windows (a correction that vanishes restarts too)
@pytest.mark.parametrize("precondition", [0, 1, 2])
@pytest.mark.parametrize("max_subspace", [3, 24])
@pytest.mark.parametrize("K,N,tsz,D,i", [(2, 2, 0, 16, 0), (4, 4, 0, 100, 1), (6, 6, 0, 12, 2), (6, 7, -1, 10, 4)])
def test_davidson_steps_on_the_device(ctx, K, N, tsz, D, i, max_subspace, precondition):
    """Against the dense matrix of the same sigma: with a residual of 1e-7 the
    energy error is below 1e-14 / gap, and rounding stays below 1e-12 |H|."""
    import torch
    h, eri, m = case(K, N, tsz, D, i)
    n = lib_load(ctx, h, eri, m)
    print(f"davidson vs dense: K={K} N={N} 2Sz={tsz} n={n} subspace={max_subspace} precond={precondition}", flush=True)
    H = np.stack([lib_sigma_flat(ctx, e) for e in np.eye(n)])
    ref, vec = np.linalg.eigh((H + H.T) / 2)
    x = np.random.default_rng(24).normal(size=n)
    psi = torch.from_numpy(x + 3 * vec[:, 0]).cuda()
    r = ctx.davidson(psi, tol=1e-7, max_iter=400, max_subspace=max_subspace, precondition=precondition)
    assert r["converged"]
    scale = np.abs(ref).max()
    gap = ref[1] - ref[0] if n > 1 else 1.0
    assert abs(r["energy"] - ref[0]) <= 1e-14 / gap + 1e-12 * scale
    out = psi.cpu().numpy()
    assert abs(np.linalg.norm(out) - 1) < 1e-12
    assert np.linalg.norm(H @ out - r["energy"] * out) <= 2e-7

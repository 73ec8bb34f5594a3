"""Spin-adapted sigma of operators that share storage: blocks of different
sizes that start at one address, the one-column ones among them, which FP64
plans copy.  Bar: that of the other spin-adapted tests (rounding only)."""
import numpy as np
import pytest

from oracle import su2
from synthetic.su2 import random_operator, sector_window

from tests.test_gpu_su2 import close, dev, oracle_sigma

pytestmark = pytest.mark.gpu


# dimensions dealt to the sectors of a side: one-column blocks of 1 to 130 rows
@pytest.mark.parametrize("dims", [(1, 3, 70, 1, 130, 2), (130, 1, 1, 17), (2, 1, 64, 33)])
@pytest.mark.parametrize("n,tS", [(8, 0), (9, 1)])
def test_blocks_of_different_heights_at_one_address(ctx, n, tS, dims):
    import torch
    print(f"su2 blocks at one address: n={n} 2S={tS} dims={dims}", flush=True)
    rng = np.random.default_rng(n + tS + len(dims))
    sides = [[(N, ts, dims[(k + q) % len(dims)]) for k, (N, ts, _) in enumerate(sec)]
             for q, sec in enumerate(sector_window(n, tS, 4, rng))]
    lsec, rsec = sides
    ops, host, pairs = ([], []), ([], []), []
    pools = [rng.normal(size=max(d for _, _, d in sec) ** 2) for sec in sides]
    tensors = [dev(p) for p in pools]
    for dn, tk in [(0, 0), (0, 2), (1, 1), (-1, 1), (2, 0)]:
        for q, sgn in ((0, 1), (1, -1)):
            dim = [d for _, _, d in sides[q]]
            keys = sorted(random_operator(sides[q], sgn * dn, tk, rng))
            host[q].append({(o, i): pools[q][:dim[o] * dim[i]].reshape(dim[o], dim[i]) for o, i in keys})
            ops[q].append(([(o, i, 0) for o, i in keys], tensors[q]))
        pairs.append((len(pairs), len(pairs), tk, abs(dn) % 2, float(rng.normal())))
    size = sum(lsec[a][2] * rsec[b][2] for a, b in su2.coupled_blocks(lsec, rsec, n, tS))
    x = rng.normal(size=size)
    ref = oracle_sigma(lsec, rsec, n, tS, host[0], host[1], pairs, x)
    psi = dev(x)
    out = torch.full_like(psi, float("nan"))
    with ctx.su2_plan(lsec, rsec, n, tS, ops[0], ops[1], pairs) as plan:
        plan.sigma(psi, out)
        torch.cuda.synchronize()
    heights = {d for sec, o in zip(sides, host) for op in o for (a, i) in op if sec[i][2] == 1 for d in [sec[a][2]]}
    assert len(heights) > 1 and close(out.cpu().numpy(), ref)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("bf16x3", 2e-5)])  # the bars of test_gpu_su2
@pytest.mark.parametrize("tile", ["", "128x64,64"])
@pytest.mark.parametrize("n,tS,dmax", [(8, 0, 3), (9, 1, 90)])
def test_blocks_in_any_order_and_more_than_once(ctx, monkeypatch, n, tS, dmax, tile, precision, tol):
    """Blocks of an operator listed in random order, some of them twice (their
    contributions add), operators without blocks and ones that no pair names."""
    import torch
    from tests.test_gpu_su2 import case_ops, pack_blocks
    print(f"su2 block order: n={n} 2S={tS} dmax={dmax} tile={tile} {precision}", flush=True)
    if tile:
        monkeypatch.setenv("DMRG_SU2_TILE", tile)
    lsec, rsec, lops, rops, pairs, size, rng = case_ops(n, tS, dmax, 90 + dmax)

    def scrambled(ops):
        out, host = [], []
        for op in ops:
            blocks, data = pack_blocks(op)
            twice = {(o, i) for o, i, _ in blocks if rng.random() < 0.2}
            lst = blocks + [b for b in blocks if b[:2] in twice]
            out.append(([lst[k] for k in rng.permutation(len(lst))], dev(data)))
            host.append({k: (2 if k in twice else 1) * v for k, v in op.items()})
        return out + [([], dev(np.zeros(1))), out[0]], host

    L, lhost = scrambled(lops)
    R, rhost = scrambled(rops)
    pairs = pairs + [(len(L) - 2, 0, 0, 0, 1.0)]  # a left operator without blocks
    x = rng.normal(size=size)
    ref = oracle_sigma(lsec, rsec, n, tS, lhost + [{}], rhost, pairs, x)
    psi = dev(x)
    out = torch.full_like(psi, float("nan"))
    with ctx.su2_plan(lsec, rsec, n, tS, L, R, pairs, precision) as plan:
        plan.sigma(psi, out)
        torch.cuda.synchronize()
    got = out.cpu().numpy()
    if precision == "fp64":
        assert np.abs(got - ref).max() <= tol * np.abs(ref).max()
    else:
        assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)

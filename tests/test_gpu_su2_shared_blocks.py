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

"""Sector lookup of a bond whose quantum numbers span any 32-bit range: the
layout check accepts them and their absence changes nothing (CPU)."""
import numpy as np
import pytest

from paper_2603_28648_amd import validate
from synthetic import make_integrals, make_mps, mps_arrays

LO, HI = -2 ** 31, 2 ** 31 - 1


def with_sectors(m, bond, extra):
    """The layout with sectors (N, 2Sz) of one state added to a bond that no site tensor outside the window reads."""
    a = dict(mps_arrays(m))
    lo, hi = a["bond_offsets"][bond], a["bond_offsets"][bond + 1]
    cols = [np.asarray(a[k]) for k in ("sector_n", "sector_2sz", "sector_dim")]
    mid = sorted([tuple(int(c[k]) for c in cols) for k in range(lo, hi)] + [(n, s, 1) for n, s in extra])
    for k, c, x in zip(("sector_n", "sector_2sz", "sector_dim"), cols, zip(*mid)):
        a[k] = np.concatenate([c[:lo], x, c[hi:]]).astype(np.int32)
    a["bond_offsets"] = np.asarray(a["bond_offsets"]).copy()
    a["bond_offsets"][bond + 1:] += len(extra)
    return a


@pytest.mark.parametrize("extra", [
    [(LO, LO), (HI, HI)],        # a product of spans of 2^64
    [(LO, -5), (HI, 2 ** 30)],   # ... of 2^63 and above
    [(LO, 0), (HI, 1)],          # one wide span
    [(0, 1 << 15), (0, -(1 << 15))],
    [(70000, 0)],
])
def test_bond_with_far_away_sectors_is_accepted(extra):
    h, eri = make_integrals(6, 6)
    m = make_mps(6, 6, 0, 12, 2, 1006)
    assert validate(h, eri, 6, 0, with_sectors(m, 3, extra), window=2) == 0

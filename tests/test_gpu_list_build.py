"""The neighbour-list build at the edges of its branches: few bins per dimension (exact tests only) and
many (FP32 offsets), more than 64 atoms in a bin, candidates beyond one register tile, several waves
per bin, single bins and runs of bins.  Forces against the FP64 oracle: a missing or doubled pair shows."""
import numpy as np
import pytest

from oracle import core
from synth import configs, fcc_lattice

pytestmark = pytest.mark.gpu

TOL = {"mixed": 1e-5, "fp64": 1e-11}      # as for every static force comparison in this suite


def kg(sizes, seed=300):
    return [configs.kg_cell([50] * (n // 50) + ([n % 50] if n % 50 else []), seed + k) for k, n in enumerate(sizes)]


def cu(ncell):
    x, H = fcc_lattice(ncell)
    x = x + np.random.default_rng(ncell).normal(0, 0.1, x.shape)
    return [dict(x=x, v=np.zeros_like(x), bonds=np.zeros((0, 2), np.int32), H0=H)]


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("name, cells, over, bins, mode", [
    ("two to four bins", lambda: kg([61, 130, 250]), dict(skin=0.6), 1, 0),
    ("five bins and more", lambda: kg([700, 1001, 2003]), dict(skin=0.4), 1, 0),
    ("half bins, six and seven", lambda: kg([180, 300, 900]), dict(skin=0.6), 2, 0),
    ("wide skin", lambda: kg([1500]), dict(skin=1.6), 1, 0),
    ("phase kernels", lambda: kg([61, 777, 4097]), dict(skin=0.55), 1, 2),
    ("runs of bins", lambda: kg([10000] * 8), dict(skin=0.3), 1, 0),
    ("copper, bins of 108 atoms", lambda: cu(6), dict(skin=2.0), 1, 0),
    ("copper, half bins", lambda: cu(8), dict(skin=1.5), 2, 2)])
def test_lists_hold_every_pair_once(prec, name, cells, over, bins, mode):
    from paper_1902_09171_amd import rcell
    cells = cells()
    params = configs.cu_params if name.startswith("copper") else configs.kg_params
    p = params(precision=prec, **over)
    g = rcell.RCellBatch(p, cells)
    g.set_bin_factor(bins)
    g.set_build_mode(mode)
    o = core.OracleBatch(p, cells)
    shift = np.random.default_rng(7)
    for k, c in enumerate(cells):            # a rebuild with the chosen bins, off the initial order
        x = c["x"] + shift.uniform(-50, 50, 3)
        s = g.get_state(k)
        g.set_state(k, x, s["v"], s["H"], s["Rprev"], s["step"])
        fg, fo = g.get_forces(k), o.get_forces(k)
        err = np.linalg.norm(fg - fo) / np.linalg.norm(fo)
        print(f"{name} {prec} cell {k}: {len(x)} atoms, force rel {err:.2e}", flush=True)
        # the shift rounds the positions at 2^-53 of 50 box units: well below the FP32 bound, and of
        # the order of 1e-13 in FP64 forces that change by ~1e3 per unit of distance
        assert err <= (TOL[prec] if prec == "mixed" else 1e-10), (name, k, err)
    assert np.all(g.status() == 0)

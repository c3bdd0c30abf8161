"""A batch of deformation gradients is committed as a whole or not at all: one refused cell leaves every
cell as it was, bit for bit, and cells that outgrow their bins or lists are committed after these have
grown.  Forces against the FP64 oracle."""
import numpy as np
import pytest

from oracle import core
from synth import configs

pytestmark = pytest.mark.gpu

TOL = {"mixed": 1e-5, "fp64": 1e-11}      # as for every static force comparison in this suite


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("ncells", [2, 70])          # 70: cells in two blocks of the commit
def test_all_cells_or_none(prec, ncells):
    from paper_1902_09171_amd import rcell
    p = configs.kg_params(precision=prec, skin=0.4)
    cells = [configs.kg_cell([20] * (8 + k % 3), 900 + k) for k in range(ncells)]
    g = rcell.RCellBatch(p, cells)
    g.set_bin_factor(2)
    g.run(3)
    last = ncells - 1
    for bad in (np.diag([0.3, 1.0, 1.0]), np.zeros((3, 3))):      # box too small; not a deformation
        before = [g.get_state(k) for k in range(ncells)]
        F = np.stack([configs.uniaxial_isochoric(0.01)] * ncells)
        F[last] = bad
        with pytest.raises(rcell.RCellError):
            g.set_deformation(F)
        for k in range(ncells):
            s = g.get_state(k)
            assert all(np.array_equal(s[q], before[k][q]) for q in ("x", "v", "H", "Rprev")), (bad[0, 0], k)
    for scale in (1.02, 1.12, 0.86, 1.0):             # kept; more bins; longer lists; back
        F = np.stack([np.eye(3)] * ncells)
        F[last] *= scale
        g.set_deformation(F)
        for k in (0, last):
            s = g.get_state(k)
            fg, fo = g.get_forces(k), core.forces(p, s["H"], s["x"], cells[k]["bonds"])[0]
            err = np.linalg.norm(fg - fo) / np.linalg.norm(fo)
            print(f"{prec} {ncells} cells, scale {scale}, cell {k}: force rel {err:.2e}", flush=True)
            assert err <= (1e-10 if prec == "fp64" else TOL[prec]), (scale, k)
        assert np.all(g.status() == 0)

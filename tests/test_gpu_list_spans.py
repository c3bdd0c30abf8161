"""The list build by spans of bins: cells rebuilt together, where a wave takes several bins at a time, against
the same cells rebuilt one by one, in short spans or single bins.  The lists hold the same pairs in the same
order, so forces and what follows are equal bit for bit; and against the FP64 oracle, where a missing or
doubled pair shows."""
import numpy as np
import pytest

from oracle import core
from synth import configs

pytestmark = pytest.mark.gpu

TOL = {"mixed": 1e-5, "fp64": 1e-10}      # FP32 forces as everywhere in this suite; FP64 ones of ~1e3 per unit of distance


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("sizes, skin, bins, stretch", [     # stretched beyond what a list survives: every cell builds
    ((10000,) * 12, 0.4, 1, 1.25),              # 1884 tiles, spans of two whole bins
    ((4000,) * 9 + (3001, 1000), 0.4, 2, 1.25),     # half bins, ~0.4 beads each: the longest spans
    ((4097, 2049, 1500), 0.7, 2, 1.35),         # the phase kernels; spans that end at a column's end
    ((333, 700, 1200), 0.3, 2, 1.2),           # few bins: spans cut by the half box, or single bins
])
def test_rebuilt_together_or_one_by_one(prec, sizes, skin, bins, stretch):
    from paper_1902_09171_amd import rcell
    p = configs.kg_params(precision=prec, skin=skin)
    melts = {n: configs.kg_cell([50] * (n // 50) + ([n % 50] if n % 50 else []), 900 + n) for n in set(sizes)}
    cells = [dict(melts[n], v=np.random.default_rng(k).standard_normal((n, 3))) for k, n in enumerate(sizes)]
    long_x = np.diag([stretch, stretch ** -0.5, stretch ** -0.5])
    F = np.stack([long_x if k % 2 else long_x[::-1, ::-1] for k in range(len(sizes))])   # and long in z
    out = []
    for together in (True, False):
        g = rcell.RCellBatch(p, cells)
        g.set_bin_factor(bins)
        n = g.rebuilds()
        g.set_deformation(F)
        assert g.rebuilds() == n + len(sizes)
        if not together:
            for k in range(len(sizes)):
                s = g.get_state(k)
                g.set_state(k, s["x"], s["v"], s["H"], s["Rprev"], s["step"])
        f = [g.get_forces(k) for k in range(len(sizes))]
        g.run(25)                         # and builds of a few cells at a time
        assert np.all(g.status() == 0)
        out.append(f + [g.get_state(k)[q] for k in range(len(sizes)) for q in ("x", "v")])
        if together:
            for k in {0, len(sizes) - 1}:
                s = g.get_state(k)
                g.set_state(k, s["x"], s["v"], s["H"], s["Rprev"], s["step"])
                fg, fo = g.get_forces(k), core.forces(p, s["H"], s["x"], cells[k]["bonds"])[0]
                err = np.linalg.norm(fg - fo) / np.linalg.norm(fo)
                print(f"{prec} {sizes[k]} beads, skin {skin}, bins {bins}: force rel {err:.2e}", flush=True)
                assert err <= TOL[prec]
    assert all(np.array_equal(a, b) for a, b in zip(*out))

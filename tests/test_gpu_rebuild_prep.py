"""The one-block-per-cell rebuild preparation at the edges of its branches (one to four atoms per thread, full
and partial; more bins than it keeps on chip) against the phase kernels: the atom order is defined by
positions alone, so whole trajectories with rebuilds are equal bit for bit."""
import numpy as np
import pytest

from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("bins", [1, 2])     # 2: the cells of 2049 atoms and more have over 4096 bins
def test_same_bits_as_the_phase_kernels(prec, bins):
    from paper_1902_09171_amd import rcell
    cells = [configs.kg_cell([50] * (n // 50) + [n % 50], 40 + k)
             for k, n in enumerate((61, 1023, 1024, 1025, 2049, 4095, 4096))]
    for c in cells:                          # hot enough that every cell rebuilds several times
        c["v"] = 2.0 * c["v"]
    p = configs.kg_params(precision=prec, skin=0.3, dt=0.004)
    out = []
    for mode in (1, 2):
        g = rcell.RCellBatch(p, cells)
        g.set_bin_factor(bins)
        g.set_build_mode(mode)
        g.run(40)
        assert np.all(g.status() == 0)
        out.append((g.get_stress(), [g.get_state(k) for k in range(len(cells))],
                    [g.get_forces(k) for k in range(len(cells))]))
    (s1, st1, f1), (s2, st2, f2) = out
    print(f"{prec} bins {bins}: stress {np.abs(s1 - s2).max():.1e}", flush=True)
    assert np.array_equal(s1, s2)
    for k in range(len(cells)):
        for q in ("x", "v", "H"):
            assert np.array_equal(st1[k][q], st2[k][q]), (k, q)
        assert np.array_equal(f1[k], f2[k]), k

"""A cell restored so dense that the neighbour list has to grow leaves the other cells of the batch as they
were: their forces at once, and their further trajectories, equal bit for bit those of a batch in which
the same cell was restored without growth."""
import numpy as np
import pytest

from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("skin", [0.4, 0.7])         # 0.4: the list grows from 48 to 64 entries, 0.7: from 64 to 80
def test_other_cells_are_untouched(prec, mode, skin):
    from paper_1902_09171_amd import rcell
    p = configs.kg_params(precision=prec, skin=skin)
    cells = [configs.kg_cell([50] * 24, 51), configs.kg_cell([37] * 30 + [1], 52), configs.kg_cell([50] * 40, 53)]
    out = []
    for scale in (1.0, 0.88):
        g = rcell.RCellBatch(p, cells)
        g.set_build_mode(mode)
        g.run(20)                                    # the atoms have left the order of the last build
        before = [(g.get_forces(k), g.get_state(k)) for k in (1, 2)]
        pe, _ = g.get_energy()
        s = g.get_state(0)
        g.set_state(0, scale * s["x"], 0.0 * s["v"], scale * s["H"], s["Rprev"], s["step"])
        pe2, _ = g.get_energy()
        for k in (1, 2):
            f, st = before[k - 1]
            now = g.get_state(k)
            assert np.array_equal(g.get_forces(k), f), (scale, k)
            assert all(np.array_equal(now[q], st[q]) for q in ("x", "v", "H")) and pe2[k] == pe[k], (scale, k)
        g.run(20)
        assert np.all(g.status()[1:] == 0)
        out.append([(g.get_forces(k), g.get_state(k)) for k in (1, 2)] + [np.array(g.get_energy())[:, 1:]])
    for k in (0, 1):
        assert np.array_equal(out[0][k][0], out[1][k][0])
        assert all(np.array_equal(out[0][k][1][q], out[1][k][1][q]) for q in ("x", "v", "H", "step"))
    assert np.array_equal(out[0][2], out[1][2])

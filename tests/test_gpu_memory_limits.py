"""Contexts short of device memory: the pruned list is optional, so it is left out, or given up again for
whatever else does not fit, and every result stays the same bit for bit."""
import numpy as np
import pytest

from oracle import core
from synth import configs, fcc_lattice

pytestmark = pytest.mark.gpu

CREATE = 37                                  # device allocations that a context cannot do without


def program(rcell, p, cells, monkeypatch, fault):
    """A run with a change of every size that memory hangs on; fault: the allocation that fails (0: none)."""
    monkeypatch.setenv("RCELL_FAULT_ALLOC", str(fault))
    g = rcell.RCellBatch(p, cells)
    monkeypatch.delenv("RCELL_FAULT_ALLOC")
    out = []
    g.set_lanes(2)
    g.run(15)
    g.autotune(use_cache=False)              # snapshot and scratch; the bins of the finer grid
    g.set_lanes(2)
    g.set_bin_factor(2)
    for scale in (1.1, 0.84, 1.0):           # more bins; longer lists; back
        F = np.stack([np.eye(3)] * len(cells))
        F[-1] *= scale
        g.set_deformation(F)
        out += [g.get_forces(k) for k in range(len(cells))]
        g.run(12)
        out += [g.get_state(k)[q] for k in range(len(cells)) for q in ("x", "v")]
        out += list(g.get_stress_ext()) + list(g.get_energy())
    assert np.all(g.status() == 0)
    g.close()
    return out


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("material", ["kg", "cu"])
def test_without_room_for_the_pruned_list(prec, material, monkeypatch):
    from paper_1902_09171_amd import rcell
    if material == "kg":
        p = configs.kg_params(precision=prec, skin=0.7, dt=0.001)
        cells = [configs.kg_cell([50] * 20, 61), configs.kg_cell([37] * 18 + [1], 62)]
    else:
        p = configs.cu_params(precision=prec)
        cells = []
        for k, n in enumerate((6, 7)):
            x, H = fcc_lattice(n)
            cells.append(dict(x=x + np.random.default_rng(k).normal(0, 0.05, x.shape), v=None,
                              bonds=np.zeros((0, 2), np.int32), H0=H))
    with pytest.raises(rcell.RCellError):    # the last one that is needed; the next two are the pruned list's
        program(rcell, p, cells, monkeypatch, CREATE)
    ref = program(rcell, p, cells, monkeypatch, 0)
    for fault in range(CREATE + 1, CREATE + 19):
        got = program(rcell, p, cells, monkeypatch, fault)
        assert all(np.array_equal(a, b) for a, b in zip(ref, got)), fault
        print(f"{material} {prec}: the same with allocation {fault} failing", flush=True)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("scale, fault", [(1.15, 1), (1.15, 4), (0.82, 1)])   # first and last array of the bins; the list
def test_refused_growth_leaves_the_batch_running(mode, scale, fault, monkeypatch):
    # no pruned list to give up: its reach does not pay at this skin
    from paper_1902_09171_amd import rcell
    p = configs.kg_params(precision="mixed", skin=0.3)
    cells = [configs.kg_cell([50] * 20, 63), configs.kg_cell([37] * 18 + [1], 64)]
    F = np.stack([np.eye(3), scale * np.eye(3)])
    out = []
    for refused in (False, True):
        monkeypatch.setenv("RCELL_FAULT_ALLOC", str(CREATE + fault))
        g = rcell.RCellBatch(p, cells)
        g.set_build_mode(mode)
        g.run(10)
        if refused:
            with pytest.raises(rcell.RCellError) as e:
                g.set_deformation(F)
            assert e.value.code == -6 and "injected" in str(e.value)
        n = g.rebuilds()
        g.run(40)
        assert g.rebuilds() > n              # on the bins and lists that it has
        out.append([g.get_state(k)[q] for k in range(2) for q in ("x", "v", "H")] + [np.array(g.get_energy())])
        assert np.all(g.status() == 0)
        if refused:                          # and the growth works once there is room
            g.set_deformation(F)
            s, f = g.get_state(1), g.get_forces(1)
            fo = core.forces(p, s["H"], s["x"], cells[1]["bonds"])[0]
            assert np.linalg.norm(f - fo) <= 1e-5 * np.linalg.norm(fo)   # as for every static force comparison
            assert np.all(g.status() == 0)
        g.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))

"""Contexts short of device memory: the pruned list is optional, so it is left out, or given up again for
whatever else does not fit, and every result stays the same bit for bit."""
import numpy as np
import pytest

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

"""k steps, a checkpoint, a load into a fresh state and k more steps against 2k steps, bit for bit, for
the variants of the cell update: what a step leaves for the next (ghosts, wave speeds) is formed anew
from a loaded state."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gks():
    import torch

    assert torch.cuda.is_available()
    import paper_2306_04467_amd as g

    g.load()
    return g


CASES = {
    "wall": (lambda: w.dam_break(25, seed=91), {}),
    "free": (lambda: w.free_outflow(20), {}),
    "coupling": (lambda: w.dam_break(25, seed=92), {"src_order": 4}),
    "discontinuous": (lambda: w.smooth_jittered(20), {"grad_mode": "discontinuous"}),
    "coupling_discontinuous": (lambda: w.smooth_jittered(20), {"src_order": 4, "grad_mode": "discontinuous"}),
    "dry": (lambda: w.dam_break_dry(30), {}),
    "dry_discontinuous": (lambda: w.dam_break_dry(30), {"grad_mode": "discontinuous"}),
}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", list(CASES))
def test_restart_is_bitwise(gks, case, precision):
    make, opts = CASES[case]
    sc = make()
    print(f"[restart] {case} {precision} T={sc.n_tri}", flush=True)
    mesh = gks.Mesh.from_scenario(sc)

    def state():
        return gks.State.from_scenario(mesh, sc, precision=precision, **opts)

    whole, first, second = state(), state(), state()
    whole.step(24)
    first.step(12)
    second.load(first.save())
    second.step(12)
    a, b = whole.read(), second.read()
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[2] == b[2]

"""The reconstruction's waves take 32 cells each: meshes that end in a wave of 2, 4, 18 or all 32
cells, with the variants of the kernel (plain, higher-order coupling, wet/dry), against the oracle
at the FP64 bound of a step, 4 steps."""
import pytest

import oracle as o
import workloads as w
from tests._parity import TOL_FP64, grad_err, state_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gks():
    import torch

    assert torch.cuda.is_available()
    import paper_2306_04467_amd as g

    g.load()
    return g


CASES = {
    "periodic_18": (lambda: w.smooth_periodic(3), {}),
    "periodic_98": (lambda: w.smooth_periodic(7), {}),
    "wall_32": (lambda: w.lake_at_rest(4, perturb=1e-2, seed=61), {}),
    "coupling_98": (lambda: w.smooth_periodic(7), {"src_order": 4}),
    "coupling_50": (lambda: w.dam_break(5, seed=62), {"src_order": 4}),
    "dry_36": (lambda: w.dam_break_dry(6), {}),
    "dry_64": (lambda: w.dam_break_dry(8), {}),
}


@pytest.mark.parametrize("case", list(CASES))
def test_last_wave_matches_oracle(gks, case):
    make, opts = CASES[case]
    sc = make()
    print(f"[waves] {case} T={sc.n_tri}", flush=True)
    st = gks.State.from_scenario(gks.Mesh.from_scenario(sc), sc, **opts)
    om = o.Mesh.from_scenario(sc)
    p = o.params_of(sc, **opts)
    W, gW = sc.W0.copy(), sc.gradW0.copy()
    for _ in range(4):
        dt = o.dt(om, p, W)
        st.stage(0, dt)
        st.stage(1)
        W, gW = o.step(om, p, dt, W, gW)
    Wg, gWg, _ = st.read()
    e, g = state_err(Wg, W), grad_err(gWg, gW, W)
    assert e.max() < 4 * TOL_FP64 and g.max() < 4 * TOL_FP64, (e, g)

"""The largest wave speeds that a step's second update leaves for the next step: meshes of one
incomplete wave, of whole waves and a remainder, and a batch whose scenarios meet inside a wave;
after an explicit step size, a checkpoint and graph replays.  Every step size against the oracle's on
the state before it (both take the maximum of the same FP64 expression: a few roundings, 1e-14)."""
import numpy as np
import pytest

import oracle as o
import workloads as w

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gks():
    import torch

    assert torch.cuda.is_available()
    import paper_2306_04467_amd as g

    g.load()
    return g


def _expected(sc, W):
    return o.dt(o.Mesh.from_scenario(sc), o.params_of(sc), W)


CASES = {
    "periodic_18": lambda: w.smooth_periodic(3),
    "wall_32": lambda: w.lake_at_rest(4, perturb=1e-2, seed=71),
    "dam_50": lambda: w.dam_break(5, seed=72),
    "dam_1250": lambda: w.dam_break(25, seed=73),
    "dry_36": lambda: w.dam_break_dry(6),
}


@pytest.mark.parametrize("case", list(CASES))
def test_single(gks, case):
    sc = CASES[case]()
    print(f"[step size] {case} T={sc.n_tri}", flush=True)
    st = gks.State.from_scenario(gks.Mesh.from_scenario(sc), sc)

    def check():
        W = st.read()[0]
        assert abs(st.step(1, want_dt=True) / _expected(sc, W) - 1) < 1e-14

    for _ in range(3):
        check()
    blob = st.save()
    st.stage(0, 0.5 * _expected(sc, st.read()[0]))
    st.stage(1)
    check()
    st.batch_step(3)
    check()
    st.load(blob)
    check()
    st.load(blob)
    W = st.read()[0]
    st.batch_step(1)
    assert abs(st.time()[1] / _expected(sc, W) - 1) < 1e-14


def test_batch(gks):
    scs = [w.dam_break(5, seed=81), w.lake_at_rest(3, perturb=1e-2, seed=82), w.dam_break(7, seed=83)]
    st = gks.State.from_scenarios(gks.Mesh.batch([gks.Mesh.from_scenario(s) for s in scs]), scs)
    for _ in range(3):
        W = st.read()[0]
        st.batch_step(1)
        c0 = 0
        for s, sc in enumerate(scs):
            dt = _expected(sc, np.ascontiguousarray(W[:, c0:c0 + sc.n_tri]))
            assert abs(st.time(s)[1] / dt - 1) < 1e-14
            c0 += sc.n_tri

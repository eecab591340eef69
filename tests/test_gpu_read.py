"""gks_state_read against the checkpoint of the same state (the raw device arrays), bit for bit, at the
sizes where the read-back changes its way: one copy through the pinned page up to 1 MiB (7,281
cells), one plain copy up to 8 MiB of a component block, copying threads beyond."""
import ctypes

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gks():
    import torch

    assert torch.cuda.is_available()
    import paper_2306_04467_amd as g

    g.load()
    return g


def _expected(st, sc, precision):
    T, TG = sc.n_tri, st.mesh.n_tri + st.mesh.n_ghost
    blob = np.frombuffer(st.save(), dtype=np.uint8)
    r = np.float64 if precision == "fp64" else np.float32
    o = blob.size - (2 * 8 + 8) - (2 * TG * 8 + 16 * TG * np.dtype(r).itemsize)
    Wh = blob[o:o + 16 * TG].view(np.float64).reshape(2, TG)[:, :T]
    o += 16 * TG
    n = 4 * TG * np.dtype(r).itemsize
    Wm = blob[o:o + n].view(r).reshape(4, TG)[:, :T].astype(np.float64)
    o += n
    n *= 3
    g = blob[o:o + n].view(r).reshape(12, TG)[:, :T].astype(np.float64)
    t = blob[o + n + 8:o + n + 16].view(np.float64)[0]
    return np.stack([Wh[0], Wm[0], Wm[1], Wh[1], Wm[2], Wm[3]]), g.reshape(6, 2, T), t


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [4, 60, 61, 170, 400])  # 32 .. 160,000 cells, flat bottom
def test_read_matches_the_checkpoint(gks, n, precision):
    if n == 400:
        sc = workloads.dam_break_dry(n)
    else:
        sc = workloads.smooth_periodic(n)
    st = gks.State.from_scenario(gks.Mesh.from_scenario(sc), sc, precision=precision)
    for steps in (0, 2):
        st.step(steps)
        W, g, t = st.read()
        We, ge, te = _expected(st, sc, precision)
        assert np.array_equal(W, We) and np.array_equal(g, ge) and t == te
    # either array alone, and neither
    lib, dp = gks.load(), ctypes.POINTER(ctypes.c_double)
    W1, g1, t1 = np.zeros_like(W), np.zeros_like(g), ctypes.c_double()
    assert lib.gks_state_read(st._h, W1.ctypes.data_as(dp), None, None) == 0
    assert lib.gks_state_read(st._h, None, g1.ctypes.data_as(dp), None) == 0
    assert lib.gks_state_read(st._h, None, None, ctypes.byref(t1)) == 0
    assert np.array_equal(W1, W) and np.array_equal(g1, g) and t1.value == t

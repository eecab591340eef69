"""The library's host code on a stub of the HIP calls: what its calls do to streams, devices and memory
that a single-GPU run does not show.  The stub's kernels do nothing, so no value is looked at."""
import ctypes
import threading

import pytest

import workloads
from tests import _stub

pytestmark = pytest.mark.skipif(not _stub.HAVE, reason="hipcc or g++ not available")


@pytest.fixture(scope="module")
def lib():
    return _stub.load()


@pytest.fixture
def stream(lib):
    _, stub = lib
    s = stub.stub_stream()
    yield ctypes.c_void_p(s)
    stub.stub_stream_free(s)


def _state(gks, stream, n=4, **kw):
    sc = workloads.lake_at_rest(n, perturb=1e-2, seed=1)
    return gks.State.from_scenario(gks.Mesh.from_scenario(sc), sc, stream=stream, **kw)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_a_new_state_leaves_its_stream_alone(lib, stream, precision):
    """Initial data are copied without the state's stream, which may be one that is being captured or
    holds other work: completing them puts nothing on it and does not wait for it."""
    gks, stub = lib
    stub.stub_capture(stream, 1)
    stub.stub_reset()
    st = _state(gks, stream, precision=precision)
    assert _stub.count(stub, "captured") == 0
    assert _stub.count(stub, "launches") > 0  # ghosts and wave speeds, elsewhere
    stub.stub_capture(stream, 0)
    st.close()


@pytest.mark.parametrize("query", ["time", "mass", "diagnostics", "check", "read"])
def test_a_query_of_a_captured_stream_queues_nothing(lib, stream, query):
    """It is refused (such a stream cannot be waited for), and leaves nothing in the caller's graph, least
    of all a copy into memory of the call."""
    gks, stub = lib
    st = _state(gks, stream)
    getattr(st, query)()
    stub.stub_capture(stream, 1)
    stub.stub_reset()
    with pytest.raises(gks.GksError):
        getattr(st, query)()
    assert _stub.count(stub, "captured") == 0
    stub.stub_capture(stream, 0)
    getattr(st, query)()
    st.close()


def test_a_step_size_asked_for_under_capture_adds_nothing_to_the_step(lib, stream):
    gks, stub = lib
    st = _state(gks, stream)
    stub.stub_capture(stream, 1)
    stub.stub_reset()
    st.step(2)
    n = _stub.count(stub, "captured")
    with pytest.raises(gks.GksError):
        st.step(2, want_dt=True)
    assert _stub.count(stub, "captured") == 2 * n > 0
    stub.stub_capture(stream, 0)
    st.close()


@pytest.mark.parametrize("n", [4, 250])  # 250: 125,000 cells, whose snapshot takes the copying threads
def test_copies_out_and_in_work_from_any_threads_device(lib, stream, n):
    """A thread of a process with several GPUs starts with device 0: what a read, a checkpoint or a query
    allocates and launches on its way goes to the state's device, and the thread's stays what it was."""
    gks, stub = lib
    stub.hipSetDevice(3)
    st = _state(gks, stream, n)
    stub.hipSetDevice(0)
    stub.stub_expect_device(3)
    stub.stub_reset()
    blob = st.save()
    st.load(blob)
    for query in ("read", "time", "check"):
        getattr(st, query)()
    assert _stub.count(stub, "wrong_device") == 0
    now = ctypes.c_int(-1)
    stub.hipGetDevice(ctypes.byref(now))
    assert now.value == 0
    stub.stub_expect_device(-1)
    st.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_reading_back_takes_no_device_memory(lib, stream, precision):
    """Neither for the call nor afterwards: a state that fills the device can be read and saved."""
    gks, stub = lib
    st = _state(gks, stream, precision=precision)
    held = _stub.count(stub, "device_bytes")
    for limit in (2 ** 62, 0):
        stub.stub_malloc_limit(limit)
        st.read()
        st.save()
        st.stage(0)
        st.read()
        st.stage(1)
        assert _stub.count(stub, "device_bytes") == held
    stub.stub_malloc_limit(2 ** 62)
    st.close()


def test_read_back_resources_belong_to_the_mesh(lib, stream):
    """Pinned pages and streams are made once for a mesh's states, not once for each of them, a bounded
    number of them is kept, and they go with the mesh."""
    gks, stub = lib
    sc = workloads.lake_at_rest(250, perturb=1e-2, seed=1)
    before = {k: _stub.count(stub, k) for k in ("pinned_bytes", "streams", "device_bytes")}
    mesh = gks.Mesh.from_scenario(sc)
    held = []
    for _ in range(3):
        states = [gks.State.from_scenario(mesh, sc, stream=stream) for _ in range(2)]
        for st in states:
            st.read()
            st.time()
        held.append({k: _stub.count(stub, k) for k in ("pinned_bytes", "streams")})
        threads = [threading.Thread(target=st.read) for st in states for _ in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for st in states:
            st.close()
    assert held[0] == {"pinned_bytes": before["pinned_bytes"] + 4 * 2 ** 20, "streams": before["streams"] + 4}
    for k, n in (("pinned_bytes", 8 * 2 ** 20), ("streams", 8)):
        assert _stub.count(stub, k) - before[k] <= n
    mesh.close()
    assert {k: _stub.count(stub, k) for k in before} == before


def test_a_checkpoint_waits_no_more_than_it_has_to(lib, stream):
    """Small ones once, to save for the arrays in their order, to load for what is formed of the state; one
    that does not fit a pinned page is loaded after the stream's earlier work."""
    gks, stub = lib
    for n, load in ((4, 1), (100, 2)):
        st = _state(gks, stream, n)
        stub.stub_reset()
        blob = st.save()
        assert _stub.count(stub, "waits") == 1
        stub.stub_reset()
        st.load(blob)
        assert _stub.count(stub, "waits") == load
        st.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_a_new_state_copies_twice(lib, stream, precision):
    """The initial data, and the scenarios' values in one block (each copy is some 8 us, a small state's
    initialisation is nothing else)."""
    gks, stub = lib
    sc = workloads.lake_at_rest(4, perturb=1e-2, seed=1)
    mesh = gks.Mesh.from_scenario(sc)
    gks.State.from_scenario(mesh, sc, stream=stream, precision=precision).close()  # the mesh's FP32 tables
    stub.stub_reset()
    st = gks.State.from_scenario(mesh, sc, stream=stream, precision=precision)
    assert _stub.count(stub, "copies") == 2
    st.close()


def test_a_new_mesh_copies_its_ghost_tables_at_once(lib):
    """One allocation and one copy a table, and the ghosts' three in one: 23 copies."""
    gks, stub = lib
    sc = workloads.lake_at_rest(4, perturb=1e-2, seed=1)
    stub.stub_reset()
    mesh = gks.Mesh.from_scenario(sc)
    assert mesh.n_ghost > 0 and _stub.count(stub, "copies") == 23
    mesh.close()

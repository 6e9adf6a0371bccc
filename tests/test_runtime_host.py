"""The library's host code without a GPU: runtime.cpp and networks.cpp linked with a stand-in for the
HIP runtime and the launchers (tests/shim/fake_hip.cpp), for what a call allocates, keeps, copies,
waits for and reports."""

import ctypes as C
import gc
import os
import shutil
import subprocess
import threading

import numpy as np
import pytest

from paper_2608_27612_amd import emr as E
from paper_2608_27612_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_27612_amd", "csrc")
SOURCES = [os.path.join(HERE, "shim", "fake_hip.cpp")] + [
    os.path.join(CSRC, s) for s in ("runtime.cpp", "networks.cpp", "plan.cpp", "pack.cpp", "sched.cpp",
                                    "jit.cpp", "record_file.cpp")]
MB = 1 << 20


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("fake") / "libfake.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-pthread",
                           "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include"]
                          + SOURCES + ["-o", path])
    return path


@pytest.fixture
def lib(built, tmp_path):
    """The binding on a copy of the stand-in library (each with caches of its own), and the stand-in's
    own calls."""
    path = str(tmp_path / "libfake.so")
    shutil.copy(built, path)
    keep = E._lib, E.LIB_PATH
    E._lib, E.LIB_PATH = None, path
    L = E.lib()
    L.emr_set_jit(E.EMR_JIT_OFF)
    for name, (res, args) in {"fake_limit": (None, [C.c_int64]),
                              "fake_hold_events": (None, [C.c_int]),
                              "fake_block_waits": (None, [C.c_int]),
                              "fake_capturing": (None, [C.c_int]), "fake_total": (None, [C.c_int64]),
                              "fake_bind_error": (None, [C.c_uint32]),
                              "fake_totals": (C.c_void_p, []),
                              "fake_held": (C.c_int64, []), "fake_size": (C.c_int64, [C.c_void_p]),
                              "fake_counts": (None, [C.c_void_p])}.items():
        fn = getattr(L, name)
        fn.restype, fn.argtypes = res, args
    yield L
    gc.collect()  # (populations go with the library that made them)
    E._lib, E.LIB_PATH = keep


def counts(lib):
    out = (C.c_int32 * 3)()
    lib.fake_counts(out)
    return dict(zip(("waits", "copies", "slow_copies"), out))


def build(pop, depth, stream=None):
    """emr_build_networks without hidden phases: (status, handle)."""
    src = W.xor_sources()
    h = C.c_void_p()
    st = E.lib().emr_build_networks(pop.handle, src.ctypes.data, len(src), depth, 0.03, 1, 0.1, 0,
                                    C.byref(h), stream)
    return st, h


def phase0(h):
    ph = E.emr_network_phase()
    assert E.lib().emr_networks_phase(h, 0, C.byref(ph)) == 0
    return ph


def test_networks_keep_records_of_the_number_found(lib):
    """A phase's first guess is 64M records (100 CPPNs, 4 sources, depth 10: 140M cells), but the
    handle keeps buffers of the records found, and one of few cells keeps its first buffers."""
    pop = E.emr_pack_population(W.population(1, 100, 6, 12))
    for found in (0, 1000, 3 << 20, 1 << 26):
        lib.fake_total(found)
        st, h = build(pop, 10)
        assert st == 0, lib.emr_last_error()
        ph = phase0(h)
        assert ph.records == found
        # (a buffer from the cache is up to twice the size asked for)
        assert 4 * found <= lib.fake_size(ph.parent) <= max(8 * found, 4096)
        assert 16 * found <= lib.fake_size(ph.w4) <= max(32 * found, 4096)
        lib.emr_free_networks(h)


def test_networks_keep_the_kept_nodes_and_edges(lib):
    """In the stand-in nothing survives pruning: a handle of 4M raw edges keeps no array of them."""
    pop = E.emr_pack_population(W.population(1, 100, 6, 12))
    lib.fake_total(4 << 20)
    st, h = build(pop, 8)
    assert st == 0, lib.emr_last_error()
    i = E.emr_network_info()
    assert lib.emr_networks_info(h, C.byref(i)) == 0
    assert i.edges == 0 and i.nodes == 0
    for p in (i.in_src, i.in_w, i.in_offset, i.node_cell):
        assert lib.fake_size(p) <= 4 * MB
    lib.emr_free_networks(h)


@pytest.mark.parametrize("spare_mb,found,ok", [(900, 1000, True), (2000, 1 << 22, True),
                                               (600, 1000, False), (9000, 1 << 26, True)])
def test_networks_under_little_memory(lib, spare_mb, found, ok):
    """Where the 64M guess (2.7 GB) does not fit, the phase runs with room for 16M records (0.7 GB),
    and reports EMR_E_NOMEM only where that does not fit either."""
    pop = E.emr_pack_population(W.population(1, 100, 6, 12))
    lib.fake_total(found)
    lib.fake_limit(spare_mb * MB)
    st, h = build(pop, 10)
    assert st == (0 if ok else E.EMR_E_NOMEM), lib.emr_last_error()
    if ok:
        assert phase0(h).records == found
        lib.emr_free_networks(h)


def discover(pop, sources, depth, ws):
    """emr_discover with no room for records and the workspace `ws` (a numpy buffer): its status."""
    n = len(sources) * pop.n_genomes
    count, offset = np.zeros(n, np.int64), np.zeros(n + 1, np.int64)
    out = E.emr_result(0, 0, 0, count.ctypes.data, offset.ctypes.data, ws.ctypes.data, ws.size)
    return E.lib().emr_discover(pop.handle, sources.ctypes.data, len(sources), None, len(sources),
                                depth, 0.03, C.byref(out), None)


def workspace(pop, sources, depth):
    n = E.emr_workspace_bytes(pop, sources, depth)
    raw = np.zeros(n + 256, np.uint8)
    at = -raw.ctypes.data % 256
    return raw[at:at + n]


@pytest.mark.parametrize("known", [True, False])
def test_a_table_error_fails_every_call_of_the_plan(lib, known):
    """A table error of the bind kernel: calls made before it is raised (`known` false) fail in their
    check, each of them and whether or not an earlier call was checked; later ones fail at once, raw
    calls among them. Another population's calls do not."""
    pop = E.emr_pack_population(W.population(2, 10, 6, 12))
    src = W.xor_sources()
    a, b, c = (workspace(pop, src, 4) for _ in range(3))
    out = np.zeros(E.emr_grid_count(4)[0] * 4 * 10, np.float32)

    def raw():
        return lib.emr_eval_raw(pop.handle, src.ctypes.data, len(src), None, len(src), 4,
                                out.ctypes.data, c.ctypes.data, c.size, None)

    lib.fake_bind_error(2)
    if not known:
        lib.fake_hold_events(1)
        assert raw() == 0 and discover(pop, src, 4, a) == 0 and discover(pop, src, 4, b) == 0
        lib.fake_hold_events(0)
        for ws in (b, a, c):
            assert lib.emr_call_check(ws.ctypes.data, 0, None, None, None) == E.EMR_E_DEVICE
    for _ in range(2):
        assert discover(pop, src, 4, b) == E.EMR_E_DEVICE
        assert "bind kernel" in lib.emr_last_error().decode()
        assert raw() == E.EMR_E_DEVICE
    lib.fake_bind_error(0)
    other = E.emr_pack_population(W.population(2, 10, 6, 12))
    assert discover(other, src, 4, a) == 0
    assert lib.emr_call_check(a.ctypes.data, 0, None, None, None) == 0


def first_call(pop, sources, depth=3):
    """The first discover call of a population's plan: it uploads the plan's tables."""
    assert discover(pop, sources, depth, workspace(pop, sources, depth)) == 0


def test_a_large_table_replaces_a_small_staging_buffer(lib):
    """Four small uploads in flight make four 1 MB staging buffers; a later table of some MB (2000
    CPPNs, 35 sources) still leaves from staging, without a wait."""
    src = W.tabular_sources(32)
    small = [E.emr_pack_population(W.population(k, 4, 4, 8)) for k in range(5)]
    large = E.emr_pack_population(W.population(9, 2000, 2, 4))
    lib.fake_hold_events(1)
    for p in small[:4]:
        first_call(p, src)
    before = counts(lib)
    first_call(small[4], src)  # all four in flight: copied from the caller's memory, with a wait
    after = counts(lib)
    assert after["slow_copies"] == before["slow_copies"] + 1 and after["waits"] > before["waits"]
    lib.fake_hold_events(0)
    first_call(E.emr_pack_population(W.population(10, 4, 4, 8)), src)
    before = counts(lib)
    first_call(large, src)
    after = counts(lib)
    assert after["copies"] == before["copies"] + 1
    assert after["slow_copies"] == before["slow_copies"]


def test_an_upload_that_waits_holds_up_no_other(lib):
    """While one thread's upload waits for its stream (all staging in flight), another thread's, which
    finds an idle buffer, goes through."""
    src = W.tabular_sources(32)
    pops = [E.emr_pack_population(W.population(k, 4, 4, 8)) for k in range(6)]
    lib.fake_hold_events(1)
    for p in pops[:4]:
        first_call(p, src)
    lib.fake_block_waits(1)
    waiting = threading.Thread(target=first_call, args=(pops[4], src))
    other = threading.Thread(target=first_call, args=(pops[5], src))
    slow = counts(lib)["slow_copies"]
    try:
        waiting.start()
        while counts(lib)["slow_copies"] == slow:
            assert waiting.is_alive()
        lib.fake_hold_events(0)
        other.start()
        other.join(20)
        assert not other.is_alive() and waiting.is_alive()
    finally:
        lib.fake_hold_events(0)
        lib.fake_block_waits(0)
        waiting.join()
        other.join()


def test_band_values_refuse_a_capture(lib):
    """The call uploads a table: recorded into a graph, the copy would read the staging buffer at
    every replay, which later calls have rewritten."""
    src = W.xor_sources()
    pop = E.emr_pack_population(W.population(3, 4, 4, 8))
    first_call(pop, src)
    n = 4 * len(src)
    b = C.c_int64()
    assert lib.emr_band_workspace_bytes(n, C.byref(b)) == 0
    raw = np.zeros(b.value + 256, np.uint8)
    ws = raw[-raw.ctypes.data % 256:]
    offset = np.zeros(n + 1, np.int64)
    conn = E.emr_connections(0, 0, 0, 0, offset.ctypes.data, 0, 0)

    def call():
        return lib.emr_band_values(pop.handle, src.ctypes.data, len(src), None, len(src), 3,
                                   C.byref(conn), None, ws.ctypes.data, b.value, None)

    lib.fake_capturing(1)
    before = counts(lib)
    assert call() == E.EMR_E_DEVICE and counts(lib) == before
    lib.fake_capturing(0)
    assert call() == 0 and counts(lib) != before


def test_counters_lie_with_the_plan(lib):
    """A record call's totals lie in the plan's memory and start at zero whatever the workspace holds
    (the stand-in's launch checks that, and leaves totals behind); calls on other streams, with the
    earlier ones in flight, have sets of their own; a capture, which may be replayed beside later
    calls, has the workspace's, cleared by the call."""
    src = W.xor_sources()
    pop = E.emr_pack_population(W.population(4, 50, 6, 12))
    ws = workspace(pop, src, 5)

    def call(stream=None):
        ws.fill(0xAB)
        n = len(src) * pop.n_genomes
        count, offset = np.zeros(n, np.int64), np.zeros(n + 1, np.int64)
        out = E.emr_result(0, 0, 0, count.ctypes.data, offset.ctypes.data, ws.ctypes.data, ws.size)
        assert lib.emr_discover(pop.handle, src.ctypes.data, len(src), None, len(src), 5, 0.03,
                                C.byref(out), stream) == 0, lib.emr_last_error()
        at = lib.fake_totals()
        return at, ws.ctypes.data <= at < ws.ctypes.data + ws.size

    own = [call() for _ in range(4)]
    assert not any(inside for _, inside in own)
    assert own[0][0] == own[2][0] != own[1][0] == own[3][0]  # two sets of totals in turn
    lib.fake_hold_events(1)
    seen = set()
    for k in range(12):  # eight sets; the other calls' streams wait for an earlier call's
        a, inside = call(C.c_void_p(1000 + k))
        assert not inside
        seen.add(a)
    assert 8 <= len(seen) <= 12
    lib.fake_hold_events(0)
    lib.fake_capturing(1)
    assert all(call()[1] for _ in range(2))
    lib.fake_capturing(0)
    assert not call()[1]

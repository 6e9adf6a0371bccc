"""The library's host code without a GPU: runtime.cpp and networks.cpp linked with a stand-in for the
HIP runtime and the launchers (tests/shim/fake_hip.cpp), for what a call allocates, keeps, copies,
waits for and reports."""

import ctypes as C
import gc
import os
import shutil
import subprocess

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
                              "fake_capturing": (None, [C.c_int]), "fake_total": (None, [C.c_int64]),
                              "fake_bind_error": (None, [C.c_uint32]),
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

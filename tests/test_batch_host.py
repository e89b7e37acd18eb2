"""Host code of batches (rx_batch.cpp) on the CPU, against a HIP runtime that records the graph instead of running it
(tests/batch_host_stub.cpp)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1901_07499_amd import build, rx

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RESET, MERGED_DEM, MERGED_EST, CLASS_DEM, CLASS_EST = 0, range(1, 5), range(5, 9), range(9, 15), range(30, 36)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("batch") / "libbatchhost.so")
    rocm = os.path.dirname(os.path.dirname(build.hipcc()))
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I", os.path.join(rocm, "include"), "-o", out, os.path.join(ROOT, "tests", "batch_host_stub.cpp"),
                    os.path.join(ROOT, "paper_1901_07499_amd", "csrc", "rx_batch.cpp")], check=True)
    return ctypes.CDLL(out)


class Batch:
    """A batch of (antennas, FFT length, used subcarriers, symbols) frames on the recording runtime."""

    def __init__(self, lib, frames):
        self.lib, self.n = lib, len(frames)
        arr = (rx.rx_params * self.n)()
        pilot = np.ones(4096, np.float32)
        for a, (A, N, U, T) in zip(arr, frames):
            a.n_ant, a.fft_len, a.cp_len, a.n_used, a.n_sym, a.bits_per_sym = A, N, 0, U, T, 4
            a.pilot = pilot.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
        self.h = ctypes.c_void_p()
        assert lib.rx_batch_create(arr, self.n, ctypes.byref(self.h)) == 0

    def process(self, base=256):
        p = [ctypes.c_void_p(base * k) for k in (1, 2, 3, 4)]
        assert self.lib.rx_batch_process(self.h, p[0], p[1], p[2], p[3], None, None) == 0
        nodes = []
        for i in range(self.lib.stub_nodes()):
            v = (ctypes.c_int64 * 6)()
            self.lib.stub_node(i, v)
            nodes.append(dict(kernel=v[0], grid=v[1], block=v[2], lds=v[3], tiles=v[4],
                              deps=[self.lib.stub_dep(i, k) for k in range(v[5])]))
        return nodes

    def config(self, N):
        v = [ctypes.c_int32() for _ in range(4)]
        assert self.lib.rx_batch_config(self.h, N, ctypes.byref(v[0]), ctypes.byref(v[1])) == 0
        assert self.lib.rx_batch_schedules(self.h, N, ctypes.byref(v[2]), ctypes.byref(v[3])) == 0
        return tuple(x.value for x in v)

    def close(self):
        self.lib.rx_batch_destroy(self.h)


MIXED = [(8, 64, 52, 4), (8, 64, 16, 4), (3, 1024, 600, 14), (5, 2048, 1900, 3), (64, 256, 180, 2)]


@pytest.mark.parametrize("frames", [[(8, 64, 16, 4)], MIXED])
def test_every_kernel_follows_the_reset(lib, frames):
    # frame completion times count from the stamp that the reset kernel sets, so no work may precede it
    b = Batch(lib, frames)
    nodes = b.process()
    assert nodes[0]["kernel"] == RESET and not nodes[0]["deps"]
    after = {0}
    for i, n in enumerate(nodes[1:], 1):
        assert after & set(n["deps"]), n
        after.add(i)
        if n["kernel"] in MERGED_DEM:               # every demod waits for an estimate kernel of its frames
            assert any(nodes[d]["kernel"] == n["kernel"] - MERGED_DEM[0] + MERGED_EST[0] for d in n["deps"])
    b.close()


@pytest.mark.parametrize("frames,T,demods", [(65536, 256, 1), (65536, 257, 2), (65536, 600, 3)])
def test_launches_hold_fewer_threads_than_the_runtime_takes(lib, frames, T, demods):
    b = Batch(lib, [(1, 64, 4, T)] * frames)
    nodes = [n for n in b.process() if n["kernel"] in MERGED_DEM]
    assert len(nodes) == demods
    assert all(0 < n["grid"] * n["block"] < 1 << 32 for n in nodes)
    assert sum(n["grid"] for n in nodes) == frames * (T - 1)
    for p, n in zip(nodes, nodes[1:]):              # the tiles continue where the launch before ended
        assert n["tiles"] == p["tiles"] + 8 * p["grid"]
    b.close()


def _kinds(nodes):
    return {"merged" if n["kernel"] in MERGED_DEM or n["kernel"] in MERGED_EST else "class" for n in nodes[1:]}


@pytest.mark.parametrize("cfg", [(4, 4, 0, 0), (8, 2, 0, 0)])
def test_configuration_says_what_runs(lib, cfg):
    lens = sorted({f[1] for f in MIXED})
    b = Batch(lib, MIXED)
    nodes = b.process()
    assert _kinds(nodes) == {"merged"}
    waves = {n["block"] // 64 for n in nodes if n["kernel"] in MERGED_DEM}
    assert {b.config(N)[0] for N in lens} == waves and {b.config(N)[1:] for N in lens} == {(2, 0, 0)}
    for N in lens:                                  # a configuration that is set is the one that runs
        assert lib.rx_batch_set_config(b.h, N, *cfg) == 0
    nodes = b.process()
    assert _kinds(nodes) == {"class"} and {b.config(N) for N in lens} == {cfg}
    assert {n["block"] for n in nodes if n["kernel"] in CLASS_DEM} == {64 * cfg[0]}
    assert lib.rx_batch_set_config(b.h, 64, 3, 4, 0, 0) != 0 and b.config(64) == cfg
    b.close()


def test_set_config_of_one_length_leaves_the_others_at_their_default(lib):
    b = Batch(lib, MIXED)
    assert lib.rx_batch_set_config(b.h, 1024, 2, 8, 1, 0) == 0
    assert _kinds(b.process()) == {"class"}
    assert b.config(1024) == (2, 8, 1, 0) and b.config(2048) == (4, 4, 0, 0)
    b.close()


@pytest.mark.parametrize("merged_ms,kind", [(1.005, "merged"), (1.02, "class")])
def test_autotune_keeps_the_faster_kernels(lib, merged_ms, kind):
    b = Batch(lib, MIXED)
    lib.stub_set_merged_ms(ctypes.c_float(merged_ms))
    p = [ctypes.c_void_p(256 * k) for k in (1, 2, 3, 4)]
    assert lib.rx_batch_autotune(b.h, p[0], p[1], p[2], p[3], None, 2, None) == 0
    lib.stub_set_merged_ms(ctypes.c_float(1.0))
    assert _kinds(b.process()) == {kind}
    assert (b.config(64)[1] == 2) or kind == "class"
    b.close()


def test_lds_allowance_does_not_depend_on_the_batch(lib):
    # kernels are shared by all batches of the process: a later, smaller batch must not lower what an earlier one needs
    big = Batch(lib, [(130, 2048, 1200, 4), (130, 64, 62, 4)])
    dem = [n for n in big.process() if n["kernel"] in MERGED_DEM]
    assert max(n["lds"] for n in dem) > 65536
    small = Batch(lib, [(130, 2048, 1200, 4), (130, 64, 50, 4)])
    small.process()
    for n in big.process(base=4096):                # rebuilt on other buffers
        if n["lds"] > 65536:
            assert n["lds"] <= lib.stub_lds(n["kernel"])
    big.close()
    small.close()

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

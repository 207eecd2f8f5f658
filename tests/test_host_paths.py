"""Error paths and host memory of the library's host code (CPU).

A stand-in for the HIP runtime (hip_host_stub.cpp) is compiled with g++ and
loaded in front of librlbm.so in a process of its own; each check below is a
function that runs there."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class Host:
    """Lattices in host memory behind the stand-in."""

    def __init__(self, stub):
        self.stub = ctypes.CDLL(stub, mode=ctypes.RTLD_GLOBAL)
        self.stub.stub_pinned.restype = ctypes.c_size_t
        self.stub.stub_pinned_limit.argtypes = [ctypes.c_size_t]
        for f in ("stub_queued", "stub_waits", "stub_frees", "stub_blocks", "stub_replays"):
            getattr(self.stub, f).restype = ctypes.c_long
        self.stub.stub_fail_launch.argtypes = [ctypes.c_long]
        sys.path.insert(0, ROOT)
        from paper_2108_07605_amd import rlbm, workloads as wl
        self.rlbm, self.wl, self.L = rlbm, wl, rlbm.lib()
        self.mech9 = wl.mechanism_h2air9()
        self.mech = rlbm.Mechanism(self.mech9)

    def lattice(self, nx, storage="f32dev", **kw):
        """(handle, memory, case) of a tube of nx nodes."""
        case = self.wl.make_case("tube", nx=nx, mech=self.mech9, **kw)
        d, keep = self.rlbm.lattice_desc(case, storage)
        n = self.rlbm.lattice_bytes(case, self.mech, storage)
        mem = np.zeros(n + 256, np.uint8)
        h = ctypes.c_void_p()
        self.rlbm._check(self.L.rlbm_lattice_create(ctypes.byref(d), self.mech.handle, (mem.ctypes.data + 255) & ~255, n,
                                                    None, ctypes.byref(h)))
        return h, mem, case

    def set_state(self, h, case):
        arrs = [np.ascontiguousarray(case["init"][k], dtype=np.float64) for k in ("rho", "u", "T", "Y")]
        return self.L.rlbm_set_state(h, *[a.ctypes.data for a in arrs], 0)


def check_pinned_memory_by_size(host):
    """A lattice holds pinned memory for its own small fields only."""
    held = host.lattice(30000)
    at = host.stub.stub_pinned()
    for nx, most in ((64, 16 << 10), (1024, 256 << 10), (4369, 513 << 10), (4370, 4 << 10), (20000, 4 << 10)):
        h, _mem, _ = host.lattice(nx)
        assert host.stub.stub_pinned() - at <= most, nx
        host.L.rlbm_lattice_destroy(h)
        at = host.stub.stub_pinned()   # what is kept is used again by a lattice of its size
        h, _mem, _ = host.lattice(nx)
        assert host.stub.stub_pinned() == at
        host.L.rlbm_lattice_destroy(h)
    host.L.rlbm_lattice_destroy(held[0])


def check_creation_without_staging(host):
    """Where no larger pinned block can be had, lattices are created without
    staging; their states are still taken."""
    host.stub.stub_pinned_limit(4096)
    for nx in (64, 4369, 5000):
        h, _mem, case = host.lattice(nx)
        assert host.set_state(h, case) == 0
        assert host.stub.stub_queued() == 0
        host.L.rlbm_lattice_destroy(h)


def check_destroy_frees_no_pinned_memory(host):
    """A free waits for the whole device: destroying lattices, the last one
    among them, leaves up to 2 MiB of blocks for the next ones, and the last
    mechanism gives those back."""
    for rounds in range(2):
        hs = [host.lattice(nx) for nx in [64] * 40 + [300] * 8 + [4000]]
        at = host.stub.stub_frees()
        for h, _mem, _ in hs:
            host.L.rlbm_lattice_destroy(h)
        assert host.stub.stub_frees() == at
        assert host.stub.stub_pinned() <= 2 << 20
    hs = [host.lattice(4000) for _ in range(9)]
    for h, _mem, _ in hs:
        host.L.rlbm_lattice_destroy(h)
    assert host.stub.stub_pinned() <= 2 << 20
    held, _mem, _ = host.lattice(64)
    host.mech.__del__()
    host.L.rlbm_lattice_destroy(held)
    assert host.stub.stub_pinned() == 0


def check_failed_set_state_leaves_no_copy_queued(host):
    """A state whose kernels cannot be launched is refused with no copy from
    the caller's arrays or the call's own still on its way."""
    for storage, kernels in (("f64", 1), ("f32dev", 3)):
        for nx in (64, 5000):
            h, _mem, case = host.lattice(nx, storage)
            for n in range(kernels):
                host.stub.stub_fail_launch(n)
                assert host.set_state(h, case) == -3, (storage, nx, n)
                assert host.stub.stub_queued() == 0, (storage, nx, n)
            host.stub.stub_fail_launch(-1)
            assert host.set_state(h, case) == 0
            host.L.rlbm_lattice_destroy(h)


def check_snapshots_wait_once(host):
    """Saving and loading a snapshot queue their copies and wait for them at
    the end (and for the lattice's own work, and a loaded header), however
    many sections there are."""
    for storage in ("f64", "f32dev"):
        for kw in ({}, {"reaction": "implicit"}):
            for nx in (4, 100):     # copied section by section, and packed
                h, _mem, case = host.lattice(nx, storage, **kw)
                assert host.set_state(h, case) == 0
                n = ctypes.c_size_t()
                host.rlbm._check(host.L.rlbm_state_bytes(h, ctypes.byref(n)))
                a = np.zeros(n.value, np.uint8)
                for f, most in ((host.L.rlbm_save_state, 2), (host.L.rlbm_load_state, 3)):
                    at = host.stub.stub_waits()
                    host.rlbm._check(f(h, a.ctypes.data, 0))
                    assert host.stub.stub_waits() - at <= most, (storage, kw, nx)
                    assert host.stub.stub_queued() == 0
                host.L.rlbm_lattice_destroy(h)


def check_finished_lattices_take_no_blocks(host):
    """Joint steps of a long tube (1 step) and two short ones: the long one's
    tiles are in the grids of its step only, wherever it stands in the batch."""
    tiles = lambda n: (n + 63) // 64                     # noqa: E731
    for sizes, steps in (((64000, 64, 128), (1, 40, 37)), ((128, 64000, 64), (37, 1, 40)), ((64, 128, 64000), (40, 37, 0))):
        hs = [host.lattice(nx) for nx in sizes]
        for h, _mem, case in hs:
            assert host.set_state(h, case) == 0
        k = len(hs)
        lats = (ctypes.c_void_p * k)(*[h.value for h, _, _ in hs])
        st = (ctypes.c_int64 * k)(*steps)
        n = ctypes.c_size_t()
        host.rlbm._check(host.L.rlbm_batch_bytes(k, ctypes.byref(n)))
        mem = np.zeros(n.value + 256, np.uint8)
        b = ctypes.c_void_p()
        host.rlbm._check(host.L.rlbm_batch_create(lats, k, (mem.ctypes.data + 255) & ~255, n.value, ctypes.byref(b)))
        # k_boundary: an inlet and an outlet node per tube, a block; k_species and k_flow: a block per tile
        want = sum(s * (1 + 2 * tiles(nx)) for nx, s in zip(sizes, steps))
        at = host.stub.stub_blocks()
        host.rlbm._check(host.L.rlbm_batch_step(b, st))
        assert host.stub.stub_blocks() - at == want and host.stub.stub_replays() == 0
        at = host.stub.stub_blocks()
        host.rlbm._check(host.L.rlbm_step_group(lats, k, st))
        assert host.stub.stub_blocks() - at == want + k     # and the table kernel's
        host.L.rlbm_batch_destroy(b)
        for h, _mem, _ in hs:
            host.L.rlbm_lattice_destroy(h)


CHECKS = {n: f for n, f in list(globals().items()) if n.startswith("check_")}


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "libhip_host_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_host_stub.cpp"), "-o", out],
                   check=True)
    return out


@pytest.mark.parametrize("name", sorted(CHECKS))
def test_host_path(stub, name):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    CHECKS[sys.argv[2]](Host(sys.argv[1]))

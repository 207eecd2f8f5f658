"""Host calls of the library around captures, transfers and snapshots."""
import ctypes

import numpy as np
import pytest

from paper_2108_07605_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _rlbm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2108_07605_amd import rlbm
    return rlbm


def test_lattices_are_destroyed_during_a_capture(mech9):
    """Steps captured in a graph while twelve other lattices are destroyed,
    more than the library keeps blocks of: the capture stays valid, and every
    replay takes the steps."""
    rlbm = _rlbm()
    import torch
    print("case destroy during a capture", flush=True)
    m = rlbm.Mechanism(mech9)
    case = wl.make_case("tube", seed=11, mech=mech9, nx=70)
    side = torch.cuda.Stream()
    lat, ref = rlbm.Lattice(case, mech=m, stream=side).set_state(), rlbm.Lattice(case, mech=m).set_state()
    small = wl.make_case("reactor", seed=1, mech=mech9, nx=16, ny=16, nz=16)
    others = [rlbm.Lattice(small, mech=m).set_state() for _ in range(12)]
    lat.step(2)
    ref.step(2)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        lat.step(2)
        for o in others:
            rlbm.lib().rlbm_lattice_destroy(o.handle)
            o.handle = None
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        ref.step(2)
        np.testing.assert_array_equal(lat.populations(), ref.populations())

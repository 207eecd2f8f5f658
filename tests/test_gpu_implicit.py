"""The linearly implicit reaction update in both storages, against the oracle.

Tolerances: those of test_gpu_tiles.  FP64 storage 1e-10 in the populations
after up to four steps (rounding differences only); FP32 deviation storage its
precision target, 1e-5 in T and Y.  A population decoded with another scale
than the one it was encoded with is off by the change of a density over a step,
which these states make percents of.
"""
import numpy as np
import pytest

from oracle import Oracle
from paper_2108_07605_amd import workloads as wl
from test_gpu_tiles import TOL, _case, _nerr, _rlbm, _three_body

pytestmark = pytest.mark.gpu


def _compare(lat, ora, species, storage, ctx):
    gf, of = lat.fields(), ora.fields()
    if storage == "f64":
        gp, op = lat.populations(), ora.populations()
        for l in range(op.shape[0]):
            assert _nerr(gp[l], op[l]) <= 1e-10, (ctx, l)
    tol = 1e-10 if storage == "f64" else TOL[storage]
    assert _nerr(gf["T"], of["T"]) <= tol, ctx
    for a in range(species):
        assert _nerr(gf["Y"][a], of["Y"][a], 1e-6) <= tol, (ctx, a)


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("species,coupling,dims,substeps", [
    (9, "strong", (1, 1, 1), 1), (9, "strong", (63, 1, 1), 3), (9, "weak", (65, 1, 1), 2), (9, "strong", (64, 2, 1), 2),
    (9, "weak", (5, 13, 3), 2), (3, "strong", (257, 1, 1), 1), (3, "weak", (11, 3, 2), 4), (2, "strong", (66, 1, 1), 1),
    (2, "weak", (3, 5, 7), 1), (4, "strong", (64, 1, 1), 3), (4, "weak", (17, 4, 1), 1)])
def test_implicit_step_at_tile_edges(species, coupling, dims, substeps, storage, mech9):
    """One, two and five steps: both buffers' scales decode and encode."""
    rlbm = _rlbm()
    print(f"case implicit step M={species} {coupling} {dims} l={substeps} {storage}", flush=True)
    case = _case(species, dims, mech9, coupling, substeps=substeps)
    case["reaction"] = "implicit"
    if species == 3:
        case["mech"] = _three_body(case["mech"])
        case["init"]["Y"][2] = 0.05
        case["init"]["Y"][1] -= 0.05
    lat, ora = rlbm.Lattice(case, storage=storage).set_state(), Oracle(case)
    done = 0
    for n in (1, 2, 5):
        lat.step(n - done)
        ora.step(n - done)
        done = n
        _compare(lat, ora, species, storage, n)
    assert lat.status() == 0


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("coupling", ["strong", "weak"])
@pytest.mark.parametrize("name,dims,steps", [("channel2d", (20, 19, 1), (3, 4)), ("channel3d", (9, 11, 9), (2, 3))])
def test_implicit_channels(name, dims, steps, coupling, storage, mech9):
    """Inlet, outlet and walls, after an odd and an even number of steps."""
    rlbm = _rlbm()
    print(f"case implicit {name} {dims} {coupling} {storage}", flush=True)
    case = wl.make_case(name, nx=dims[0], ny=dims[1], nz=dims[2], mech=mech9, coupling=coupling, reaction="implicit")
    lat, ora = rlbm.Lattice(case, storage=storage).set_state(), Oracle(case)
    done = 0
    for n in steps:
        lat.step(n - done)
        ora.step(n - done)
        done = n
        _compare(lat, ora, 9, storage, n)


@pytest.mark.parametrize("coupling", ["strong", "weak"])
def test_implicit_snapshot_resumes_bit_exactly(coupling, mech9):
    """A run saved after an odd number of steps and one resumed from it in a
    lattice of the other buffer parity stay the same bits."""
    rlbm = _rlbm()
    print(f"case implicit snapshot {coupling}", flush=True)
    case = wl.make_case("channel2d", nx=33, ny=9, nz=1, mech=mech9, coupling=coupling, reaction="implicit")
    lat = rlbm.Lattice(case, storage="f32dev").set_state()
    lat.step(5)
    back = rlbm.Lattice(case, storage="f32dev").set_state()
    back.step(2)
    back.load_state(lat.save_state())
    np.testing.assert_array_equal(back.populations(), lat.populations())
    back.step(3)
    lat.step(3)
    np.testing.assert_array_equal(back.populations(), lat.populations())


@pytest.mark.parametrize("coupling", ["strong", "weak"])
@pytest.mark.parametrize("species", [9, 3, 2])
def test_snapshots_between_the_updates(species, coupling, mech9):
    """A lattice takes a snapshot of the other reaction update's lattice (a
    linearly implicit one keeps the scales of f and g in the species' row where
    they fit, an explicit one apart): the same populations, the same bits in
    the next snapshot's, and runs within the storage's precision of the FP64
    ones."""
    rlbm = _rlbm()
    print(f"case snapshots between updates M={species} {coupling}", flush=True)
    ex = _case(species, (66, 5, 3), mech9, coupling)
    im = dict(ex, reaction="implicit")
    for a, b in ((ex, im), (im, ex)):
        lat = rlbm.Lattice(a, storage="f32dev").set_state()
        lat.step(3)
        other = rlbm.Lattice(b, storage="f32dev").set_state()
        f64 = rlbm.Lattice(b, storage="f64").set_state()
        snap = lat.save_state()
        row = (lat.L + 3) // 4 == (lat.L + 1) // 4     # f and g fit in the species' row of scales
        assert snap[:8].view(np.uint32)[1] == (1 if a is im and row else 2)
        other.load_state(snap)
        pops = lat.populations()
        np.testing.assert_array_equal(other.populations(), pops)
        f64.write_populations(pops)
        back = rlbm.Lattice(a, storage="f32dev").load_state(other.save_state())
        np.testing.assert_array_equal(back.populations(), pops)
        for n in (1, 2):
            other.step(n)
            f64.step(n)
            _fields_close(other, f64, species)


def _fields_close(lat, f64, species):
    a, b = lat.fields(), f64.fields()
    assert _nerr(a["T"], b["T"]) <= TOL["f32dev"]
    for s in range(species):
        assert _nerr(a["Y"][s], b["Y"][s], 1e-6) <= TOL["f32dev"], s


@pytest.mark.parametrize("coupling", ["strong", "weak"])
def test_step_after_written_populations(coupling, mech9):
    """FP32 storage: populations of a state far from the lattice's own are
    rounded once when they are written.  The step after encodes with scales of
    their own size, so its deviations are small and their rounding too; scales
    left from the old state would round every population a second time as
    coarsely, an error of sqrt(2) times the first where the other way leaves
    it as it is.  The line is at the root of that, 2^(1/4)."""
    rlbm = _rlbm()
    base = wl.make_case("bbbox", seed=2, mech=mech9, nx=16, ny=8, nz=6, coupling=coupling, reaction="implicit")
    print(f"case step after written populations {coupling}", flush=True)
    _after_write(rlbm, base)


def _after_write(rlbm, base):
    rng = np.random.default_rng(5)
    init = {k: np.array(v, dtype=np.float64) for k, v in base["init"].items()}
    N = init["rho"].size
    Y = init["Y"].reshape(9, N)
    sl = int(np.argmax(Y.mean(1)))
    base["slaved"] = sl
    Y = Y * np.exp(0.7 * rng.uniform(-1.0, 1.0, (9, 1))) + 1e-3
    Y /= Y.sum(0)
    Y[sl] += 1.0 - Y.sum(0)
    init.update(Y=Y.reshape(init["Y"].shape), T=1.1 * init["T"], rho=1.2 * init["rho"])
    pops = rlbm.Lattice(base, storage="f64").set_state(init).populations()
    f64, f32 = (rlbm.Lattice(base, storage=s).set_state() for s in ("f64", "f32dev"))
    f64.write_populations(pops)
    f32.write_populations(pops)

    def err():
        p, q = f64.populations(), f32.populations()
        return max(np.sqrt(((p[l] - q[l]) ** 2).mean() / (p[l] ** 2).mean()) for l in range(p.shape[0]))

    first = err()
    for n in (1, 2):
        f64.step(1)
        f32.step(1)
        assert err() <= 2.0 ** 0.25 * first, n

"""Kernels at the edges of their tiles, against the oracle.

The kernels take 64 nodes per tile (the invariants 256 per block); a lattice
that ends inside, at or just past a tile exercises their remainders.

Tolerances.  FP64 storage: sums of 27 populations and a Newton solve differ
from the oracle's only in rounding order, about 30 roundings of 1.1e-16 each,
amplified in T by the ratio of the formation energies to c_v T (below 100):
1e-11.  FP32 deviation storage: its precision target, 1e-5.
"""
import numpy as np
import pytest

from oracle import Oracle
from paper_2108_07605_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-11, "f32dev": 1e-5}


def _rlbm():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2108_07605_amd import rlbm
    return rlbm


def _nerr(a, b, floor=0.0):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), floor, 1e-300))


def _mech(species, mech9):
    return {2: None, 3: wl.mechanism_abc(), 4: wl.mechanism_abcd(), 9: mech9}[species]


def _case(species, dims, mech9, coupling="strong", **kw):
    """A periodic box of the given size with seeded modes in every field."""
    name = {2: "binary", 9: "bbbox"}.get(species, "abc_box")
    m = _mech(species, mech9)
    kw = dict(kw, **({"mech": m} if m else {}))
    c = wl.make_case(name, nx=dims[0], ny=dims[1], nz=dims[2], coupling=coupling, **kw)
    c["faces"] = wl.periodic_faces()
    rng = np.random.default_rng([7, species, *dims])
    c["init"]["u"] = 1e-2 * rng.uniform(-1.0, 1.0, c["init"]["u"].shape)
    c["init"]["T"] = c["init"]["T"] * (1.0 + 0.05 * rng.uniform(-1.0, 1.0, c["init"]["T"].shape))
    return c


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("species,coupling,dims", [
    (9, "strong", (1, 1, 1)), (9, "strong", (63, 1, 1)), (9, "weak", (64, 1, 1)), (9, "strong", (13, 5, 1)),
    (3, "strong", (16, 4, 4)), (3, "weak", (257, 1, 1)), (2, "strong", (51, 5, 1)), (4, "weak", (7, 11, 13))])
def test_readout_at_tile_edges(species, coupling, dims, storage, mech9):
    """Initial populations, fields, invariants and a round trip of the
    populations."""
    rlbm = _rlbm()
    print(f"case readout M={species} {coupling} {dims} {storage}", flush=True)
    case = _case(species, dims, mech9, coupling)
    lat, ora = rlbm.Lattice(case, storage=storage).set_state(), Oracle(case)
    tol = TOL[storage]
    gp, op = lat.populations(), ora.populations()
    for l in range(op.shape[0]):
        assert _nerr(gp[l], op[l]) <= tol, l
    gf, of = lat.fields(), ora.fields()
    for k in ("rho", "T", "P"):
        assert _nerr(gf[k], of[k]) <= tol, k
    assert _nerr(gf["u"], of["u"]) <= tol
    for a in range(species):
        assert _nerr(gf["Y"][a], of["Y"][a], 1e-6) <= tol, a
    gi, oi = lat.invariants(), ora.invariants()
    scale = np.abs(op).sum()
    assert np.abs(gi[:-1] - oi[:-1]).max() <= tol * scale and gi[-1] == 0.0
    if storage == "f64":
        lat.write_populations(gp[:, ::-1].copy())
        assert np.array_equal(lat.populations(), gp[:, ::-1])


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
def test_invariants_flag_any_velocity(storage, mech9):
    """A single non-finite population raises the flag, whichever wave of the
    block sums it and wherever its node lies in the block."""
    rlbm = _rlbm()
    print(f"case invariants flag {storage}", flush=True)
    case = _case(9, (259, 1, 1), mech9)
    lat = rlbm.Lattice(case, storage=storage).set_state()
    pops = lat.populations()
    for l, i, n in ((0, 0, 0), (3, 13, 64), (8, 26, 258), (9, 9, 255)):
        bad = pops.copy()
        bad[l, i, n] = np.nan
        lat.write_populations(bad)
        assert lat.invariants()[-1] == 1.0, (l, i, n)
    lat.write_populations(pops)
    assert lat.invariants()[-1] == 0.0


def _three_body(mech):
    """The one-reaction mechanism with a reversible three-molecule reaction
    A + B + C <-> 3 C and one that is switched off (ln A = -inf)."""
    m = dict(mech)
    m["nu_f"] = [*mech["nu_f"], [1, 1, 1], [1, 1, 0]]
    m["nu_r"] = [*mech["nu_r"], [0, 0, 3], [0, 0, 2]]
    m["lnA"] = [*mech["lnA"], mech["lnA"][0] - 1.0, -np.inf]
    m["beta"] = [*mech["beta"], 0.5, 0.0]
    m["Ta"] = [*mech["Ta"], 0.5 * mech["Ta"][0], 100.0]
    m["reversible"] = [*mech["reversible"], 1, 1]
    return m


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("species,coupling,dims,substeps", [
    (9, "strong", (1, 1, 1), 1), (9, "strong", (63, 1, 1), 3), (9, "weak", (65, 1, 1), 2), (9, "strong", (64, 2, 1), 2),
    (9, "strong", (5, 13, 3), 2), (3, "strong", (257, 1, 1), 1), (3, "weak", (11, 3, 2), 4), (2, "strong", (66, 1, 1), 1),
    (2, "weak", (3, 5, 7), 1), (4, "strong", (64, 1, 1), 3), (4, "weak", (17, 4, 1), 1)])
def test_step_at_tile_edges(species, coupling, dims, substeps, storage, mech9):
    """One and four steps with every species count, both couplings and
    several sub-step counts; the three-species mechanism with more than two
    molecules on a side.  FP64: 1e-10, the rounding differences of the
    readout times the steps; FP32: 1e-5 in Y and T."""
    rlbm = _rlbm()
    print(f"case step M={species} {coupling} {dims} l={substeps} {storage}", flush=True)
    case = _case(species, dims, mech9, coupling, substeps=substeps)
    if species == 3:
        case["mech"] = _three_body(case["mech"])
        case["init"]["Y"][2] = 0.05
        case["init"]["Y"][1] -= 0.05
    lat, ora = rlbm.Lattice(case, storage=storage).set_state(), Oracle(case)
    done = 0
    for n in (1, 4):
        lat.step(n - done)
        ora.step(n - done)
        done = n
        gf, of = lat.fields(), ora.fields()
        if storage == "f64":
            gp, op = lat.populations(), ora.populations()
            for l in range(op.shape[0]):
                assert _nerr(gp[l], op[l]) <= 1e-10, (n, l)
        tol = 1e-10 if storage == "f64" else TOL[storage]
        assert _nerr(gf["T"], of["T"]) <= tol
        for a in range(species):
            assert _nerr(gf["Y"][a], of["Y"][a], 1e-6) <= tol, a
    assert lat.status() == 0


@pytest.mark.parametrize("storage,coupling", [("f64", "strong"), ("f32dev", "strong"), ("f32dev", "weak")])
def test_first_snapshot_format_still_loads(storage, coupling, mech9):
    """A snapshot in the first format (one scale vector per node, no second
    copy of the reference shapes) holds the same populations, and a run
    resumed from it stays with the run it was taken from."""
    rlbm = _rlbm()
    print(f"case snapshot v1 {storage} {coupling}", flush=True)
    case = wl.make_case("channel2d", nx=33, ny=9, nz=1, mech=mech9, coupling=coupling)
    lat = rlbm.Lattice(case, storage=storage).set_state()
    lat.step(5)
    snap, N, L, M = lat.save_state(), lat.N, lat.L, 9
    pops = lat.populations()
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    head = snap[:256].copy()
    ints = head.view(np.int32)
    assert ints[1] == 2
    ints[1] = 1
    if storage == "f64":
        old = snap.copy()
        old[:256] = head
    else:
        rss, rss1, nsp = int(ints[6]), (L + 3) // 4 * 4, L - 2
        n_ref1 = (L * 27 + L + 27 + 2) * 8
        n_ref = n_ref1 + L * 27 * 8
        P = (N + lat.n_interface + 63) // 64 * 64
        n_pops, n_sc = L * 27 * P * 4, rss * N * 4
        o = up(256 - 255)
        ref = snap[o:o + n_ref1]; o = up(o + n_ref)
        body = snap[o:o + n_pops]; o = up(o + n_pops)
        sc = snap[o:o + n_sc].view(np.float32).reshape(N, rss); o = up(up(o + n_sc) + n_sc)
        fs = snap[o:o + 8 * N].view(np.float32).reshape(N, 2); o = up(o + 8 * N)
        rest = snap[o:]
        one = np.zeros((N, rss1), np.float32)
        one[:, :nsp], one[:, nsp:L] = sc[:, :nsp], fs
        ints[6] = rss1
        pad = lambda b: np.concatenate([b, np.zeros(up(len(b)) - len(b), np.uint8)])  # noqa: E731
        old = np.concatenate([pad(head), pad(ref), pad(body), pad(one.reshape(-1).view(np.uint8)), rest])
    back = rlbm.Lattice(case, storage=storage).load_state(old)
    assert np.array_equal(back.populations(), pops)
    back.step(6)
    lat.step(6)
    a, b = back.fields(), lat.fields()
    for k in ("T", "rho"):
        assert _nerr(a[k], b[k]) <= TOL[storage], k
    for s in range(M):
        assert _nerr(a["Y"][s], b["Y"][s], 1e-6) <= TOL[storage], s


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("name,dims,coupling", [
    ("channel2d", (20, 19, 1), "strong"),      # 17 inlet nodes: a block of 16 and one node
    ("channel2d", (20, 18, 1), "weak"),        # 16: one block of 16
    ("channel3d", (9, 11, 9), "strong"),       # an inlet plane of 9 x 7 nodes in four blocks
    ("channel2d", (2100, 9, 1), "strong")])    # more than 64 wall blocks: inlet blocks of 32
def test_boundary_blocks(name, dims, coupling, storage, mech9):
    """Inlet and outlet runs cut into boundary blocks of 16 and 32 nodes."""
    rlbm = _rlbm()
    print(f"case boundary blocks {name} {dims} {coupling} {storage}", flush=True)
    case = wl.make_case(name, nx=dims[0], ny=dims[1], nz=dims[2], mech=mech9, coupling=coupling)
    lat, ora = rlbm.Lattice(case, storage=storage).set_state(), Oracle(case)
    lat.step(3)
    ora.step(3)
    gf, of = lat.fields(), ora.fields()
    if storage == "f64":
        gp, op = lat.populations(), ora.populations()
        for l in range(op.shape[0]):
            assert _nerr(gp[l], op[l]) <= 1e-10, l
    tol = 1e-10 if storage == "f64" else TOL[storage]
    assert _nerr(gf["T"], of["T"]) <= tol
    for a in range(9):
        assert _nerr(gf["Y"][a], of["Y"][a], 1e-6) <= tol, a


@pytest.mark.parametrize("nx", [1, 300, 4369, 4370])
def test_host_and_device_transfers_agree(mech9, nx):
    """Fields read to the host and to the device, all of them and a few, are
    the same bits, and so are the populations set from host and from device
    arrays: up to 4369 nodes of nine species the host's go through pinned
    memory, beyond through the idle population buffer."""
    rlbm = _rlbm()
    import ctypes
    import torch
    case = wl.make_case("tube", seed=nx, mech=mech9, nx=max(nx, 4)) if nx > 1 else wl.make_case(
        "reactor", seed=3, mech=mech9, nx=1, ny=1, nz=1)
    print(f"case transfers nx={nx}", flush=True)
    lat = rlbm.Lattice(case, storage="f32dev").set_state()
    first = lat.populations()
    keys = ("rho", "u", "T", "Y")
    dev = [torch.as_tensor(np.ascontiguousarray(case["init"][k], dtype=np.float64), device="cuda") for k in keys]
    lat.step(1)
    rlbm._check(rlbm.lib().rlbm_set_state(lat.handle, *[ctypes.c_void_p(d.data_ptr()) for d in dev], 1))
    np.testing.assert_array_equal(lat.populations(), first)
    lat.step(3)
    host = lat.fields()
    on = {k: torch.empty(v.size, dtype=torch.float64, device="cuda") for k, v in host.items()}
    rlbm._check(rlbm.lib().rlbm_read_fields(lat.handle, *[ctypes.c_void_p(v.data_ptr()) for v in on.values()], 1))
    for k, v in host.items():
        np.testing.assert_array_equal(v.ravel(), on[k].cpu().numpy())
    T, P = np.full_like(host["T"], -1.0), np.full_like(host["P"], -1.0)
    rlbm._check(rlbm.lib().rlbm_read_fields(lat.handle, None, None, ctypes.c_void_p(T.ctypes.data), None,
                                            ctypes.c_void_p(P.ctypes.data), 0))
    np.testing.assert_array_equal(T, host["T"])
    np.testing.assert_array_equal(P, host["P"])


@pytest.mark.parametrize("at", [0, 255, 256, 511, 600])
@pytest.mark.parametrize("key,value,word", [("rho", -1.0, "rho and T"), ("T", np.inf, "rho and T"),
                                            ("Y", np.nan, "mass fractions must be finite"),
                                            ("Y", 0.5, "sum to 1"), ("u", np.nan, "velocity")])
def test_set_state_refuses_a_bad_node(mech9, key, value, word, at):
    """One bad value at the edges of the checked chunks is refused with its
    own message, and the lattice keeps the state it had."""
    rlbm = _rlbm()
    case = wl.make_case("tube", seed=5, mech=mech9, nx=601)
    lat = rlbm.Lattice(case, storage="f64").set_state()
    before = lat.populations()
    init = {k: np.array(v, dtype=np.float64) for k, v in case["init"].items()}
    flat = init[key].reshape(-1, 601)
    flat[-1, at] = flat[-1, at] + value if key == "Y" else value
    with pytest.raises(rlbm.RlbmError) as e:
        lat.set_state(init)
    assert e.value.code == -1 and word in str(e.value)
    np.testing.assert_array_equal(lat.populations(), before)


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("name,dims", [
    ("reactor", (64, 5, 4)),       # a tile is a whole periodic row: both outer columns wrap
    ("reactor", (128, 3, 2)),      # a wrapped and an inner column beside each tile
    ("channel3d", (64, 9, 5)),     # an inlet and an outlet beside each tile
    ("channel3d", (128, 5, 4)),
    ("channel3d", (63, 9, 5)),     # a row one short of a tile
    ("channel3d", (64, 65, 3)),    # planes of 65 tiles: a strip of 64 and one of a single tile
    ("channel3d", (96, 64, 3))])   # planes of 96 tiles that cross rows
def test_flow_tiles(name, dims, storage, mech9):
    """Stencil and collision of f and g where tiles meet rows, faces and the
    ends of strips."""
    rlbm = _rlbm()
    print(f"case flow tiles {name} {dims} {storage}", flush=True)
    case = wl.make_case(name, seed=dims[0], nx=dims[0], ny=dims[1], nz=dims[2], mech=mech9)
    lat, ora = rlbm.Lattice(case, storage=storage).set_state(), Oracle(case)
    lat.step(2)
    ora.step(2)
    gp, op = lat.populations(), ora.populations()
    for l in range(op.shape[0]):
        assert _nerr(gp[l], op[l]) <= (1e-10 if storage == "f64" else TOL[storage]), l


@pytest.mark.parametrize("reaction", ["explicit", "implicit"])
@pytest.mark.parametrize("storage", ["f64", "f32dev"])
def test_negative_temperature_is_flagged(mech9, storage, reaction):
    """A state whose energy stands for a temperature below zero, which the
    Newton iteration reaches, has no rates: the lattice's flag is set within
    three steps."""
    rlbm = _rlbm()
    print(f"case negative temperature {storage} {reaction}", flush=True)
    case = wl.make_case("reactor", seed=4, mech=mech9, nx=4, ny=4, nz=4, reaction=reaction)
    lat = rlbm.Lattice(case, storage=storage).set_state()
    pops = lat.populations()
    T0 = lat.fields()["T"].mean()
    x0, t0, x, t = 1.0, T0, 1.0 + 1e-3, None
    for _ in range(20):      # secant for the energy of -0.3 T0
        p = pops.copy()
        p[-1] *= x
        lat.write_populations(p)
        t = lat.fields()["T"].mean()
        if -0.6 * T0 < t < -0.1 * T0:
            break
        x0, t0, x = x, t, x + np.clip((-0.3 * T0 - t) * (x - x0) / (t - t0), -0.5, 0.5)
    assert -0.6 * T0 < t < -0.1 * T0
    assert lat.status() == 0
    lat.step(3)
    assert lat.status() == 1


def test_creation_waits_for_earlier_work_on_its_memory(mech9):
    """A lattice on a side stream, in memory that the allocator took back from
    a tensor still being written on the default stream, has its tables intact."""
    rlbm = _rlbm()
    import torch
    case = wl.make_case("tube", seed=8, mech=mech9, nx=300)
    ref = rlbm.Lattice(case, storage="f64").set_state()
    ref.step(2)
    want = ref.populations()
    side = torch.cuda.Stream()
    for _ in range(3):
        block = torch.empty(ref.nbytes + 256, dtype=torch.uint8, device="cuda")
        a = torch.randn(4096, 4096, device="cuda")
        for _ in range(20):
            a = (a @ a).clamp_(-1.0, 1.0)       # a few milliseconds ahead of the fill
        block.fill_(255)
        del block
        lat = rlbm.Lattice(case, storage="f64", stream=side).set_state()
        lat.step(2)
        np.testing.assert_array_equal(lat.fields()["T"], ref.fields()["T"])
        np.testing.assert_array_equal(lat.populations(), want)

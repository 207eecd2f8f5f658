"""Host-side checks of the C ABI: the library loads, exports every symbol the
header declares, and validates descriptors.  No call here touches a GPU."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2108_07605_amd import rlbm, workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "rlbm.h")


def _declared():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(rlbm_\w+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = rlbm.lib()
    names = _declared()
    assert len(names) >= 15
    for name in names:
        assert hasattr(L, name), name
    assert set(names) == set(rlbm.EXPORTS)


def test_library_exports_no_other_plain_name():
    """Functions with C linkage beside the declared ones would stand in for
    another library's of the same name in the process."""
    out = subprocess.run(["nm", "-D", "--defined-only", rlbm.LIB_PATH], check=True, capture_output=True, text=True).stdout
    names = [ln.split()[-1] for ln in out.splitlines() if " T " in ln]
    assert set(n for n in names if not n.startswith(("_Z", "_init", "_fini"))) == set(rlbm.EXPORTS)


def test_mechanism_validation(mech9):
    m = rlbm.Mechanism(mech9)
    assert m.M == 9 and m.R == len(mech9["lnA"]) and m.E == 3
    bad = dict(mech9)
    bad["molar_mass"] = [-1.0] + list(mech9["molar_mass"][1:])
    with pytest.raises(rlbm.RlbmError) as e:
        rlbm.Mechanism(bad)
    assert e.value.code == -1
    D = np.array(mech9["transport"]["D_ref"])
    D[0, 1] *= 2.0                       # not symmetric
    bad = dict(mech9)
    bad["transport"] = dict(mech9["transport"], D_ref=D.tolist())
    with pytest.raises(rlbm.RlbmError):
        rlbm.Mechanism(bad)


def test_reaction_must_conserve_mass(mech_abc):
    bad = dict(mech_abc)
    bad["molar_mass"] = [2.0, 32.0, 18.0]        # A + B -> 2C with 34 != 36
    with pytest.raises(rlbm.RlbmError) as e:
        rlbm.Mechanism(bad)
    assert e.value.code == -1


def test_unsupported_species_count():
    mech = wl.mechanism_abc()
    five = dict(mech)
    five["M"] = 5
    for k in ("molar_mass",):
        five[k] = list(mech[k]) + [10.0, 20.0]
    five["nasa"] = list(mech["nasa"]) + [mech["nasa"][0]] * 2
    five["composition"] = list(mech["composition"]) + [[1, 0], [0, 1]]
    five["nu_f"] = [list(r) + [0, 0] for r in mech["nu_f"]]
    five["nu_r"] = [list(r) + [0, 0] for r in mech["nu_r"]]
    D = np.full((5, 5), 1e-3)
    five["transport"] = dict(mech["transport"], D_ref=D.tolist())
    with pytest.raises(rlbm.RlbmError) as e:
        rlbm.Mechanism(five)
    assert e.value.code == -4


def test_lattice_bytes_plan(mech9):
    m = rlbm.Mechanism(mech9)
    case = wl.make_case("channel2d", nx=64, ny=16, nz=1, mech=mech9)
    b64 = rlbm.lattice_bytes(case, m, "f64")
    b32 = rlbm.lattice_bytes(case, m, "f32dev")
    N, L = 64 * 16, 10
    assert b64 >= 2 * L * 27 * N * 8 and b32 >= 2 * L * 27 * N * 4
    # FP32 storage adds two buffers of per-node reference scales (12 floats)
    assert b64 - b32 >= 2 * L * 27 * N * 4 - 2 * 12 * N * 4 - 4096


@pytest.mark.parametrize("mutate,code", [
    (lambda c: c["faces"].__setitem__(3, {"type": "periodic"}), -1),   # y axis half periodic
    (lambda c: c["faces"].__setitem__(0, {"type": "outlet", "P_inf": 1.0, "sigma": 0.25}), -4),
    (lambda c: c.__setitem__("substeps", 0), -1),
    (lambda c: c["faces"].__setitem__(1, dict(c["faces"][0], type="inlet_local")), -4),   # inlet on x+
    (lambda c: c.__setitem__("nx", 2 ** 27), -4),                         # 9 N s beyond 2^32
    (lambda c: c.__setitem__("nx", 0), -1),
])
def test_lattice_descriptor_validation(mech9, mutate, code):
    m = rlbm.Mechanism(mech9)
    case = wl.make_case("channel2d", nx=32, ny=8, nz=1, mech=mech9)
    mutate(case)
    with pytest.raises(rlbm.RlbmError) as e:
        rlbm.lattice_bytes(case, m, "f64")
    assert e.value.code == code


def test_boundary_variants_accepted(mech9):
    """Bounce-back walls and the simplified inlet are valid descriptors; a
    bounce-back x- face with an outlet on x+ is a valid channel end."""
    m = rlbm.Mechanism(mech9)
    for case in (wl.make_case("bbbox", mech=mech9),
                 wl.make_case("channel2d", nx=32, ny=8, nz=1, mech=mech9, inlet="inlet_local")):
        assert rlbm.lattice_bytes(case, m, "f64") > 0
    case = wl.make_case("channel2d", nx=32, ny=8, nz=1, mech=mech9)
    case["faces"][0] = {"type": "bounceback"}
    assert rlbm.lattice_bytes(case, m, "f32dev") > 0


def test_reaction_scheme_validation(mech9):
    m = rlbm.Mechanism(mech9)
    case = wl.make_case("channel2d", nx=32, ny=8, nz=1, mech=mech9, reaction="implicit")
    assert rlbm.lattice_bytes(case, m, "f64") > 0
    d, _keep = rlbm.lattice_desc(case, "f64")
    assert d.reaction == rlbm.REACTION_LINEARLY_IMPLICIT
    d.reaction = 2
    n = ctypes.c_size_t()
    assert rlbm.lib().rlbm_lattice_bytes(ctypes.byref(d), m.handle, ctypes.byref(n)) == -1
    with pytest.raises(KeyError):
        rlbm.lattice_desc(dict(case, reaction="rk4"), "f64")


def test_weak_coupling_stores_every_species(mech9):
    """RLBM_SLAVED_NONE: L = M + 2 lattices (one more population buffer pair
    and reference scale per node than with a slaved species)."""
    m = rlbm.Mechanism(mech9)
    strong = wl.make_case("channel2d", nx=32, ny=8, nz=1, mech=mech9)
    weak = wl.make_case("channel2d", nx=32, ny=8, nz=1, mech=mech9, coupling="weak")
    d, _keep = rlbm.lattice_desc(weak, "f64")
    assert d.slaved == rlbm.SLAVED_NONE
    N = 32 * 8
    for st, s in (("f64", 8), ("f32dev", 4)):
        extra = rlbm.lattice_bytes(weak, m, st) - rlbm.lattice_bytes(strong, m, st)
        assert extra >= 2 * 27 * N * s                  # two population buffers of one more lattice
        assert extra <= 2 * 27 * N * s + 27 * 256 * 8 + 2 * 4 * N * 4 + 8 * 4096
    d.slaved = -3
    n = ctypes.c_size_t()
    assert rlbm.lib().rlbm_lattice_bytes(ctypes.byref(d), m.handle, ctypes.byref(n)) == -1
    with pytest.raises(KeyError):
        rlbm.lattice_desc(dict(weak, coupling="loose"), "f64")


def test_inlet_composition_must_sum_to_one(mech9):
    m = rlbm.Mechanism(mech9)
    case = wl.make_case("channel2d", nx=32, ny=8, nz=1, mech=mech9)
    y = list(case["faces"][0]["Y"])
    y[0] += 0.1
    case["faces"][0] = dict(case["faces"][0], Y=y)
    with pytest.raises(rlbm.RlbmError) as e:
        rlbm.lattice_bytes(case, m, "f64")
    assert e.value.code == -1


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
def test_record_of_the_explicit_update(mech9, storage):
    """The explicit step hands on 12 rows of doubles per node, the linearly
    implicit one 14 + 6 M + 6: a lattice is charged for its own."""
    m = rlbm.Mechanism(mech9)
    kw = dict(nx=64, ny=16, nz=1, mech=mech9)
    ex = rlbm.lattice_bytes(wl.make_case("channel2d", **kw), m, storage)
    im = rlbm.lattice_bytes(wl.make_case("channel2d", reaction="implicit", **kw), m, storage)
    N = 64 * 16
    assert abs(im - ex - (14 + 6 * 9 + 6 - 12) * 8 * N) <= 8 * 256

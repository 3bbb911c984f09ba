"""Interfaces that are not boxes (re-entrant corners, staircases, balls),
interfaces that a body cuts into, and equilibrium and Neumann faces on one
level: in place against two buffers, bit for bit after odd and even step
counts, levels in one launch against one launch each, and all of them against
the oracle at the FP64 bounds of every parity test.

Which kernels that runs: with two buffers the collide explodes (with children
missing, child by child) and, in the BGK, RR and polynomial models, fills the
Neumann cells of a level, while the boundary kernel is left its equilibrium
cells; Newton models and in-place runs launch the kernels for all of it."""
import numpy as np
import pytest

from gpu_util import assert_within, compare, run_pair, say
from interface_cases import cut_cases, open_cases, patch_cases
from paper_2504_04465_amd import lbm as B
from paper_2504_04465_amd import workloads as W

pytestmark = pytest.mark.gpu


CASES = patch_cases() + cut_cases() + open_cases()
IDS = [c[0] for c in CASES]
# (FP16 storage is refused with two distributions)
STORED = [(n, w, s) for n, w in CASES for s in ("fp64", "fp32", "fp16") if s != "fp16" or not w.collision.startswith("DDF")]


def same_state(a, b, what):
    assert np.array_equal(a.moments(), b.moments(), equal_nan=True), what
    for p, q in zip(a.get_state(), b.get_state()):
        assert p is None or np.array_equal(p, q), what
    assert np.array_equal(a.sensor(), b.sensor(), equal_nan=True), what
    cells = np.arange(0, a.n, 7)
    for p, q in zip(a.get_cells(cells), b.get_cells(cells)):
        assert p is None or np.array_equal(p, q), what


@pytest.mark.parametrize("name,w,storage", STORED, ids=[f"{n} {s}" for n, _, s in STORED])
def test_in_place_equals_two_buffers(name, w, storage):
    a = B.LBM.from_workload(w, storage=storage)
    b = B.LBM.from_workload(w, storage=storage, in_place=True)
    c = B.LBM.from_workload(w, storage=storage)
    c.level_fusion(False)
    m0 = w.initial_moments(*a.coords_levels())
    for s in (a, b, c):
        s.init(m0)
    for n in (1, 1, 2, 5):
        for s in (a, b, c):
            s.step(n)
        same_state(a, b, (name, n, "in place"))
        same_state(a, c, (name, n, "a launch per level"))
    say(f"[shapes] {name} {storage}: identical")
    for s in (a, b, c):
        s.close()


@pytest.mark.parametrize("in_place", [False, True], ids=["two buffers", "in place"])
@pytest.mark.parametrize("name,w", CASES, ids=IDS)
def test_against_oracle(name, w, in_place):
    w.newton_tol = 1e-14  # (both sides stop well below the bound compared at)
    mg, mo, level, s, o = run_pair(w, 5, "fp64", lib_over={"in_place": in_place})
    err = compare(mg, mo, level, len(w.ext))
    say(f"[shapes] {name} in_place={in_place}: {err}")
    assert_within(err, 1e-12)
    s.close()


@pytest.mark.parametrize("in_place", [False, True], ids=["two buffers", "in place"])
def test_wide_boundary_layer_of_a_newton_model(in_place):
    """66,000 boundary cells on one level, half Neumann and half equilibrium:
    the boundary kernel with several populations per lane"""
    w = W.shear(n=16, levels=1, lattice="D2Q21", collision="DDF_NEWTON", kind="random", u0=0.03, nu_finest=0.05,
                T0=0.65)
    w.ext = (11000, 20)
    w.newton_tol = 1e-14
    w.faces = [W.Face(), W.Face(), W.Face("neumann"),
               W.Face("equilibrium", u=(0.03, 0.01, 0.0), T=0.65, extrapolate_rho=True), W.Face(), W.Face()]
    mg, mo, level, s, o = run_pair(w, 3, "fp64", lib_over={"in_place": in_place})
    err = compare(mg, mo, level, 2)
    say(f"[shapes] wide boundary layer in_place={in_place}: {err}")
    assert_within(err, 1e-12)
    s.close()

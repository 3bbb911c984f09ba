"""Interfaces and boundary layers of 65536 lanes and more, where the
coalescence, the explosion and the Neumann fill give a lane several
populations instead of one: against the oracle, with two buffers and in
place.  FP64 storage, relative L2 1e-12 and 1e-11 in the worst cell (the
bounds of every FP64 parity test).  The Newton case solves to 1e-14 on both
sides: a residual of 1e-12 in the momentum is 3e-11 of the largest velocity
here (0.03), and where each side stops below its tolerance is decided by
rounding."""
import pytest

from gpu_util import assert_within, compare, run_pair, say
from paper_2504_04465_amd import workloads as W

pytestmark = pytest.mark.gpu


def boxed(lattice, collision, ext, lo, hi, faces=None, T0=1.0, newton_tol=1e-12):
    dim = len(ext)
    w = W.shear(n=16, levels=2, lattice=lattice, collision=collision, kind="random", u0=0.03, nu_finest=0.05, T0=T0)
    w.ext = ext
    w.refine = [W._box_mask(ext, dim, 0, lo, hi)]
    w.newton_tol = newton_tol
    if faces:
        w.faces = faces
    return w


NEUMANN_Y = [W.Face(), W.Face(), W.Face("neumann"), W.Face("neumann"), W.Face(), W.Face()]
# lanes of one population: ghosts x children (76 k, 264 k, 72 k), and 66 k
# boundary cells in the second case
CASES = [("D3Q27 cube", lambda: boxed("D3Q27", "RR", (64, 64, 64), (12, 12, 12), (52, 52, 52))),
         ("D2Q9 strip, Neumann", lambda: boxed("D2Q9", "BGK", (33000, 20), (0, 6), (33000, 14), NEUMANN_Y)),
         ("D2Q21 Newton strip", lambda: boxed("D2Q21", "DDF_NEWTON", (3000, 32), (0, 10), (3000, 22), T0=0.65,
                                             newton_tol=1e-14))]


@pytest.mark.parametrize("in_place", [False, True], ids=["two buffers", "in place"])
@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_wide_interface_against_oracle(name, make, in_place):
    mg, mo, level, s, o = run_pair(make(), 2, "fp64", lib_over={"in_place": in_place})
    err = compare(mg, mo, level, len(make().ext))
    say(f"[wide] {name} in_place={in_place}: {err}")
    assert_within(err, 1e-12)
    s.close()

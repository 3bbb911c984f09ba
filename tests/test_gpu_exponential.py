"""The exponential of the numerical equilibrium over its whole range: a
surrogate network with zero weights hands every cell the multipliers
(lambda_0, 0, ..., 0), whose equilibrium is rho exp(-(1 + lambda_0)) for every
population, and at tau = 1 a collision returns the equilibrium.

FP64: relative 1e-14 of |f| + |f_eq| (f - (f - f_eq) rounds by half an ulp of
either three times, the exponential by an ulp).  FP32: 1e-6 of the same.
Arguments beyond the range, also where 64 s / ln 2 no longer fits 32 or 37
bits, give 0 and infinity."""
import numpy as np
import pytest

from gpu_util import say
from paper_2504_04465_amd import lbm as B
from paper_2504_04465_amd import workloads as W

pytestmark = pytest.mark.gpu

LN2 = float(np.log(2.0))
NEAR = [0.0, 0.3, 1.0, 5.5, 20.0, 60.0, 86.0]
FAR = [300.0, 700.0, 705.0, 709.0, 712.0, 744.0, 800.0, 1e4, 2.0 ** 25 * LN2, 2.5e7, 1e9, 1.4e9, 1.45e9, 1.6e9, 2e9,
       3e9, 2.0 ** 32 * LN2, 2.0 ** 33 * LN2, 1e11, 1e13, 1e16, 1e20]


@pytest.mark.parametrize("before", [0, 1], ids=["first step", "second step"])
@pytest.mark.parametrize("storage,tol", [("fp64", 1e-14), ("fp32", 1e-6)])
def test_exponential_over_its_range(storage, tol, before):
    w = W.shear(n=16, levels=1, lattice="D2Q21", collision="DDF_MLP", T0=0.65)
    s = B.LBM("D2Q21", "DDF_MLP", storage, nu_finest=0.5 * 0.65, T0=0.65)
    s.grid(w.dim, w.ext, 1, [], None, w.faces)
    real = np.float64 if storage == "fp64" else np.float32
    m0 = np.zeros((4, s.n))
    m0[0], m0[3] = 1.0, 0.65
    for a in sorted(set(NEAR + FAR)):
        for sign in (1.0, -1.0):
            p = np.zeros(9176, np.float32)
            s.init(m0)
            if before:  # a step at a harmless point, so that the next one pulls
                p[9160] = 1.0
                s.mlp_set_weights(p)
                s.step(1)
            f, _, _ = s.get_state()
            p[9160] = np.float32(sign * a)
            s.mlp_set_weights(p)
            s.step(1)
            got, _, _ = s.get_state()
            arg = 1.0 + float(p[9160])
            with np.errstate(over="ignore", under="ignore", invalid="ignore"):
                rho = f.sum(0)
                feq = (rho.astype(real) * real(np.exp(-arg))).astype(np.float64)
                feq = np.broadcast_to(feq, f.shape)
                if np.isfinite(feq).all():
                    err = np.max(np.abs(got - feq) / (np.abs(f) + np.abs(feq)))
                    assert err <= tol, (a, sign, err)
                else:
                    assert np.all(np.isposinf(got)), (a, sign, got.min(), got.max())
    say(f"[exp] {storage}: right from 0 to 1e20 of both signs")
    s.close()


@pytest.mark.parametrize("lattice", ["D2Q13", "D2Q21", "D2Q37"])
def test_solve_whose_first_step_overflows(lattice):
    """warm starts with lambda_0 far too large: the residual is that of an
    empty cell, the first full step is e^b long and its exponentials overflow
    (up to |s| = 4e9), and the line search comes back from it.  The collision
    then equals that of a warm start at the solution, to the solver's
    tolerance (1e-12 in the moments, times 1e2 for the multipliers'
    conditioning)."""
    T0 = 0.35 if lattice == "D2Q13" else 0.65
    w = W.shear(n=16, levels=1, lattice=lattice, collision="DDF_NEWTON", T0=T0, u0=0.05)
    out = []
    for b in (0.0, 10.0, 16.0, 20.0, 22.0):
        s = B.LBM.from_workload(w, storage="fp64")
        s.init(w.initial_moments(*s.coords_levels()))
        f, g, lam = s.get_state()
        lam[0] += b
        s.set_state(f, g, lam)
        s.step(1)
        st = s.stats()
        assert st["newton_failures"] == 0, (b, st)
        out.append(s.get_state()[0])
        say(f"[exp] {lattice} b={b}: {st['newton_iterations'] / s.n:.2f} steps a solve")
        s.close()
    for f in out[1:]:
        assert np.max(np.abs(f - out[0])) <= 1e-10

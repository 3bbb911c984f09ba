"""Small grids whose refinement interfaces are not boxes, shared by the host
and GPU tests: re-entrant corners and staircases, where the coalescence
reads children that keep a population for want of a source."""
import numpy as np

from paper_2504_04465_amd import workloads as W


def _patched(mask, lattice, collision, T0=1.0):
    w = W.shear(n=max(mask.shape), levels=1, lattice=lattice, collision=collision, nu_finest=0.05, kind="random",
                u0=0.03, T0=T0)
    w.ext = tuple(reversed(mask.shape))
    w.n_levels = 2
    w.refine = [W.Mask(mask.astype(np.uint8), (0,) * mask.ndim)]
    w.solid = [None, None]
    return w


def l_shape(n, a, b, c):
    """cells [a, c)^2 without [b, c)^2"""
    m = np.zeros((n, n), bool)
    m[a:c, a:c] = True
    m[b:c, b:c] = False
    return m


def ball(n, r, dim):
    x = np.arange(n) + 0.5 - n / 2
    return sum(q * q for q in np.meshgrid(*[x] * dim, indexing="ij")) < r * r


def patch_cases():
    return [("L D2Q9", _patched(l_shape(24, 4, 12, 20), "D2Q9", "RR")),
            ("disc D2Q9", _patched(ball(48, 18.0, 2), "D2Q9", "BGK")),
            ("L D2Q21", _patched(l_shape(48, 8, 24, 40), "D2Q21", "DDF_NEWTON", T0=0.65)),
            ("disc D2Q37", _patched(ball(48, 16.0, 2), "D2Q37", "DDF_POLY")),
            ("ball D3Q27", _patched(ball(20, 7.0, 3), "D3Q27", "RR"))]

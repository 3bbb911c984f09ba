"""Small grids shared by the host and GPU tests, whose interfaces and faces are
less simple than the workloads':
- interfaces that are not boxes: re-entrant corners and staircases, where the
  coalescence reads children that keep a population for want of a source;
- interfaces that a body cuts into: coarse ghosts some of whose children are
  solid;
- equilibrium faces (density imposed and extrapolated) and Neumann faces on the
  same level, with shared corners."""
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


def cut_cases():
    """a box refined once, with solid fine cells in its outermost ring: one, two
    and three (in 3-D up to seven) of the children of several coarse ghosts"""
    out = []
    for lattice, collision, ext, lo, hi, T0 in (
            ("D2Q9", "RR", (24, 20), (6, 5), (18, 15), 1.0),
            ("D2Q9", "BGK", (21, 17), (5, 4), (16, 13), 1.0),
            ("D2Q21", "DDF_NEWTON", (48, 40), (10, 9), (38, 31), 0.65),
            ("D2Q37", "DDF_POLY", (48, 40), (10, 9), (38, 31), 1.0),
            ("D3Q27", "RR", (14, 13, 12), (3, 3, 3), (11, 10, 9), 1.0)):
        dim = len(ext)
        m = np.zeros(ext[::-1], bool)
        m[tuple(slice(lo[a], hi[a]) for a in reversed(range(dim)))] = True
        w = _patched(m, lattice, collision, T0)
        body = np.zeros(tuple(2 * e for e in ext[::-1]), np.uint8)

        def cut(ghost, octants):
            for o in octants:
                body[tuple(2 * ghost[a] + ((o >> a) & 1) for a in reversed(range(dim)))] = 1

        mid = [(a + b) // 2 for a, b in zip(lo, hi)]
        cut([lo[0]] + mid[1:], [0])
        cut([lo[0]] + [q + 3 for q in mid[1:]], [1, 2])
        cut([mid[0], lo[1]] + mid[2:], range((1 << dim) - 1))
        cut([hi[0] - 1] + mid[1:], [1, 3])
        cut([h - 1 for h in hi], [0])  # a corner of the box
        w.solid = [None, W.Mask(body, (0,) * dim)]
        out.append((f"cut {lattice} {collision}", w))
    return out


def _open(w, T0):
    u = (0.03, 0.01, 0.0)
    w.faces = [W.Face("equilibrium", rho=1.01, u=u, T=T0), W.Face("neumann"),
               W.Face("neumann"), W.Face("equilibrium", u=u, T=T0, extrapolate_rho=True),
               W.Face("neumann"), W.Face("equilibrium", rho=0.99, u=u, T=T0)]
    return w


def open_cases():
    """both kinds of open face on the coarse level (a refined patch inside), or
    on the fine one (a coarse hole inside); in 2-D the z faces are ignored"""
    def boxed(ext, lo, hi, hole):
        m = np.full(ext[::-1], hole)
        m[tuple(slice(lo[a], hi[a]) for a in reversed(range(len(ext))))] = not hole
        return m

    out = []
    for lattice, collision, ext, lo, hi, T0 in (
            ("D2Q9", "RR", (24, 20), (8, 7), (17, 14), 1.0),
            ("D2Q13", "RR", (36, 32), (11, 10), (25, 22), 1.0),
            ("D3Q27", "BGK", (14, 13, 12), (4, 4, 4), (10, 9, 8), 1.0),
            ("D2Q37", "DDF_POLY", (48, 40), (14, 12), (34, 28), 1.0),
            ("D2Q21", "DDF_NEWTON", (48, 40), (14, 12), (34, 28), 0.65)):
        for hole in (False, True):
            w = _open(_patched(boxed(ext, lo, hi, hole), lattice, collision, T0), T0)
            out.append((f"open {lattice} {collision}{', hole' if hole else ''}", w))
    w = _open(W.shear(n=19, levels=1, lattice="D2Q9", collision="BGK", nu_finest=0.05, kind="random", u0=0.03), 1.0)
    out.append(("open D2Q9 BGK, one level", w))
    return out

"""In-place streaming on the CPU, word by word: the rules of
csrc/inplace.h, which the kernels use, on the pull sources of host-built
grids.  In the odd step, whose cells run in no order, no word of the buffer
may be read by a cell other than the one that writes it, nor have two
writers; and an even step, an odd step and the reads between them must give
every cell the populations that a pull from two buffers gives it."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from edge_cases import edge_cases
from interface_cases import cut_cases, open_cases, patch_cases
from oracle.oracle import Oracle
from paper_2504_04465_amd import lbm as B
from paper_2504_04465_amd import workloads as W

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_04465_amd", "csrc")
CODE = r"""
#include <cstdint>
#include <vector>
#include "inplace.h"
using namespace lbm;
// src[i - 1][cell]: source slot of link i (nslot and above: the cell's coalesced slot), negative: a wall
extern "C" void check(int64_t n, int64_t nslot, int64_t nvirtual, int Q, const int32_t *opp, const int32_t *slot,
                      const int32_t *src, int64_t *out) {
  const int64_t S = nslot + nvirtual;
  std::vector<int64_t> writer(Q * S, -1), reader(Q * S, -1), held(Q * S, -1);
  auto w = [&](Word a) { return a.slot * Q + a.row; };
  auto tag = [&](int i, int64_t s) { return s * Q + i; };  // population i of slot s
  auto link = [&](int i, int64_t k) { return (int64_t)src[(i - 1) * n + k]; };
  // after an even step: the cells' own populations, and the coalesced slots swapped
  for (int64_t k = 0; k < n; ++k) {
    const int64_t c = slot[k];
    held[w(Word{0, c})] = tag(0, c);
    for (int i = 1; i < Q; ++i) {
      const Word to = even_store(opp[i], link(opp[i], k), c);
      if (to.row >= 0) held[w(to)] = tag(i, c);
      if (keeps(link(i, k), c)) held[w(Word{i, c})] = tag(i, c);
    }
  }
  for (int64_t v = nslot; v < S; ++v)
    for (int i = 1; i < Q; ++i) held[w(Word{opp[i], v})] = tag(i, v);
  // the odd step pulls; what it pushes, the next even step reads in its own rows
  int64_t races = 0, wrong = 0, kept = 0;
  std::vector<int64_t> next(Q * S, -1);
  for (int64_t k = 0; k < n; ++k) {
    const int64_t c = slot[k];
    for (int i = 1; i < Q; ++i) {
      const int64_t s = link(i, k), t = link(opp[i], k);
      const int64_t r = w(odd_pull(i, opp[i], s, c));
      if (held[r] != (s < 0 ? tag(opp[i], c) : tag(i, s))) ++wrong;
      if (reader[r] >= 0 && reader[r] != k) ++races;
      reader[r] = k;
      kept += s == c;
      Word to[2] = {odd_store(i, opp[i], t, c), keeps(s, c) ? Word{i, c} : Word{-1, c}};
      for (Word a : to) {
        if (a.row < 0) continue;
        if (writer[w(a)] >= 0) ++races;
        writer[w(a)] = k;
        next[w(a)] = tag(i, c);
      }
    }
  }
  for (int64_t a = 0; a < Q * S; ++a) races += reader[a] >= 0 && writer[a] >= 0 && reader[a] != writer[a];
  for (int64_t k = 0; k < n; ++k)
    for (int i = 1; i < Q; ++i) {
      const int64_t c = slot[k], s = link(i, k);
      if (s >= nslot) continue;  // the coalescence writes these anew
      if (next[w(Word{i, c})] != (s < 0 ? tag(opp[i], c) : tag(i, s))) ++wrong;
    }
  out[0] = races;
  out[1] = wrong;
  out[2] = kept;
}
"""


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    d = tmp_path_factory.mktemp("words")
    src, so = d / "check.cpp", d / "check.so"
    src.write_text(CODE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so)).check


def sources(s):
    """pull source of every link over slots, and the slots of the cells"""
    e, d = s.export(("nbr",)), s.layout_export()
    slot, row, n = d["slot_of"], d["xrow_of"], s.n
    nbr = e["nbr"].reshape(n, -1).T
    src = np.where(nbr >= 0, slot[np.maximum(nbr, 0)], nbr).astype(np.int32)
    has = row >= 0
    x = d["xnbr"].reshape(src.shape[0], -1)
    src[:, has] = x[:, row[has]]
    return np.ascontiguousarray(src), np.ascontiguousarray(slot, np.int32)


def grids():
    base = [("cavity", W.cavity(n=64, steps=1)), ("shear, 3 levels", W.shear(n=32, levels=3, steps=1)),
            ("D2Q13", W.shear(n=32, levels=3, lattice="D2Q13", collision="DDF_NEWTON", T0=0.35)),
            ("cylinder", W.cylinder(scale=16, steps=1)), ("sphere", W.sphere(scale=8, steps=1)),
            ("airfoil", W.airfoil(scale=16, steps=1)), ("Sod", W.sod(nx=256, ny=8, steps=1))]
    return base + edge_cases() + patch_cases() + cut_cases() + open_cases()


@pytest.mark.parametrize("name,w", grids(), ids=[g[0] for g in grids()])
def test_odd_step_words_have_one_user(name, w, check):
    s = B.LBM.from_workload(w, storage="fp32", host_only=True)
    src, slot = sources(s)
    opp = np.ascontiguousarray(Oracle.from_workload(w).opp, np.int32)
    ns = s.layout()["slots"]
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    out = np.zeros(3, np.int64)
    check(ctypes.c_int64(s.n), ctypes.c_int64(ns), ctypes.c_int64(s.n_ghosts), len(opp), ptr(opp), ptr(slot), ptr(src),
          ptr(out))
    races, wrong, kept = out
    assert races == 0 and wrong == 0
    if s.n_ghosts:
        assert kept > 0  # fine ghosts at the edge of their level
    s.close()


@pytest.mark.parametrize("name,w", cut_cases(), ids=[c[0] for c in cut_cases()])
def test_cut_cases_cut(name, w):
    """the grids meant to have coarse ghosts with one to all but one of their
    children missing do"""
    s = B.LBM.from_workload(w, storage="fp32", host_only=True)
    missing = (s.export(("child",))["child"] < 0).sum(1)
    assert {1, 2, (1 << len(w.ext)) - 1} <= set(missing.tolist()) and (missing == 0).sum() > 0
    s.close()

"""The row GEMMs' cut into units, as the library computes it: csrc/row_units.h
compiled for the host (it is plain arithmetic, shared by kernels and launchers)."""
from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile
from typing import NamedTuple

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_11867_amd", "csrc")
SOURCE = """
#include "row_units.h"
using namespace foremoe;
extern "C" {
void units(int n, const int* rows, int N0, int K0, int N1, int K1, int phases, int G, int ws, int* out) {
  int tiles[3] = {0, 0, 0};
  for (int i = 0; i < n; ++i) {
    const SlotTiles t = slot_tiles(rows[i]);
    tiles[0] += t.full;
    tiles[1] += t.is_short;
    tiles[2] += t.is_thin;
  }
  const LaunchUnits l = launch_units(tiles[0], tiles[1] + tiles[2], N0, K0, N1, K1, phases, G, ws);
  for (const PhaseUnits* u : {&l.u0, &l.u1})
    for (int v : {u->nt, u->kt, u->small, u->plain, u->full_cut, u->h, u->s, u->total}) *out++ = v;
  for (int v : tiles) *out++ = v;
}
int max_cut(int G) { return cut_units(G); }
int fits(int G) { return rows_workspace_fits(G); }
size_t bytes(int G) { return rows_workspace_bytes(G); }
size_t used(int G) { return rows_workspace_used(G); }
}
"""


class Phase(NamedTuple):
    nt: int
    kt: int
    small: int
    plain: int
    full_cut: int
    h: int
    s: int
    total: int

    @property
    def small_cut(self) -> int:
        """Small tiles among the cut ones."""
        return (self.total - self.plain) // self.s - self.full_cut * self.h


class Tiles(NamedTuple):
    full: int
    short: int
    thin: int


@functools.lru_cache(maxsize=None)
def lib() -> ctypes.CDLL:
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "units.cpp"), os.path.join(d, "units.so")
        with open(src, "w") as f:
            f.write("#include <initializer_list>\n" + SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", f"-I{CSRC}", src, "-o", so],
                       check=True, timeout=60)
        h = ctypes.CDLL(so)
    h.bytes.restype = h.used.restype = ctypes.c_size_t
    return h


def units(rows, first, second, phases=3, G=256, ws=True):
    """(Phase, Phase, Tiles) of a launch over slots of `rows` rows: `first` and
    `second` are (N, K) of its GEMMs."""
    out = (ctypes.c_int * 19)()
    lib().units(len(rows), (ctypes.c_int * max(len(rows), 1))(*[int(r) for r in rows]), *first, *second, phases, G,
                int(ws), out)
    v = list(out)
    return Phase(*v[:8]), Phase(*v[8:16]), Tiles(*v[16:])


def forward(rows, d, F, **kw):
    """The forward: gate/up (N = 2F, K = d), then down (N = d, K = F)."""
    return units(rows, (2 * F, d), (d, F), **kw)


def dgrad(rows, d, F, **kw):
    """The input gradients: down (N = F, K = d), then gate/up (N = d, K = 2F)."""
    return units(rows, (F, d), (d, 2 * F), **kw)

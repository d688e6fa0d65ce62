"""Storage of the interior factor (csrc/band.hpp, compiled here for the host): every entry that the
factorisation, the mirror and the solves touch lies inside the block, and no two of them share a place."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NB, PANEL, WIDE = 128, 256, 512   # block columns, a panel's columns, the widest block read as a rectangle
MAIN = r"""
#include "band.hpp"
#include <cstdio>
int main() {
  long long n, bs, wide, k;
  while (std::scanf("%lld %lld %lld %lld", &n, &bs, &wide, &k) == 4) {
    std::vector<int64_t> rend(k);
    for (auto& r : rend) { long long v; if (std::scanf("%lld", &v) != 1) return 1; r = v; }
    const rpf::FactorLayout f = rpf::factor_layout(n, rend, bs, wide);
    std::printf("%lld %lld %lld\n", (long long)f.ld, (long long)f.len, (long long)f.hw);
  }
}
"""


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("layout")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "layout")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1208_6387_amd", "csrc"),
                    str(d / "main.cpp"), "-o", exe], check=True)

    def call(n, rend):
        text = " ".join(str(int(v)) for v in (n, NB, WIDE, len(rend), *rend))
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return tuple(int(v) for v in out.split())
    return call


def _blocks(first):
    """rend and cstart of every block of NB columns (rows), from the first column of every row."""
    n = len(first)
    nblk = -(-n // NB)
    mx = np.zeros(nblk, int)
    np.maximum.at(mx, first // NB, np.arange(n) + 1)
    ends = np.minimum(n, NB * np.arange(1, nblk + 1))
    rend = np.maximum(np.maximum.accumulate(mx), ends)
    cstart = np.array([first[t * NB:(t + 1) * NB].min() for t in range(nblk)])
    return rend, cstart


def _rectangles(n, rend, cstart):
    """(rows, columns) of every rectangle that a kernel addresses, as half-open ranges."""
    nblk = len(rend)
    for t in range(nblk):                                       # diagonal block, panel, mirror
        yield (t * NB, rend[t]), (t * NB, min(n, (t + 1) * NB))
        yield (t * NB, min(n, (t + 1) * NB)), (t * NB, rend[t])
        yield (t * NB, min(n, (t + 1) * NB)), (max(0, cstart[t]), t * NB)
        yield (max(0, cstart[t]), t * NB), (t * NB, min(n, (t + 1) * NB))
    for p0 in range(0, n, PANEL):                               # the update right of a panel
        p1 = min(p0 + PANEL, n)
        pend = max(rend[p0 // NB:-(-p1 // NB)])
        yield (p1, pend), (p0, p1)
        yield (p1, pend), (p1, pend)
    for j0 in range(0, n, WIDE):                                # solves through the block inverses
        j1, b = min(j0 + WIDE, n), slice(j0 // NB, -(-min(j0 + WIDE, n) // NB))
        yield (j0, max(j1, rend[b][-1])), (j0, j1)
        cs = min(j0, max(0, cstart[b].min()))
        yield (cs, j1), (j0, j1)
        yield (j0, j1), (cs, j1)


def _brick(a, b, c, dpn):
    """First columns of the interior rows of a box of a x b x c elements."""
    s = [x - 1 for x in (a, b, c) if x > 1]
    node = np.arange(int(np.prod(s)))
    stride = np.cumprod([1] + s[:-1])
    at = np.stack([node // st % m for st, m in zip(stride, s)])
    low = sum(np.maximum(v - 1, 0) * st for v, st in zip(at, stride))
    return np.repeat(low * dpn, dpn)


CASES = {"12^3": _brick(12, 12, 12, 3), "18^3": _brick(18, 18, 18, 3), "20^3": _brick(20, 20, 20, 3),
         "heat 30 x 1000": _brick(30, 1000, 1, 1), "heat 8 x 400": _brick(8, 400, 1, 1),
         "heat 1000 x 8": _brick(1000, 8, 1, 1), "3 x 3 x 300": _brick(3, 3, 300, 3), "7 x 11 x 5": _brick(7, 11, 5, 3),
         "one dof": np.zeros(1, int), "129 dofs": np.maximum(np.arange(129) - 3, 0)}
for _k in range(6):
    _g = np.random.default_rng(_k)
    _n = int(_g.integers(1300, 6000))
    _w = _g.integers(0, int(_g.integers(2, 900)), _n)
    CASES[f"ragged {_n}"] = np.maximum(np.arange(_n) - _w, 0)


@pytest.mark.parametrize("name", list(CASES))
def test_every_touched_entry_has_a_place_of_its_own(layout, name):
    first = CASES[name]
    n = len(first)
    rend, cstart = _blocks(first)
    ld, length, hw = layout(n, rend)
    assert (n - 1) * (ld + 1) < length          # the last diagonal entry
    for (r0, r1), (c0, c1) in _rectangles(n, rend, cstart):
        if r0 >= r1 or c0 >= c1:
            continue
        assert 0 <= r0 and r1 <= n and 0 <= c0 and c1 <= n
        assert 0 <= r0 + c0 * ld and (r1 - 1) + (c1 - 1) * ld < length
        if hw:                                  # columns of the band do not overlap
            assert max(r1 - 1 - c0, c1 - 1 - r0) < hw and 2 * hw <= ld + 1
        else:
            assert ld == n and length == n * n


def test_thin_patterns_are_stored_in_a_band(layout):
    """The cases above cover bands that are many times longer than they are wide."""
    long = 0
    for first in CASES.values():
        _, _, hw = layout(len(first), _blocks(first)[0])
        long += hw > 0 and len(first) > 3 * hw
    assert long >= 5

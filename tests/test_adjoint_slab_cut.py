"""How the transposes cut a block level into slabs (csrc/adjoint_slab.h), on
the CPU: the header is compiled by itself.  Every node is summed once, all
the blocks that cover it have their contributions in the scratch then, and
the scratch keeps its bound.  (Large values of "bytes per value" make small
grids take many slabs.)"""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_00205_amd", "csrc")

SHIM = """
#include "adjoint_slab.h"
extern "C" void cut(const int64_t* nb, int64_t b, int64_t esize, int64_t* o) {
  const bm::SlabCut c = bm::slab_cut(nb, b, size_t(esize));
  const int64_t v[7] = {c.layers, c.ring, c.cut[0], c.run[0], c.cut[1], c.run[1], c.blocks()};
  for (int i = 0; i < 7; ++i) o[i] = v[i];
}
extern "C" void strip(int64_t n, int64_t cut, int64_t k, int64_t* o) {
  const bm::BlockRange r = bm::strip(n, cut, k);
  o[0] = r.run;
  o[1] = r.lo;
  o[2] = r.hi;
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("slab")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.run([shutil.which("g++") or "c++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC,
                    str(d / "shim.cpp"), "-o", so], check=True)
    return C.CDLL(so)


def _bound(b):
    return (128 if b < 33 else 256) << 20


def _cut(shim, nb, b, esize):
    o = (C.c_int64 * 7)()
    shim.cut((C.c_int64 * 3)(*nb), C.c_int64(b), C.c_int64(esize), o)
    return dict(zip(("layers", "ring", "cut_y", "run_y", "cut_x", "run_x", "blocks"), o))


def _strips(shim, n, cut):
    o, out = (C.c_int64 * 3)(), []
    for k in range((n + cut - 1) // cut):
        shim.strip(C.c_int64(n), C.c_int64(cut), C.c_int64(k), o)
        out.append(tuple(o))
    return out


# dims in blocks of grids up to the largest a card holds: cubes, flat, one row
@pytest.mark.parametrize("nb", [(1, 1, 1), (32, 32, 32), (7, 75, 75), (64, 64, 32), (4, 128, 128), (1, 512, 512),
                                (1, 1000, 1000), (1, 1, 1 << 21), (1, 1 << 21, 1), (1 << 21, 1, 1), (2, 13, 388),
                                (2, 60, 400), (129, 129, 2)])
@pytest.mark.parametrize("b", [9, 17, 33])
@pytest.mark.parametrize("esize", [4, 8])
def test_scratch_keeps_its_bound(shim, nb, b, esize):
    c = _cut(shim, nb, b, esize)
    assert c["blocks"] * b ** 3 * esize <= _bound(b)
    assert c["blocks"] == c["ring"] * c["run_y"] * c["run_x"]
    # blocks run more than once: at most a quarter more than there are (x and y cut)
    runs = [sum(hi - run for run, _, hi in _strips(shim, n, c["cut_" + a])) for n, a in ((nb[1], "y"), (nb[2], "x"))]
    assert runs[0] * runs[1] <= 1.25 * nb[1] * nb[2]
    # a level that fits takes one slab and no more than its own blocks
    if nb[0] * nb[1] * nb[2] * b ** 3 * esize <= _bound(b):
        assert c["blocks"] == nb[0] * nb[1] * nb[2]


@pytest.mark.parametrize("seed", range(60))
def test_every_node_is_summed_from_all_its_blocks(shim, seed):
    rng = random.Random(seed)
    b = 9
    nb = [rng.randint(1, 7), rng.randint(1, 30), rng.randint(1, 30)]
    fit = rng.choice([8, 12, 20, 50, 120, 400])
    esize = _bound(b) // (fit * b ** 3)
    c = _cut(shim, nb, b, esize)
    assert c["blocks"] <= _bound(b) // (b ** 3 * esize)
    done, slot = set(), {}                               # faces summed; block in each slot

    def covering(f, n):                                  # blocks that cover face coordinate f (node f (b - 1))
        return [k for k in (f - 1, f) if 0 <= k < n]

    for ry, ly, hy in _strips(shim, nb[1], c["cut_y"]):
        for rx, lx, hx in _strips(shim, nb[2], c["cut_x"]):
            for k0 in range(0, nb[0], c["layers"]):
                k1 = min(nb[0], k0 + c["layers"])
                for z in range(k0, k1):
                    for y in range(ry, hy):
                        for x in range(rx, hx):
                            s = ((z % c["ring"]) * (hy - ry) + y - ry) * (hx - rx) + x - rx
                            assert 0 <= s < c["blocks"]
                            slot[s] = (z, y, x)
                for z in range(k0, k1 + (k1 == nb[0])):
                    for y in range(ly, hy + (hy == nb[1])):
                        for x in range(lx, hx + (hx == nb[2])):
                            assert (z, y, x) not in done
                            done.add((z, y, x))
                            for bz in covering(z, nb[0]):
                                for by in covering(y, nb[1]):
                                    for bx in covering(x, nb[2]):
                                        s = ((bz % c["ring"]) * (hy - ry) + by - ry) * (hx - rx) + bx - rx
                                        assert slot[s] == (bz, by, bx)
    assert len(done) == (nb[0] + 1) * (nb[1] + 1) * (nb[2] + 1)

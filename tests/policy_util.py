"""cache_policy.hpp compiled with the host compiler: the cache policy that a step
takes for given lattices, without a GPU."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

import numpy as np

from paper_0912_4230_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STREAM, REUSE, KEEP = 0, 1, 2
STORED = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2, "bf16s": 2, "f16s": 2}

SHIM = """
#include "cache_policy.hpp"
using namespace plbm;
extern "C" {
size_t lattice_size() { return sizeof(CacheLattice); }
void add(double *step, const CacheLattice *l, int n)
{
    CacheStep s = {step[0], step[1]};
    add_launch(s, l, n);
    step[0] = s.keep;
    step[1] = s.reuse;
}
int policy(const CacheLattice *l, int n, const double *step) { return cache_policy(l, n, CacheStep{step[0], step[1]}); }
}
"""


class CacheLattice(C.Structure):
    _fields_ = [("physics", C.c_int), ("storage", C.c_int), ("nx", C.c_int), ("solutes", C.c_int),
                ("links", C.c_bool), ("tensor", C.c_bool), ("cells", C.c_double), ("bytes", C.c_double),
                ("medium", C.c_double), ("bounced", C.c_double)]


@functools.lru_cache(maxsize=None)
def _lib():
    d = tempfile.mkdtemp()
    src, out = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_0912_4230_amd", "csrc"),
                    src, "-o", out], check=True)
    L = C.CDLL(out)
    L.lattice_size.restype = C.c_size_t
    assert L.lattice_size() == C.sizeof(CacheLattice)
    return L


def lattice(physics, storage, shape, links=False, tensor=False, species=1, uniform=None, bounced=None):
    """physics: single, miscible, immiscible or freesurf.  uniform: no medium planes (by default in the models
    without one in their problems here).  bounced: the share of cells with a link cut by the mask (links), by
    default as with a fifth of them solid.  The planes' padding is left out of the bytes."""
    k = {"single": B.LBM_SINGLE, "miscible": B.LBM_MISCIBLE, "immiscible": B.LBM_IMMISCIBLE, "freesurf": B.LBM_FREESURF}
    cells = float(np.prod(shape))
    copies = 1 if physics in ("single", "freesurf") else 1 + species
    each = 2 * (19 * STORED[storage] + (4 if storage.endswith("s") else 0))
    uniform = physics in ("single", "immiscible") if uniform is None else uniform
    planes = (0 if uniform else (8 if tensor else 4)) + (physics == "immiscible")
    medium = cells * (planes * (8 if storage == "f64" else 4) + (4 if links else 0))
    return CacheLattice(k[physics], B.STORAGE_NAMES[storage], shape[0], species, links, tensor, cells, cells * copies * each, medium,
                        (0.28 if bounced is None else bounced) if links else 0.0)


def policies(groups):
    """The policy of every group (a list of lattices) of a batch in one step."""
    arrays = [(CacheLattice * len(g))(*g) for g in groups]
    step = (C.c_double * 2)()
    for a in arrays:
        _lib().add(step, a, len(a))
    return [_lib().policy(a, len(a), step) for a in arrays]

"""The regrid's data remap (Sec. 2.2: copy, prolong, restrict) and the
gradient criterion over what the kernels are specialised for: precision,
dimension, block size, ghost width and number of variables, each against the
FP64 oracle without tolerance.  FP32 states hold FP32 values that the oracle
starts from, and both do their sums in FP64, so the oracle's result rounded
once to FP32 is the expectation."""
import sys

import numpy as np
import pytest

from oracle import OracleMesh
from tests.gpu_helpers import gpu_state, interior

pytestmark = pytest.mark.gpu

# (ndim, block size, ghost width): every block size with every ghost width
# that it admits (block size >= 2 ghost widths)
SHAPES = [(d, N, g) for d in (2, 3) for N in (8, 16, 32) for g in (2, 3, 4)]


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def f4():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_07612_amd as f4
    f4.lib()
    return f4


def fill(gm, om, prec, seed):
    """The same rough state in both: independent values in every cell, with
    equal neighbours and sign changes of the slopes among them."""
    import torch
    r = np.random.default_rng(seed)
    shape = om.interior().shape
    u = 1.0 + 0.25 * r.integers(-3, 4, shape) + r.uniform(-0.1, 0.1, shape) * r.integers(0, 2, shape)
    u[:, -1] += 4.0
    if prec == 0:
        u = u.astype(np.float32).astype(np.float64)
    om.u[...] = 0.0
    om.interior()[...] = u
    gm.interior().copy_(torch.from_numpy(u).to(gm.dtype).cuda())


@pytest.mark.parametrize("physics", ["euler", "advection"])
@pytest.mark.parametrize("prec", [0, 1], ids=["f32", "f64"])
@pytest.mark.parametrize("ndim,N,g", SHAPES)
def test_remap_and_criterion_bit_exact(f4, ndim, N, g, prec, physics):
    """Four trees in a row, all neighbours of equal level where a stencil
    reaches into ghost cells: the first regrid refines tree 0, the second
    coarsens it again, refines tree 2 and copies the rest.  The remapped data
    and the criterion's flags before and after equal the oracle's."""
    kw = dict(physics=physics, velocity=(1.0, 0.5, 0.25)[:ndim]) if physics == "advection" else {}
    trees = (4, 1, 1)
    gm = f4.Mesh(ndim, trees, N, g, 1.0, max_level=1, max_blocks=4 + 2 * (1 << ndim), prec=prec, **kw)
    om = OracleMesh(ndim, trees, N, g, 1.0, **kw)

    def same(what):
        a, b = interior(gpu_state(gm), g, N, ndim), om.interior()
        if prec == 0:
            b = b.astype(np.float32).astype(np.float64)
        say("remap", what, ndim, N, g, prec, physics, "blocks", len(b), "differ", int(np.sum(a != b)))
        assert np.array_equal(a, b)

    def flags_same():
        om.ghost_fill()
        assert np.array_equal(gm.refine_flags(), om.lohner_flags())

    fill(gm, om, prec, 1)
    flags_same()
    f = np.array([1, 0, 0, 0], np.int8)
    assert gm.regrid(f) and om.regrid(f, 0, 1) is not None
    same("refine")
    fill(gm, om, prec, 2)
    lev, tree, _ = gm.export()
    f = np.where(lev == 1, -1, np.where(tree == 2, 1, 0)).astype(np.int8)
    assert gm.regrid(f)
    res = om.regrid(f, 0, 1)
    assert sorted(set(res[0].tolist())) == [0, 1, 2]
    assert all(np.array_equal(x, y) for x, y in zip(gm.export(), om.forest.export()))
    same("coarsen, refine and copy")

"""The FP64 arithmetic of the stage kernels at single-operation accuracy.
Every expectation is exact (no tolerance)."""
import sys

import numpy as np
import pytest

import synth
from tests.gpu_helpers import build_pair, gpu_state, interior
from tests.test_gpu_parity import small_uniform

pytestmark = pytest.mark.gpu


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


CFL_CASES = {
    "8": small_uniform(8, (4, 3, 2)),
    "16": small_uniform(16, (3, 2, 1)),
    "32": small_uniform(32, (1, 2, 1)),
    "2d": small_uniform(16, (3, 2), ndim=2),
    "vanleer-hll": dict(small_uniform(16, (2, 2, 2)), limiter="vanleer", flux="hll"),
    "gravity": dict(small_uniform(16, (2, 2, 2)), gravity=(0.0, 0.1, -0.2)),
    "weno5": dict(small_uniform(16, (2, 2, 1)), limiter="weno5", g=3),
    "weno5-2d": dict(small_uniform(8, (3, 2), ndim=2), limiter="weno5", g=3),
    "two-level": synth.two_level_blast(base_trees=4, block=8),
}


@pytest.mark.parametrize("form", ["plain", "batch"])
@pytest.mark.parametrize("name", list(CFL_CASES))
def test_step_dt_is_the_plain_evaluation(f4, name, form):
    """The time step that a step leaves behind (the CFL limits of the stage
    epilogue and the flux fix) is the one that foap4_compute_dt and the
    oracle's plain FP64 evaluation give for the same state, bit for bit."""
    w = CFL_CASES[name]
    gm, om = build_pair(w, 1)
    b = f4.Batch([gm]) if form == "batch" else None
    for step in range(3):
        (b or gm).step(1)
        left = gm.time()[1]
        om.u[...] = 0.0
        om.interior()[...] = interior(gpu_state(gm), w["g"], w["N"], w["ndim"])
        plain = om.dt()
        gm.compute_dt()
        say("step dt", name, form, step, left.hex(), gm.time()[1].hex(), plain.hex())
        assert left == plain
        assert gm.time()[1] == plain


@pytest.mark.parametrize("integrator", ["ssprk3", "ssprk43", "rk4"])
def test_step_dt_of_the_other_integrators(f4, integrator):
    w = small_uniform(16, (2, 2, 1))
    from paper_2605_07612_amd import layout
    gm = f4.Mesh(3, w["trees"], 16, 2, w["tree_size"], prec=f4.F64, gamma=w["gamma"], cfl=w["cfl"],
                 integrator=integrator)
    layout.set_from_field(gm, w["field"])
    gm.step(2)
    left = gm.time()[1]
    gm.compute_dt()
    assert left == gm.time()[1]


def test_wave_speed_root_is_correctly_rounded(f4):
    """d_bar of Rusanov's flux is a correctly rounded square root.  A shear
    layer on a gas at rest, rho = 1, v_z = 0 for x < 1/2 and 1 beyond, leaves
    one inexact step at a time: every slope is zero, u_bar is zero, sqrt(rho)
    is one, d_bar = sqrt(gamma p), and the only z-momentum flux of the cells at
    rest next to the layers is d_bar / 2, so that the first Heun stage leaves
    (dt / dx) d_bar / 2 in them (dx a power of two).  The energy, and with it
    p = (gamma - 1) E, differs from row to row in y, where nothing couples the
    z momenta of cells at rest."""
    from paper_2605_07612_amd import layout
    rows, gamma = 64, 1.4
    m = f4.Mesh(3, (2, rows, 1), 8, 2, 1.0, prec=f4.F64, gamma=gamma)
    e = 1.0 + np.random.default_rng(5).integers(0, 3 << 20, rows * 8) / (1 << 20)

    def field(x, y, z):
        vz = (x > 1.0).astype(float)
        E = e[np.floor(y * 8.0).astype(int)] + 0.5 * vz
        return np.stack([np.ones_like(x), 0 * x, 0 * x, vz, E])

    layout.set_from_field(m, field)
    m.compute_dt()
    dt = m.time()[1]
    m.step(1)
    _, G = layout.global_coords(m)
    u1 = m.interior(state=1 - m.cur).cpu().numpy()  # the first stage's result
    off = 0
    for n, g in enumerate(np.asarray(G)):
        if g[0] == 0:  # the blocks at rest, a layer on either side
            p = (gamma - 1.0) * e[8 * g[1]:8 * g[1] + 8]
            want = (dt * 8.0) * (0.5 * np.sqrt(gamma * p))
            for i in (0, 7):
                off += int(np.sum(u1[n, 3, :, :, i] != want[None, :]))
    say("shear layer: cells off the correctly rounded value:", off, "of", rows * 128)
    assert off == 0


@pytest.mark.parametrize("flux", ["rusanov", "hll"])
@pytest.mark.parametrize("k", [-600, 600])
def test_density_range(f4, flux, k):
    """The Euler equations scale with the density at fixed velocities: the
    conserved variables times 2^k (k even, far from the range's ends) take the
    same time steps and give the same states times 2^k, bit for bit."""
    w = small_uniform(16, (2, 2, 1))
    ms = []
    for s in (0, k):
        m = f4.Mesh(3, w["trees"], 16, 2, w["tree_size"], prec=f4.F64, gamma=w["gamma"], cfl=w["cfl"], flux=flux)
        from paper_2605_07612_amd import layout
        layout.set_from_field(m, lambda *x: np.ldexp(w["field"](*x), s))
        m.step(3)
        ms.append(m)
    a, b = (m.interior().cpu().numpy() for m in ms)
    say("density 2^", k, flux, "times", ms[0].time(), ms[1].time())
    assert ms[0].time() == ms[1].time()
    assert np.array_equal(np.ldexp(a, k), b)

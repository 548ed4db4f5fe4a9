"""Boxes around the largest that a 2D workgroup's tile holds (70 nodes in FP64, 114 in FP32): one
wave of nearly resting particles in a row of `cells` cells, a box of 3 (cells + 2) nodes, and the
same across the periodic seam.  Against the CPU oracle, tolerances as in
test_gpu_orbit_quadrature.py."""
import numpy as np
import pytest

import oracle as O
from paper_2609_36383_amd import workloads as W
from test_gpu_parity import _gpu, _rel, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seam", [False, True])
@pytest.mark.parametrize("shape", [2, 1])
@pytest.mark.parametrize("cells", [19, 20, 21, 22, 34, 35, 36, 37])
def test_box_at_the_tile_limit(cells, shape, seam):
    G = _gpu()
    n, h, dt, num = (64, 8), 0.2, 0.1, 64
    length = tuple(h * v for v in n)
    gphi, An, Anp1, _ = W.random_fields(2, n, length, seed=150, amp=0.3)
    Uh = (Anp1 - An) / dt
    rng = np.random.default_rng(151)
    first = 64 - cells // 2 if seam else 5
    col = first + np.sort(np.concatenate([np.arange(cells), rng.integers(0, cells, num - cells)]))
    x = np.stack([(h * (col + rng.uniform(-0.4, 0.4, num))) % length[0], h * (3.0 + rng.uniform(-0.4, 0.4, num))])
    q = -0.01 * rng.uniform(0.5, 1.5, num)
    P = rng.normal(size=(3, num)) * 0.01 * np.abs(q)[None, :]
    vbar = rng.uniform(-0.1, 0.1, (3, num))  # a twentieth of a cell
    kw = dict(dim=2, n=n, lo=(0.0, 0.0), length=length, dt=dt, shape_order=shape)
    osim = O.OracleSim(O.make_config(**kw, gl_order=8))
    u = np.zeros((3, num))
    osim.load_particles(x, u, q)
    osim.set_particle_state(x, P, vbar)
    ref = osim.orbit_pass(gphi, An, Anp1, Uh, vbar, iterate=False)
    for prec, tol in ((G.FP64, 1e-12), (G.FP32_BULK, 2e-5)):
        sim = G.Simulation(G.make_config(**kw, precision=prec), num)
        sim.load_particles(x, u, q)
        sim.set_particle_state(x, P, vbar)
        sim.set_frozen_fields(gphi, An, Anp1, Uh)
        rep = sim.orbit_pass_frozen(iterate=False)
        vout, Pn1, J = sim.read_pass()
        sim.close()
        err = (_rel(vout, ref["vout"]), _rel(Pn1, ref["Pnp1"]), _rel(J, ref["J"]))
        _say(f"{cells} cells S{shape} seam={seam} prec={prec}: v {err[0]:.1e} P {err[1]:.1e} J {err[2]:.1e}")
        assert rep["failed"] == 0 and max(err) < tol

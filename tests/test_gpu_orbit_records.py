"""3D orbit pass where the deposit's records follow the parked particle constants in the same
LDS: waves whose particles have charges decades apart and converge after different numbers
of evaluations, so a constant read after a record was written would show.

Tolerances: the frozen inner loop's 1e-11 (each side stops within tol 1e-12 of its own fixed
point), and the same bits from a second pass."""
import numpy as np
import pytest

import oracle as O
from paper_2609_36383_amd import workloads as W
from test_gpu_parity import _gpu, _rel, _say
from test_gpu_point_passes import MESH, _particles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("num", [64, 4033])
def test_mixed_charges_and_evaluation_counts(num):
    G = _gpu()
    dim, dt, seed = 3, 0.1, 70
    n, length = MESH[dim]
    gphi, An, Anp1, _ = W.random_fields(dim, n, length, seed=seed, amp=0.2)
    Uh = (Anp1 - An) / dt
    x, u, q = _particles(dim, num, "cells", seed + 1)
    rng = np.random.default_rng(seed + 2)
    q = q * 10.0 ** rng.uniform(-3.0, 0.0, num) * rng.choice([-1.0, 1.0], num)
    P = rng.normal(size=(3, num)) * 0.3 * np.abs(q)[None, :]
    vbar = rng.uniform(-0.5, 0.5, (3, num))
    kw = dict(dim=dim, n=n, lo=(0.0,) * dim, length=length, dt=dt)
    osim = O.OracleSim(O.make_config(**kw, gl_order=8))
    osim.load_particles(x, u, q)
    osim.set_particle_state(x, P, vbar)
    ref = osim.orbit_pass(gphi, An, Anp1, Uh, vbar, iterate=True)
    got = []
    for _ in range(2):
        sim = G.Simulation(G.make_config(**kw), num)
        sim.load_particles(x, u, q)
        sim.set_particle_state(x, P, vbar)
        sim.set_frozen_fields(gphi, An, Anp1, Uh)
        rep = sim.orbit_pass_frozen(iterate=True)
        got.append(sim.read_pass(iters=True))
        sim.close()
        assert rep["failed"] == 0
    vout, Pn1, J, it = got[0]
    err = (_rel(vout, ref["vout"]), _rel(Pn1 / np.abs(q), ref["Pnp1"] / np.abs(q)), _rel(J, ref["J"]))
    _say(f"np={num}: evaluations {it.min()}..{it.max()}, v {err[0]:.1e} P/|q| {err[1]:.1e} J {err[2]:.1e}")
    assert it[:64].max() > it[:64].min()
    assert max(err) < 1e-11
    assert all(np.array_equal(a, b) for a, b in zip(got[0], got[1]))

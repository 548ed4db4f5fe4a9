"""Rounding error of one FP32-bulk orbit evaluation against the FP64 oracle.

The bounds are those of quadrature at Gauss-Legendre points with both potentials kept as FP32
(root mean square over four seeded fields, of the largest value: v_out, P^{n+1}, J), and a
twentieth more, several times what other roundings of the same arithmetic move them by.  The
closed form with the difference of the two potentials gives P^{n+1} 1.10 (2D) and 1.27 (3D) of
them; with each potential's own weights 1.00 in 1D and 2D, 1.09 in 3D."""
import numpy as np
import pytest

import oracle as O
from paper_2609_36383_amd import workloads as W
from test_gpu_parity import _gpu, _say
from test_gpu_point_passes import MESH, _particles

pytestmark = pytest.mark.gpu

RMS = {  # (dim, shape): v_out, P^{n+1}, J
    (1, 2): (3.678e-8, 12.47e-8, 1.009e-8), (1, 1): (3.535e-8, 12.42e-8, 1.013e-8),
    (2, 2): (3.661e-8, 4.271e-8, 1.747e-8), (2, 1): (3.295e-8, 3.930e-8, 0.875e-8),
    (3, 2): (4.173e-8, 3.788e-8, 0.991e-8), (3, 1): (3.311e-8, 3.270e-8, 1.035e-8),
}


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("shape", [2, 1])
@pytest.mark.parametrize("gl", [0, 8])
def test_fp32_evaluation_error(dim, shape, gl):
    G = _gpu()
    n, length = MESH[dim]
    num, square = 6000, np.zeros(3)
    for seed in range(4):
        dt = (0.05, 0.2)[seed % 2]
        gphi, An, Anp1, _ = W.random_fields(dim, n, length, seed=seed, amp=0.3)
        Uh = (Anp1 - An) / dt
        x, u, q = _particles(dim, num, "cells", seed + 1)
        rng = np.random.default_rng(seed + 2)
        P = rng.normal(size=(3, num)) * 0.01 * np.abs(q)[None, :]
        vbar = rng.uniform(-0.9, 0.9, (3, num))
        kw = dict(dim=dim, n=n, lo=(0.0,) * dim, length=length, dt=dt, shape_order=shape)
        osim = O.OracleSim(O.make_config(**kw, gl_order=8))
        osim.load_particles(x, u, q)
        osim.set_particle_state(x, P, vbar)
        ref = osim.orbit_pass(gphi, An, Anp1, Uh, vbar, iterate=False)
        sim = G.Simulation(G.make_config(**kw, gl_order=gl, precision=G.FP32_BULK), num)
        sim.load_particles(x, u, q)
        sim.set_particle_state(x, P, vbar)
        sim.set_frozen_fields(gphi, An, Anp1, Uh)
        sim.orbit_pass_frozen(iterate=False)
        got = sim.read_pass()
        sim.close()
        square += [np.mean(((a - b) / np.abs(b).max()) ** 2) for a, b in
                   zip(got, (ref["vout"], ref["Pnp1"], ref["J"]))]
    rms = np.sqrt(square / 4)
    _say(f"d={dim} S{shape} gl={gl}: rms v {rms[0]:.3e} P {rms[1]:.3e} J {rms[2]:.3e}")
    assert all(r <= 1.05 * b for r, b in zip(rms, RMS[dim, shape]))

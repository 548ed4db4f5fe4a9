"""The passes over particles at one time on both sides of the rules that split their work: storage
order and the order by cell (from 65,536 particles and four to eight per cell on), windows of one
to four waves, several windows per workgroup (from 2,097,152 particles on), rows of one cell and
scattered particles in one workgroup.  Against the CPU oracle.

Tolerances as in test_gpu_point_passes.py: 1e-13 for momenta and velocities; sums of N values in
another order, N eps: 1e-11 up to 65,536 particles, 5e-10 at 2.1e6."""
import numpy as np
import pytest

import oracle as O
from paper_2609_36383_amd import workloads as W
from test_gpu_parity import _gpu, _rel, _say
from test_gpu_point_passes import MESH, _particles

pytestmark = pytest.mark.gpu


def _check(dim, shape, x, u, q, sums):
    G = _gpu()
    n, length = MESH[dim]
    _, A0, U0, _ = W.random_fields(dim, n, length, seed=95 + dim, amp=0.2)
    kw = dict(dim=dim, n=n, lo=(0.0,) * dim, length=length, dt=0.05, shape_order=shape)
    ref = O.OracleSim(O.make_config(**kw, gl_order=8))
    sim = G.Simulation(G.make_config(**kw), q.size)
    for s in (ref, sim):
        s.load_particles(x, u, q)
        s.load_potentials(A0, U0)
        s.initialize()
    (_, Po, vo), (_, P, v) = ref.read_particles(), sim.read_particles()
    do, d = ref.diagnostics(), sim.diagnostics()
    err = [_rel(P, Po), _rel(v, vo)]
    err += [_rel(sim.read_field(f), ref.read_field(f)) for f in ("rho", "J")]
    err += [abs(d[k] / do[k] - 1.0) for k in ("kinetic", "vperp_rms")]
    sim.close()
    _say(f"d={dim} S{shape} np={q.size}: P {err[0]:.1e} v {err[1]:.1e} rho {err[2]:.1e} J {err[3]:.1e} K {err[4]:.1e}")
    assert max(err[:2]) < 1e-13 and max(err[2:]) < sums


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("shape", [2, 1])
@pytest.mark.parametrize("num,order", [(65535, "random"), (65536, "random"), (65536, "cells")])
def test_order_by_cell(dim, shape, num, order):
    _check(dim, shape, *_particles(dim, num, order, 75 + dim), 1e-11)


@pytest.mark.parametrize("dim,num", [(1, 131073), (1, 262145), (1, 400001), (2, 524289)])
def test_window_lengths(dim, num):
    _check(dim, 2, *_particles(dim, num, "seam", 85 + dim), num * 2.3e-16)


@pytest.mark.parametrize("dim", [1, 2, 3])
def test_several_windows(dim):
    """A workgroup's windows: one cell's rows across several, and scattered stretches between
    (every third stretch of 256 particles shuffled over the whole box; the kinetic energy takes
    the storage order)."""
    num = 2 ** 21 + 4099
    x, u, q = _particles(dim, num, "cells", 105 + dim)
    rng = np.random.default_rng(115 + dim)
    at = np.flatnonzero((np.arange(num) // 256) % 3 == 1)
    o = np.arange(num)
    o[at] = rng.permutation(at)
    _check(dim, 2, *(np.ascontiguousarray(a[..., o]) for a in (x, u, q)), 5e-10)

"""The initial deposit does not depend on the particles' order: its sums are exact (fixed point), in
rows of one cell, for scattered particles and across workgroups alike, so the fields of the same
particles loaded in any order are equal to the bit.  Cell order, reversed and shuffled, on both
sides of the rule for the order by cell, with whole and cut windows; charges decades apart, so that a
rounded sum would depend on its order."""
import numpy as np
import pytest

from paper_2609_36383_amd import workloads as W
from test_gpu_parity import _gpu
from test_gpu_point_passes import MESH, _particles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("shape", [2, 1])
@pytest.mark.parametrize("num", [1, 999, 30011, 70001, 600000])
def test_fields_do_not_depend_on_the_order(dim, shape, num):
    G = _gpu()
    n, length = MESH[dim]
    x, u, q = _particles(dim, num, "cells", 160 + dim)
    rng = np.random.default_rng(170 + dim)
    q = q * 10.0 ** rng.uniform(-6.0, 0.0, num) * rng.choice([-1.0, 1.0], num)
    _, A0, U0, _ = W.random_fields(dim, n, length, seed=180 + dim, amp=0.2)
    ref = None
    for order in (np.arange(num), np.arange(num)[::-1], rng.permutation(num)):
        sim = G.Simulation(G.make_config(dim=dim, n=n, lo=(0.0,) * dim, length=length, dt=0.05, shape_order=shape), num)
        sim.load_particles(*(np.ascontiguousarray(a[..., order]) for a in (x, u, q)))
        sim.load_potentials(A0, U0)
        sim.initialize()
        got = [sim.read_field(f) for f in ("rho", "J", "phi")]
        sim.close()
        ref = ref or got
        assert all(np.array_equal(a, b) for a, b in zip(got, ref))

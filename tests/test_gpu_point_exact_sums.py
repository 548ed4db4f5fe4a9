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


def test_more_values_than_one_exact_sum_takes():
    """Above 8,192 particles per workgroup (67,108,864 in all) a row's sums are put away in between:
    here all particles sit in two cells, so that rows go on with one cell throughout."""
    import ctypes as C

    import torch
    G = _gpu()
    num, dev, f64 = 8192 * 8192 + 300007, "cuda:0", torch.float64
    n, length = MESH[1]
    g = torch.Generator(device=dev).manual_seed(190)
    h = length[0] / n[0]
    x = (31.5 + torch.rand(num, generator=g, device=dev, dtype=f64)) * h
    x[num // 2:] += h
    u = torch.rand(3, num, generator=g, device=dev, dtype=f64) - 0.5
    q = -(0.5 + torch.rand(num, generator=g, device=dev, dtype=f64)) / num
    # without the projector, which takes the Nyquist mode out of the fields read
    sim = G.Simulation(G.make_config(dim=1, n=n, lo=(0.0,), length=length, dt=0.05, project_nyquist=0), num, device=dev)
    ref = None
    for _ in range(2):
        sim.stream.wait_stream(torch.cuda.current_stream())
        ptr = [C.c_void_p(t.data_ptr()) for t in (x, u, q)]
        assert sim.lib.gmhc_load_particles(sim.h, *ptr, G.DEVICE) == G.OK
        sim.initialize()
        got = [sim.read_field(f) for f in ("rho", "J")]
        ref = ref or got
        x, u, q = x.flip(0), u.flip(1).contiguous(), q.flip(0)
    sim.close()
    assert all(np.array_equal(a, b) for a, b in zip(got, ref))
    # the charge of the two cells' nodes, against the sum over the particles
    total = float(got[0].sum() - got[0][0] * n[0]) * h
    assert abs(total / float(q.sum()) - 1.0) < 1e-12

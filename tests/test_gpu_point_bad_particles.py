"""A bad particle among good ones at initialization.  Positions are not checked
at load; the passes over particles at one time take a coordinate that is not finite (or 1e9
cells away) as the origin's on that axis, whatever the particle's place in its batch, and leave
the other particles as they are.  A particle whose velocity is not finite (a momentum that is
not, or no charge) deposits no current.  The reference is the oracle's run with the coordinate
put there, or with the particle at rest.

Tolerances as in test_gpu_point_passes.py: 1e-13 for momenta, N eps for sums, 1.5e-11 at these N."""
import numpy as np
import pytest

import oracle as O
from paper_2609_36383_amd import workloads as W
from test_gpu_parity import _gpu, _rel, _say

pytestmark = pytest.mark.gpu

N = {1: (16,), 2: (8, 16), 3: (8, 4, 8)}
H = 0.25  # a power of two: whole cells away is exact


def _inputs(dim, num, seed, i0):
    """Particles in cell order, and the first particle of the cell (i0, n1 / 2, n2 / 2)."""
    n = N[dim]
    length = tuple(H * v for v in n)
    x, u, q = W.random_particles(dim, n, length, num, seed, umax=0.5)
    key = np.zeros(num, dtype=np.int64)
    for i in reversed(range(dim)):
        key = key * n[i] + np.floor(x[i] / H + 0.5).astype(np.int64) % n[i]
    o = np.argsort(key, kind="stable")
    x, u, q, key = x[:, o], u[:, o], q[o], key[o]
    mid = i0 + sum((n[i] // 2) * int(np.prod(n[:i])) for i in range(1, dim))
    return n, length, np.ascontiguousarray(x), np.ascontiguousarray(u), np.ascontiguousarray(q), int(np.argmax(key >= mid))


def _state(cls, cfg, x, u, q, A0, U0):
    sim = cls(cfg, q.size) if cls is not O.OracleSim else cls(cfg)
    sim.load_particles(x, u, q)
    sim.load_potentials(A0, U0)
    sim.initialize()
    return sim, sim.read_particles(), {f: sim.read_field(f) for f in ("rho", "J")}


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("shape", [2, 1])
@pytest.mark.parametrize("num", [1543, 65543])  # in storage order, and in the order by cell
@pytest.mark.parametrize("bad", ["nan", "inf", "far", "cells_away"])
def test_bad_position(dim, shape, num, bad):
    G = _gpu()
    # its cell as the passes take it: column 0, or its own
    n, length, x, u, q, b = _inputs(dim, num, 50 + dim, N[dim][0] // 2 if bad == "cells_away" else 0)
    _, A0, U0, _ = W.random_fields(dim, n, length, seed=60 + dim, amp=0.2)
    xg, xo = x.copy(), x.copy()
    if bad == "cells_away":  # 2^28 cells: wrapped like any other position
        xo[0, b] = H * (round(x[0, b] / H) + 0.125)
        xg[0, b] = xo[0, b] + H * 2.0 ** 28
    else:
        xg[0, b] = {"nan": np.nan, "inf": -np.inf, "far": 1e300}[bad]
        xo[0, b] = 0.0
    kw = dict(dim=dim, n=n, lo=(0.0,) * dim, length=length, dt=0.05, shape_order=shape)
    _, (_, Po, vo), fo = _state(O.OracleSim, O.make_config(**kw, gl_order=8), xo, u, q, A0, U0)
    sim, (_, Pg, vg), fg = _state(G.Simulation, G.make_config(**kw), xg, u, q, A0, U0)
    sim.close()
    err = [_rel(Pg, Po), _rel(vg, vo)] + [_rel(fg[f], fo[f]) for f in ("rho", "J")]
    _say(f"d={dim} S{shape} {bad} particle {b} of {num}: P {err[0]:.1e} v {err[1]:.1e} rho {err[2]:.1e} J {err[3]:.1e}")
    assert max(err[:2]) < 1e-13 and max(err[2:]) < 1.5e-11


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("shape", [2, 1])
@pytest.mark.parametrize("num", [1543, 65543])
@pytest.mark.parametrize("bad", ["momentum_nan", "momentum_inf", "no_charge"])
def test_velocity_not_finite(dim, shape, num, bad):
    G = _gpu()
    n, length, x, u, q, b = _inputs(dim, num, 70 + dim, N[dim][0] // 2)
    _, A0, U0, _ = W.random_fields(dim, n, length, seed=80 + dim, amp=0.2)
    ug, uo, qg, qo = u.copy(), u.copy(), q.copy(), q.copy()
    uo[:, b] = 0.0
    if bad == "no_charge":
        qg[b], qo[b] = 0.0, 1e-40
    else:
        ug[1, b] = np.nan if bad == "momentum_nan" else np.inf
    kw = dict(dim=dim, n=n, lo=(0.0,) * dim, length=length, dt=0.05, shape_order=shape)
    _, (_, Po, vo), fo = _state(O.OracleSim, O.make_config(**kw, gl_order=8), x, uo, qo, A0, U0)
    sim, (_, Pg, vg), fg = _state(G.Simulation, G.make_config(**kw), x, ug, qg, A0, U0)
    sim.close()
    good = np.arange(num) != b
    err = [_rel(Pg[:, good], Po[:, good]), _rel(vg[:, good], vo[:, good])] + [_rel(fg[f], fo[f]) for f in ("rho", "J")]
    _say(f"d={dim} S{shape} {bad} of {num}: P {err[0]:.1e} v {err[1]:.1e} rho {err[2]:.1e} J {err[3]:.1e}")
    assert max(err[:2]) < 1e-13 and max(err[2:]) < 1.5e-11

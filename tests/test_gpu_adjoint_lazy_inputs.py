"""Device particles whose tensors carry a lazy negation (torch's negative bit, as of the imaginary
part of a conjugate) load as the values they stand for: energy and gradients to the bit."""
import pytest
import torch

from paper_2609_36383_amd import adjoint as A
from paper_2609_36383_amd import gmhc as G
from paper_2609_36383_amd import workloads as W
from test_gpu_adjoint_inputs import _grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", [0, 1, 2])
def test_negative_bit(which):
    w = W.spec("weibel2d", n=(8, 8), ppc=9)
    cfg = G.config_from_dict(W.config_dict(w))
    x, u, q = (torch.as_tensor(a).cuda() for a in W.particles(w))
    u = u + 0.1 * torch.linspace(0.0, 1.0, u.numel(), dtype=torch.float64, device=u.device).reshape(u.shape)
    ref = _grads(x, u, q, cfg)
    lazy = [x, u, q]
    lazy[which] = torch._neg_view(-lazy[which])
    assert lazy[which].is_neg()
    leaves = [t.detach().requires_grad_(True) for t in lazy]
    assert leaves[which].is_neg()
    e = A.field_energy_run(*leaves, cfg, 2, 1, "cuda:0")
    e.backward()
    got = [e.detach()] + [t.grad.cpu() for t in leaves]
    assert all(torch.equal(a, b) for a, b in zip(got, ref))

"""The 1-D MGE kernels' division of the work (32 lanes per amplitude, a wave per
component's derivatives, a bounded grid): one profile and more than the grid
takes at once, one Gaussian and the most, fewer and more terms than lanes.  A
profile's results do not depend on the others', bit for bit, and keep the 1e-9 of
the largest that the transform's cancellation allows against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import mge1d as omge
from paper_2504_01302_amd import binding

pytestmark = pytest.mark.gpu


def _run(comp, sig, cot, P, dev):
    c, w = (torch.as_tensor(v, device=dev) for v in (comp, cot))
    amp = binding.jam_mge1d(c, sig, P)
    grad = binding.jam_mge1d_vjp(c, sig, w, P)
    return amp.cpu().numpy(), grad.cpu().numpy()


@pytest.mark.parametrize("n_prof,n_sigma,P", [(1, 1, 10), (3, 64, 12), (9000, 64, 10), (70, 5, 20)])
def test_many_profiles(n_prof, n_sigma, P):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n_prof + P)
    sig = omge.sigma_grid(0.02, 20.0, n_sigma) if n_sigma > 1 else np.array([0.5])
    comp = np.zeros((n_prof, 3, 3))
    comp[:, :, 0] = rng.uniform(-1.0, 1.0, (n_prof, 3))
    comp[:, :, 1] = rng.uniform(0.05, 2.0, (n_prof, 3))
    comp[:, :, 2] = rng.uniform(0.5, 1.5, (n_prof, 3))
    cot = rng.standard_normal((n_prof, n_sigma))
    amp, grad = _run(comp, sig, cot, P, dev)
    assert np.isfinite(amp).all() and np.isfinite(grad).all()
    for i in sorted({0, n_prof // 2, n_prof - 1}):
        a1, g1 = _run(comp[i:i + 1], sig, cot[i:i + 1], P, dev)
        assert np.array_equal(amp[i], a1[0]) and np.array_equal(grad[i], g1[0])
        if P > 12:      # the Euler sum's cancellation grows tenfold per three terms
            continue
        leaf = torch.tensor(comp[i], requires_grad=True)
        ref = omge.mge_amplitudes(leaf, sig, P)
        (g,) = torch.autograd.grad(torch.sum(ref * torch.as_tensor(cot[i])), [leaf])
        ref = ref.detach().numpy()
        assert np.max(np.abs(amp[i] - ref)) <= 1e-9 * np.max(np.abs(ref))
        assert np.max(np.abs(grad[i] - g.numpy())) <= 1e-9 * np.max(np.abs(g.numpy()))

"""The spherical model's polar potential grid (form 0) against the direct sums
over the (j, u) terms at every node (form 1), at the sizes where its kernels'
divisions of the work begin, end or leave a remainder."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from test_gpu_sph import KEYS, _dev, _eval  # noqa: E402

from paper_2504_01302_amd import binding, inputs  # noqa: E402

pytestmark = pytest.mark.gpu


def _workload(n_lum, n_mass, n_u, kind, seed):
    g = inputs.small_geometry(seed=seed, n_lum=n_lum, n_mass=n_mass, nx=8, ny=7, ss=1, psf_n=3,
                              n_bins=4, n_u=n_u)
    if kind == "round":             # q' = 1 throughout: the columns' scale s0 = 1
        g.lum_q[:] = 1.0
        g.mass_q[:] = 1.0
    if kind == "narrow":            # nothing left of all tracers but one over most radii
        g.lum_sigma[1:] *= 0.02
    p = inputs.small_params(g, seed=seed)
    if kind == "thin":              # axial ratios down to 0.04, at 87.5 degrees
        g.mass_q[0] = 0.06
        p = inputs.with_overrides(p, inc=float(np.radians(87.5)))
    return g, inputs.Workload("w", [g], np.zeros(1, np.int32), [p])


@pytest.mark.parametrize("n_lum,n_mass,n_u,kind", [
    (1, 1, 16, "plain"),      # one tracer, one group, terms below one 64-term chunk
    (2, 3, 100, "plain"),     # a full cotangent group; 400 terms, one slice
    (3, 8, 98, "thin"),       # a half-filled group; 882 terms: two slices, uneven chunks
    (5, 8, 64, "round"),
    (6, 5, 64, "narrow"),     # (tracer, radius) pairs that are left out
    (21, 4, 64, "plain"),     # two tracers per moments wave, the last alone
    (41, 16, 60, "plain"),    # three tracers per cotangent group; 1020 terms: 512-term tiles
])
def test_polar_grid_vs_direct_sums(n_lum, n_mass, n_u, kind):
    """Both forms take FP32 exponentials of the same coefficients; they differ
    by the rounding of the exponents' squared coordinates (up to 20 x 6e-8 of a
    term) and the grid's interpolation (1e-7).  Forward bar 2e-6 per bin, the
    bar of the other comparison of the two forms; gradient 1e-5 of the norm,
    five times that for the sums of both signs."""
    dev = _dev()
    g, w = _workload(n_lum, n_mass, n_u, kind, seed=n_lum + n_mass)
    out = []
    for form in (0, 1):
        ctx = binding.Context([g], alignment=1, form=form)
        V, st = _eval(ctx, w, dev)
        assert int(st[0]) == 0
        pk = binding.pack_params(w, dev, amplitudes=True)
        Vd, _ = ctx.eval_batch(w.geom_idx, pk["inc"], pk["mass_scale"], pk["m_bh"], pk["beta"],
                               pk["lum_I0"], pk["mass_S0"])
        cot = torch.as_tensor(np.random.default_rng(3).standard_normal(len(V)), device=dev)
        gr = ctx.vjp(w.geom_idx, pk["inc"], pk["mass_scale"], pk["m_bh"], pk["beta"],
                     pk["lum_I0"], pk["mass_S0"], Vd, cot)
        out.append((V, np.concatenate([np.atleast_1d(gr[k].cpu().numpy()) for k in KEYS])))
        ctx.close()
    (Va, ga), (Vb, gb) = out
    err = np.max(np.abs(Va / Vb - 1))
    gerr = np.linalg.norm(ga - gb) / np.linalg.norm(gb)
    print(f"K={n_lum} J={n_mass} n_u={n_u} {kind}: forward {err:.2e}, gradient {gerr:.2e}")
    assert err <= 2e-6
    assert gerr <= 1e-5


def test_polar_grid_is_the_same_in_any_batch():
    """Values and gradients of a model alone and among others, bit for bit."""
    dev = _dev()
    g, w1 = _workload(7, 6, 90, "plain", seed=2)
    ps = [inputs.small_params(g, seed=s) for s in (5, 2, 9)]
    w3 = inputs.Workload("w3", [g], np.zeros(3, np.int32), ps)
    ctx = binding.Context([g], alignment=1)
    res = []
    for w, at in ((w1, 0), (w3, 1)):
        pk = binding.pack_params(w, dev, amplitudes=True)
        args = (w.geom_idx, pk["inc"], pk["mass_scale"], pk["m_bh"], pk["beta"], pk["lum_I0"],
                pk["mass_S0"])
        V, _ = ctx.eval_batch(*args)
        nb = g.n_bins
        cot = torch.ones_like(V)
        gr = ctx.vjp(*args, V, cot)
        sel = [V.cpu().numpy()[at * nb:(at + 1) * nb]]
        for k in KEYS:
            a = gr[k].cpu().numpy()
            n = a.size // len(w.params)
            sel.append(a.reshape(-1)[at * n:(at + 1) * n])
        res.append(np.concatenate(sel))
    ctx.close()
    assert np.array_equal(res[0], res[1])


@pytest.mark.parametrize("n_lum", [3, 64, 70])
def test_gradient_does_not_depend_on_the_tracers_order(n_lum):
    """The node scale follows the tracer of the smallest sigma q, found over 64
    lanes: at the front, at the back and, with 70 tracers, in a lane's second
    turn.  Only the order of FP64 sums differs: 1e-9 of the gradient's norm."""
    dev = _dev()
    g, w = _workload(n_lum, 3, 40, "plain", seed=4)
    order = np.arange(n_lum)[::-1]
    rev = g.__class__(**{**g.__dict__, **{k: getattr(g, k)[order].copy()
                                          for k in ("lum_sigma", "lum_q", "lum_I0")}})
    out = []
    for geom, perm in ((g, np.arange(n_lum)), (rev, order)):
        p = inputs.with_overrides(w.params[0], beta=np.asarray(w.params[0].beta)[perm])
        wl = inputs.Workload("w", [geom], np.zeros(1, np.int32), [p])
        ctx = binding.Context([geom], alignment=1)
        pk = binding.pack_params(wl, dev, amplitudes=True)
        args = (wl.geom_idx, pk["inc"], pk["mass_scale"], pk["m_bh"], pk["beta"], pk["lum_I0"],
                pk["mass_S0"])
        V, st = ctx.eval_batch(*args)
        assert int(st[0]) == 0
        gr = ctx.vjp(*args, V, torch.ones_like(V))
        res = {k: np.atleast_1d(gr[k].cpu().numpy()) for k in KEYS}
        for k in ("beta", "lum_I0"):
            res[k] = res[k][np.argsort(perm)]
        out.append(res)
        ctx.close()
    for k in KEYS:
        a, b = out[0][k], out[1][k]
        assert np.linalg.norm(a - b) <= 1e-9 * np.linalg.norm(b), k


@pytest.mark.parametrize("margin", [1e-4, 1e-6, 1e-8, 1e-12])
def test_near_the_deprojection_limit(margin):
    """The flattest mass Gaussian's q^2 down to 1e-12: the grid's columns have to
    follow the terms' 1 / h, which u < 1 bounds.  Against the direct sums, at the
    bars against the oracle (1e-5 per bin, 1e-4 of the gradient's norm)."""
    dev = _dev()
    g = inputs.small_geometry(seed=3, n_lum=3, n_mass=4, nx=15, ny=15, n_bins=5, n_u=100,
                              pixsize=0.06)
    p = inputs.small_params(g, seed=12)
    q = float(np.concatenate([g.lum_q, g.mass_q]).min())
    p = inputs.with_overrides(p, inc=float(np.arccos(q - margin)))
    w = inputs.Workload("l", [g], np.zeros(1, np.int32), [p])
    out = []
    for form in (0, 1):
        ctx = binding.Context([g], alignment=1, form=form)
        pk = binding.pack_params(w, dev, amplitudes=True)
        args = (w.geom_idx, pk["inc"], pk["mass_scale"], pk["m_bh"], pk["beta"], pk["lum_I0"],
                pk["mass_S0"])
        V, st = ctx.eval_batch(*args)
        assert int(st[0]) == 0
        gr = ctx.vjp(*args, V, torch.ones_like(V))
        out.append((V.cpu().numpy(), np.concatenate([gr[k].cpu().numpy() for k in KEYS])))
        ctx.close()
    (Va, ga), (Vb, gb) = out
    err, gerr = np.max(np.abs(Va / Vb - 1)), np.linalg.norm(ga - gb) / np.linalg.norm(gb)
    print(f"{margin:.0e} inside: forward {err:.2e}, gradient {gerr:.2e}")
    assert err <= 1e-5 and gerr <= 1e-4


def test_flattening_that_rounds_to_zero():
    """q^2 = q'^2 - cos^2 i above zero, but 1 - e^2 = 0 in FP64: a valid model, whose
    grid must not lose its columns."""
    dev = _dev()
    g, w = _workload(2, 3, 64, "plain", seed=5)
    g.mass_q[0] = 0.01
    inc = float(np.arccos(0.01))
    seen = 0
    for _ in range(40):                       # a few ulp around the limit
        p = inputs.with_overrides(w.params[0], inc=inc)
        one = inputs.Workload("z", [g], np.zeros(1, np.int32), [p])
        ctx = binding.Context([g], alignment=1)
        V, st = _eval(ctx, one, dev)
        if int(st[0]) == 0:
            assert np.all(np.isfinite(V)), inc
            seen += 1
        ctx.close()
        inc = np.nextafter(inc, np.pi)
    assert seen > 10


def test_tracers_that_just_underflow():
    """Tracers whose exponent at one of the table's radii is that from which a
    (tracer, radius) is left out, to the last bit: the moments and the spread have to
    agree on which are, or the spread reads nodes that nothing wrote (the workspace
    is filled with NaN)."""
    dev = _dev()
    g = inputs.small_geometry(seed=8, n_lum=60, n_mass=3, nx=9, ny=9, psf_n=1, n_bins=4, n_u=32)
    g.lum_q[:] = 1.0
    g.lum_sigma[0] = 2.0
    x = (np.arange(9) - 4) * g.pixsize
    rs = np.hypot(x[:, None], x[None, :])
    lo, hi = 0.5 * rs[rs > 0].min(), 12.0 * 2.0
    r = np.exp(np.log(lo) + np.arange(128) * (np.log(hi) - np.log(lo)) / 127)
    # exponent r^2 / 2 sigma^2 = 750, a few ulp to either side
    g.lum_sigma[1:] = r[20:79] / np.sqrt(1500.0) * (1.0 + 1.1e-16 * (np.arange(59) % 9 - 4))
    p = inputs.small_params(g, seed=8)
    w = inputs.Workload("u", [g], np.zeros(1, np.int32), [p])
    ctx = binding.Context([g], alignment=1)
    pk = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, pk["inc"], pk["mass_scale"], pk["m_bh"], pk["beta"], pk["lum_I0"],
            pk["mass_S0"])
    V, st = ctx.eval_batch(*args)
    assert int(st[0]) == 0
    ctx.workspace(w.geom_idx, True, dev).fill_(255)
    gr = ctx.vjp(*args, V, torch.ones_like(V))
    for k in KEYS:
        assert torch.isfinite(gr[k]).all(), k
    ctx.close()

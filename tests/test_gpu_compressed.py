"""The compressed cylindrical form (terms interpolated onto Chebyshev nodes of
their exponents, all FP64) against the FP64 oracle, forward and adjoint, where
it can go wrong: tile edges, off-centre and elongated fields, more than 256
columns, the widest node sets (inclination at the deprojection limit), the
black hole alone, tracers whose light ends inside the field, a batch mixed
with the other forms.

Bars: the interpolants of one term are within 2 rho^-8, rho = 9 (eight nodes
an octave in v: exp(-z e^s) is bounded by 1 for |Im s| < pi / 2), about 5e-8 of
the term, with alternating signs over the terms; V per bin within 1e-7, the
gradient in norm within 1e-7 (the FP32 forms are held to 1e-5 and 1e-4)."""
import json
import os

import numpy as np
import pytest
import torch

from oracle import jam as ojam
from paper_2504_01302_amd import binding, inputs

pytestmark = pytest.mark.gpu

KEYS = ("inc", "beta", "mass_scale", "m_bh", "lum_I0", "mass_S0")


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


# name: geometry sizes, inclination as cos i = q_min - margin (None: drawn)
CASES = {
    "33x33": (dict(n_lum=2, n_mass=13, nx=64, ny=64, n_u=160, pixsize=0.05, psf_n=3), None),
    "32x129": (dict(n_lum=2, n_mass=14, nx=62, ny=256, n_u=160, pixsize=0.05, psf_n=3), None),
    "off_centre": (dict(n_lum=2, n_mass=13, nx=70, ny=41, n_u=150, pixsize=0.04, psf_n=3,
                        xc=0.013, yc=-0.007), None),
    "off_the_galaxy": (dict(n_lum=3, n_mass=13, nx=40, ny=66, n_u=150, pixsize=0.04, psf_n=1,
                            xc=2.5, yc=1.1), None),
    "over_256_columns": (dict(n_lum=2, n_mass=13, nx=290, ny=35, n_u=160, pixsize=0.03, psf_n=3,
                              xc=0.011), None),
    "black_hole_alone": (dict(n_lum=3, n_mass=0, nx=140, ny=140, n_u=1024, pixsize=0.05, psf_n=3), None),
    "limit_1e-2": (dict(n_lum=3, n_mass=13, nx=66, ny=70, n_u=160, pixsize=0.05, psf_n=3), 1e-2),
    "limit_1e-4": (dict(n_lum=3, n_mass=13, nx=66, ny=70, n_u=160, pixsize=0.05, psf_n=3), 1e-4),
    "limit_1e-8": (dict(n_lum=3, n_mass=13, nx=66, ny=70, n_u=160, pixsize=0.05, psf_n=3), 1e-8),
}


def _model(name, seed=0):
    kw, margin = CASES[name]
    g = inputs.small_geometry(seed=300 + seed, n_bins=5, **kw)
    p = inputs.small_params(g, seed=400 + seed)
    if margin is not None:
        q = float(np.concatenate([g.lum_q, g.mass_q]).min())
        p = inputs.with_overrides(p, inc=float(np.arccos(q - margin)))
    return g, p


def _run(g, p, cot, dev, n=1000):
    """The model as the last of a batch of n copies with other black holes (a
    batch large enough for the compressed form to be chosen)."""
    ps = [inputs.with_overrides(p, m_bh=p.m_bh * (1.0 + 0.001 * (n - 1 - m))) for m in range(n)]
    w = inputs.Workload("compressed", [g], np.zeros(n, np.int32), ps)
    ctx = binding.Context([g])
    kernel = ctx.plan_info(w.geom_idx)["num_kernel"]
    t = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, t["inc"], t["mass_scale"], t["m_bh"], t["beta"], t["lum_I0"], t["mass_S0"])
    V, st = ctx.eval_batch(*args)
    cot = torch.as_tensor(np.tile(cot, n), device=dev)
    gr = ctx.vjp(*args, V, cot)
    gr2 = ctx.vjp(*args, None, cot)         # V recomputed inside
    torch.cuda.synchronize()
    assert np.all(st.cpu().numpy() == 0)
    for k in KEYS:
        assert torch.equal(gr[k], gr2[k]), k
    out = V.cpu().numpy()[-g.n_bins:], {k: v.cpu().numpy()[len(v) // n * (n - 1):]
                                        for k, v in gr.items()}, kernel
    ctx.close()
    return out


def _check(name, g, p, cot, V, grad):
    ref, gref = ojam.vrms2_and_grad(g, p, cot)
    rel = np.max(np.abs(V / ref.numpy() - 1))
    a = np.concatenate([np.atleast_1d(grad[k]) for k in KEYS])
    b = np.concatenate([np.atleast_1d(gref[k].numpy()) for k in KEYS])
    gerr = np.linalg.norm(a - b) / np.linalg.norm(b)
    print(f"{name}: V {rel:.2e}, gradient {gerr:.2e}")
    assert rel <= 1e-7 and gerr <= 1e-7


@pytest.mark.parametrize("name", list(CASES))
def test_compressed_matches_oracle(name):
    dev = _dev()
    g, p = _model(name)
    cot = np.random.default_rng(5).standard_normal(g.n_bins)
    V, grad, kernel = _run(g, p, cot, dev)
    assert kernel == 4
    _check(name, g, p, cot, V, grad)


def test_compact_light_on_a_wide_field():
    """Tracers that end inside the field (units that reach no outer tile), with
    a wide one that carries the outer bins."""
    dev = _dev()
    g, p = _model("33x33", seed=1)
    g.lum_sigma[:] = (0.02, 1.5)
    cot = np.random.default_rng(6).standard_normal(g.n_bins)
    V, grad, kernel = _run(g, p, cot, dev)
    assert kernel == 4
    _check("compact light", g, p, cot, V, grad)


@pytest.mark.parametrize("q,n_u,margin", [(0.03, 160, None), (0.005, 160, None), (0.005, 1024, None),
                                          (None, 160, 1e-3), (None, 160, 1e-6)])
def test_thin_mass_seen_edge_on(q, n_u, margin):
    """Mass Gaussians whose exponents in y exceed those in x by 1 / q^2 (the
    linear panel's stretches): all of them thin and seen edge-on, or one, as
    wide as the field, next to the deprojection limit."""
    dev = _dev()
    g = inputs.small_geometry(seed=320, n_lum=2, n_mass=13, nx=100, ny=100, n_u=n_u,
                              pixsize=0.054, psf_n=3, n_bins=5)
    p = inputs.small_params(g, seed=420)
    g.lum_q[:] = 0.8
    if q is not None:
        g.mass_q[:] = q
        p = inputs.with_overrides(p, inc=np.pi / 2)
    else:
        j = int(np.argmin(g.mass_q))
        g.mass_sigma[j] = 0.9 * 50 * 0.054
        p = inputs.with_overrides(p, inc=float(np.arccos(g.mass_q[j] - margin)))
    cot = np.random.default_rng(7).standard_normal(g.n_bins)
    V, grad, kernel = _run(g, p, cot, dev)
    assert kernel == 4
    _check(f"thin {q} {n_u} {margin}", g, p, cot, V, grad)


def test_mixed_batch_and_invalid_model():
    """Compressed, small-map and invalid models in one batch: each as it is
    alone; the invalid one NaN."""
    dev = _dev()
    a, pa = _model("off_centre")
    b, pb = _model("33x33")
    c = inputs.small_geometry(seed=9)
    pc = inputs.small_params(c, seed=9)
    bad = inputs.with_overrides(pb, inc=0.2)
    n = 600
    gs, gi, ps = [a, b, c], [0, 1, 2, 1] * n, [pa, pb, pc, bad] * n
    rng = np.random.default_rng(7)
    cots = [rng.standard_normal(gs[i].n_bins) for i in gi]
    w = inputs.Workload("mixed", gs, np.asarray(gi, np.int32), ps)
    ctx = binding.Context(gs)
    t = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, t["inc"], t["mass_scale"], t["m_bh"], t["beta"], t["lum_I0"], t["mass_S0"])
    V, st = ctx.eval_batch(*args)
    g = ctx.vjp(*args, V, torch.as_tensor(np.concatenate(cots), device=dev))
    torch.cuda.synchronize()
    assert st.cpu().tolist() == [0, 0, 0, 2] * n
    V = V.cpu().numpy()
    nb = [gs[i].n_bins for i in gi]
    o = np.cumsum([0] + nb)
    assert np.all(np.isnan(V[o[3]:o[4]])) and np.isnan(g["inc"][3].item())
    ol = np.cumsum([0] + [gs[i].n_lum for i in gi])
    om = np.cumsum([0] + [gs[i].n_mass for i in gi])
    for m in range(2):
        gm = dict(inc=g["inc"][m].item(), mass_scale=g["mass_scale"][m].item(),
                  m_bh=g["m_bh"][m].item(), beta=g["beta"][ol[m]:ol[m + 1]].cpu().numpy(),
                  lum_I0=g["lum_I0"][ol[m]:ol[m + 1]].cpu().numpy(),
                  mass_S0=g["mass_S0"][om[m]:om[m + 1]].cpu().numpy())
        _check(f"model {m}", gs[gi[m]], ps[m], cots[m], V[o[m]:o[m + 1]], gm)
    ctx.close()


def test_noalloc_takes_what_the_direct_forms_fit():
    """A composition whose direct forms fit the allocation-free entry point's
    scratch stays accepted by it: the compressed models then share their
    workspace in groups, with the same results bit for bit."""
    dev = _dev()
    g = inputs.small_geometry(seed=320, n_lum=20, n_mass=9, nx=70, ny=41, n_u=120, pixsize=0.04,
                              psf_n=3, n_bins=5, xc=0.013, yc=-0.007)
    n = 36
    ps = [inputs.small_params(g, seed=500 + m) for m in range(n)]
    w = inputs.Workload("many", [g], np.zeros(n, np.int32), ps)
    ctx = binding.Context([g])
    t = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, t["inc"], t["mass_scale"], t["m_bh"], t["beta"], t["lum_I0"], t["mass_S0"])
    V, st = ctx.eval_batch(*args)
    assert ctx.plan_info(w.geom_idx)["num_kernel"] == 4
    ws = binding.jam_workspace_size(ctx.handle, w.geom_idx, False)
    assert 40 << 20 < ws <= 64 << 20
    V2, st2 = torch.full_like(V, float("nan")), torch.empty_like(st)
    binding.jam_eval_batch_noalloc(ctx.handle, *args, V2, st2,
                                   torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(V, V2) and torch.equal(st, st2)
    ctx.close()


def _best_us(call):
    best = np.inf
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(10):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, 100.0 * a.elapsed_time(b))
    return best


def _call_us(g, n, form, dev):
    ps = [inputs.small_params(g, seed=600 + m) for m in range(n)]
    w = inputs.Workload("timed", [g], np.zeros(n, np.int32), ps)
    ctx = binding.Context([g], form=form)
    t = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, t["inc"], t["mass_scale"], t["m_bh"], t["beta"], t["lum_I0"], t["mass_S0"])
    best = _best_us(lambda: ctx.eval_batch(*args))
    ctx.close()
    return best


@pytest.mark.parametrize("nx,n,n_mass,n_u", [(84, 232, 12, 100), (130, 70, 12, 100),
                                             (130, 150, 12, 100), (280, 200, 4, 60),
                                             (430, 36, 6, 40)])
def test_automatic_form_is_not_the_slower_one(nx, n, n_mass, n_u):
    """Maps of two and three blocks a side with 1300 terms per tracer and of five and
    seven with 300, near the break-even of the compressed form: the automatic choice
    within a tenth of the direct forms (the compressed one took a third longer), also
    where its workspace exceeds the allocation-free scratch and the direct forms' does
    not (in many groups of models it took a fifth longer)."""
    dev = _dev()
    g = inputs.small_geometry(seed=330, n_lum=10, n_mass=n_mass, nx=nx, ny=nx, n_u=n_u,
                              pixsize=0.05 if nx < 200 else 0.025, psf_n=9, n_bins=20)
    auto, direct = _call_us(g, n, 0, dev), _call_us(g, n, 2, dev)
    print(f"{nx} x {nx}, {n} models: automatic {auto:.0f} us, direct {direct:.0f} us")
    assert auto <= 1.1 * direct


def test_uneven_adjoint_is_not_the_slower_one():
    """Off-centre maps of 67 to 203 pixels a side with few terms, of which some gain in
    the compressed form by themselves: beside the others' launches they do not (the
    adjoint took 1.3 times as long as the direct one)."""
    dev = _dev()
    rng = np.random.default_rng(8)
    gs = [inputs.small_geometry(seed=340 + m, n_lum=int(rng.integers(2, 6)),
                                n_mass=int(rng.integers(2, 8)), nx=int(rng.integers(67, 204)),
                                ny=int(rng.integers(67, 204)), n_u=int(rng.integers(24, 161)),
                                pixsize=0.04, psf_n=9, n_bins=20, xc=0.011, yc=-0.007)
          for m in range(63)]
    ps = [inputs.small_params(g, seed=700 + m) for m, g in enumerate(gs)]
    w = inputs.Workload("uneven", gs, np.arange(63, dtype=np.int32), ps)
    t = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, t["inc"], t["mass_scale"], t["m_bh"], t["beta"], t["lum_I0"], t["mass_S0"])
    us = {}
    for form in (0, 2):
        ctx = binding.Context(gs, form=form)
        V, _ = ctx.eval_batch(*args)
        us[form] = _best_us(lambda: ctx.vjp(*args, V, torch.ones_like(V)))
        ctx.close()
    print(f"automatic {us[0]:.0f} us, direct {us[2]:.0f} us")
    assert us[0] <= 1.1 * us[2]


def _golden(name):
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", name)
    if not os.path.exists(path):
        pytest.skip(f"{name} not generated")
    return json.load(open(path))


@pytest.mark.parametrize("name,make", [("cfg2_seed0.json", inputs.config2),
                                       ("composite_seed0.json", inputs.config_composite)])
def test_full_size_maps_in_the_automatic_form(name, make):
    """The IFU-scale and the composite model's sampled maps."""
    dev = _dev()
    gd = _golden(name)
    w = make(seed=0)
    g = w.geometries[0]
    ctx = binding.Context(w.geometries)
    assert ctx.plan_info(w.geom_idx)["num_kernel"] == 4
    p = binding.pack_params(w, dev)
    N, I, st = ctx.eval_maps(w.geom_idx, p["inc"], p["mass_scale"], p["m_bh"], p["beta"])
    torch.cuda.synchronize()
    assert int(st.cpu()[0]) == 0
    shape = (g.ny * g.supersample + g.psf_n - 1, g.nx * g.supersample + g.psf_n - 1)
    at = np.array(gd["pix_iy"]), np.array(gd["pix_ix"])
    rN = np.abs(N.cpu().numpy().reshape(shape)[at] / np.array(gd["N"]) - 1).max()
    rI = np.abs(I.cpu().numpy().reshape(shape)[at] / np.array(gd["I"]) - 1).max()
    print(f"{name}: N {rN:.2e}, I {rI:.2e}")
    ctx.close()
    assert rN <= 1e-7 and rI <= 1e-12


def test_full_size_model_from_recorded_graphs():
    """The IFU-scale model: all bins against the stored oracle values, and forward
    and adjoint replayed from recorded graphs against the eager calls."""
    dev = _dev()
    ref = np.array(_golden("cfg2_seed0.json")["vrms2"])
    w = inputs.config2(seed=0)
    p = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, p["inc"], p["mass_scale"], p["m_bh"], p["beta"], p["lum_I0"], p["mass_S0"])
    cot = torch.as_tensor(inputs.cotangent(len(ref), 1)[0], device=dev)
    eager = binding.Context(w.geometries)
    assert eager.plan_info(w.geom_idx)["num_kernel"] == 4
    V, st = eager.eval_batch(*args)
    want = eager.vjp(*args, V, cot)
    torch.cuda.synchronize()
    rel = np.abs(V.cpu().numpy() / ref - 1).max()
    print(f"all bins: {rel:.2e}")
    assert int(st.cpu()[0]) == 0 and rel <= 1e-7
    ctx = binding.Context(w.geometries, graph=1)
    out = torch.empty_like(V)
    for rep in range(4):
        out.fill_(-1.0)
        ctx.eval_batch(*args, out=out, status=st)
        got = ctx.vjp(*args, out, cot)
        torch.cuda.synchronize()
        assert torch.equal(out, V), rep
        for k in KEYS:
            assert torch.equal(got[k], want[k]), (rep, k)
        eager.eval_batch(*args)               # eager work of the program between replays
        torch.cuda.synchronize()
    ctx.close()
    eager.close()

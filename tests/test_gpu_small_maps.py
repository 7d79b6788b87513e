"""Small maps (one 32 x 32 block of distinct pixels) in batches, forward and
adjoint, against the FP64 oracle at the edges of the 4 x 4 tilings (12, 20, 24
distinct columns or rows, remainders of four, the sizes beyond) and of the
adjoint's groups of four rows; and the adjoint's items, whole tracers in a batch
and rows of one tracer for a single model.

Bars: the sums are FP32 with FP32 exponentials whose rounded coefficients shift
an exponent by up to 6e-8 of itself, 20 where a term still counts: 1.2e-6 of such
a term, 1e-7 of the sum.  Per bin 1e-6, the gradient's norm (sums of both signs)
1e-5."""
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


def _flat(g):
    return np.concatenate([np.ravel(np.asarray(g[k])) for k in KEYS])


def _model(nx, ny, n_u):
    # off centre: every column and row distinct
    g = inputs.small_geometry(seed=nx + 40 * ny, n_lum=3, n_mass=5, nx=nx, ny=ny, psf_n=1,
                              n_bins=3, n_u=n_u, pixsize=0.06, xc=0.007, yc=-0.011)
    return g, inputs.small_params(g, seed=nx + ny)


def _run(g, ps, cot, dev):
    n = len(ps)
    w = inputs.Workload("s", [g], np.zeros(n, np.int32), ps)
    ctx = binding.Context([g])
    par = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, par["inc"], par["mass_scale"], par["m_bh"], par["beta"], par["lum_I0"],
            par["mass_S0"])
    V, st = ctx.eval_batch(*args)
    gr = ctx.vjp(*args, V, torch.as_tensor(np.tile(cot, n), device=dev))
    torch.cuda.synchronize()
    assert (st.cpu().numpy() == 0).all()
    out = (V.cpu().numpy()[-g.n_bins:],
           {k: gr[k].cpu().numpy().reshape(n, -1)[-1] for k in KEYS})
    ctx.close()
    return out


@pytest.mark.parametrize("nx,ny,n_u", [
    (4, 4, 40), (12, 12, 40), (13, 5, 33), (20, 20, 40), (21, 12, 40), (24, 24, 47), (5, 23, 40),
    (25, 9, 40), (9, 32, 40), (3, 17, 64)])
@pytest.mark.parametrize("n", [1, 2000])
def test_tilings_vs_oracle(nx, ny, n_u, n):
    dev = _dev()
    g, p = _model(nx, ny, n_u)
    cot = np.random.default_rng(5).standard_normal(g.n_bins)
    ps = [inputs.with_overrides(p, m_bh=p.m_bh * (1.0 + 1e-3 * (n - 1 - m))) for m in range(n)]
    V, gr = _run(g, ps, cot, dev)
    rV, rg = ojam.vrms2_and_grad(g, p, cot)
    err = np.max(np.abs(V / rV.numpy() - 1))
    a, b = _flat(gr), _flat({k: v.numpy() for k, v in rg.items()})
    gerr = np.linalg.norm(a - b) / np.linalg.norm(b)
    print(f"{nx} x {ny}, {n}: forward {err:.2e}, gradient {gerr:.2e}")
    assert err <= 1e-6 and gerr <= 1e-5


@pytest.mark.parametrize("nx,ny,n_u,n", [
    (33, 33, 40, 400),     # two items a side, one column of pixels past the block
    (39, 21, 40, 400),     # 6 x 5 tiles; the last item's padding
    (40, 24, 40, 400),     # whole items
    (79, 33, 100, 40),     # four by two; several slices
    (70, 67, 12, 150),     # three by three
])
def test_items_of_tiles_vs_oracle(nx, ny, n_u, n):
    """Maps of more than one block whose items of 4 x 4 tiles read the terms
    from their table: the last of n models."""
    test_tilings_vs_oracle(nx, ny, n_u, n)


def test_items_of_tiles_in_a_mixed_batch():
    """Two geometries of tiles and one of blocks in one batch equal each alone:
    the values are sums of the same terms in an order that may differ between
    the two forms (FP32 over 64 terms), 1e-6."""
    dev = _dev()
    gs, ps = zip(*[_model(nx, ny, 40) for nx, ny in ((33, 33), (39, 21), (28, 40))])
    ctx = binding.Context(list(gs))
    idx = np.repeat(np.arange(3, dtype=np.int32), 200)
    w = inputs.Workload("m", list(gs), idx, [ps[i] for i in idx])
    par = binding.pack_params(w, dev, amplitudes=True)
    keys = ("inc", "mass_scale", "m_bh", "beta", "lum_I0", "mass_S0")
    V = ctx.eval_batch(idx, *[par[k] for k in keys])[0].cpu().numpy().reshape(600, -1)
    for i in range(3):
        one = inputs.Workload("o", list(gs), np.array([i], np.int32), [ps[i]])
        par = binding.pack_params(one, dev, amplitudes=True)
        r = ctx.eval_batch(one.geom_idx, *[par[k] for k in keys])[0].cpu().numpy()
        assert (V[200 * i:200 * (i + 1)] == V[200 * i]).all()
        assert np.max(np.abs(V[200 * i] / r - 1)) <= 1e-6
    ctx.close()


def _mixed(sizes, n_u, dev):
    """(context, index list, device arguments, models) of a batch of several
    sizes of small maps, count of them each."""
    gs, ps = zip(*[_model(nx, ny, n_u) for nx, ny, _ in sizes])
    idx = np.repeat(np.arange(len(sizes), dtype=np.int32), [c for _, _, c in sizes])
    w = inputs.Workload("x", list(gs), idx, [ps[i] for i in idx])
    par = binding.pack_params(w, dev, amplitudes=True)
    return binding.Context(list(gs)), idx, (idx, par["inc"], par["mass_scale"], par["m_bh"],
                                            par["beta"], par["lum_I0"], par["mass_S0"]), gs, ps


def test_few_maps_run_in_the_larger_ones_kernels():
    """Sizes with few models share the tilings, blocks and adjoint kernels of
    larger ones: each against the oracle."""
    dev = _dev()
    sizes = ((24, 24, 900), (12, 12, 3), (5, 23, 2), (20, 9, 2), (32, 9, 2), (3, 31, 2))
    ctx, idx, args, gs, ps = _mixed(sizes, 40, dev)
    cot = np.random.default_rng(8).standard_normal(3)
    V, st = ctx.eval_batch(*args)
    gr = ctx.vjp(*args, V, torch.as_tensor(np.tile(cot, len(idx)), device=dev))
    torch.cuda.synchronize()
    assert (st.cpu().numpy() == 0).all()
    V = V.cpu().numpy().reshape(len(idx), 3)
    gr = {k: gr[k].cpu().numpy().reshape(len(idx), -1) for k in KEYS}
    for i, (g, p) in enumerate(zip(gs, ps)):
        m = int(np.flatnonzero(idx == i)[-1])
        rV, rg = ojam.vrms2_and_grad(g, p, cot)
        a, b = _flat({k: gr[k][m] for k in KEYS}), _flat({k: v.numpy() for k, v in rg.items()})
        assert np.max(np.abs(V[m] / rV.numpy() - 1)) <= 1e-6, sizes[i]
        assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b), sizes[i]
    ctx.close()


def test_mixed_sizes_take_no_longer_than_the_largest():
    """256 models on rectangles of all small sizes against 256 on the largest:
    less work, so no more than half as long again (a launch for every tiling one
    after the other took five times as long)."""
    dev = _dev()
    rng = np.random.default_rng(4)
    mixed = [(int(a), int(b), 2) for a, b in rng.integers(8, 33, (128, 2))]
    took = []
    for sizes in (mixed, [(32, 32, 256)]):
        ctx, _, args, _, _ = _mixed(sizes, 400, dev)
        for _ in range(3):
            ctx.eval_batch(*args)
        best = np.inf
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                ctx.eval_batch(*args)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        took.append(best)
        ctx.close()
    print(f"mixed {took[0] * 100:.1f} us, largest {took[1] * 100:.1f} us")
    assert took[0] <= 1.5 * took[1]


@pytest.mark.parametrize("nx,ny,n_u,n", [
    (28, 40, 20, 700),     # one 32 x 64 tile
    (64, 64, 12, 400),     # whole blocks
    (76, 45, 12, 400),     # 64 and 32 wide tiles, both with remainders
])
def test_single_slice_of_blocks_vs_oracle(nx, ny, n_u, n):
    """A batch large enough for one slice per model: the tiles go straight into
    the map."""
    test_tilings_vs_oracle(nx, ny, n_u, n)


@pytest.mark.parametrize("n_lum,n_mass", [(3, 2), (4, 63), (17, 70)])
def test_gradients_of_many_models_equal_a_single_ones(n_lum, n_mass):
    """Beyond 256 models the reductions run on four waves a model instead of
    sixteen: fewer and more tracers than waves, more mass Gaussians than lanes.
    The sums differ in order, and the batch's sensitivities in their grouping of
    FP32 sums: 1e-6 of the norm."""
    dev = _dev()
    g = inputs.small_geometry(seed=n_mass, n_lum=n_lum, n_mass=n_mass, nx=9, ny=7, psf_n=1,
                              n_bins=3, n_u=16, pixsize=0.06, xc=0.007, yc=-0.011)
    p = inputs.small_params(g, seed=n_lum)
    cot = np.random.default_rng(2).standard_normal(g.n_bins)
    (V1, g1), (Vn, gn) = (_run(g, [p] * n, cot, dev) for n in (1, 257))
    assert np.max(np.abs(Vn / V1 - 1)) <= 1e-6
    a, b = _flat(gn), _flat(g1)
    assert np.linalg.norm(a - b) <= 1e-6 * np.linalg.norm(b)

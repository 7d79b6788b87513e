"""The spherical model's line-of-sight kernels: pixel counts around their
64-pixel items, the pixel on the axis, and blocks whose range of items crosses
models."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from test_gpu_sph import KEYS, RTOL, _dev, _eval  # noqa: E402

from oracle import jam_sph as osph  # noqa: E402
from paper_2504_01302_amd import binding, inputs  # noqa: E402

pytestmark = pytest.mark.gpu

# odd maps have a pixel at x = y = 0; PSF of one pixel: unique pixels nx x ny
SIZES = [(1, 1), (9, 7), (8, 8), (13, 5), (17, 15)]


def _geom(nx, ny, seed=4):
    return inputs.small_geometry(seed=seed, n_lum=3, n_mass=2, nx=nx, ny=ny, ss=1, psf_n=1,
                                 n_bins=1, n_u=24)


@pytest.mark.parametrize("nx,ny", SIZES)
def test_pixel_counts_vs_oracle(nx, ny):
    dev = _dev()
    g = _geom(nx, ny)
    p = inputs.small_params(g, seed=4)
    w = inputs.Workload("s", [g], np.zeros(1, np.int32), [p])
    ctx = binding.Context([g], alignment=1)
    V, st = _eval(ctx, w, dev)
    err = np.max(np.abs(V / osph.vrms2(g, p) - 1))
    print(f"{nx} x {ny}: max rel err {err:.2e}")
    assert st[0] == 0 and err <= RTOL
    ctx.close()


def _values_and_gradients(ctx, w, dev):
    pk = binding.pack_params(w, dev, amplitudes=True)
    args = (w.geom_idx, pk["inc"], pk["mass_scale"], pk["m_bh"], pk["beta"], pk["lum_I0"],
            pk["mass_S0"])
    V, st = ctx.eval_batch(*args)
    gr = ctx.vjp(*args, V, torch.ones_like(V))
    return V.cpu().numpy(), st.cpu().numpy(), {k: gr[k].cpu().numpy().reshape(-1) for k in KEYS}


def test_items_across_models():
    """400 models of five geometries (more items than blocks, so that ranges
    cross models, geometries and an inadmissible model): each, bit for bit, as
    evaluated alone."""
    dev = _dev()
    geoms = [_geom(nx, ny) for nx, ny in SIZES]
    idx = np.array([(3 * i) % len(geoms) for i in range(400)], np.int32)
    ps = [inputs.small_params(geoms[i], seed=n % 7) for n, i in enumerate(idx)]
    ps[5] = inputs.with_overrides(ps[5], inc=0.05)        # not deprojectable
    ctx = binding.Context(geoms, alignment=1)
    V, st, gr = _values_and_gradients(ctx, inputs.Workload("w", geoms, idx, ps), dev)
    assert st[5] != 0 and (np.delete(st, 5) == 0).all()
    for m in (0, 4, 6, 133, 399):
        w1 = inputs.Workload("w1", geoms, idx[m:m + 1], [ps[m]])
        V1, _, g1 = _values_and_gradients(ctx, w1, dev)
        assert np.array_equal(V[m:m + 1], V1)             # one bin per model
        for k in KEYS:
            n = g1[k].size
            assert np.array_equal(gr[k][m * n:(m + 1) * n], g1[k]), (m, k)
    ctx.close()

"""Gradients of the spherically aligned model where they cancel.

A single model's derivative with respect to the inclination is one number in
which terms hundreds of times larger cancel, so the rounding of the adjoint's
term sums shows in it first.  IFU-scale models drawn as the timed case draws
them, chosen for that cancellation (FP32 sums left 1.4e-5, 3.0e-6 and 9.5e-6 of
these derivatives), against the 64-bit gradients of plain torch; the bar is the
timed case's own tolerance."""
import importlib.util
import pathlib

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _cases():
    path = pathlib.Path(__file__).resolve().parents[1] / "perf" / "cases.py"
    spec = importlib.util.spec_from_file_location("timed_cases", path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("seed", [205, 216, 222])
def test_gradients_of_single_models_against_64_bits(seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cases = _cases()
    case = next(c for c in cases.listed() if c["name"] == "spherical ifu model, gradient")
    state = cases.prepare(case, seed)
    got = cases.run(state)
    want = cases.exact(case, seed)
    torch.cuda.synchronize()
    bar = cases.tolerance(case)["rel"]
    for name, a, b in zip(("V", "status") + cases.PARAMS, got, want):
        a = a.detach().double().cpu().numpy()
        b = b.detach().double().cpu().numpy()
        assert np.linalg.norm(a - b) <= bar * np.linalg.norm(b), name
    state["ctx"].close()

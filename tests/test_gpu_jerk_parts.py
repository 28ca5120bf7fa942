"""The batched FP64 jerk pass gives every lane at most one particle: Hermite steps with work
units and splits whose parts end anywhere against the fixed rules' plan, on systems of no, one
and a few particles, of whole workgroups, and of one particle more or less."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TUNING = os.path.join(ROOT, "paper_1406_4254_amd", "etics_tuning.json")
SIZES = [0, 1, 7, 255, 256, 257, 0, 1024, 1025, 5003]


@pytest.fixture(autouse=True)
def clean_table():
    from paper_1406_4254_amd import etics as E
    E.etics_tuning_clear()
    yield
    if os.path.exists(TUNING):
        E.etics_tuning_load(TUNING)
    else:
        E.etics_tuning_clear()


def steps(nmax, lmax):
    from paper_1406_4254_amd import etics as E
    rng = np.random.default_rng(8)
    n = sum(SIZES)
    d = rng.normal(size=(3, n))
    x = d / np.linalg.norm(d, axis=0) * rng.uniform(0.2, 3.0, n)
    s = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (*x, *(0.3 * rng.normal(size=(3, n))))]
    m = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    off = torch.tensor(np.concatenate([[0], np.cumsum(SIZES)]), dtype=torch.int64, device="cuda")
    E.etics_hermite_scf_batched(*s, m, off, nmax, lmax, 0.01, 3, E.ETICS_FP64)
    return torch.stack(s).cpu().numpy()


@pytest.mark.parametrize("nmax,lmax", [(4, 3), (3, 12)])
@pytest.mark.parametrize("shape", [{"unit": 256, "split": 1}, {"unit": 320, "split": 5}, {"unit": 1000, "split": 3},
                                   {"unit": 1 << 20, "split": 16}])
def test_hermite_parts(nmax, lmax, shape):
    """Other units sum a system's coefficients in other groups: FP64 rounding, times three steps."""
    from paper_1406_4254_amd import etics as E
    ref = steps(nmax, lmax)
    E.etics_tuning_set(nmax, lmax, E.ETICS_FP64, sum(SIZES), shape, batched=True)
    info = E.etics_plan_info(sum(SIZES), nmax, lmax, E.ETICS_FP64, batched=True)
    assert info["tuned"] and info["unit"] == shape["unit"] and info["split"] == shape["split"]
    np.testing.assert_allclose(steps(nmax, lmax), ref, rtol=1e-11, atol=1e-13)

"""FP64 sigmoid and 10^y of the emulators at the ends of their ranges: gates
saturated on both sides (|beta t| from 1e-3 to 1e6) and outputs 10^y that
overflow, underflow or are subnormal, in the one-kernel narrow network, the
layer-by-layer one and the wide one on digits.

Tolerance: 1e-11 of the entry plus the row's largest entry, as for every FP64
theory vector; beyond a double's range the oracle's infinities and zeros."""
import sys

import numpy as np
import pytest
import torch

import workloads as W
from oracle.cmb import model_vector

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("hidden", [(64, 64), (128, 128), (512, 512)])
def test_saturated_gates(hidden):
    print(f"case saturated gates {hidden}", flush=True)
    from paper_2509_13307_amd import Model
    m = W.cmb_diag_structure(hidden=hidden, n_out=40)
    net = m["nets"][0]
    rng = np.random.default_rng(5)
    for l, w in enumerate(hidden):
        net["beta"][l] = rng.choice([-1.0, 1.0], w) * 10.0 ** rng.uniform(-3, 6, w)
    m.update(data=np.zeros(40), sigma=np.ones(40))
    g = Model(m)
    th = W.prior_draws(m, 37, tag=41)
    got = g.theory(torch.tensor(th, device=DEV)).cpu().numpy()
    with np.errstate(over="ignore"):
        ref = model_vector(th, m)
    err = np.abs(got - ref) / (np.abs(ref) + np.max(np.abs(ref), axis=1, keepdims=True))
    print(f"  max error {err.max():.2e}", flush=True)
    assert err.max() <= 1e-11
    g.close()


@pytest.mark.parametrize("hidden", [(64, 64), (512, 512)])
def test_powers_at_the_ends_of_the_range(hidden):
    print(f"case powers {hidden}", flush=True)
    from paper_2509_13307_amd import Model
    mu = np.array([-1e9, -400.0, -330.0, -315.0, -309.0, -307.0, -20.0, 0.0, 20.0, 307.0, 309.0, 330.0, 1e9])
    m = W.cmb_cv_structure(n_ell=mu.size, hidden=hidden)
    m["nets"][0]["out_mu"] = mu
    m["data"] = np.ones(mu.size)
    g = Model(m)
    th = W.prior_draws(m, 33, tag=42)
    got = g.theory(torch.tensor(th, device=DEV)).cpu().numpy()
    with np.errstate(over="ignore"):
        ref = model_vector(th, m)
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.array_equal(got == 0, ref == 0)
    normal = np.isfinite(ref) & (ref > 1e-307)
    err = np.abs(got[normal] - ref[normal]) / ref[normal]
    sub = (ref > 0) & (ref <= 1e-307)
    off = np.abs(got[sub] - ref[sub])
    print(f"  max relative error {err.max():.2e}, subnormal {off.max():.2e}", flush=True)
    # |y| to 320: an argument's rounding is worth 320 ln 10 2^-53 = 8e-14 of the power in either computation
    assert err.max() <= 1e-12
    assert np.all(off <= 1e-12 * ref[sub] + 2 * 5e-324)
    g.close()

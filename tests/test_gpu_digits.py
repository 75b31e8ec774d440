"""The FP64 form of wide emulators, whose layers run as int8 digit products:
layer by layer (split tiles, whole tiles, several input blocks) and in one
kernel from 104 row blocks of 32 on (the adjoint from 80), at the edges of their tiles.

Tolerances: the theory vector as in test_gpu_theory.py (1e-11 of the entry plus
the spectrum's largest entry: a few thousand roundings; the digit products'
own error is below that of an FP64 product), the gradient as in
test_gpu_gradient.py (1e-8 of the row's largest component, against the complex
step).  A row's results are bitwise independent of the batch: the integer sums
are exact and both paths use the same scales and expressions."""
import sys

import numpy as np
import pytest
import torch

import workloads as W
from oracle.cmb import model_vector
from oracle.gradient import loglike_grad

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def tt_model(hidden, n_ell):
    m = W.cmb_cv_structure(n_ell=n_ell, hidden=hidden)
    fid = W.fiducial_cmb()
    m["data"] = model_vector(fid[None, :], m)[0] * (1.0 + 0.01 * W.noise(n_ell, tag=77))
    m["theta_fid"] = fid
    return m


def check_theory(m, g, th):
    got = g.theory(torch.tensor(th, device=DEV)).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(min(8, len(th))), np.arange(max(0, len(th) - 8), len(th))]))
    ref = model_vector(th[rows], m)
    s = np.max(np.abs(ref), axis=1, keepdims=True)
    err = np.abs(got[rows] - ref) / (np.abs(ref) + s)
    say(f"  max theory error {err.max():.2e}")
    assert err.max() <= 1e-11


@pytest.mark.parametrize("hidden,n_ell,B", [
    ((256, 256), 33, 1), ((320, 256), 65, 31), ((512, 512, 512), 31, 33), ((512, 512), 420, 300),
    ((1024, 512), 100, 40), ((512, 1024, 256), 70, 1100),
    ((512, 512, 512, 512), 2500, 97), ((512, 512, 512, 512), 2500, 1500),
    ((512, 512), 97, 4576), ((512, 512), 97, 4577), ((512, 512, 512), 300, 9000),
    ((512, 512), 97, 3296), ((512, 512), 97, 3297)])
def test_digit_layers_match_oracle(hidden, n_ell, B):
    say(f"case digits {hidden} n_ell={n_ell} B={B}")
    from paper_2509_13307_amd import Model
    m = tt_model(hidden, n_ell)
    g = Model(m)
    check_theory(m, g, W.prior_draws(m, B, tag=31))
    g.close()


@pytest.mark.parametrize("n_ell", [97, 600, 2500])
def test_digit_gradient_and_batch_independence(n_ell):
    """Gradient against the complex step; logL and gradient of 40 rows bitwise
    the same alone (layer by layer) and within a batch for the one-kernel form."""
    say(f"case digits gradient n_ell={n_ell}")
    from paper_2509_13307_amd import Model
    m = tt_model((512, 512, 512), n_ell)
    g = Model(m)
    th = torch.tensor(W.prior_draws(m, 4700, tag=32), device=DEV)
    big_l, big_g = g.loglike_grad(th)
    big = g.loglike(th)
    for n in (1, 33, 40, 1030, 2528, 2529, 3297):
        l, gr = g.loglike_grad(th[:n].contiguous())
        assert torch.equal(l, big_l[:n]) and torch.equal(gr, big_g[:n])
        assert torch.equal(g.loglike(th[:n].contiguous()), big[:n])
    _, ref = loglike_grad(th[:4].cpu().numpy(), m)
    got = big_g[:4].cpu().numpy()
    err = np.abs(got - ref) / np.max(np.abs(ref), axis=1, keepdims=True)
    say(f"  max gradient error {err.max():.2e}")
    assert err.max() < 1e-8
    g.close()


@pytest.mark.parametrize("B", [40, 4700])
def test_digit_rows_are_independent_of_nan_rows(B):
    say(f"case digits nan B={B}")
    from paper_2509_13307_amd import Model
    m = tt_model((512, 512), 97)
    g = Model(m)
    th = W.prior_draws(m, B, tag=33)
    clean = g.loglike(torch.tensor(th, device=DEV)).cpu().numpy()
    bad = th.copy()
    bad[5, 2] = np.nan
    got = g.loglike(torch.tensor(bad, device=DEV)).cpu().numpy()
    assert np.isnan(got[5])
    keep = np.arange(B) != 5
    np.testing.assert_array_equal(got[keep], clean[keep])
    g.close()


def test_uneven_weights_stay_in_fp64():
    """One weight a thousand times its neighbours: digits of a common scale
    would lose the others' last bits, so the network keeps FP64 products.  Its
    zero-weight unit and a zero input row pass through both."""
    say("case digits uneven weights")
    from paper_2509_13307_amd import Model
    m = tt_model((512, 512), 97)
    for scale in (1.0, 1e3):
        m["nets"][0]["W"][1][3, 7] *= scale
        m["nets"][0]["W"][1][9, :] = 0.0
        g = Model(m)
        check_theory(m, g, W.prior_draws(m, 70, tag=34))
        g.close()

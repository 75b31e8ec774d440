"""Four-spectrum models whose networks differ in the evenness of their weights:
FP64 likelihood, theory vector and gradient against the oracle, at a batch for
the layer-by-layer kernels and one for the one-kernel forms.

Tolerances as in test_gpu_likelihood.py, test_gpu_theory.py and
test_gpu_gradient.py: logL 1e-6, theory 1e-11 of the entry plus the
spectrum's largest entry, gradient 1e-8 of the row's largest component."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.cmb import model_vector
from oracle.gradient import loglike_grad
from oracle.likelihood import loglike

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("uneven", [(0,), (2,), (3, 1)])
@pytest.mark.parametrize("B", [33, 4700])
def test_networks_that_differ_in_evenness(uneven, B):
    print(f"case mixed networks, uneven {uneven}, B={B}", flush=True)
    from paper_2509_13307_amd import Model
    n = 70
    m = W.cmb_block_structure(n_ell=n, hidden=(512, 512))
    fid = W.fiducial_cmb()
    for i in uneven:
        m["nets"][i]["W"][1][3, 7] *= 1e3
    c = model_vector(fid[None, :], m)[0]
    f = np.abs(c).reshape(4, n) * 0.05 + 0.05 * np.abs(c).reshape(4, n).max(axis=1, keepdims=True)
    m["data"] = c + f.ravel() * W.noise(4 * n, tag=78)
    m["cov_blocks"] = np.einsum("sl,tl,st->lst", f[:3], f[:3], 0.5 * np.eye(3) + 0.5)
    m["sigma_pp"] = f[3]
    g = Model(m)
    th = W.prior_draws(m, B, tag=35)
    rows = np.r_[0:6, B - 6:B]
    td = torch.tensor(th, device=DEV)
    got = g.loglike(td).cpu().numpy()[rows]
    ref = loglike(th[rows], m)
    print(f"  max |dlogL| {np.abs(got - ref).max():.2e}", flush=True)
    assert np.all(np.abs(got - ref) <= 1e-6)
    got = g.theory(td).cpu().numpy()[rows].reshape(-1, 4, n)
    ref = model_vector(th[rows], m).reshape(-1, 4, n)
    err = np.abs(got - ref) / (np.abs(ref) + np.max(np.abs(ref), axis=2, keepdims=True))
    print(f"  max theory error {err.max():.2e}", flush=True)
    assert err.max() <= 1e-11
    l, gr = (x.cpu().numpy()[rows] for x in g.loglike_grad(td))
    rl, rg = loglike_grad(th[rows], m)
    err = np.abs(gr - rg) / np.max(np.abs(rg), axis=1, keepdims=True)
    print(f"  max gradient error {err.max():.2e}", flush=True)
    assert np.all(np.abs(l - rl) <= 1e-6) and err.max() < 1e-8
    g.close()

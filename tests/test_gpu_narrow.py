"""The one-kernel FP64 forward of narrow networks at the edges of its row
groups (four, eight and sixteen rows per workgroup), output tiles and padded
inputs: against the oracle (1e-11 of the entry plus the spectrum's largest, a
few thousand roundings) and bitwise against the layer-by-layer launches."""
import os

import numpy as np
import pytest
import torch

import workloads as W
from oracle.cmb import model_vector

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_out,n_hidden", [(200, 3), (128, 1), (129, 2), (17, 6), (256, 2)])
def test_row_groups(n_out, n_hidden):
    print(f"case narrow n_out={n_out} hidden={n_hidden}", flush=True)
    from paper_2509_13307_amd import Model
    m = W.load_model("cmb6") if (n_out, n_hidden) == (200, 3) else narrow(n_out, n_hidden)
    g = Model(m)
    th = W.prior_draws(m, 2100, tag=61)
    th[3, 0] = -5.0                                     # outside the support
    t = torch.tensor(th, device=DEV)
    ref = model_vector(th[:5], m)
    got = g.theory(t[:5].contiguous()).cpu().numpy()
    s = np.max(np.abs(ref), axis=1, keepdims=True)
    assert np.max(np.abs(got - ref) / (np.abs(ref) + s)) <= 1e-11
    os.environ["NSMI_NO_FUSED_MLP"] = "1"
    try:
        base_l, base_t = g.loglike(t), g.theory(t)
    finally:
        os.environ.pop("NSMI_NO_FUSED_MLP")
    assert base_l[3] == -float("inf")
    for B in (1, 3, 4, 5, 1023, 1024, 1025, 1029, 2047, 2048, 2049, 2100):
        assert torch.equal(g.loglike(t[:B].contiguous()), base_l[:B]), B
        assert torch.equal(g.theory(t[:B].contiguous()), base_t[:B]), B
    g.close()


def narrow(n_out, n_hidden):
    m = dict(W.load_model("cmb6"))
    rng = np.random.default_rng(n_out)
    net = dict(m["nets"][0])
    n_in = net["W"][0].shape[1]
    dims = [n_in] + [128] * (n_hidden + 1) + [n_out]
    net["W"] = [rng.normal(size=(o, i)) / np.sqrt(i) for i, o in zip(dims[:-1], dims[1:])]
    net["b"] = [0.1 * rng.normal(size=o) for o in dims[1:]]
    net["beta"] = [1.0 + 0.1 * rng.normal(size=o) for o in dims[1:-1]]
    net["gamma"] = [0.5 + 0.1 * rng.normal(size=o) for o in dims[1:-1]]
    net["out_mu"] = rng.normal(size=n_out)
    net["out_sigma"] = 0.1 + rng.random(n_out)
    m["nets"] = [net]
    m["data"] = rng.normal(size=n_out)
    m["sigma"] = 0.5 + rng.random(n_out)
    return m

"""Gradients of the BF16-operand forms with the one-kernel forward that keeps
the pre-activations: bitwise the layer-by-layer forward's gradients, for every
launch shape (shapes that split the output blocks fall back to the first), at
batches with a partly filled last row block."""
import os

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def grads(g, th, prec, **env):
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        l, gr = g.loglike_grad(th, prec)
        return l.cpu().numpy(), gr.cpu().numpy()
    finally:
        for k, v in old.items():
            if v is None:
                os.environ.pop(k)
            else:
                os.environ[k] = v


@pytest.mark.parametrize("name,B", [("cmb6", 1), ("cmb6", 130), ("cmbtt_cv", 97), ("cmb4x2500", 65), ("shear10", 9)])
@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
def test_saved_forward_gives_the_same_gradient(name, B, prec):
    print(f"case fused gradient {name} {prec} B={B}", flush=True)
    from paper_2509_13307_amd import Model
    m = W.load_model(name)
    g = Model(m)
    th = torch.tensor(W.prior_draws(m, B, tag=51), device=DEV)
    ref = grads(g, th, prec, NSMI_NO_FUSED_MLP="1")
    width = m["nets"][0]["W"][0].shape[0]
    for c in [None] + list(range(8 if width == 512 and prec == "bf16x3" else 10)):
        got = grads(g, th, prec, **({} if c is None else {"NSMI_FUSED_CFG": str(c)}))
        np.testing.assert_array_equal(got[0], ref[0])
        np.testing.assert_array_equal(got[1], ref[1])
    g.close()

"""The FP32 layers' 64- and 128-wide tiles: both run the same K order, so a
row's logL and gradient are bitwise the same alone and within a batch large
enough for the wide tiles, at rows and columns that do not fill a tile."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("name,prec,big", [("cmb4x2500", "fp32", 4133), ("cmb6", "fp32", 33000)])
def test_rows_do_not_depend_on_the_tile(name, prec, big):
    print(f"case fp32 tiles {name} {big}", flush=True)
    from paper_2509_13307_amd import Model
    m = W.load_model(name)
    g = Model(m)
    th = torch.tensor(W.prior_draws(m, big, tag=71), device=DEV)
    wide_l, (wide_gl, wide_g) = g.loglike(th, prec), g.loglike_grad(th, prec)
    for B in (1, 63, 64, 65, 129, 300):
        part = th[:B].contiguous()
        l, gr = g.loglike_grad(part, prec)
        assert torch.equal(g.loglike(part, prec), wide_l[:B])
        assert torch.equal(l, wide_gl[:B]) and torch.equal(gr, wide_g[:B])
    g.close()

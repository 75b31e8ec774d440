"""FP64 calls of wide networks with more rows than one launch takes at a time
(65536 per part): every row as in a small batch, and beside the same network on
FP64 products no more device memory than a part's digits (twice their bytes
allowed: large allocations are rounded up)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.cmb import model_vector

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def model(uneven):
    m = W.cmb_diag_structure(hidden=(256, 320), n_out=33)
    m["nets"][0] = W.net_dict(W.draw_mlp((6, 256, 320, 33), 5, 98, "wide"), np.full(6, 0.5), np.full(6, 0.5),
                              np.zeros(33), np.ones(33))
    if uneven:
        m["nets"][0]["W"][1][3, 7] *= 1e3
    m.update(data=np.zeros(33), sigma=np.ones(33))
    return m


@pytest.mark.parametrize("B", [65536, 65537, 600_000])
def test_rows_beyond_one_part(B):
    print(f"case large batch B={B}", flush=True)
    from paper_2509_13307_amd import Model
    m = model(False)
    base = torch.tensor(W.prior_draws(m, 5000, tag=55), device=DEV)
    th = base.repeat((B + 4999) // 5000, 1)[:B].contiguous()
    big = torch.empty(B, dtype=torch.float64, device=DEV)
    grown = []
    for uneven in (True, False):
        g = Model(model(uneven))
        small = g.loglike(base)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        big.copy_(g.loglike(th))
        torch.cuda.synchronize()
        grown.append(free - torch.cuda.mem_get_info()[0])
        if uneven:
            g.close()
            torch.cuda.empty_cache()
    print(f"  {grown[1] / 2**20:.0f} MiB more in use, on FP64 products {grown[0] / 2**20:.0f}", flush=True)
    assert grown[1] - grown[0] <= 2 * 65536 * (320 * 7 + 16)
    for r0 in (0, B - 5000, 63000):
        idx = torch.arange(r0, min(r0 + 5000, B), device=DEV)
        assert torch.equal(big[idx], small[idx % 5000])
    y = model_vector(base[:8].cpu().numpy(), m)
    ref = -0.5 * np.sum(y * y, axis=1) - 0.5 * 33 * np.log(2.0 * np.pi)
    assert np.all(np.abs(small[:8].cpu().numpy() - ref) <= 1e-9)
    l, gr = g.loglike_grad(th)
    ls, gs = g.loglike_grad(base)
    idx = torch.arange(B - 5000, B, device=DEV)
    assert torch.equal(l[idx], ls[idx % 5000]) and torch.equal(gr[idx], gs[idx % 5000])
    g.close()

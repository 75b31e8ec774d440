"""Error of the FP64 gate: theta sigmoid(theta) through a network whose first
layer hands the parameter on and whose output picks one unit, against 80-bit
values.

Bound: the rms error of the sigmoid with the library's exp and division is
0.6696 x 2^-53 for normal arguments (measured on this GPU), and the product with
theta adds the rms of one rounding (taken here from the exact sigmoid's
products).  The rms of 2^22 values scatters by 0.05%."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def test_gate_is_no_worse_than_the_library():
    print("case gate accuracy", flush=True)
    from paper_2509_13307_amd import Model
    w = 64
    one = [(np.zeros((w, 1)), np.zeros(w), np.ones(w), np.zeros(w)), (np.zeros((1, w)), np.zeros(1), None, None)]
    one[0][0][:, 0] = 1.0
    one[1][0][0, 5] = 1.0
    net = W.net_dict(one, [0.0], [1.0], np.zeros(1), np.ones(1))
    m = dict(kind="cmb_diag", d=1, prior_kind=np.zeros(1, dtype=np.int32), prior_a=-np.full(1, 9.0), prior_b=np.full(1, 9.0),
             nets=[net], spec_log=[False], data=np.zeros(1), sigma=np.ones(1))
    g = Model(m)
    th = np.random.default_rng(6).normal(size=(1 << 22, 1))
    got = g.theory(torch.tensor(th, device="cuda:0")).cpu().numpy()[:, 0]
    t = th[:, 0].astype(np.longdouble)
    s = 1 / (1 + np.exp(-t))
    error = float(np.sqrt(np.mean((((got - t * s) / (t * s)).astype(float) * 2.0 ** 53) ** 2)))
    p = t * s.astype(np.float64)
    product = float(np.sqrt(np.mean((((p.astype(np.float64) - p) / p).astype(float) * 2.0 ** 53) ** 2)))
    bound = (0.6696 ** 2 + product ** 2) ** 0.5
    print(f"  rms error {error:.4f}, bound {bound:.4f}", flush=True)
    assert error <= 1.0005 * bound
    g.close()

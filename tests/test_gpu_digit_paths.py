"""Which kernels an FP64 call of a wide network runs, by the names in the trace
report: digit products for even weights, layer by layer and in one kernel, FP64
products for uneven ones; and rows of zeros through both."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.cmb import model_vector

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def tt_model(hidden, n_ell):
    m = W.cmb_cv_structure(n_ell=n_ell, hidden=hidden)
    m["data"] = model_vector(W.fiducial_cmb()[None, :], m)[0]
    return m


def traced(g, call):
    g.trace(True)
    call()
    names = set(g.trace_report())
    g.trace(False)
    return names


@pytest.mark.parametrize("B,forward,adjoint", [
    (70, {"gemm_i8_f64_hidden", "gemm_i8_f64_out"}, {"adj_gemm_i8_f64"}), (4700, {"mlp_i8_f64"}, {"mlp_i8_f64_adjoint"})])
def test_even_weights_run_on_digits(B, forward, adjoint):
    print(f"case digit path B={B}", flush=True)
    from paper_2509_13307_amd import Model
    m = tt_model((512, 512), 300)
    g = Model(m)
    th = torch.tensor(W.prior_draws(m, B, tag=61), device=DEV)
    names = traced(g, lambda: g.theory(th))
    assert forward <= names and not any(k.startswith("gemm_f64") for k in names)
    names = traced(g, lambda: g.loglike_grad(th))
    assert forward | adjoint <= names and not any("gemm_f64" in k for k in names)
    g.close()


@pytest.mark.parametrize("B", [70, 4700])
def test_uneven_weights_run_on_fp64_products(B):
    print(f"case digit path, uneven B={B}", flush=True)
    from paper_2509_13307_amd import Model
    m = tt_model((512, 512), 300)
    m["nets"][0]["W"][1][3, 7] *= 1e3
    g = Model(m)
    th = torch.tensor(W.prior_draws(m, B, tag=62), device=DEV)
    names = traced(g, lambda: (g.theory(th), g.loglike_grad(th)))
    assert {"gemm_f64_hidden", "gemm_f64_out", "adj_gemm_f64"} <= names and not any("_i8" in k for k in names)
    g.close()


def test_shear_output_adjoint_runs_on_fp64_products():
    print("case digit path, shear", flush=True)
    from paper_2509_13307_amd import Model
    m = W.load_model("shear10")
    g = Model(m)
    th = torch.tensor(W.prior_draws(m, 500, tag=63), device=DEV)
    names = traced(g, lambda: g.loglike_grad(th))
    assert {"mlp_i8_f64", "adj_gemm_f64", "mlp_i8_f64_adjoint"} <= names and "adj_gemm_i8_f64" not in names
    g.close()


@pytest.mark.parametrize("uneven", [False, True])
@pytest.mark.parametrize("B", [70, 4700])
def test_rows_and_units_of_zeros(uneven, B):
    """Parameters at the input shift and no first biases: a first layer of zeros;
    and a unit whose weights are zeros."""
    print(f"case digit zeros uneven={uneven} B={B}", flush=True)
    from paper_2509_13307_amd import Model
    m = tt_model((512, 512), 97)
    net = m["nets"][0]
    net["b"][0][:] = 0.0
    net["W"][1][9, :] = 0.0
    if uneven:
        net["W"][1][3, 7] *= 1e3
    g = Model(m)
    th = W.prior_draws(m, B, tag=64)
    th[[0, 40, B - 1]] = net["in_shift"]
    rows = np.r_[0:4, 38:42, B - 3:B]
    got = g.theory(torch.tensor(th, device=DEV)).cpu().numpy()[rows]
    ref = model_vector(th[rows], m)
    err = np.abs(got - ref) / (np.abs(ref) + np.max(np.abs(ref), axis=1, keepdims=True))
    print(f"  max error {err.max():.2e}", flush=True)
    assert err.max() <= 1e-11
    g.close()

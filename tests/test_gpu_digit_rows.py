"""Rows that digits of one scale do not serve: the FP64 form of wide networks
against extended precision, beside the same network on FP64 products.

Two models of one function are compared: one whose weights the digits admit,
and a twin with one more output, whose weights are uneven and send the whole
model to FP64 products (that output is left out of the comparison).  A row is
made uneven by scaling one unit of the first hidden layer, whose gate is open
(the activation is linear), the adjoint's rows by one small error bar.

Tolerance: the digits' error is to be no larger than the FP64 products'.  Both
are rms values over at least 32 rows of 130 outputs (or 6 gradient components),
which scatter by up to 1 / sqrt(2 x 180) = 5%, so 1.15."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from oracle.cmb import model_vector
from paper_2509_13307_amd import _capi
from paper_2509_13307_amd.model import Model

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
L = np.longdouble
N_OUT = 130


def plan(desc):
    f = ctypes.CDLL(_capi.LIB_PATH).nsmi_digit_plan
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_void_p]
    m = Model.__new__(Model)
    D = m._describe(desc)
    return f(ctypes.addressof(D))


def diag(net, sigma):
    n = net["W"][-1].shape[0]
    return dict(kind="cmb_diag", d=6, prior_kind=np.zeros(6, dtype=np.int32), prior_a=np.zeros(6), prior_b=np.ones(6),
                nets=[net], spec_log=[False], data=np.zeros(n), sigma=sigma)


def pair(hidden, spike=1.0, dead=False, sigma=None, few=0, n_out=N_OUT):
    """(model on digits, twin on FP64 products with one more output); `few`:
    first-layer units that are not zero."""
    layers = [[np.array(x) for x in l] for l in W.draw_mlp((6, *hidden, n_out + 1), 5, 99, "wide")]
    layers[0][3][:] = 1.0
    layers[0][0][7] *= spike
    layers[0][1][7] *= spike
    if dead:
        layers[1][0][:, 7] = 0.0
    if few:
        layers[0][0][few:] = 0.0
        layers[0][1][few:] = 0.0
        layers[0][0][:few, 0] = 1.0 + 0.01 * np.arange(few)
        layers[0][0][:few, 1:] *= 0.01
    sigma = np.ones(n_out) if sigma is None else sigma
    out = []
    for n in (n_out, n_out + 1):
        ls = [tuple(l) for l in layers[:-1]] + [(layers[-1][0][:n].copy(), layers[-1][1][:n].copy(), *layers[-1][2:])]
        if n > n_out:
            ls[-1][0][-1, 0] = 1e4
        net = W.net_dict(ls, np.full(6, 0.5), np.full(6, 0.5), np.zeros(n), np.ones(n))
        out.append(diag(net, np.append(sigma, np.full(n - n_out, 1e150))))
    assert plan(out[0]) & 1 and plan(out[1]) == 0
    return out


def forward(th, net):
    """(outputs, pre-activations) in extended precision."""
    h = (th.astype(L) - net["in_shift"].astype(L)) / net["in_scale"].astype(L)
    ts = []
    for Wl, b, be, ga in zip(net["W"], net["b"], net["beta"], net["gamma"]):
        t = h @ Wl.T.astype(L) + b
        ts.append(t)
        h = (ga + (1 - ga.astype(L)) / (1 + np.exp(-be.astype(L) * t))) * t
    return h @ net["W"][-1].T.astype(L) + net["b"][-1], ts


def gradient(th, m):
    net = m["nets"][0]
    y, ts = forward(th, net)
    d = (m["data"] - y) / m["sigma"].astype(L) ** 2
    for Wl, be, ga, t in zip(net["W"][:0:-1], net["beta"][::-1], net["gamma"][::-1], ts[::-1]):
        s = 1 / (1 + np.exp(-be.astype(L) * t))
        d = (d @ Wl.astype(L)) * (ga + (1 - ga.astype(L)) * (s + be * t * s * (1 - s)))
    return (d @ net["W"][0].astype(L)) / net["in_scale"]


def rms_error(got, ref):
    return float(np.sqrt(np.mean((((got - ref) / np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True))) ** 2).astype(float))))


@pytest.mark.parametrize("B", [40, 4700])
@pytest.mark.parametrize("spike,dead", [(1.0, False), (6.0, False), (30.0, False), (100.0, False), (1000.0, False),
                                        (1e6, False), (1e6, True)])
def test_forward_is_no_worse_than_fp64_products(B, spike, dead):
    print(f"case digit rows spike={spike} dead={dead} B={B}", flush=True)
    models = pair((512, 512), spike, dead)
    th = W.prior_draws(models[0], B, tag=51)
    rows = np.r_[0:16, B - 16:B]
    ref, _ = forward(th[rows], models[0]["nets"][0])
    err = []
    for m in models:
        g = Model(m)
        err.append(rms_error(g.theory(torch.tensor(th, device=DEV)).cpu().numpy()[rows, :N_OUT], ref))
        g.close()
    print(f"  digits {err[0]:.3e}, FP64 products {err[1]:.3e}", flush=True)
    assert err[0] <= 1.15 * err[1]


@pytest.mark.parametrize("B", [40, 4700])
@pytest.mark.parametrize("few", [1, 2, 3, 5, 9])
def test_rows_of_few_entries(B, few):
    """Rows of zeros but for a few entries of one size, of which FP64 sums round
    almost nowhere; one hidden layer, so that nothing covers their error."""
    print(f"case digit rows few={few} B={B}", flush=True)
    models = pair((512,), few=few)
    th = W.prior_draws(models[0], B, tag=56)
    rows = np.r_[0:32, B - 8:B]
    ref, _ = forward(th[rows], models[0]["nets"][0])
    err = []
    for m in models:
        g = Model(m)
        err.append(rms_error(g.theory(torch.tensor(th, device=DEV)).cpu().numpy()[rows, :N_OUT], ref))
        g.close()
    print(f"  digits {err[0]:.3e}, FP64 products {err[1]:.3e}", flush=True)
    assert err[0] <= 1.15 * err[1]


@pytest.mark.parametrize("B", [40, 4700])
@pytest.mark.parametrize("spike", [1.0, 30.0, 1e3, 1e6])
@pytest.mark.parametrize("n_out", [N_OUT, 600])
def test_gradient_is_no_worse_than_fp64_products(B, spike, n_out):
    """Output deltas of one block of inputs and of two."""
    print(f"case digit rows, gradient, delta spike={spike} B={B} n_out={n_out}", flush=True)
    sigma = np.ones(n_out)
    sigma[11] /= np.sqrt(spike)
    models = pair((512, 512, 512), sigma=sigma, n_out=n_out)
    assert plan(models[0]) == 7
    th = W.prior_draws(models[0], B, tag=52)
    rows = np.r_[0:16, B - 16:B]
    ref = gradient(th[rows], models[0])
    err = []
    for m in models:
        g = Model(m)
        err.append(rms_error(g.loglike_grad(torch.tensor(th, device=DEV))[1].cpu().numpy()[rows], ref))
        g.close()
    print(f"  digits {err[0]:.3e}, FP64 products {err[1]:.3e}", flush=True)
    assert err[0] <= 1.15 * err[1]


@pytest.mark.parametrize("hidden", [(512, 512), (1024, 512), (256, 320, 256)])
def test_uneven_rows_do_not_depend_on_the_batch(hidden):
    """Even and uneven rows in one tile (a gate that opens one unit wide on half
    of the rows): bitwise the same alone and within a large batch, forward and
    gradient."""
    print(f"case digit rows batch {hidden}", flush=True)
    m, _ = pair(hidden)
    net = m["nets"][0]
    net["W"][0][7] = 0.0
    net["W"][0][7, 0] = 400.0
    net["beta"][0][7], net["gamma"][0][7] = 50.0, 0.0
    m["sigma"][5] = 1e-4
    assert plan(m) & 1
    g = Model(m)
    th = torch.tensor(W.prior_draws(m, 4700, tag=53), device=DEV)
    big, (bl, bg) = g.theory(th), g.loglike_grad(th)
    for n in (1, 33, 1000, 2529):
        assert torch.equal(g.theory(th[:n].contiguous()), big[:n])
        l, gr = g.loglike_grad(th[:n].contiguous())
        assert torch.equal(l, bl[:n]) and torch.equal(gr, bg[:n])
    ref = model_vector(th[:40].cpu().numpy(), m)
    err = np.abs(big[:40].cpu().numpy() - ref) / (np.abs(ref) + np.abs(ref).max(axis=1, keepdims=True))
    print(f"  max error {err.max():.2e}", flush=True)
    assert err.max() <= 1e-11
    g.close()


@pytest.mark.parametrize("B", [40, 4700])
def test_infinite_and_huge_rows(B):
    """Rows with infinite, and with finite activations up to 1e290, give what
    FP64 products give: the oracle's infinities and values (positive weights, so
    that no infinities of both signs meet)."""
    print(f"case digit rows, infinities B={B}", flush=True)
    m, _ = pair((512, 512))
    for Wl in m["nets"][0]["W"][1:]:
        np.abs(Wl, out=Wl)
    m["nets"][0]["W"][0][:, 0] = 1.0
    assert plan(m) & 1
    th = W.prior_draws(m, B, tag=54)
    th[3, 0], th[20, 0], th[B - 1, 0], th[25, 0] = np.inf, 1e290, 1e280, 1e200
    g = Model(m)
    got = g.theory(torch.tensor(th, device=DEV)).cpu().numpy()
    rows = np.r_[0:32, B - 4:B]
    ref = model_vector(th[rows], m)
    assert np.all(np.isposinf(ref[3])) and np.all(np.isposinf(got[3]))
    fin = np.isfinite(ref)
    assert np.array_equal(fin, np.isfinite(got[rows]))
    err = np.abs(got[rows][fin] - ref[fin]) / np.abs(ref[fin])
    print(f"  max error {err.max():.2e}", flush=True)
    assert err.max() <= 1e-11
    g.close()


@pytest.mark.parametrize("B", [40, 4700])
@pytest.mark.parametrize("bits", [0x7ff8000000000000, 0x7ff800007f7f7f7f, 0x7fffffffffffffff, 0x7ff80000007fffff])
def test_nan_rows_of_any_payload(B, bits):
    """A NaN is a NaN in every output and in the gradient, whatever its low bits
    read as digits, and the rows beside it are what they are without it."""
    print(f"case digit rows, NaN {bits:x} B={B}", flush=True)
    m, _ = pair((512, 512))
    th = torch.tensor(W.prior_draws(m, B, tag=57), device=DEV)
    bad = th.clone()
    bad.view(torch.int64)[[3, 20, B - 1], 2] = bits
    rest = torch.ones(B, dtype=torch.bool, device=DEV)
    rest[[3, 20, B - 1]] = False
    g = Model(m)
    y, (l, gr) = g.theory(th), g.loglike_grad(th)
    yb, (lb, gb) = g.theory(bad), g.loglike_grad(bad)
    assert torch.isnan(yb[~rest]).all() and torch.isnan(lb[~rest]).all() and torch.isnan(gb[~rest]).all()
    assert torch.equal(yb[rest], y[rest]) and torch.equal(lb[rest], l[rest]) and torch.equal(gb[rest], gr[rest])
    g.close()

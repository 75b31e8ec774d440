"""The shear spectra at the edges of the Limber kernel: the smallest wavenumber
grids (the four-column gather moved inside the grid at both ends), one to ten
bins (one or two pairs per thread, with a last odd pair), partial node chunks
and several of them, more than 20 multipoles.  Reference: the oracle's FP64
spectra; bounds as for the emulator's theory vectors, 1e-11 of the largest entry
in FP64 (a few thousand roundings) and 1e-4 in FP32 (2^-24 on log10 P of order
one, amplified by ln 10 and the spline, over the sums)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_k,n_bins,n_a,n_ell,z_interp,n_z", [
    (4, 1, 64, 20, "cubic", 5), (5, 2, 257, 21, "linear", 12), (6, 3, 255, 1, "cubic", 16),
    (60, 5, 256, 20, "cubic", 17), (61, 10, 513, 22, "linear", 40), (64, 6, 300, 19, "cubic", 70)])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-11), ("fp32", 1e-4)])
def test_spectra_at_kernel_edges(n_k, n_bins, n_a, n_ell, z_interp, n_z, prec, tol):
    print(f"case limber n_k={n_k} bins={n_bins} n_a={n_a} n_ell={n_ell} {z_interp} {prec}", flush=True)
    from oracle import shear as oshear
    from paper_2509_13307_amd import Model
    m = W.shear_structure(n_z=n_z, n_bins=n_bins, n_extra=0, hidden=(64, 64), n_a=n_a, n_k=n_k, n_ell=n_ell,
                          z_interp=z_interp)
    C0 = oshear.spectra(m["theta_fid"][None], m)[0][0]
    m["data"] = C0
    m["cov"] = np.diag((0.05 * np.abs(C0) + 1e-3 * np.abs(C0).max()) ** 2)
    width = np.where(m["prior_kind"] == 0, m["prior_b"] - m["prior_a"], 1.0)
    th = W.posterior_draws(m["theta_fid"], 0.02 * width, 3, tag=41)
    th[:, 2] = np.clip(th[:, 2], 0.65, None)
    ref = oshear.spectra(th, m)[0]
    g = Model(m)
    got = g.theory(torch.tensor(th, device=DEV), prec).cpu().numpy()
    g.close()
    err = np.max(np.abs(got.reshape(ref.shape) - ref) / np.max(np.abs(ref), axis=1, keepdims=True))
    print(f"  max error {err:.2e}", flush=True)
    assert err < tol


@pytest.mark.parametrize("B", [1, 31, 33, 65])
def test_support_of_every_coordinate(B):
    """The dense likelihood's support test, eight lanes per walker: a coordinate
    outside its uniform prior gives -inf for that walker alone, a NaN does not."""
    print(f"case dense support B={B}", flush=True)
    from paper_2509_13307_amd import Model
    m = W.load_model("shear10")
    g = Model(m)
    base = np.repeat(m["theta_fid"][None], B, axis=0)
    ref = g.loglike(torch.tensor(base, device=DEV)).cpu().numpy()
    assert np.all(np.isfinite(ref))
    for j in range(m["d"]):
        if m["prior_kind"][j] != 0:
            continue
        th = base.copy()
        r = (7 * j + 3) % B
        th[r, j] = m["prior_b"][j] + 1e-6 * (m["prior_b"][j] - m["prior_a"][j])
        got = g.loglike(torch.tensor(th, device=DEV)).cpu().numpy()
        assert got[r] == -np.inf
        np.testing.assert_array_equal(np.delete(got, r), np.delete(ref, r))
    g.close()

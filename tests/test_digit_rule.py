"""Which models run their FP64 layers as int8 digit products: the host's
decision alone (no GPU needed)."""
import ctypes
import os

import numpy as np
import pytest

import workloads as W
from paper_2509_13307_amd import _capi
from paper_2509_13307_amd.model import Model


@pytest.fixture(scope="module")
def admitted():
    if not os.path.exists(_capi.LIB_PATH):
        from paper_2509_13307_amd.build import build
        build()
    _capi.lib()
    f = ctypes.CDLL(_capi.LIB_PATH).nsmi_digit_plan
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_void_p]

    def ask(desc):
        m = Model.__new__(Model)
        D = m._describe(desc)
        return f(ctypes.addressof(D))
    return ask


def four(hidden=(512, 512), n_ell=140):
    m = W.cmb_block_structure(n_ell=n_ell, hidden=hidden)
    m.update(data=np.ones(4 * n_ell), cov_blocks=np.tile(np.eye(3), (n_ell, 1, 1)), sigma_pp=np.ones(n_ell))
    return m


FORWARD, HIDDEN_ADJOINT, OUTPUT_ADJOINT = 1, 2, 4


def test_even_networks_are_admitted(admitted):
    assert admitted(four()) == FORWARD | HIDDEN_ADJOINT | OUTPUT_ADJOINT
    assert admitted(four(hidden=(256, 320))) == FORWARD | HIDDEN_ADJOINT | OUTPUT_ADJOINT
    assert admitted(four(n_ell=70)) == FORWARD | HIDDEN_ADJOINT     # sums of fewer than 128 products
    assert not admitted(four(hidden=(512, 128)))


def test_shear_output_adjoint_stays_on_fp64(admitted):
    m = W.shear_structure(n_z=10, hidden=(256, 256))
    n = m["n_bins"] * (m["n_bins"] + 1) // 2 * m["n_ell"]
    m.update(data=np.ones(n), cov=np.eye(n))
    assert admitted(m) == FORWARD | HIDDEN_ADJOINT


@pytest.mark.parametrize("what", ["sparse", "faint inputs", "heavy tails", "zero unit", "scaled units"])
def test_weights_of_unlike_size(admitted, what):
    """Mostly zero units, inputs whose weights are a millionth of the others'
    (the row's large entries may be those) and tails that reach ten times the
    rms are refused; a unit of zeros, and units of other scales, are not."""
    rng = np.random.default_rng(3)
    m = four()
    Wl = m["nets"][1]["W"][1]
    if what == "sparse":
        Wl *= rng.random(Wl.shape) < 0.4
    elif what == "faint inputs":
        Wl[:, 100:120] *= 1e-6
    elif what == "heavy tails":
        Wl[:] = rng.standard_t(4, size=Wl.shape) / 30.0
    elif what == "zero unit":
        Wl[9] = 0.0
    else:
        Wl *= 10.0 ** rng.uniform(-0.3, 0.3, size=(Wl.shape[0], 1))
    assert bool(admitted(m)) == (what in ("zero unit", "scaled units"))


@pytest.mark.parametrize("net", [0, 1, 2, 3])
@pytest.mark.parametrize("spoil", ["large", "nan"])
def test_one_uneven_network_decides_for_all(admitted, net, spoil):
    """The four networks are launched as one group: an uneven one among them,
    wherever it stands, keeps the whole model on FP64 products."""
    m = four()
    Wl = m["nets"][net]["W"][1]
    Wl[3, 7] = 1e3 * Wl[3, 7] if spoil == "large" else np.nan
    assert not admitted(m)

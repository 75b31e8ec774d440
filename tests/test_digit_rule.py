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
    f = ctypes.CDLL(_capi.LIB_PATH).nsmi_digits_admitted
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_void_p]

    def ask(desc):
        m = Model.__new__(Model)
        D = m._describe(desc)
        return bool(f(ctypes.addressof(D)))
    return ask


def four(hidden=(512, 512), n_ell=70):
    m = W.cmb_block_structure(n_ell=n_ell, hidden=hidden)
    m.update(data=np.ones(4 * n_ell), cov_blocks=np.tile(np.eye(3), (n_ell, 1, 1)), sigma_pp=np.ones(n_ell))
    return m


def test_even_networks_are_admitted(admitted):
    assert admitted(four())
    assert admitted(four(hidden=(256, 320)))
    assert not admitted(four(hidden=(512, 128)))


@pytest.mark.parametrize("net", [0, 1, 2, 3])
@pytest.mark.parametrize("spoil", ["large", "nan"])
def test_one_uneven_network_decides_for_all(admitted, net, spoil):
    """The four networks are launched as one group: an uneven one among them,
    wherever it stands, keeps the whole model on FP64 products."""
    m = four()
    Wl = m["nets"][net]["W"][1]
    Wl[3, 7] = 1e3 * Wl[3, 7] if spoil == "large" else np.nan
    assert not admitted(m)

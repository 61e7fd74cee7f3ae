"""The fine SAP pass on its smallest lattices and over its options (steps per
block solve, batch sizes across the groups of six fields that share an XCD,
unequal extents), against the oracle's sweep.  Tolerances: those of the other
smoother tests, 1e-12 in FP64 and 1e-5 in FP32."""
import numpy as np
import pytest

import workloads as W
from oracle.sap import sap_sweep
from tests.test_gpu_batched import Setup, _p
from tests.gpu_util import dev, host, relerr, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dd():
    from paper_1307_6101_amd import ddamg
    ddamg.load_library()
    return ddamg


@pytest.mark.parametrize("dims,mr,nrhs", [((8, 8, 8, 8), 3, 1), ((8, 8, 8, 16), 2, 2), ((8, 16, 8, 24), 1, 7),
                                          ((16, 8, 8, 8), 5, 13)])
def test_sap_pass(dd, dims, mr, nrhs):
    S = Setup(dd, dims, dict(_p(2, [(4, 4, 4, 4)], [4], n_inv=0), mr_iters=mr), m0=-0.25, seed=71)
    b = W.gaussian_spinor(dims, 601, nrhs=nrhs)
    z0 = W.gaussian_spinor(dims, 602, nrhs=nrhs)
    ref = [sap_sweep(S.op, b[r], z0[r], (2, 2, 2, 2), mr) for r in range(nrhs)]
    for prec, tol in ((dd.F64, 1e-12), (dd.F32, 1e-5)):
        z = dev(z0)
        dd.sap_smooth(S.H, 0, dev(b), z, 1, nrhs=nrhs, prec=prec)
        zz = host(z)
        e = max(relerr(zz[r], ref[r]) for r in range(nrhs))
        say(f"  {dims} mr={mr} x {nrhs} prec={prec}: relerr {e:.2e}")
        assert e < tol

"""P and the Galerkin operator from imported test vectors, against the oracle,
where the matrix-core tiles of the construction end unevenly: test-vector
counts on both sides of a 16-wide tile, aggregates of 256 sites that are not
4^4 (faces of 128, 64 and 32 sites), and a coarse level whose vectors do not
fill 16-element runs.

Tolerance 1e-12 relative, as for the other FP64 setup products: sums of at
most 3072 products in FP64 (sqrt(3072) 2^-53 = 6e-15) after an
orthonormalisation whose conditioning for random vectors costs a digit or
two."""
import numpy as np
import pytest

import workloads as W
from oracle.aggregation import Aggregation
from oracle.dirac import WilsonClover
from oracle.galerkin import galerkin
from tests.gpu_util import dev, export_Dc, export_P, oracle_from_gpu, relerr, say, to_params
from tests.test_gpu_hierarchy import _p

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def dd():
    from paper_1307_6101_amd import ddamg
    ddamg.load_library()
    return ddamg


def _blocks(Dc):
    return np.concatenate([Dc.S[..., None, :, :], np.moveaxis(Dc.F, 0, -3), np.moveaxis(Dc.B, 0, -3)], axis=-3)


@pytest.mark.parametrize("dims,agg,n", [((8, 8, 8, 8), (4, 4, 4, 4), 1), ((8, 8, 8, 8), (4, 4, 4, 4), 16),
                                        ((8, 8, 8, 8), (4, 4, 4, 4), 32), ((8, 8, 8, 16), (2, 4, 4, 8), 17),
                                        ((16, 8, 8, 8), (8, 4, 4, 2), 13), ((8, 8, 16, 8), (4, 2, 8, 4), 5)])
def test_rebuild_fine(dd, dims, agg, n):
    say(f"rebuild dims={dims} agg={agg} N={n}")
    U = W.links(dims, 0.5, 61)
    tv = W.test_vectors(dims, 12, n, 62)
    ctx = dd.create(dims, -0.3, 1.0, dev(U))
    H = dd.build_hierarchy(ctx, to_params(dd, _p(2, [agg], [n], n_inv=0), dd.F32), dev(tv))
    dd.import_test_vectors(H, 0, dev(tv))
    A = Aggregation(dims, agg, tv)
    assert relerr(export_P(dd, H, 0, n), A.columns()) <= TOL
    e = relerr(export_Dc(dd, H, 1), _blocks(galerkin(WilsonClover(U, -0.3, 1.0), A)))
    say(f"  D_c relerr {e:.2e}")
    assert e <= TOL


@pytest.mark.parametrize("n0,n1", [(5, 7), (9, 18)])
def test_rebuild_coarse(dd, n0, n1):
    dims = (16, 16, 16, 16)
    say(f"rebuild level 1 N={n0}, {n1}")
    U = W.links(dims, 0.5, 63)
    p = _p(3, [(4, 4, 4, 4), (2, 2, 2, 2)], [n0, n1], n_inv=0)
    ctx = dd.create(dims, -0.3, 1.0, dev(U))
    extra = W.gaussian_field((4, 4, 4, 4), 2 * n0, 65, nrhs=n1 - n0)
    H = dd.build_hierarchy(ctx, to_params(dd, p), dev(W.test_vectors(dims, 12, n0, 64)), dev(extra))
    tv = W.gaussian_field((4, 4, 4, 4), 2 * n0, 66, nrhs=n1)
    dd.import_test_vectors(H, 1, dev(tv))
    A = Aggregation((4, 4, 4, 4), (2, 2, 2, 2), tv)
    assert relerr(export_P(dd, H, 1, n1), A.columns()) <= TOL
    OH = oracle_from_gpu(dd, H, WilsonClover(U, -0.3, 1.0), p)
    assert relerr(export_Dc(dd, H, 2), _blocks(galerkin(OH.ops[1], A))) <= TOL

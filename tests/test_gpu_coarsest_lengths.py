"""The coarsest solve on both sides of the vector length up to which a
workgroup holds a system's vector (53248 bytes: 3328 FP64 components, 6656
FP32), against the oracle's cycle: the one-launch steps and the separate ones
follow the same iteration, so a cycle agrees with the oracle to the 1e-9 of
the other FP64 cycle tests, and an FP32 cycle with an FP64 one to 1e-4 (the
coarsest solve stops at 5e-2 of its right-hand side, so an iteration count
that differs would show as more than that)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.dirac import WilsonClover
from tests.gpu_util import dev, empty, host, oracle_from_gpu, relerr, say, to_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dd():
    from paper_1307_6101_amd import ddamg
    ddamg.load_library()
    return ddamg


# coarsest sites x 40 / 2 unknowns of the odd-even system: 160 sites -> 3200
# (short in both), 192 -> 3840 (short in FP32 only), 352 -> 7040 (long in
# both); 16 sites of 12 components -> 96, fewer than a workgroup's threads
@pytest.mark.parametrize("dims,ntv,oracle", [((8, 8, 8, 80), 20, True), ((8, 8, 8, 96), 20, True),
                                             ((8, 8, 16, 88), 20, False), ((8, 8, 8, 8), 6, True)])
def test_coarsest_vector_lengths(dd, dims, ntv, oracle):
    p = dict(W.DEFAULT_PARAMS)
    p.update(levels=2, agg=[(4, 4, 4, 4)], ntv=[ntv], n_inv=1, nu=2)
    U = W.links(dims, 0.5, 991)
    op = WilsonClover(U, -0.3, 1.0)
    ctx = dd.create(dims, -0.3, 1.0, dev(U))
    tv = dev(W.test_vectors(dims, 12, ntv, 992))
    b = W.gaussian_spinor(dims, 993, nrhs=3)
    out = {}
    for prec in (dd.F64, dd.F32):
        P = to_params(dd, p, prec)
        P.coarse_dense = 0
        H = dd.build_hierarchy(ctx, P, tv)
        z = empty(b.shape)
        dd.precondition(H, dev(b), z, nrhs=3)
        out[prec] = host(z)
        if oracle and prec == dd.F64:
            OH = oracle_from_gpu(dd, H, op, p)
            for r in range(3):
                e = relerr(out[prec][r], OH.cycle(0, b[r]))
                say(f"  {dims} ntv={ntv} rhs {r}: cycle against the oracle {e:.2e}")
                assert e < 1e-9
    for r in range(3):
        e = relerr(out[dd.F32][r], out[dd.F64][r])
        say(f"  rhs {r}: FP32 cycle against FP64 {e:.2e}")
        assert e < 1e-4


# The dispatch goes by the whole level's length, sites x 2N, also where the
# odd-even system has half as many unknowns: 80 sites x 40 = 3200 (short in both),
# 96 -> 3840 and 160 -> 6400 (short in FP32 only), 176 -> 7040 (long in both)
@pytest.mark.parametrize("dims,sides", [((8, 8, 8, 40), (True, True)), ((8, 8, 8, 48), (False, True)),
                                        ((8, 8, 8, 80), (False, True)), ((8, 8, 8, 88), (False, False))])
def test_coarsest_lengths_at_the_limit(dd, dims, sides):
    """As above, with the side of the line checked from the level's size."""
    p = dict(W.DEFAULT_PARAMS)
    p.update(levels=2, agg=[(4, 4, 4, 4)], ntv=[20], n_inv=1, nu=2)
    U = W.links(dims, 0.5, 991)
    op = WilsonClover(U, -0.3, 1.0)
    ctx = dd.create(dims, -0.3, 1.0, dev(U))
    tv = dev(W.test_vectors(dims, 12, 20, 992))
    b = W.gaussian_spinor(dims, 993, nrhs=2)
    out = {}
    for prec, size, short in ((dd.F64, 16, sides[0]), (dd.F32, 8, sides[1])):
        P = to_params(dd, p, prec)
        P.coarse_dense = 0
        H = dd.build_hierarchy(ctx, P, tv)
        cdims, dof = dd.level_info(H, 1)
        assert (int(np.prod(cdims)) * dof * size <= 53248) == short
        z = empty(b.shape)
        dd.precondition(H, dev(b), z, nrhs=2)
        out[prec] = host(z)
        if prec == dd.F64:
            OH = oracle_from_gpu(dd, H, op, p)
            for r in range(2):
                e = relerr(out[prec][r], OH.cycle(0, b[r]))
                say(f"  {dims} rhs {r}: cycle against the oracle {e:.2e}")
                assert e < 1e-9
    for r in range(2):
        e = relerr(out[dd.F32][r], out[dd.F64][r])
        say(f"  rhs {r}: FP32 cycle against FP64 {e:.2e}")
        assert e < 1e-4

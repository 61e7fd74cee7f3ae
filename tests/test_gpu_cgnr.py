"""FP64 CGNR on the GPU against the oracle's CGNR (Sec. 4): same iteration
count up to rounding, solutions agreeing to the tolerance's scale, the
residual bound met with the oracle's operator; a batch equals its systems
solved alone; the iteration limit and a zero right-hand side."""
import gc
import time

import numpy as np
import pytest
import torch

import workloads as W
from oracle.dirac import WilsonClover
from oracle.krylov import cgnr, norm
from tests.gpu_util import dev, empty, host, relerr, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dd():
    from paper_1307_6101_amd import ddamg
    ddamg.load_library()
    return ddamg


@pytest.fixture(autouse=True)
def _release():
    """The library allocates beside torch: what torch keeps cached of the large
    fields goes back after each test."""
    yield
    gc.collect()
    torch.cuda.empty_cache()


@pytest.fixture(scope="module")
def lat(dd):
    dims = (8, 8, 8, 8)
    U = W.links(dims, 0.5, 811)
    op = WilsonClover(U, -0.2, 1.0)
    ctx = dd.create(dims, -0.2, 1.0, dev(U))
    b = W.gaussian_spinor(dims, 812, nrhs=3)
    return dims, op, ctx, b


def test_cgnr_matches_oracle(dd, lat):
    dims, op, ctx, b = lat
    st = {}
    xo = cgnr(op.apply, op.apply_dagger, b[0], 1e-10, 5000, stats=st)
    z = empty(b[:1].shape)
    rc, sg = dd.cgnr(ctx, dev(b[:1]), z, tol=1e-10)
    zz = host(z)[0]
    say(f"  CGNR iterations: oracle {st['iters']}, GPU {sg[0]['outer_iters']}, rel. diff {relerr(zz, xo):.1e}")
    assert rc == dd.OK
    assert abs(sg[0]["outer_iters"] - st["iters"]) <= 2
    assert relerr(zz, xo) <= 1e-8
    res = norm(b[0] - op.apply(zz)) / norm(b[0])
    assert res <= 1e-10 and abs(res - sg[0]["true_relres"]) <= 1e-12


def test_cgnr_batch_equals_alone(dd, lat):
    dims, op, ctx, b = lat
    z3 = empty(b.shape)
    rc, s3 = dd.cgnr(ctx, dev(b), z3, nrhs=3, tol=1e-10)
    assert rc == dd.OK
    zz3 = host(z3)
    for r in range(3):
        z1 = empty(b[:1].shape)
        rc1, s1 = dd.cgnr(ctx, dev(b[r:r + 1]), z1, tol=1e-10)
        assert s1[0]["outer_iters"] == s3[r]["outer_iters"]
        assert relerr(zz3[r], host(z1)[0]) <= 1e-13
        assert norm(b[r] - op.apply(zz3[r])) / norm(b[r]) <= 1e-10


def test_cgnr_limits(dd, lat):
    dims, op, ctx, b = lat
    z = empty(b[:1].shape)
    rc, st = dd.cgnr(ctx, dev(b[:1]), z, tol=1e-10, max_iter=5)
    assert rc == dd.ENOCONV and st[0]["outer_iters"] == 5 and st[0]["status"] == dd.ENOCONV
    zb = np.zeros_like(b[:2])
    zb[1] = b[1]
    z2 = empty(zb.shape)
    rc, st = dd.cgnr(ctx, dev(zb), z2, nrhs=2, tol=1e-10)
    assert rc == dd.OK and st[0]["outer_iters"] == 0
    assert np.all(host(z2)[0] == 0)
    with pytest.raises(dd.DDAMGError):
        dd.cgnr(ctx, dev(b[:1]), z, tol=0.0)


def test_cgnr_many_norm_parts(dd):
    """A lattice with more tiles than the update kernels sum themselves (the
    stencil's norm parts are folded first), two systems of which one starts at
    its solution.  A residual of 1e-8 leaves an error of at most 1e-8 times the
    condition number of D, below 100 for this massive operator."""
    dims = (16, 16, 32, 36)
    say(f"cgnr dims={dims}")
    ctx = dd.create(dims, -0.3, 1.0, dev(W.links(dims, 0.5, 91)))
    zs = dev(W.gaussian_spinor(dims, 92, nrhs=2))
    b, z = torch.empty_like(zs), torch.zeros_like(zs)
    dd.apply_D(ctx, zs, b, nrhs=2)
    z[1] = zs[1]
    rc, st = dd.cgnr(ctx, b, z, nrhs=2, tol=1e-8)
    assert rc == dd.OK and st[1]["outer_iters"] == 0 and st[0]["outer_iters"] > 50
    assert st[0]["true_relres"] <= 1e-8
    assert float((z[0] - zs[0]).norm() / zs[0].norm()) <= 1e-6
    assert torch.equal(z[1], zs[1])


def test_cgnr_short_run_time(dd):
    """A run that its tolerance ends after one iteration takes the time of one that
    max_iter ends there (32^3x64: 2.3 ms an iteration beside 5.7 ms for the norms,
    residuals and vectors of a call), not that of iterations issued ahead."""
    dims = (32, 32, 32, 64)
    g = torch.Generator(device="cuda").manual_seed(5)
    shape = dims[::-1]
    ctx = dd.create(dims, 1.0, 1.0, 0.1 * torch.randn(shape + (4, 3, 3), generator=g, device="cuda", dtype=torch.complex128))
    b = torch.randn(shape + (12,), generator=g, device="cuda", dtype=torch.complex128)
    z = torch.zeros_like(b)
    times = {}
    for name, tol, limit in (("tol", 0.9, 50), ("limit", 1e-12, 1)) * 6:
        z.zero_()
        torch.cuda.synchronize()
        t = time.perf_counter()
        rc, st = dd.cgnr(ctx, b, z, tol=tol, max_iter=limit)
        dt = time.perf_counter() - t
        assert st[0]["outer_iters"] == 1 and rc == (dd.OK if name == "tol" else dd.ENOCONV)
        times[name] = min(dt, times.get(name, 1e30))
    say(f"cgnr one iteration: {1e3 * times['tol']:.2f} ms by tolerance, {1e3 * times['limit']:.2f} ms by limit")
    assert times["tol"] <= 1.25 * times["limit"]


def test_cgnr_streamed_operator(dd):
    """One system on a lattice whose FP64 operator does not fit the last-level
    cache (it is read past the caches), against its known solution; tolerance as
    for the many norm parts."""
    dims = (16, 16, 32, 36)
    say(f"cgnr dims={dims}, one system")
    ctx = dd.create(dims, -0.3, 1.0, dev(W.links(dims, 0.5, 91)))
    zs = dev(W.gaussian_spinor(dims, 92, nrhs=2))[:1].contiguous()
    b, z = torch.empty_like(zs), torch.zeros_like(zs)
    dd.apply_D(ctx, zs, b)
    rc, st = dd.cgnr(ctx, b, z, tol=1e-8)
    assert rc == dd.OK and st[0]["outer_iters"] > 50 and st[0]["true_relres"] <= 1e-8
    assert float((z - zs).norm() / zs.norm()) <= 1e-6

"""Batched coarse-level operator and SAP smoother on the matrix cores, against
the FP64 oracle on the operator the kernels store (rounded to FP16 where the
hierarchy has FP16 storage, so that only the arithmetic differs).

Sizes: components per site that fill their 16-row tiles (64), end inside one
(40, 56) or inside a step of four columns (26); batches at the edges of the
dispatch and of a 16-field chunk; SAP blocks of 16 sites and of one site.

Tolerance: a component is a sum of 9d complex products in FP32, whose rounding
errors add to about sqrt(4 * 9d) 2^-24 <= 3e-6 of it; a smoother step stacks a
few such products: 1e-5 for both."""
import gc

import numpy as np
import pytest
import torch

import workloads as W
from oracle.sap import smooth
from oracle.stencil import BlockStencil
from tests.gpu_util import dev, empty, export_Dc, host, relerr, say, to_params
from tests.test_gpu_hierarchy import _p

pytestmark = pytest.mark.gpu

DIMS = (16, 16, 16, 16)
TOL = 1e-5


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


def _half(a):
    return a.real.astype(np.float16).astype(np.float64) + 1j * a.imag.astype(np.float16).astype(np.float64)


@pytest.mark.parametrize("n,half,nrhs", [(20, False, (3, 17)), (20, True, (5, 16)), (13, True, (3,)), (28, False, (16,)),
                                         (32, True, (3, 14))])
def test_batched_coarse_level(dd, n, half, nrhs):
    say(f"coarse batch d={2 * n} half={half} nrhs={nrhs}")
    p = _p(3, [(4, 4, 4, 4), (2, 2, 2, 2)], [n, 4], n_inv=0)
    ctx = dd.create(DIMS, -0.3, 1.0, dev(W.links(DIMS, 0.5, 71)))
    H = dd.build_hierarchy(ctx, to_params(dd, p, dd.F32, half=half), dev(W.test_vectors(DIMS, 12, n, 72)))
    G = export_Dc(dd, H, 1)
    if half:
        G = _half(G)
    op = BlockStencil((4, 4, 4, 4), G[..., 0, :, :], np.moveaxis(G[..., 1:5, :, :], -3, 0),
                      np.moveaxis(G[..., 5:9, :, :], -3, 0))
    for nb in nrhs:
        b = W.gaussian_field(op.dims, op.d, 80 + nb, nrhs=nb)
        z0 = 0.3 * W.gaussian_field(op.dims, op.d, 81 + nb, nrhs=nb)
        out = empty(b.shape)
        dd.apply_Dc(H, 1, dev(b), out, nrhs=nb, prec=dd.F32)
        got = host(out)
        for r in range(nb):
            assert relerr(got[r], op.apply(b[r])) <= TOL, (nb, r)
        for block in ((2, 2, 2, 2), (1, 1, 1, 1)):
            dd.set_sap_block(H, 1, block)
            z = dev(z0)
            dd.sap_smooth(H, 1, dev(b), z, 2, nrhs=nb, prec=dd.F32)
            got = host(z)
            e = max(relerr(got[r], smooth(op, b[r], z0[r], 2, block)) for r in range(nb))
            say(f"  nrhs={nb} block={block} relerr {e:.2e}")
            assert e <= TOL
    torch.cuda.synchronize()


@pytest.mark.parametrize("dims,n,nb", [((16, 16, 16, 16), 20, 4), ((16, 16, 16, 16), 6, 3), ((32, 32, 16, 32), 8, 2)])
def test_half_storage_batch_against_single(dd, dims, n, nb):
    """FP16 storage, batches on both sides of the dispatch's lines (nb = 2 goes
    to the matrix cores from 2048 sites), against the same fields one by one on
    the vector kernels; and fields of very different scale, a zero field and
    one with a NaN in it, none of which may touch another.  Tolerance: two
    results with TOL of the exact one each."""
    p = _p(2, [(4, 4, 4, 4)], [n], n_inv=0)
    g = torch.Generator(device="cuda").manual_seed(5)

    def field(sites, dof, k):
        return torch.randn((k,) + sites + (dof,), generator=g, device="cuda", dtype=torch.complex128)

    shape = tuple(dims)[::-1]
    ctx = dd.create(dims, -0.3, 1.0, dev(W.links(dims, 0.5, 71)))
    H = dd.build_hierarchy(ctx, to_params(dd, p, dd.F32, half=True), field(shape, 12, n))
    cs = tuple(e // 4 for e in shape)
    b = field(cs, 2 * n, nb)
    scale = [1.0, 1e-30, 1e30, 0.0][:nb]
    for r in range(nb):
        b[r] *= scale[r]
    out = torch.zeros_like(b)
    dd.apply_Dc(H, 1, b, out, nrhs=nb, prec=dd.F32)
    for r in range(nb):
        one = torch.zeros_like(b[r])
        dd.apply_Dc(H, 1, b[r].contiguous(), one, prec=dd.F32)
        assert float((out[r] - one).norm()) <= 2 * TOL * float(one.norm()), r
    b = field(cs, 2 * n, nb)
    b.view(nb, -1)[nb - 1, 3] = float("nan")
    z = torch.zeros_like(b)
    dd.apply_Dc(H, 1, b, z, nrhs=nb, prec=dd.F32)
    assert bool(torch.isnan(torch.view_as_real(z[nb - 1])).any())
    for r in range(nb - 1):
        one = torch.zeros_like(b[r])
        dd.apply_Dc(H, 1, b[r].contiguous(), one, prec=dd.F32)
        assert float((z[r] - one).norm()) <= 2 * TOL * float(one.norm()), r
    torch.cuda.synchronize()


# groups of wavefronts per row tile (1, 2, 4) and lanes per staged row (8, 16, 32,
# 64) of the matrix-core kernels over d and the number of sites: 4^4 sites take
# the most groups, 8^4 the fewest; 16 FP32 fields of d = 56 the even pitch
@pytest.mark.parametrize("e,n,half,nb", [(16, 4, True, 5), (16, 4, False, 16), (16, 7, True, 9), (16, 10, False, 3),
                                         (16, 28, False, 16), (32, 4, True, 3), (32, 4, False, 17), (32, 8, True, 9),
                                         (32, 13, False, 3), (32, 13, True, 9), (32, 20, False, 5), (32, 22, True, 11),
                                         (32, 28, False, 16), (32, 32, True, 3)])
def test_batch_shapes_against_single(dd, e, n, half, nb):
    """Operator and two SAP sweeps of a batch against its fields one by one (the
    vector kernels).  Tolerance: two results with TOL of the exact one each."""
    say(f"coarse shapes e={e} d={2 * n} half={half} nb={nb}")
    g = torch.Generator(device="cuda").manual_seed(11)

    def field(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.complex128)

    dims = (e,) * 4
    p = _p(3, [(4, 4, 4, 4), (2, 2, 2, 2)], [n, 4], n_inv=0)
    ctx = dd.create(dims, 1.0, 1.0, 0.3 * field(e, e, e, e, 4, 3, 3))
    H = dd.build_hierarchy(ctx, to_params(dd, p, dd.F32, half=half), field(n, e, e, e, e, 12))
    b, z0 = (field(nb, *((e // 4,) * 4), 2 * n) for _ in range(2))
    out, z = torch.zeros_like(b), z0.clone()
    dd.apply_Dc(H, 1, b, out, nrhs=nb, prec=dd.F32)
    dd.sap_smooth(H, 1, b, z, 2, nrhs=nb, prec=dd.F32)
    for r in range(nb):
        one, zr = torch.zeros_like(b[r]), z0[r].clone()
        dd.apply_Dc(H, 1, b[r].contiguous(), one, prec=dd.F32)
        dd.sap_smooth(H, 1, b[r].contiguous(), zr, 2, prec=dd.F32)
        assert float((out[r] - one).norm()) <= 2 * TOL * float(one.norm()), r
        assert float((z[r] - zr).norm()) <= 2 * TOL * float(zr.norm()), r


@pytest.mark.parametrize("e,n,nb,bound", [(16, 4, 16, 2.5), (16, 8, 12, 2.5), (32, 8, 16, 4.0)])
def test_batch_time(dd, e, n, nb, bound):
    """A batch of small blocks costs little more than one field: on 4^4 sites, where
    latency counts, less than 2.5 times its time, on 8^4 sites (the fields' bytes
    are a third of the operator's) less than 4 times."""
    g = torch.Generator(device="cuda").manual_seed(12)

    def field(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.complex128)

    dims = (e,) * 4
    p = _p(3, [(4, 4, 4, 4), (2, 2, 2, 2)], [n, 4], n_inv=0)
    ctx = dd.create(dims, 1.0, 1.0, 0.3 * field(e, e, e, e, 4, 3, 3))
    H = dd.build_hierarchy(ctx, to_params(dd, p, dd.F32, half=True), field(n, e, e, e, e, 12))
    b = field(nb, (e // 4) ** 4, 2 * n).to(torch.complex64)
    z = torch.zeros_like(b)

    def time(call, k):
        best = 1e30
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for _ in range(8):
            ev[0].record()
            for _ in range(20):
                call(k)
            ev[1].record()
            torch.cuda.synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]) / 20)
        return best

    for name, call in (("apply", lambda k: dd.apply_Dc(H, 1, b, z, k, dd.F16, dd.NATIVE)),
                       ("sap", lambda k: dd.sap_smooth(H, 1, b, z, 1, k, dd.F16, dd.NATIVE))):
        t1, tn = time(call, 1), time(call, nb)
        say(f"  {name} e={e} d={2 * n}: one field {1e3 * t1:.1f} us, {nb} fields {1e3 * tn:.1f} us")
        assert tn <= bound * t1

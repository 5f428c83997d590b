"""The pencil kernels of the collapsed shapes with per-element factors: every order, at counts around
their groups (1 to 21 elements by shape, order and type), and as items of the persistent mixed kernel,
with work items whose last groups are short or empty.

Against the FP64 oracle, normwise per element, at the bars of the operator tests (FP64 1e-12, FP32
2e-4); the values after the batch must stay what they were; the persistent kernel runs the same device
code as the standalone pencil kernels, so its results are theirs bit for bit.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import geometry as og, operators as op
from paper_2606_20917_amd import nir
from tests.gpu_util import elem_relerr, small_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda"
TOL = {nir.F64: 1e-12, nir.F32: 2e-4}


def _batch(shape, P, ne, dtype):
    real = torch.float64 if dtype == nir.F64 else torch.float32
    verts = small_mesh(shape, 3, 7 + P, 0.03 if shape == nir.TET else 0.0, 0.0)
    verts = np.ascontiguousarray(np.tile(verts, (-(-ne // len(verts)), 1, 1))[:ne])
    basis = nir.Basis(shape, P)
    helm = torch.empty(ne, 7, dtype=torch.float64, device=DEV)
    nir.nir_geom_from_vertices(nir.batch(shape, P, ne, nir.F64, 0), basis, torch.tensor(verts, device=DEV), nir.MAP_VERTEX,
                               0.0, helm64=helm)
    c = torch.tensor(np.random.default_rng(P).uniform(-1, 1, (ne, nir.nir_nmodes(shape, P))), device=DEV).to(real)
    return verts, basis, nir.geom(helm=helm.to(real)), c


def _ref(shape, P, verts, lam, c):
    return op.helmholtz(op.Tables(shape, P, P + 1), og.Geometry(shape, P + 1, verts, 0.0), lam, c.double().cpu().numpy())


@pytest.mark.parametrize("dtype", [nir.F64, nir.F32])
@pytest.mark.parametrize("P", range(2, 11))
@pytest.mark.parametrize("shape", [nir.PRISM, nir.TET, nir.PYR])
def test_counts_around_a_group(shape, P, dtype):
    verts, basis, g, c = _batch(shape, P, 24, dtype)
    ref = _ref(shape, P, verts, 0.7, c)
    try:
        nir.nir_set_helmholtz_variant(shape, P, dtype, nir.VARIANT_PENCIL)
        for ne in (1, 2, 4, 5, 7, 8, 11, 13, 15, 22, 24):
            out = torch.full((ne + 3, c.shape[1]), 7.0, dtype=c.dtype, device=DEV)
            nir.nir_helmholtz_apply(nir.batch(shape, P, ne, dtype, 0), basis, g, 0.7, c, out)
            assert elem_relerr(out[:ne].cpu().numpy(), ref[:ne]) <= TOL[dtype], ne
            assert bool((out[ne:] == 7.0).all()), ne
    finally:
        nir.nir_set_helmholtz_variant(shape, P, dtype, nir.VARIANT_AUTO)


@pytest.mark.parametrize("dtype", [nir.F64, nir.F32])
@pytest.mark.parametrize("P", range(2, 9))
def test_persistent_items(P, dtype):
    """Hexahedra, prisms and tetrahedra of one order; a count of one leaves every group of its item but
    the first empty."""
    shapes = (nir.HEX, nir.PRISM, nir.TET)
    try:
        for shape in shapes:
            nir.nir_set_helmholtz_variant(shape, P, dtype, nir.VARIANT_PENCIL)
        for counts in ((1, 1, 1), (27, 54, 100), (64, 37, 41)):
            parts = [_batch(shape, P, ne, dtype) for shape, ne in zip(shapes, counts)]
            bs = [nir.batch(shape, P, ne, dtype, 0) for shape, ne in zip(shapes, counts)]
            plan = nir.MixedPlan(bs, [p[1] for p in parts], [p[2] for p in parts])
            plan.set_strategy(nir.MIXED_PERSISTENT)
            ys = [torch.full((len(p[3]) + 3, p[3].shape[1]), 7.0, dtype=p[3].dtype, device=DEV) for p in parts]
            nir.nir_mixed_helmholtz_apply(plan, 0.7, [p[3] for p in parts], ys)
            for (verts, basis, g, c), b, y, shape in zip(parts, bs, ys, shapes):
                one = torch.empty_like(c)
                nir.nir_helmholtz_apply(b, basis, g, 0.7, c, one)
                assert torch.equal(y[:len(c)], one), (shape, counts)
                assert bool((y[len(c):] == 7.0).all()), (shape, counts)
                assert elem_relerr(one.cpu().numpy(), _ref(shape, P, verts, 0.7, c)) <= TOL[dtype], (shape, counts)
    finally:
        for shape in shapes:
            nir.nir_set_helmholtz_variant(shape, P, dtype, nir.VARIANT_AUTO)

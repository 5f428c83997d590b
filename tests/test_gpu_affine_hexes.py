"""Affine hexahedra (per-element factors), whose default is the folded kernel with its own blocks of 1
to 28 elements: counts around a block, every order and both types, against the oracle's explicit
operators, the values after the batch untouched.

Bars of the operator tests (normwise per element): FP64 1e-12, FP32 2e-4.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import geometry as og, operators as op
from paper_2606_20917_amd import nir
from tests.gpu_util import elem_relerr, small_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("variant", [nir.VARIANT_AUTO, nir.VARIANT_PENCIL_EO, nir.VARIANT_PENCIL_EO_SPLIT])
@pytest.mark.parametrize("dtype", [nir.F64, nir.F32])
@pytest.mark.parametrize("P", range(2, 11))
def test_counts_around_a_block(P, dtype, variant):
    real = torch.float64 if dtype == nir.F64 else torch.float32
    # boxes of differing sides, sheared
    verts = small_mesh(nir.HEX, 4, 3, 0.0, 0.0) ** 2 @ np.array([[1.0, 0.1, 0.0], [0.3, 1.2, 0.2], [0.0, -0.2, 0.9]])
    tab, basis = op.Tables(nir.HEX, P, P + 1), nir.Basis(nir.HEX, P)
    geo = og.Geometry(nir.HEX, P + 1, verts, 0.0)
    ne = len(verts)
    c = torch.tensor(np.random.default_rng(P).uniform(-1, 1, (ne, tab.M)), device=DEV).to(real)
    helm = torch.empty(ne, 7, dtype=torch.float64, device=DEV)
    nir.nir_geom_from_vertices(nir.batch(nir.HEX, P, ne, nir.F64, 0), basis, torch.tensor(verts, device=DEV),
                               nir.MAP_VERTEX, 0.0, helm64=helm)
    helm = helm.to(real)
    ref = op.helmholtz(tab, geo, 0.7, c.double().cpu().numpy())
    try:
        nir.nir_set_helmholtz_variant(nir.HEX, P, dtype, variant)
        for n in (1, 2, 3, 4, 5, 6, 27, 28, 29, 57, ne):
            out = torch.full((n + 3, tab.M), 7.0, dtype=real, device=DEV)
            nir.nir_helmholtz_apply(nir.batch(nir.HEX, P, n, dtype, 0), basis, nir.geom(helm=helm), 0.7, c, out)
            assert elem_relerr(out[:n].cpu().numpy(), ref[:n]) <= (1e-12 if dtype == nir.F64 else 2e-4), n
            assert bool((out[n:] == 7.0).all()), n
    finally:
        nir.nir_set_helmholtz_variant(nir.HEX, P, dtype, nir.VARIANT_AUTO)

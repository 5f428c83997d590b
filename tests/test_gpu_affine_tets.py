"""Affine tetrahedra through the gradient tables, at counts around the kernel's blocks of 16 to 96
elements, every order and both types, against the oracle's explicit operators.

Bars of the operator tests (normwise per element): FP64 1e-12, FP32 2e-4.  The values after the batch
must stay what they were.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import geometry as og, operators as op
from paper_2606_20917_amd import nir
from tests.gpu_util import elem_relerr, small_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype", [nir.F64, nir.F32])
@pytest.mark.parametrize("P", range(2, 11))
def test_counts_around_a_block(P, dtype):
    real = torch.float64 if dtype == nir.F64 else torch.float32
    verts = small_mesh(nir.TET, 3, 11 + P, 0.05, 0.0)   # 162 elements
    tab, basis = op.Tables(nir.TET, P, P + 1), nir.Basis(nir.TET, P)
    geo = og.Geometry(nir.TET, P + 1, verts, 0.0)
    ne = len(verts)
    c = torch.tensor(np.random.default_rng(P).uniform(-1, 1, (ne, tab.M)), device=DEV).to(real)
    helm = torch.empty(ne, 7, dtype=torch.float64, device=DEV)
    nir.nir_geom_from_vertices(nir.batch(nir.TET, P, ne, nir.F64, 0), basis, torch.tensor(verts, device=DEV),
                               nir.MAP_VERTEX, 0.0, helm64=helm)
    helm = helm.to(real)
    for lam in (1.0, 0.0):
        ref = op.helmholtz(tab, geo, lam, c.double().cpu().numpy())
        for n in (1, 15, 16, 17, 33, 48, 49, 64, 65, 97, 129, ne):
            out = torch.full((n + 3, tab.M), 7.0, dtype=real, device=DEV)
            nir.nir_helmholtz_apply(nir.batch(nir.TET, P, n, dtype, 0), basis, nir.geom(helm=helm), lam, c, out)
            assert elem_relerr(out[:n].cpu().numpy(), ref[:n]) <= (1e-12 if dtype == nir.F64 else 2e-4), (n, lam)
            assert bool((out[n:] == 7.0).all()), n

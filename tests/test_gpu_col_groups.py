"""Collapsed-shape Helmholtz kernels at element counts around their groups (1 to 21 elements by shape,
order and type): the lanes past the batch end read zeros or nothing, and never write.

FP64 bar 1e-12, FP32 bar 2e-4 (the bars of the operator tests, normwise per element); the values
after the batch must stay what they were.
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
@pytest.mark.parametrize("P", [2, 5, 7, 8, 10])
@pytest.mark.parametrize("shape", [nir.PRISM, nir.TET, nir.PYR])
def test_counts_around_a_group(shape, P, dtype):
    Q, amp = P + 1, 0.05
    real = torch.float64 if dtype == nir.F64 else torch.float32
    verts = small_mesh(shape, 3, 7 + P, 0.03, 0.0)
    tab, basis = op.Tables(shape, P, Q), nir.Basis(shape, P)
    rng = np.random.default_rng(P)
    for ne in (1, 4, 5, 7, 8, 13, 15, 22):
        v = verts[:ne]
        helm = torch.empty(ne, 7, Q ** 3, dtype=torch.float64, device=DEV)
        b = nir.batch(shape, P, ne, dtype, 1)
        nir.nir_geom_from_vertices(b, basis, torch.tensor(v, device=DEV), nir.MAP_VERTEX_SIN, amp, helm64=helm)
        c = torch.tensor(rng.uniform(-1, 1, (ne, tab.M)), device=DEV).to(real)
        out = torch.full((ne + 3, tab.M), 7.0, dtype=real, device=DEV)
        nir.nir_helmholtz_apply(b, basis, nir.geom(helm=helm.to(real)), 1.0, c, out)
        ref = op.helmholtz(tab, og.Geometry(shape, Q, v, amp), 1.0, c.double().cpu().numpy())
        assert elem_relerr(out[:ne].cpu().numpy(), ref) <= (1e-12 if dtype == nir.F64 else 2e-4), ne
        assert bool((out[ne:] == 7.0).all()), ne

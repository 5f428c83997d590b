"""Affine hexahedra at P = 5, 9 and 10 on both sides of the counts where the blocks change: against the FP64
oracle, normwise per element at the operator tests' bars (FP64 1e-12, FP32 2e-4), on a mesh of 8 elements
repeated with coefficients of 24, with the values after the batch untouched."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import geometry as og, operators as op
from paper_2606_20917_amd import nir
from tests.gpu_util import elem_relerr, small_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda"
COUNTS = {5: (6144, 6145, 7168, 7169), 9: (256, 257, 512, 513, 1280, 1281, 5120, 5121), 10: (256, 257, 513, 1281, 1536, 1537)}


@pytest.mark.parametrize("dtype", [nir.F64, nir.F32])
@pytest.mark.parametrize("P", sorted(COUNTS))
def test_counts_where_the_blocks_change(P, dtype):
    few, top = 24, max(COUNTS[P])
    real = torch.float64 if dtype == nir.F64 else torch.float32
    verts = np.tile(small_mesh(nir.HEX, 2, P, 0.0, 0.0), (3, 1, 1))
    tab, basis = op.Tables(nir.HEX, P, P + 1), nir.Basis(nir.HEX, P)
    helm = torch.empty(few, 7, dtype=torch.float64, device=DEV)
    nir.nir_geom_from_vertices(nir.batch(nir.HEX, P, few, nir.F64, 0), basis, torch.tensor(verts, device=DEV),
                               nir.MAP_VERTEX, 0.0, helm64=helm)
    c = torch.tensor(np.random.default_rng(P).uniform(-1, 1, (few, P ** 3)), device=DEV).to(real)
    ref = op.helmholtz(tab, og.Geometry(nir.HEX, P + 1, verts, 0.0), 0.7, c.double().cpu().numpy())
    reps = -(-top // few)
    helm, x, ref = helm.to(real).repeat(reps, 1), c.repeat(reps, 1), np.tile(ref, (reps, 1))
    for ne in COUNTS[P]:
        out = torch.full((ne + 3, P ** 3), 7.0, dtype=real, device=DEV)
        nir.nir_helmholtz_apply(nir.batch(nir.HEX, P, ne, dtype, 0), basis, nir.geom(helm=helm), 0.7, x, out)
        assert elem_relerr(out[:ne].cpu().numpy(), ref[:ne]) <= (1e-12 if dtype == nir.F64 else 2e-4), ne
        assert bool((out[ne:] == 7.0).all()), ne

"""FP64 tetrahedra and pyramids at P = 7 on both sides of the counts where the launch shape changes (2,048,
3,584 and 4,096 elements): against the FP64 oracle at the operator tests' bar, 1e-12 normwise per element,
on a mesh of 24 elements repeated, with the values after the batch untouched."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import geometry as og, operators as op
from paper_2606_20917_amd import nir
from tests.gpu_util import elem_relerr, small_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("shape", [nir.TET, nir.PYR])
def test_counts_where_the_launch_shape_changes(shape):
    P, Q, few, top = 7, 8, 24, 4097
    verts = small_mesh(shape, 3, 1, 0.03, 0.0)[:few]
    tab, basis = op.Tables(shape, P, Q), nir.Basis(shape, P)
    helm = torch.empty(few, 7, Q ** 3, dtype=torch.float64, device=DEV)
    nir.nir_geom_from_vertices(nir.batch(shape, P, few, nir.F64, 1), basis, torch.tensor(verts, device=DEV),
                               nir.MAP_VERTEX_SIN, 0.05, helm64=helm)
    c = np.random.default_rng(P).uniform(-1, 1, (few, tab.M))
    ref = op.helmholtz(tab, og.Geometry(shape, Q, verts, 0.05), 0.7, c)
    reps = -(-top // few)
    helm, x, ref = helm.repeat(reps, 1, 1), torch.tensor(c, device=DEV).repeat(reps, 1), np.tile(ref, (reps, 1))
    for ne in (2047, 2048, 2049, 3584, 3585, 4096, 4097):
        out = torch.full((ne + 3, tab.M), 7.0, dtype=torch.float64, device=DEV)
        nir.nir_helmholtz_apply(nir.batch(shape, P, ne, nir.F64, 1), basis, nir.geom(helm=helm), 0.7, x, out)
        assert elem_relerr(out[:ne].cpu().numpy(), ref[:ne]) <= 1e-12, ne
        assert bool((out[ne:] == 7.0).all()), ne

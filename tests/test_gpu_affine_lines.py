"""Where affine batches pass from the pencil kernel to the matrix cores: the default is the pencil
kernel's result up to the line and the dense variant's from it, bit for bit, with the values after
the batch untouched; and the dense variant itself, which small batches no longer reach by default, at
counts around its blocks.  The two kernels agree within the operator tests' bars (normwise per
element, FP64 1e-12, FP32 2e-4).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2606_20917_amd import nir
from tests.gpu_util import elem_relerr, small_mesh

pytestmark = pytest.mark.gpu
DEV = "cuda"
F32, F64 = nir.F32, nir.F64
LINES = [(nir.TET, 6, F64, 0), (nir.TET, 7, F64, 2048), (nir.TET, 8, F64, 1792), (nir.TET, 9, F64, 6144),
         (nir.TET, 10, F64, 2560), (nir.TET, 7, F32, 0), (nir.TET, 8, F32, 4096), (nir.TET, 9, F32, 6144),
         (nir.TET, 10, F32, 3840), (nir.PYR, 4, F64, 0), (nir.PYR, 5, F64, 4096), (nir.PYR, 6, F64, 8192),
         (nir.PYR, 5, F32, 8192), (nir.PYR, 6, F32, 8192), (nir.PRISM, 3, F32, 0), (nir.PRISM, 4, F64, None),
         (nir.PRISM, 4, F32, None)]


@pytest.mark.parametrize("shape,P,dtype,line", LINES)
def test_default_on_both_sides_of_the_line(shape, P, dtype, line):
    real = torch.float64 if dtype == F64 else torch.float32
    verts = small_mesh(shape, 3, P, 0.05 if shape == nir.TET else 0.0, 0.0)
    basis, M, few = nir.Basis(shape, P), nir.nir_nmodes(shape, P), len(verts)
    helm = torch.empty(few, 7, dtype=torch.float64, device=DEV)
    nir.nir_geom_from_vertices(nir.batch(shape, P, few, F64, 0), basis, torch.tensor(verts, device=DEV),
                               nir.MAP_VERTEX, 0.0, helm64=helm)
    counts = [1, 15, 16, 17, 49, 97, few] + ([] if not line else [line - 1, line])
    top = max(counts)
    helm = helm.repeat(-(-top // few), 1)[:top].to(real).contiguous()
    c = torch.tensor(np.random.default_rng(P).uniform(-1, 1, (top, M)), device=DEV).to(real)

    def run(variant, n):
        out = torch.full((n + 3, M), 7.0, dtype=real, device=DEV)
        nir.nir_set_helmholtz_variant(shape, P, dtype, variant)
        nir.nir_helmholtz_apply(nir.batch(shape, P, n, dtype, 0), basis, nir.geom(helm=helm), 0.7, c, out)
        assert bool((out[n:] == 7.0).all()), n
        return out[:n]

    try:
        for n in counts:
            auto, dense, pencil = (run(v, n) for v in (nir.VARIANT_AUTO, nir.VARIANT_DENSE, nir.VARIANT_PENCIL))
            assert torch.equal(auto, pencil if line is None or n < line else dense), n
            assert elem_relerr(dense.cpu().numpy(), pencil.double().cpu().numpy()) <= (1e-12 if dtype == F64 else 2e-4), n
    finally:
        nir.nir_set_helmholtz_variant(shape, P, dtype, nir.VARIANT_AUTO)

"""The fused CG iteration: the element apply that gathers by itself, in every hex kernel family and
order, and the scatter-reduce and reductions at counts around their thread and row groups.

A solution is judged by its residual formed through the public gather, apply and scatter-add, which
share no gather or reduction with the solver: ||b - A x|| <= 1.5e-10 ||b|| for a solve to 1e-10.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2606_20917_amd import nir
from tests.test_gpu_solver import DEV, _gpu_rhs, _problem

pytestmark = pytest.mark.gpu

FAMILIES = [nir.VARIANT_GENERIC, nir.VARIANT_PENCIL, nir.VARIANT_PENCIL_PF, nir.VARIANT_PENCIL_SPLIT_GP,
            nir.VARIANT_PENCIL_EO, nir.VARIANT_PENCIL_EO_SPLIT]


def _public_residual(pr, b, x):
    g = nir.geom(None, None, pr["helm"])
    xl = torch.empty(pr["ne"], pr["P"] ** 3, dtype=torch.float64, device=DEV)
    yl, yg = torch.empty_like(xl), torch.empty_like(b)
    nir.nir_gather(pr["A"], nir.F64, x, xl)
    nir.nir_helmholtz_apply(pr["b64"], pr["basis"], g, pr["lam"], xl, yl)
    nir.nir_scatter_add(pr["A"], nir.F64, yl, yg)
    return float((b - yg).norm() / b.norm())


@pytest.mark.parametrize("variant", FAMILIES)
@pytest.mark.parametrize("P", range(2, 11))
def test_solution_through_the_public_operators(P, variant):
    pr = _problem(3 if P < 6 else 2, P)   # 27 or 8 elements: no whole number of groups
    b = _gpu_rhs(pr)
    if float(b.norm()) == 0.0:
        pytest.skip("zero right-hand side")
    try:
        for dt in (nir.F64, nir.F32):
            nir.nir_set_helmholtz_variant(nir.HEX, P, dt, variant)
        plan = nir.CGPlan(pr["b64"], pr["basis"], nir.geom(None, None, pr["helm"]), pr["helm32"], pr["A"], pr["lam"])
        for mode in (nir.CG_FP64, nir.CG_MIXED_F32):
            x = torch.zeros(pr["ng"], dtype=torch.float64, device=DEV)
            _, info = nir.nir_cg_solve(plan, mode, b, x, rtol=1e-10, maxit=20000)
            res = _public_residual(pr, b, x)
            assert res <= 1.5e-10 and abs(res - info.rel_residual) <= 1e-11, (mode, res, info.rel_residual)
    finally:
        for dt in (nir.F64, nir.F32):
            nir.nir_set_helmholtz_variant(nir.HEX, P, dt, nir.VARIANT_AUTO)


@pytest.mark.parametrize("dtype", [nir.F64, nir.F32])
@pytest.mark.parametrize("ng,nelmt,M", [(1, 1, 1), (255, 64, 4), (257, 300, 3), (1025, 41, 25), (70000, 20000, 7)])
def test_scatter_rows_of_any_length(ng, nelmt, M, dtype):
    """Rows of 1 to many entries in no order, at counts around a block and a thread's rows: the
    FP64 sums are bincount's (the same order), the FP32 ones a sequential FP32 sum."""
    rng = np.random.default_rng(ng)
    l2g = rng.integers(0, ng, nelmt * M)
    if nelmt * M >= ng:
        l2g[rng.permutation(nelmt * M)[:ng]] = np.arange(ng)   # every row has an entry
    used = np.unique(l2g)
    l2g = np.searchsorted(used, l2g).astype(np.int32)
    ng = len(used)
    A = nir.Assembly(torch.tensor(l2g.reshape(nelmt, M), device=DEV), ng)
    npdt = np.float64 if dtype == nir.F64 else np.float32
    yl = rng.uniform(-1, 1, nelmt * M).astype(npdt)
    yg = torch.empty(ng, dtype=torch.float64 if dtype == nir.F64 else torch.float32, device=DEV)
    nir.nir_scatter_add(A, dtype, torch.tensor(yl, device=DEV), yg)
    ref = np.zeros(ng, npdt)
    np.add.at(ref, l2g, yl)
    assert np.array_equal(yg.cpu().numpy(), ref)

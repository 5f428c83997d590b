"""Mixed-precision solves whose last group of elements is short: the staged-factor groups (FP32, P = 2..4)
hold 7, 4 and 2 elements, and the gathered coefficients of a short group end before its threads do.
Judged by the residual formed through the public gather, apply and scatter-add, as in
test_gpu_cg_kernels."""
import pytest

torch = pytest.importorskip("torch")

from paper_2606_20917_amd import nir
from tests.test_gpu_cg_kernels import _public_residual
from tests.test_gpu_solver import DEV, _gpu_rhs, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,n", [(2, 4), (3, 3), (3, 5), (4, 3), (4, 5)])   # 64, 27, 125, 27, 125 elements
def test_short_last_group(P, n):
    pr = _problem(n, P)
    b = _gpu_rhs(pr)
    plan = nir.CGPlan(pr["b64"], pr["basis"], nir.geom(None, None, pr["helm"]), pr["helm32"], pr["A"], pr["lam"])
    x = torch.zeros(pr["ng"], dtype=torch.float64, device=DEV)
    _, info = nir.nir_cg_solve(plan, nir.CG_MIXED_F32, b, x, rtol=1e-10, maxit=20000)
    res = _public_residual(pr, b, x)
    assert res <= 1.5e-10 and abs(res - info.rel_residual) <= 1e-11, (res, info.rel_residual)

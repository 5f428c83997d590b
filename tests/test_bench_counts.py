"""Matrix-core FLOPs that bench.py prices affine batches with, counted here from the sizes of the operands."""
import pytest

from oracle import operators as op
from tests.test_bench_host import PRISM, PYR, TET, _bench


@pytest.mark.parametrize("P", [2, 3, 5, 8, 10])
def test_tetrahedra_are_priced_by_their_two_contractions(P):
    M = op.Tables(TET, P, P + 1).M
    G = sum(1 for i in range(P - 1) for j in range(P - 1 - i) for k in range(P - 1 - i - j))
    # X (1 x M) to three gradients (M x G each), back (3 G x M), and the mass matrix (M x M)
    assert _bench().matrix_core_flops(TET, P) == 2 * (3 * M * G + 3 * G * M + M * M)


@pytest.mark.parametrize("shape,P", [(PRISM, 2), (PRISM, 3), (PYR, 4), (PYR, 6)])
def test_prisms_and_pyramids_by_the_stacked_matrices(shape, P):
    M = op.Tables(shape, P, P + 1).M
    assert _bench().matrix_core_flops(shape, P) == 2 * 7 * (-(-M // 4) * 4) * (-(-M // 16) * 16)

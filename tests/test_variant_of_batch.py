"""The variant query of a batch against the rules that nir.h states: what per-element factors, the element
count, an explicit choice and the 256 modes of the dense tables make of the selection."""
import pytest

from paper_2606_20917_amd import nir

F64, F32 = nir.F64, nir.F32
EO, EOS, D, PC, G = (nir.VARIANT_PENCIL_EO, nir.VARIANT_PENCIL_EO_SPLIT, nir.VARIANT_DENSE, nir.VARIANT_PENCIL,
                     nir.VARIANT_GENERIC)


def _of(shape, P, ne, dtype, deformed, **kw):
    return nir.nir_get_helmholtz_variant_of(nir.batch(shape, P, ne, dtype, deformed, **kw))


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("P", range(2, 11))
def test_built_in_choices(P, dtype):
    for ne in (1, 1000, 100000):
        assert _of(nir.HEX, P, ne, dtype, 1) == nir.nir_get_helmholtz_variant(nir.HEX, P, dtype)
        assert _of(nir.HEX, P, ne, dtype, 0) == (EOS if P == 6 and dtype == F64 else EO)
        for shape in (nir.PRISM, nir.TET, nir.PYR):
            assert _of(shape, P, ne, dtype, 1) == PC
        assert _of(nir.PRISM, P, ne, dtype, 0) == (D if P <= 3 else PC)
    assert _of(nir.TET, P, 100000, dtype, 0) == D
    assert _of(nir.TET, P, 1000, dtype, 0) == (PC if P >= (8 if dtype == F32 else 7) else D)
    assert _of(nir.PYR, P, 100000, dtype, 0) == (D if P <= 6 else PC)
    assert _of(nir.PYR, P, 1000, dtype, 0) == (D if P <= 4 else PC)


def test_explicit_choices():
    try:
        for shape, P, want in ((nir.TET, 8, D), (nir.PYR, 8, D), (nir.PYR, 9, PC), (nir.PRISM, 4, D)):   # 285 modes at P = 9
            nir.nir_set_helmholtz_variant(shape, P, F64, D)
            assert _of(shape, P, 1, F64, 0) == want and _of(shape, P, 1, F64, 1) == PC
        nir.nir_set_helmholtz_variant(nir.TET, 8, F64, G)
        assert _of(nir.TET, 8, 1, F64, 0) == G == _of(nir.TET, 8, 1, F64, 1)
    finally:
        for shape, P in ((nir.TET, 8), (nir.PYR, 8), (nir.PYR, 9), (nir.PRISM, 4)):
            nir.nir_set_helmholtz_variant(shape, P, F64, nir.VARIANT_AUTO)


def test_invalid_batches():
    assert _of(nir.HEX, 11, 1, F64, 1) == -1
    assert _of(nir.HEX, 4, 1, F64, 1, Q=6) == -1
    assert _of(nir.HEX, 4, -1, F64, 1) == -1
    assert _of(nir.HEX, 4, 1, F64, 2) == -1
    assert _of(nir.HEX, 4, 1, F32, 1, math=nir.MATH_F16SPLIT) == -1
    assert nir.lib().nir_get_helmholtz_variant_of(None) == -1

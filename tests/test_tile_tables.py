"""The shapes of the tile tests reach every tile that the products' rules can
choose (no GPU: the rules are read from the sources)."""
import pytest

import tile_tables as tt


@pytest.mark.parametrize("function", ["gauss_f64", "real_f64", "cheb_f32_cplx", "cheb_f32_real"])
def test_every_tile_of_a_table_has_a_shape(function):
    t = tt.table(function)
    assert {tt.choose(t, n, k) for n, k in tt.SHAPES} == {e[:2] for e in t}
    # one tile runs with more waves while there is at most one of it per compute unit
    double = {"gauss_f64": (48, 32), "real_f64": (64, 64)}.get(function)
    if double:
        assert {tt.tiles(n, k, *double) <= tt.NCU for n, k in tt.SHAPES
                if tt.choose(t, n, k) == double} == {True, False}


@pytest.mark.parametrize("planes", [42, 14])
def test_every_int8_width_has_a_shape(planes):
    t = tt.int8_widths()
    assert {tt.int8_width(t, n, k, planes) for n, k in tt.INT8_SHAPES} == {e[0] for e in t}

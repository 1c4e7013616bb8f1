"""Units of the passes beside the look-ups of a fast search: sized as if up to as many tiles again were theirs."""
import pytest

from test_gpu_fast_pruned import P  # noqa: F401  (the module's fixture)
from test_gpu_routes import searched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,bits,n,units", [
    ([(470, 6256), (8056, 104)], 7, 985, 4028), ([(8056, 104)], 7, 985, 8056),        # 8526 tiles: two to a unit; 8056: one
    ([(470, 6256), (7721, 104)], 7, 985, 7721), ([(471, 6256), (7721, 104)], 7, 985, 3861),        # 8191 and 8192
    ([(20000, 300), (3000, 17)], 4, 100, 3000), ([(20000, 300), (4096, 104)], 4, 100, 2048)])       # no more than as many again
def test_units(P, shapes, bits, n, units):  # noqa: F811
    assert searched(P, shapes, bits, n, fast=True).endswith("k_search")
    assert P.last_search_shape()["units"] == units

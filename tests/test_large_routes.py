"""Which kernel, shape and order large layouts get, without a GPU (tests/host_route_driver.cpp)."""

import os

import pytest

from test_host_abi import _route_answers

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "large_routes.txt")


@pytest.mark.parametrize("layout", ["long", "short", "ordinary11", "ordinary20"])
def test_routes_of_large_layouts(tmp_path, layout):
    """Steps, mixing, mixing with the error and accumulation of 4 to 96 rows of 2 to 7 sources, both types, over one long segment or
    segments of 1100 elements that stream (1.2e8 elements of all rows), and one that does not (1.1e7, 2e7): the tile's
    wavefronts x vectors and tiles to a die's block, or the order of the rows.  The reasons stand at the rules in dadam_host.cpp."""
    want = dict(line.split(" | ", 1)[1].rstrip("\n").split(": ", 1) for line in open(GOLDEN) if line.startswith(layout + " | "))
    assert len(want) == 34
    got = _route_answers(tmp_path, layout)
    assert got == want, {k: (got.get(k), want.get(k)) for k in want if got.get(k) != want.get(k)}

"""Injection at the border of its two kernels: 24 particles per node.

Bars: as in test_gpu_inject, whose check this is.
"""
import pytest

from test_gpu_inject import test_injection_matches_its_definition as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells,per_node,fp", [
    (2, 24, 32), (2, 24, 64), (255, 24, 32), (600, 24, 64), (4096, 24, 32), (8191, 24, 32), (8192, 24, 64),
    (16384, 24, 32),
])
@pytest.mark.parametrize("past", [-1, 0, 1])
def test_injection_around_the_border(cells, per_node, fp, past):
    check(cells, per_node * (cells + 1) + past, fp)

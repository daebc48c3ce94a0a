"""Node sums in rows at the border of their rule's gap count (eight): as in test_gpu_rows,
whose check this is."""
import pytest

from test_gpu_rows import test_rows_change_nothing as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells,gaps", [(300, 8), (2559, 8), (300, 9)])
def test_rows_of_several_gaps_change_nothing(cells, gaps):
    check(cells, gaps, {})

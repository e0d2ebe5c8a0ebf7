"""The number of stencil launches that bench.py expects of a plan run in the row form, against
launches counted by hand: one a step and chunk width, problems leaving as their degree ends."""
import pytest

import bench


@pytest.mark.parametrize("rows,deg,nbytes,cplx,want", [
    ([48] * 8, [20] * 8, 8, True, 20),               # one width
    ([24, 17, 40], [6, 5, 3], 8, False, 6 + 5),      # 16-byte and one-value chunks
    ([24, 17, 17], [3, 6, 4], 8, False, 3 + 6),
    ([40, 42, 43], [5, 4, 3], 4, False, 5 + 4 + 3),  # four, two and one floats
    ([33, 45], [4, 4], 8, True, 4),                  # a complex double is a whole chunk
    ([32, 33], [4, 2], 4, True, 4 + 2)])
def test_plan_launches(rows, deg, nbytes, cplx, want):
    assert bench.plan_launches(rows, deg, nbytes, cplx) == want

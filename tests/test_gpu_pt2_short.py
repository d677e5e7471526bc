"""The correction from the accumulator for short vectors, whose few sums a row queue in LDS, with one, some and most
slots of a row in use, and rows cut in stretches (few long rows): the check of the longer ones."""
import pytest

from test_gpu_pt2_dense import test_dense_form as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,nnz", [(18, 2, 5, 1), (18, 2, 5, 30), (18, 2, 5, 2000), (20, 1, 4, 3), (12, 6, 6, 2),
                                         (12, 6, 6, 200), (16, 1, 6, 5), (9, 4, 4, 3)])
def test_short(n, na, nb, nnz):
    check(n, na, nb, nnz)

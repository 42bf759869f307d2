"""Adjoint products on parts tiles that read the output's cotangent and the other
operand where they lie: rows and sums at random address bits (lowest bit of either
kind), 128 and 64 columns, both operand roles. The check and its bound are those of
the few-column products."""
import pytest

from tests import test_gpu_rowsum as rowsum
from tests.test_gpu_rowsum import torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k,n,sl", [(8, 7, 8, 7), (7, 8, 4, 7), (4, 8, 7, 7), (9, 6, 7, 8), (7, 7, 9, 7), (10, 5, 10, 5)])
def test_adjoint_parts_in_place(torch, m, k, n, sl):  # noqa: F811
    rowsum.test_adjoint_products_in_place(torch, m, k, n, sl)

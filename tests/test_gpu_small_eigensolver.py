"""Environments of at most 128 rows, diagonalised whole (Householder reduction
with one or two columns per lane, divide and conquer, back-transform of the
rows kept), against the oracle's projector at the sizes where the kernels'
layouts change: the smallest, one below, at and above 64 rows, and at 128.

Tolerances as for the larger environments (tests/test_gpu_projector.py): a
backward-stable solver's errors are a few n u (n u = 1.4e-14 at n = 128), two
orders below them.
"""

import numpy as np
import pytest

from tests.inputs import graded_gram, orthogonal_with_spectrum
from tests.test_gpu_projector import _check, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [(3, 1), (4, 4), (5, 2), (16, 16), (17, 8), (63, 9), (64, 8), (64, 64), (65, 8),
         (100, 40), (127, 10), (128, 11), (128, 128)]


@pytest.mark.parametrize("n, d_new", SIZES)
def test_graded(torch_cuda, n, d_new):  # noqa: F811
    from paper_2306_00358_amd import Context

    with Context(0) as ctx:
        _check(torch_cuda, ctx, graded_gram(n, n, 8.0, 100 + n), d_new, spec_len=n,
               label="graded", iterative=False)


@pytest.mark.parametrize("n, d_new", [(16, 4), (64, 8), (65, 20), (128, 12)])
def test_diagonal_and_multiplets(torch_cuda, n, d_new):  # noqa: F811
    from paper_2306_00358_amd import Context

    vals = 10.0 ** (-np.arange(n) / 12.0)
    with Context(0) as ctx:
        # nothing to reduce: every reflector is the identity
        _check(torch_cuda, ctx, np.diag(vals[::-1]).copy(), d_new, spec_len=n, label="diagonal",
               iterative=False)
        # equal groups of four: the tridiagonal splits, equal poles deflate
        vals = np.repeat(vals[: n // 4 + 1], 4)[:n]
        _check(torch_cuda, ctx, orthogonal_with_spectrum(vals, 300 + n), d_new, spec_len=n,
               label="multiplets", iterative=False)

"""Environments of at most 128 rows, diagonalised whole (Householder reduction
with one or two columns per lane, divide and conquer from leaves of at most 8
rows, back-transform of the rows kept), against the oracle's projector at the
sizes where the kernels' layouts change: the smallest, one below, at and above
8 and 64 rows, and at 128; spectra with equal groups rotate and deflate.

Tolerances as for the larger environments (tests/test_gpu_projector.py): a
backward-stable solver's errors are a few n u (n u = 1.4e-14 at n = 128), two
orders below them.
"""

import numpy as np
import pytest

from tests.inputs import graded_gram, orthogonal_with_spectrum
from tests.test_gpu_projector import _check, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [(3, 1), (4, 4), (5, 2), (7, 3), (8, 8), (9, 4), (16, 16), (17, 8), (33, 5), (63, 9),
         (64, 8), (64, 64), (65, 8), (100, 40), (127, 10), (128, 11), (128, 128)]


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


@pytest.mark.parametrize("n", [8, 40, 64, 128])
def test_one_eigenvalue_and_two(torch_cuda, n):  # noqa: F811
    from paper_2306_00358_amd import Context

    with Context(0) as ctx:
        # all poles of every merge equal
        _check(torch_cuda, ctx, 0.5 * np.eye(n), n, spec_len=n, label="identity", iterative=False)
        # two groups of n / 2 equal eigenvalues, in a random basis: long chains
        # of rotations, one pole per group left
        vals = np.repeat([1.0, 0.25], n // 2)
        _check(torch_cuda, ctx, orthogonal_with_spectrum(vals, 500 + n), n // 2, spec_len=n,
               label="two groups", iterative=False)


def _tridiagonals(n):
    rng = np.random.default_rng(n)
    yield "random", rng.standard_normal(n), rng.standard_normal(n - 1)
    yield "graded", 10.0 ** (-8.0 * np.arange(n) / n), 10.0 ** (-8.0 * (np.arange(n - 1) + 0.5) / n)
    yield "wilkinson", np.abs(np.arange(n) - (n - 1) / 2.0), np.ones(n - 1)
    yield "split", rng.standard_normal(n), rng.standard_normal(n - 1) * (np.arange(n - 1) % 3 > 0)
    yield "clustered", np.round(rng.standard_normal(n)), 1e-3 * rng.standard_normal(n - 1)
    yield "zero diagonal", np.zeros(n), np.ones(n - 1)


@pytest.mark.parametrize("n", [3, 8, 9, 17, 33, 64, 65, 128])
def test_tridiagonals(torch_cuda, n):  # noqa: F811
    # matrices that are tridiagonal from the start, made positive by a shift: the
    # spectra the divide and conquer finds hard (1e-12: the other tests' bound)
    from paper_2306_00358_amd import Context, hotrg_projector

    with Context(0) as ctx:
        for label, d, e in _tridiagonals(n):
            print(label, n, flush=True)
            T = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
            T += np.eye(n) * (np.abs(d).max() + 2.0 * np.abs(e).max() + 1.0)
            U = torch_cuda.empty((n, n), dtype=torch_cuda.float64, device="cuda")
            kept, err, spec = hotrg_projector(ctx, torch_cuda.from_numpy(T).to("cuda"), U, n,
                                              spec_len=n)
            s, u = np.linalg.eigvalsh(T)[::-1], U.cpu().numpy()
            assert np.abs(np.array(spec) - s / s[0]).max() <= 1e-12
            assert np.abs(u.T @ u - np.eye(n)).max() <= 1e-12
            assert np.abs(T @ u - u * s).max() <= 1e-12 * s[0]


@pytest.mark.parametrize("n", [4, 8, 16, 64, 65, 128])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_not_finite_is_an_error(torch_cuda, n, value):  # noqa: F811
    from paper_2306_00358_amd import Context, HotrgError, hotrg_projector

    M = graded_gram(n, n, 8.0, 100 + n)
    M[n // 2, n - 1] = M[n - 1, n // 2] = value
    U = torch_cuda.empty((n, 2), dtype=torch_cuda.float64, device="cuda")
    with Context(0) as ctx:
        print("not finite", n, value, flush=True)
        with pytest.raises(HotrgError) as e:
            hotrg_projector(ctx, torch_cuda.from_numpy(M).to("cuda"), U, 2, spec_len=2)
        assert e.value.status == 4  # HOTRG_ERR_NUMERIC
        # the context is as good as before
        M = graded_gram(n, n, 8.0, 100 + n)
        hotrg_projector(ctx, torch_cuda.from_numpy(M).to("cuda"), U, 2, spec_len=2)

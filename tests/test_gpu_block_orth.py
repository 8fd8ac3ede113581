"""The block eigensolver's orthonormalisation at each block size p (a multiple of
16: 32 to 128, with and without a second wave of columns, 4 and 8 waves) through
hotrg_projector, in buffers that a larger block left full, and a matrix whose
Gram pivots fail (rank far below the block: the dense solver takes over).

The projector's columns are orthonormal and the spectrum is right to 1e-12 of
the leading value, the bounds of the other projector tests."""

import numpy as np
import pytest

from oracle import hotrg
from tests.inputs import graded_gram

pytestmark = pytest.mark.gpu


# d_new -> p = max(2 d_new, d_new + 17) rounded up to 16
@pytest.mark.parametrize("order", [[64, 56, 48, 40, 33, 32, 20, 14, 4]])
def test_block_sizes(order):
    import torch

    from paper_2306_00358_amd import Context, hotrg_projector

    with Context(0) as ctx:
        for d in order:
            for n in (320, 577):
                print("block for", d, "of", n, flush=True)
                M = graded_gram(n, n, 8.0, seed=d + n)
                U = torch.empty((n, d), dtype=torch.float64, device="cuda")
                kept, err, spec = hotrg_projector(ctx, torch.from_numpy(M).to("cuda"), U, d,
                                                  spec_len=d + 1)
                assert ctx.last_eig()[0] > 0  # the block solver converged
                _, s, _, want = hotrg.projector(M, d, "plain", 1e-10)
                u = U.cpu().numpy()
                assert kept == want
                assert np.abs(u.T @ u - np.eye(d)).max() <= 1e-12
                assert np.abs(np.array(spec) - s[:d + 1] / s[0]).max() <= 1e-12


def test_rank_below_the_block():
    import torch

    from paper_2306_00358_amd import Context, hotrg_projector

    n, d, r = 400, 32, 5
    X = np.random.default_rng(3).standard_normal((n, r))
    M = X @ X.T
    U = torch.empty((n, d), dtype=torch.float64, device="cuda")
    with Context(0) as ctx:
        print("rank", r, flush=True)
        kept, err, spec = hotrg_projector(ctx, torch.from_numpy(M).to("cuda"), U, d, spec_len=d)
    u, s = U.cpu().numpy(), np.linalg.eigvalsh(M)[::-1]
    assert np.abs(u[:, :r].T @ u[:, :r] - np.eye(r)).max() <= 1e-12
    assert np.abs(np.array(spec) - s[:d] / s[0]).max() <= 1e-12
    assert np.abs(u[:, :kept] @ (u[:, :kept].T @ M) - M).max() <= 1e-11 * np.abs(M).max()


@pytest.mark.parametrize("cuts", [[13], [13, 15, 21], [13, 16, 24], [16, 20]])
def test_lockstep_odd_environments(cuts):
    # odd D: rows of odd length, copied into LDS 4 bytes a lane, alone and beside
    # even ones (16 bytes a lane; each product of the table takes its own)
    import torch  # noqa: F401  (one HIP runtime for the process)

    from paper_2306_00358_amd import Context, hotrg_run, hotrg_run_grouped, make_opts, model_params

    P = [model_params("ising", beta=0.42 + 0.01 * i) for i in range(len(cuts))]
    O = [make_opts(d, 12) for d in cuts]
    print("lockstep", cuts, flush=True)
    with Context(0) as ctx:
        got, statuses = hotrg_run_grouped(ctx, P, O)
        assert statuses == [0] * len(cuts)
        for p, o, g in zip(P, O, got):
            want = hotrg_run(ctx, p, o)["lnz_per_site"]
            assert abs(g["lnz_per_site"] - want) <= 1e-12 * abs(want)


@pytest.mark.parametrize("ratio, scale", [(5e7, 1.0), (2e8, 1.0), (5e7, 2.0**-260), (5e7, 2.0**260),
                                          (2e8, 2.0**260)])
def test_two_products_per_orthonormalisation(ratio, scale):
    # one eigenvalue `ratio` times the 64th, the others a slow decay (2 over the 31
    # vectors of the block past the needed ones): several sweeps after the first
    # check, paired below a ratio of 1e8 where the fourth powers of the eigenvalues
    # are in range, and not else; the block solver converges in each case
    import torch

    from paper_2306_00358_amd import Context, hotrg_projector
    from tests.inputs import orthogonal_with_spectrum

    n, d = 640, 32
    i = np.arange(n)
    vals = np.where(i < 64, 2.0 ** ((63 - i) / 31.0), 10.0 ** (-(i - 63) / 200.0)) / ratio
    vals[0] = 1.0
    M = scale * orthogonal_with_spectrum(vals, 7)
    U = torch.empty((n, d), dtype=torch.float64, device="cuda")
    with Context(0) as ctx:
        print("ratio", ratio, "scale", scale, flush=True)
        kept, err, spec = hotrg_projector(ctx, torch.from_numpy(M).to("cuda"), U, d, spec_len=d + 1)
        sweeps = ctx.last_eig()[0]
        print("sweeps", sweeps, flush=True)
    assert sweeps >= 3 + 4
    u = U.cpu().numpy()
    assert np.abs(np.array(spec) - vals[:d + 1]).max() <= 1e-12
    assert np.abs(u.T @ u - np.eye(d)).max() <= 1e-12
    assert np.linalg.norm(M @ u - u * (scale * vals[:d]), axis=0).max() <= 1e-12 * scale


@pytest.mark.parametrize("n, d", [(256, 4), (625, 14), (641, 14), (1025, 32), (2048, 14), (2064, 14),
                                  (2048, 64), (2064, 64), (3498, 64), (3500, 64), (4097, 64),
                                  (4225, 64), (4240, 20), (5184, 48), (5472, 48)])
def test_block_product_by_tiles_and_by_chunks(n, d):
    # either side of the lines between the two ways of V M: even and odd rows, a
    # tile a compute unit, and past the small tiles' 2^19 outputs; M of rank 256
    # with known eigenpairs (formed to 256 u, two orders below the bounds)
    import torch

    from paper_2306_00358_amd import Context, hotrg_projector

    r = min(n, 256)
    Q = np.linalg.qr(np.random.default_rng(n + d).standard_normal((n, r)))[0]
    vals = 10.0 ** (-8.0 * np.arange(r) / r)
    M = (Q * vals) @ Q.T
    U = torch.empty((n, d), dtype=torch.float64, device="cuda")
    with Context(0) as ctx:
        print("block product", n, d, flush=True)
        kept, err, spec = hotrg_projector(ctx, torch.from_numpy(M).to("cuda"), U, d, spec_len=d + 1)
        assert ctx.last_eig()[0] > 0
    u = U.cpu().numpy()
    assert kept == d
    assert np.abs(np.array(spec) - vals[:d + 1]).max() <= 1e-12
    assert np.abs(u.T @ u - np.eye(d)).max() <= 1e-12
    assert np.linalg.norm(M @ u - u * vals[:d], axis=0).max() <= 1e-12

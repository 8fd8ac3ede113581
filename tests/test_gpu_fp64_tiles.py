"""The FP64 contraction kernels at the edges of their tiles, against the oracle:
the 64 x 64, 128 x 128 and 64 x 32 LDS tiles forced one at a time, and the environment's
symmetric products (64 x 64 tiles, both halves in one launch) around multiples
of the tile.  Element-wise within 1e-12 of the largest element, the bound of the
other FP64 parity tests (a sum of K products of magnitude at most s has an error
of at most K u s: 3e-13 s at the largest K here, 2500)."""

import os
import subprocess
import sys

import numpy as np
import pytest

from oracle import hotrg
from tests.inputs import random_tensor

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("variant", ["6", "7", "8"])
def test_forced_lds_tile(variant):
    print("forced", variant, flush=True)
    env = dict(os.environ, HOTRG_GEMM_VARIANT=variant)
    r = subprocess.run([sys.executable, "-m", "tests.variant_child", "fp64"], cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=600)
    print(r.stdout, r.stderr[-2000:], flush=True)
    assert r.returncode == 0, r.stderr[-2000:]


# P = dx dy: the smallest of the symmetric launch (400), one tile more or less
# than a multiple of 64, and legs that differ
@pytest.mark.parametrize("dx, dy", [(20, 20), (25, 16), (16, 28), (24, 24), (36, 16), (13, 48),
                                    (32, 32), (33, 32)])
def test_environment(dx, dy):
    import torch

    from paper_2306_00358_amd import Context, hotrg_environment

    print("environment", dx, dy, flush=True)
    T = random_tensor(dx, dy, seed=40 + dx + dy)
    M = torch.full((dx * dx, dx * dx), float("nan"), dtype=torch.float64, device="cuda")
    with Context(0) as ctx:
        hotrg_environment(ctx, torch.from_numpy(T).to("cuda"), M)
    want = hotrg.environment(T)
    assert np.abs(M.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()


# the small tiles (K split over the waves of a workgroup): one slab and less,
# remainders past a slab, odd strides, more slabs than waves, both tile sizes
@pytest.mark.parametrize("dx, dy, dn", [(2, 2, 2), (3, 2, 9), (4, 4, 7), (5, 5, 5), (8, 8, 8),
                                        (7, 11, 13), (16, 16, 16), (9, 17, 20), (21, 21, 21),
                                        (23, 23, 23), (1, 2, 1), (2, 22, 3), (3, 26, 5),
                                        (18, 9, 11), (18, 18, 18), (22, 22, 5)])
def test_coarse_and_environment_small(dx, dy, dn):
    import torch

    from paper_2306_00358_amd import Context, hotrg_coarse, hotrg_environment
    from tests.inputs import random_projector

    print("small", dx, dy, dn, flush=True)
    T, U = random_tensor(dx, dy, seed=70 + dx), random_projector(dx, dn, seed=90 + dn)
    Tg, Ug = torch.from_numpy(T).to("cuda"), torch.from_numpy(U).to("cuda")
    M = torch.full((dx * dx, dx * dx), float("nan"), dtype=torch.float64, device="cuda")
    Tt = torch.full((dn, dy, dn, dy), float("nan"), dtype=torch.float64, device="cuda")
    mx = torch.zeros(1, dtype=torch.float64, device="cuda")
    with Context(0) as ctx:
        hotrg_environment(ctx, Tg, M)
        hotrg_coarse(ctx, Tg, Ug, Tt, mx)
    for got, want in ((M, hotrg.environment(T)), (Tt, hotrg.coarse_tensor(T, U))):
        assert np.abs(got.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    assert mx.item() == Tt.abs().max().item()


# contracted indices of 128 and more not a multiple of 16: rows padded with
# zeros, odd and even strides, in buffers that the shape before left full
RAGGED = [(27, 31, 29), (12, 11, 13), (11, 12, 7), (15, 17, 16), (13, 13, 13), (41, 40, 9),
          (12, 12, 12), (3, 43, 9), (20, 33, 20)]


@pytest.mark.parametrize("prec, tol", [("fp64", 1e-12), ("fp32", 2e-5), ("bf16x3", 2e-4)])
def test_ragged_sizes(prec, tol):
    # (FP32: K <= 1681 products of 2^-24 each way, 1e-4 at worst and about 1e-6
    # in practice; split BF16 drops products below 2^-16 of the largest.  Both
    # far below an element lost or doubled by wrong padding.)
    import torch

    from paper_2306_00358_amd import Context, hotrg_coarse, hotrg_environment
    from tests.inputs import random_projector

    with Context(0) as ctx:
        for dx, dy, dn in RAGGED:
            print("ragged", prec, dx, dy, dn, flush=True)
            T, U = random_tensor(dx, dy, seed=dx + 3 * dy), random_projector(dx, dn, seed=dn)
            Tg, Ug = torch.from_numpy(T).to("cuda"), torch.from_numpy(U).to("cuda")
            M = torch.full((dx * dx, dx * dx), float("nan"), dtype=torch.float64, device="cuda")
            Tt = torch.full((dn, dy, dn, dy), float("nan"), dtype=torch.float64, device="cuda")
            hotrg_environment(ctx, Tg, M, prec=prec)
            hotrg_coarse(ctx, Tg, Ug, Tt, prec=prec)
            for got, want in ((M, hotrg.environment(T)), (Tt, hotrg.coarse_tensor(T, U))):
                assert np.abs(got.cpu().numpy() - want).max() <= tol * np.abs(want).max()


def test_more_tiles_than_a_grid_row():
    # one leg of 1 beside one of 23184: the operand layouts are over 2^24 tiles of 256
    # threads, more than one grid dimension holds.  T = a b^T, so that M = |a|^2 |b|^2
    # (a . b)^2; 2^29 terms summed in 32 chains: 2^24 2^-53 at most
    import torch

    from paper_2306_00358_amd import Context, hotrg_environment

    dy = 23184
    g = torch.Generator(device="cuda").manual_seed(3)
    a, b = (torch.rand(dy, dtype=torch.float64, device="cuda", generator=g) + 0.5 for _ in range(2))
    T = (a[:, None] * b).reshape(1, dy, 1, dy)
    M = torch.zeros((1, 1), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    print("long leg", dy, flush=True)
    with Context(0) as ctx:
        hotrg_environment(ctx, T, M)
    want = float((a @ a) * (b @ b) * (a @ b) ** 2)
    assert abs(float(M[0, 0]) - want) <= 2.0 ** -29 * want

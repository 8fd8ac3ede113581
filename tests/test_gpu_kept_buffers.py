"""Whole runs and single operations that share one context, which keeps the last
one's operand buffers: other sizes and precisions in between change nothing, a
context with a budget keeps nothing, and inputs off 16-byte alignment or
overwritten by the result are read as before.  Bounds: those of the other
parity tests (FP64 1e-12; a run's value is the same within rounding)."""

import numpy as np
import pytest

from oracle import hotrg
from tests.inputs import random_projector, random_tensor

pytestmark = pytest.mark.gpu


def _close(got, want, tol=1e-12):
    assert np.abs(got.cpu().numpy() - want).max() <= tol * np.abs(want).max()


def test_one_context_many_operations():
    import torch

    from paper_2306_00358_amd import (Context, hotrg_coarse, hotrg_environment, hotrg_run,
                                      make_opts, model_params)

    p = model_params("ising", beta=0.43)
    o = [make_opts(16, 10, spec_len=4), make_opts(13, 8, prec="fp32"), make_opts(8, 12)]
    alone = []
    for q in o:
        with Context(0) as ctx:
            alone.append(hotrg_run(ctx, p, q)["lnz_per_site"])
    with Context(0) as ctx, Context(0, hbm_budget=1 << 30) as tight:
        for c in (ctx, tight):
            for turn in range(2):
                for q, want, (dx, dy, dn) in zip(o, alone, [(5, 4, 7), (15, 17, 16), (16, 16, 9)]):
                    print("kept", turn, dx, dy, dn, flush=True)
                    assert abs(hotrg_run(c, p, q)["lnz_per_site"] - want) <= 1e-12 * abs(want)
                    T, U = random_tensor(dx, dy, seed=dx), random_projector(dx, dn, seed=dn)
                    Tg, Ug = torch.from_numpy(T).to("cuda"), torch.from_numpy(U).to("cuda")
                    M = torch.empty((dx * dx, dx * dx), dtype=torch.float64, device="cuda")
                    Tt = torch.empty((dn, dy, dn, dy), dtype=torch.float64, device="cuda")
                    hotrg_environment(c, Tg, M)
                    hotrg_coarse(c, Tg, Ug, Tt)
                    _close(M, hotrg.environment(T))
                    _close(Tt, hotrg.coarse_tensor(T, U))
                if turn == 0:
                    held = c.bytes_in_use()
            assert c.bytes_in_use() == held
        assert tight.bytes_in_use() < ctx.bytes_in_use()


@pytest.mark.parametrize("D", [5, 16])
def test_unaligned_and_overwritten_inputs(D):
    import torch

    from paper_2306_00358_amd import Context, hotrg_coarse, hotrg_environment

    T, U = random_tensor(D, D, seed=D), random_projector(D, D, seed=D + 1)
    n = D ** 4
    with Context(0) as ctx:
        for off in (0, 1):
            print("unaligned", D, off, flush=True)
            buf = torch.zeros(n + 2, dtype=torch.float64, device="cuda")
            Tg = buf[off:off + n].view(D, D, D, D)
            Ug = torch.from_numpy(U).to("cuda")
            Tg.copy_(torch.from_numpy(T))
            hotrg_coarse(ctx, Tg, Ug, Tg)
            _close(Tg, hotrg.coarse_tensor(T, U))
            Tg.copy_(torch.from_numpy(T))
            hotrg_environment(ctx, Tg, Tg.view(D * D, D * D))
            _close(Tg.view(D * D, D * D), hotrg.environment(T))


def test_large_operands_are_given_back():
    # FP32 operands of D = 88: five arrays of 240 MB, over the 1 GiB that a context
    # keeps; the two environment halves (workspace) stay
    import torch

    from paper_2306_00358_amd import Context, hotrg_environment

    D = 88
    T = torch.ones((D, D, D, D), dtype=torch.float64, device="cuda")
    M = torch.empty((D * D, D * D), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    with Context(0) as ctx:
        for _ in range(2):
            print("given back", D, flush=True)
            hotrg_environment(ctx, T, M, prec="fp32")
            assert ctx.bytes_in_use() <= 2 * 4 * D**4 + (1 << 20)
        # D^2 equal terms in FP32: D^2 2^-24
        assert float((M / float(D) ** 6 - 1.0).abs().max()) <= D * D * 2.0 ** -24

"""The admission footprint: no more than the unpadded buffers of a problem and
the solver margin, also where the initial legs are larger than D_cut (raw
tensors, long character expansions), so that what fitted a budget without
padded operands still does; and a pool with no more than that budget runs
ragged problems, to the same value."""

import numpy as np
import pytest

from tests.inputs import random_tensor


def _unpadded(d0, d_cut, steps):
    # 8 bytes times the largest of each kind of buffer over the steps (FP64, one side)
    peak = {"state": 3 * d0**4}

    def need(name, count):
        peak[name] = max(peak.get(name, 0), count)

    dx = dy = d0
    for _ in range(steps):
        n, P, dn = dx * dx, dx * dy, min(d_cut, dx * dx)
        p = (min(128, max(2 * dn, dn + 17)) + 15) // 16 * 16
        need("M", n * n)
        need("WE", 2 * n)
        need("U", 3 * n * dn)
        # vectors, Ritz vectors, at most 16 partial products, small matrices
        need("eig", (5 + 16) * p * n + 4 * p * p + 4 * p + 16)
        need("dense", n * n if n > 128 else 0)
        need("A12", 2 * P * P)
        need("X12", 2 * dn * P * P)
        need("Tt", (dn * dy) ** 2)
        need("state", 6 * (dy * dn) ** 2)  # operands before and after
        dx, dy = dy, dn
    return 8 * sum(peak.values()) + (256 << 20)


@pytest.mark.parametrize("d0, d_cut, steps", [(64, 8, 1), (64, 16, 10), (41, 16, 10), (31, 12, 8),
                                              (45, 45, 3), (2, 50, 20), (3, 45, 20), (7, 23, 12)])
def test_no_more_than_unpadded_buffers(d0, d_cut, steps):
    from paper_2306_00358_amd import hotrg_footprint, make_opts, model_params

    raw = np.ones((d0, d0, d0, d0))
    fp = hotrg_footprint(model_params("raw", raw=raw), make_opts(d_cut, steps))
    assert fp <= _unpadded(d0, d_cut, steps)


@pytest.mark.gpu
@pytest.mark.parametrize("d0, d_cut, steps", [(41, 16, 4), (3, 23, 8)])
def test_pool_of_one_footprint(d0, d_cut, steps):
    import torch  # noqa: F401  (one HIP runtime for the process)

    from paper_2306_00358_amd import (Context, Ticket, hotrg_footprint, hotrg_run, make_opts,
                                      model_params)

    p = model_params("raw", raw=random_tensor(d0, d0, seed=d0, positive=True))
    o = make_opts(d_cut, steps)
    fp = hotrg_footprint(p, o)
    with Context(0) as ctx:
        want = hotrg_run(ctx, p, o)["lnz_per_site"]
    for budget in (fp, 2 * fp):  # unpadded rows, padded ones
        print("pool", d0, d_cut, budget, flush=True)
        with Context(0, hbm_budget=budget) as ctx:
            ctx.set_workers(2)
            for _ in range(2):
                got = Ticket(ctx, p, o).value()["lnz_per_site"]
                assert abs(got - want) <= 1e-12 * abs(want)
            assert ctx.sched_stats()["peak_reserved"] <= budget

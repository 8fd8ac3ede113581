"""Contexts whose memory budget is what a call's own buffers take: the small dense
eigensolver's vectors share the contractions' buffers, or, without room for
them, the solver that works in place takes over.  Bounds: those of the projector
and parity tests."""

import numpy as np
import pytest

from oracle import hotrg, tensors
from tests.inputs import graded_gram

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, d", [(9, 3), (64, 8), (128, 11), (128, 128)])
@pytest.mark.parametrize("room", [False, True])
def test_projector_in_place(n, d, room):
    import torch

    from paper_2306_00358_amd import Context, hotrg_projector

    M = graded_gram(n, n, 8.0, seed=n)
    U = torch.empty((n, d), dtype=torch.float64, device="cuda")
    # M, and 4 KB for eigenvalues, spectrum and scalars; with room M once more
    with Context(0, hbm_budget=n * n * 8 * (2 if room else 1) + 4096) as ctx:
        print("in place", n, d, room, flush=True)
        kept, err, spec = hotrg_projector(ctx, torch.from_numpy(M).to("cuda"), U, d, spec_len=d)
    _, s, _, want = hotrg.projector(M, d, "plain", 1e-10)
    u = U.cpu().numpy()
    assert kept == want
    assert np.abs(u.T @ u - np.eye(d)).max() <= 1e-12
    assert np.abs(np.array(spec) - s[:d] / s[0]).max() <= 1e-12


@pytest.mark.parametrize("iso, budget", [("one", 3434496), ("two", 3786752)])
def test_run_in_its_contractions_buffers(iso, budget):
    # D = 11: what the operands, the environments (one or two), the eigenvalues and
    # the intermediates take
    import torch  # noqa: F401  (one HIP runtime for the process)

    from paper_2306_00358_amd import Context, hotrg_run, make_opts, model_params

    print("run", iso, budget, flush=True)
    with Context(0, hbm_budget=budget) as ctx:
        got = hotrg_run(ctx, model_params("ising", beta=0.43), make_opts(11, 10, isometry=iso))
    want = hotrg.run(tensors.ising(0.43), 11, 10, isometry=iso)
    assert abs(got["lnz_per_site"] - want.lnz_per_site) <= 1e-12 * abs(want.lnz_per_site)

"""dk_spectral_bounds where the squarings of both sequences run 64 x 64 tiles (from 1409 rows
on) and, once one has converged, 32 x 32 ones, with a ragged last tile of either.  The
spectrum is given; tolerance as for the bounds elsewhere (1e-11)."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1407, 1441])
def test_bounds(n):
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context
    from workloads import custom_spec, make_problem
    ctx = Context(make_problem(custom_spec("bounds", 62, 6.0, 1, 13, 4, 2.0, basis="sc",
                                           noise=False), with_block=False))
    try:
        ctx.ensure_workspace(n, 16)
        rng = np.random.default_rng(n)
        lam = np.sort(rng.uniform(-3, 9, n))
        lam[0], lam[-1] = -3.5, 9.1  # of different gaps: one sequence ends first
        H = np.diag(lam)
        for _ in range(4):
            v = rng.standard_normal(n)
            v /= np.linalg.norm(v)
            H -= 2 * np.outer(v, v @ H)
            H -= 2 * np.outer(H @ v, v)
        H = torch.as_tensor(0.5 * (H + H.T), device="cuda").contiguous()
        print(f"bounds {n}", flush=True)
        lo, hi, steps = L.dk_spectral_bounds(ctx.h, H)
        assert abs(lo - lam[0]) < 1e-11 and abs(hi - lam[-1]) < 1e-11 and steps > 0
    finally:
        ctx.close()

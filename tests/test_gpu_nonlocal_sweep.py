"""H X and one filter pass where the nonlocal term's tables and tiles have edges:
grids that are no multiple of the 64-point blocks, odd leading dimensions,
blocks of 1, 17 and 130 columns, one group, the last group counts of the dense
runs (32 and 64 groups) and the first of the compact ones (65 and more live
groups in a block), a cell with points no projector reaches, and run counts on both sides
of the reduction's two widths (64 and fewer, 167, 216).  Oracle: the FP64 Hamiltonian; tolerances as for H X elsewhere (FP64 1e-12, FP32 blocks 2e-5)."""

import numpy as np
import pytest
import torch

from oracle.filter import chebyshev_filter
from oracle.hamiltonian import Hamiltonian
from workloads import custom_spec, make_problem

pytestmark = pytest.mark.gpu

# name, a0, reps, n, basis, columns
CASES = [("one", 6.0, 1, 13, "sc", 17),         # one atom, 2197 points
         ("apart", 24.0, 1, 24, "sc", 1),       # one atom in a large cell: dead blocks
         ("g27", 4.0, 3, 17, "sc", 130),
         ("g32", 5.0, 2, 14, "fcc", 33),        # the dense runs' last count in FP64
         ("g64", 3.5, 4, 15, "sc", 70),         # and in the mixed path
         ("r64", 5.0, 1, 16, "fcc", 5),         # runs of one block: 64 of them
         ("r167", 7.0, 1, 22, "fcc", 65),
         ("g108", 4.5, 3, 19, "fcc", 18)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name,a0,reps,n,basis,n_s", CASES)
def test_nonlocal_edges(name, a0, reps, n, basis, n_s, precision):
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context
    spec = custom_spec(name, 70 + reps, a0, reps, n, n_s, 2.0, basis=basis, noise=False)
    p = make_problem(spec, with_block=False)
    H = Hamiltonian(p)
    X = np.random.default_rng(31).standard_normal((p.n_grid, n_s))
    X = X.astype(np.float32).astype(np.float64)
    ctx = Context(p, precision)
    try:
        ctx.ensure_workspace(n_s, 16)
        # a leading dimension past the grid: columns start off every alignment
        ld = p.n_grid + 3
        buf = torch.zeros((n_s, ld), dtype=ctx.dtype, device=ctx.device)
        out = torch.full_like(buf, 7.0)
        buf[:, :p.n_grid] = torch.as_tensor(X.T.copy(), device=ctx.device).to(ctx.dtype)
        ws = torch.empty(L.dk_workspace_bytes(ctx.h, n_s, ld, 16) // 8 + 64, dtype=torch.float64,
                         device=ctx.device)
        L.dk_set_workspace(ctx.h, ws)
        print(f"H X {name} {precision}", flush=True)
        L.dk_apply_h(ctx.h, buf[:, :p.n_grid], out[:, :p.n_grid])
        got = out[:, :p.n_grid].double().cpu().numpy().T
        ref = H.apply(X)
        tol = 1e-12 if precision == "fp64" else 2e-5
        assert np.abs(got - ref).max() / np.abs(ref).max() < tol
        assert torch.all(out[:, p.n_grid:] == 7.0)
        print(f"filter {name} {precision}", flush=True)
        a, b, a0f = 4.0, ctx.upper, -2.0
        L.dk_filter(ctx.h, buf[:, :p.n_grid], 5, a, b, a0f)
        got = buf[:, :p.n_grid].double().cpu().numpy().T
        ref = chebyshev_filter(H, X, 5, a, b, a0f)
        assert np.abs(got - ref).max() / np.abs(ref).max() < tol
        assert torch.all(buf[:, p.n_grid:] == 0.0)
    finally:
        ctx.close()

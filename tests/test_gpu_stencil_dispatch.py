"""H X and filter steps (Y_{k+1} over Y_{k-1} in place) in every kernel of the local part that
blocks of a few columns do not reach: the row-rotation kernel (48 points a row in FP32,
workgroups that fill the chip) at planes that are no multiple of its waves, of fewer than
twelve rows and in z-chunks of unequal length; the whole-plane kernel (rows of 81 points and
more, planes of at most 4096) in both of its sizes; the slab kernel in FP32 and FP64; the
one-point form for short ragged rows in large blocks.  Leading dimensions of the grid, and
off every alignment, which sends FP32 rows to the general kernels.  Oracle: the FP64
Hamiltonian on some of the columns; tolerances as for H X elsewhere (FP64 1e-12, FP32 2e-5)."""

import numpy as np
import pytest
import torch

from oracle.filter import chebyshev_filter
from oracle.hamiltonian import Hamiltonian
from workloads import custom_spec, make_problem

pytestmark = pytest.mark.gpu

H0 = 0.32
CASES = [("mixed", (48, 48, 13), 500), ("mixed", (48, 47, 14), 512),   # row rotation
         ("mixed", (48, 9, 26), 256), ("mixed", (48, 7, 30), 250),
         ("mixed", (48, 41, 50), 128), ("mixed", (48, 34, 61), 103),
         ("mixed", (100, 25, 8), 1), ("mixed", (100, 25, 25), 37),     # whole plane
         ("mixed", (116, 20, 9), 3), ("mixed", (116, 20, 30), 5), ("mixed", (124, 33, 8), 2),
         ("mixed", (116, 40, 9), 3), ("mixed", (116, 62, 8), 2),       # slab
         ("mixed", (96, 52, 26), 4), ("fp64", (114, 12, 9), 3), ("fp64", (114, 14, 9), 3), ("fp64", (116, 30, 8), 2), ("fp64", (130, 50, 25), 2),
         ("mixed", (7, 30, 300), 64), ("fp64", (7, 30, 300), 64),      # short ragged rows
         ("mixed", (7, 100, 90), 80), ("fp64", (7, 100, 90), 80),
         ("mixed", (9, 43, 163), 70), ("fp64", (9, 60, 61), 123), ("mixed", (10, 47, 69), 129)]


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("precision,dims,n_s", CASES,
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_dispatch(precision, dims, n_s, pad):
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context
    lens = tuple(d * h for d, h in zip(dims, (H0, 1.1 * H0, 0.95 * H0)))
    spec = custom_spec("dispatch", 65, lens[0], 1, dims[0], 4, 1.0, basis="sc", dims=dims,
                       lens=lens, noise=False)
    p = make_problem(spec, positions=np.array([[0.3, 0.4, 0.2]]), with_block=False)
    H = Hamiltonian(p)
    ctx = Context(p, precision)
    try:
        ld = p.n_grid + pad
        gen = torch.Generator("cuda").manual_seed(n_s)
        buf = torch.full((n_s, ld), 7.0, dtype=ctx.dtype, device=ctx.device)
        buf[:, :p.n_grid] = torch.randn((n_s, p.n_grid), generator=gen, device="cuda")
        out = torch.full_like(buf, 7.0)
        some = sorted({0, n_s // 2, n_s - 1})
        X = buf[some, :p.n_grid].double().cpu().numpy().T
        ws = torch.empty(L.dk_workspace_bytes(ctx.h, n_s, ld, 16) // 8 + 64, dtype=torch.float64,
                         device=ctx.device)
        L.dk_set_workspace(ctx.h, ws)
        tol = 1e-12 if precision == "fp64" else 2e-5
        print(f"H X {dims} x {n_s} ld +{pad} {precision}", flush=True)
        L.dk_apply_h(ctx.h, buf[:, :p.n_grid], out[:, :p.n_grid])
        ref = H.apply(X)
        got = out[some, :p.n_grid].double().cpu().numpy().T
        assert np.abs(got - ref).max() / np.abs(ref).max() < tol
        assert torch.all(out[:, p.n_grid:] == 7.0)
        print(f"filter {dims} x {n_s} ld +{pad} {precision}", flush=True)
        a, b, a0 = 4.0, ctx.upper, -2.0
        L.dk_filter(ctx.h, buf[:, :p.n_grid], 5, a, b, a0)
        ref = chebyshev_filter(H, X, 5, a, b, a0)
        got = buf[some, :p.n_grid].double().cpu().numpy().T
        assert np.abs(got - ref).max() / np.abs(ref).max() < tol
        assert torch.all(buf[:, p.n_grid:] == 7.0)
    finally:
        ctx.close()

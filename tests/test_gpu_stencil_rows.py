"""H X where the local part's row kernel has edges: row lengths on both sides of its vectors
(four points in FP32, two in FP64), of its three LDS pitches (32, 33, 80, 81) and of its
last row length (112, 113), the smallest grid, slabs whose last one is shorter, planes of one slab,
z-chunks of unequal length, odd leading dimensions.  Oracle: the FP64 Hamiltonian;
tolerances as for H X elsewhere (FP64 1e-12, FP32 blocks 2e-5)."""

import numpy as np
import pytest
import torch

from oracle.hamiltonian import Hamiltonian
from workloads import custom_spec, make_problem

pytestmark = pytest.mark.gpu

H0 = 0.32
DIMS = [(7, 7, 7), (8, 9, 10), (9, 7, 25), (10, 30, 8), (11, 13, 17), (12, 25, 19),
        (31, 14, 9), (32, 40, 13), (33, 41, 12), (34, 26, 11), (48, 48, 14), (63, 50, 9),
        (80, 31, 8), (81, 16, 9), (96, 21, 8), (96, 52, 8), (112, 16, 9), (113, 14, 8)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
def test_rows(dims, precision):
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context
    lens = tuple(d * h for d, h in zip(dims, (H0, 1.1 * H0, 0.95 * H0)))
    spec = custom_spec("rows", 64, lens[0], 1, dims[0], 4, 1.0, basis="sc", dims=dims, lens=lens,
                       noise=False)
    p = make_problem(spec, positions=np.array([[0.3, 0.4, 0.2]]), with_block=False)
    H = Hamiltonian(p)
    for n_s in (1, 37):
        X = np.random.default_rng(n_s).standard_normal((p.n_grid, n_s))
        X = X.astype(np.float32).astype(np.float64)
        ctx = Context(p, precision)
        try:
            ctx.ensure_workspace(n_s, 16)
            for pad in (0, 1):
                ld = p.n_grid + pad
                buf = torch.full((n_s, ld), 7.0, dtype=ctx.dtype, device=ctx.device)
                out = buf.clone()
                buf[:, :p.n_grid] = torch.as_tensor(X.T.copy(), device=ctx.device).to(ctx.dtype)
                ws = torch.empty(L.dk_workspace_bytes(ctx.h, n_s, ld, 16) // 8 + 64,
                                 dtype=torch.float64, device=ctx.device)
                L.dk_set_workspace(ctx.h, ws)
                print(f"H X {dims} x {n_s} ld +{pad} {precision}", flush=True)
                L.dk_apply_h(ctx.h, buf[:, :p.n_grid], out[:, :p.n_grid])
                got = out[:, :p.n_grid].double().cpu().numpy().T
                ref = H.apply(X)
                tol = 1e-12 if precision == "fp64" else 2e-5
                assert np.abs(got - ref).max() / np.abs(ref).max() < tol
                assert torch.all(out[:, p.n_grid:] == 7.0)
        finally:
            ctx.close()

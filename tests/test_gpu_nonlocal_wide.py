"""The nonlocal term's remaining forms: the filter's integrals in 256-column tiles (from 2048
blocks of 64 points and tiles on, 65 to 128 projectors) with clamped columns, idle waves, a
ragged last block and a short last run, sums straight on and apart; the 128-column tiles with
sums apart; more than 1024 groups, whose order stays as it is.  Oracle: the FP64 Hamiltonian
on some of the columns; tolerances as for H X elsewhere (FP64 1e-12, FP32 blocks 2e-5)."""

import numpy as np
import pytest
import torch

from oracle.filter import chebyshev_filter
from oracle.hamiltonian import Hamiltonian
from workloads import custom_spec, make_problem

pytestmark = pytest.mark.gpu


def _check(n_atoms, dims, n_s, precision):
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context
    lens = tuple(0.4 * d for d in dims)
    spec = custom_spec("wide", 76, lens[0], 1, dims[0], 4, 1.0, basis="sc", dims=dims, lens=lens,
                       noise=False)
    pos = np.random.default_rng(n_atoms).uniform(0, 1, (n_atoms, 3)) * np.array(lens)
    p = make_problem(spec, positions=pos, with_block=False)
    H = Hamiltonian(p)
    ctx = Context(p, precision)
    try:
        ctx.ensure_workspace(n_s, 16)
        x = torch.randn((n_s, p.n_grid), generator=torch.Generator("cuda").manual_seed(n_s),
                        device="cuda").to(ctx.dtype)
        y = torch.full_like(x, 7.0)
        some = sorted({0, n_s // 2, n_s - 1})
        X = x[some].double().cpu().numpy().T
        tol = 1e-12 if precision == "fp64" else 2e-5
        print(f"H X {n_atoms} atoms {dims} x {n_s} {precision}", flush=True)
        L.dk_apply_h(ctx.h, x, y)
        ref = H.apply(X)
        assert np.abs(y[some].double().cpu().numpy().T - ref).max() / np.abs(ref).max() < tol
        print(f"filter {n_atoms} atoms {dims} x {n_s} {precision}", flush=True)
        a, b, a0 = 4.0, ctx.upper, -2.0
        L.dk_filter(ctx.h, x, 4, a, b, a0)
        ref = chebyshev_filter(H, X, 4, a, b, a0)
        assert np.abs(x[some].double().cpu().numpy().T - ref).max() / np.abs(ref).max() < tol
        assert bool(torch.isfinite(x).all()) and bool(torch.isfinite(y).all())
    finally:
        ctx.close()


@pytest.mark.parametrize("n_atoms,dims,n_s", [(17, (51, 52, 53), 130),   # 256 columns, straight on
                                              (32, (51, 52, 53), 290),   # apart
                                              (20, (48, 49, 51), 200)])  # 128 columns, apart
def test_filter_tiles(n_atoms, dims, n_s):
    _check(n_atoms, dims, n_s, "mixed")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_more_than_1024_groups(precision):
    _check(1027, (11, 12, 13), 19, precision)

"""The nonlocal term over 33 to 64 atom groups, where FP64 runs take the groups in two sets
of 32 slots: uneven and full sets, ragged grids, columns on both sides of a tile, and the
workspace, which depends on the sizes alone up to 64 groups (atoms may move).  Oracle: the
FP64 Hamiltonian; tolerances as for H X elsewhere (FP64 1e-12, FP32 blocks 2e-5)."""

import numpy as np
import pytest
import torch

from oracle.hamiltonian import Hamiltonian
from workloads import custom_spec, make_problem

pytestmark = pytest.mark.gpu


def _problem(n_atoms, dims, box):
    """n_atoms at random places of the lower `box` share of the cell."""
    lens = tuple(0.4 * d for d in dims)
    spec = custom_spec("sets", 75, lens[0], 1, dims[0], 4, 1.0, basis="sc", dims=dims, lens=lens,
                       noise=False)
    pos = np.random.default_rng(n_atoms).uniform(0, 1, (n_atoms, 3)) * np.array(lens) * box
    return make_problem(spec, positions=pos, with_block=False)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n_atoms,dims,n_s", [(33, (16, 16, 16), 1), (33, (24, 25, 26), 17),
                                              (47, (13, 15, 17), 130), (64, (20, 18, 21), 129)])
def test_two_sets(n_atoms, dims, n_s, precision):
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context
    p = _problem(n_atoms, dims, 1.0)
    X = np.random.default_rng(5).standard_normal((p.n_grid, n_s)).astype(np.float32)
    ctx = Context(p, precision)
    try:
        ctx.ensure_workspace(n_s, 16)
        x = torch.as_tensor(X.T.copy(), device=ctx.device).to(ctx.dtype)
        y = torch.full_like(x, 7.0)
        print(f"H X {n_atoms} atoms {dims} x {n_s} {precision}", flush=True)
        L.dk_apply_h(ctx.h, x, y)
        ref = Hamiltonian(p).apply(X.astype(np.float64))
        got = y.double().cpu().numpy().T
        tol = 1e-12 if precision == "fp64" else 2e-5
        assert np.abs(got - ref).max() / np.abs(ref).max() < tol
    finally:
        ctx.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n_atoms", [32, 33, 48, 64])
def test_workspace_does_not_follow_the_atoms(n_atoms, precision):
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context
    sizes = []
    for box in (1.0, 0.2):
        p = _problem(n_atoms, (24, 24, 24), box)
        ctx = Context(p, precision)
        try:
            sizes.append([L.dk_workspace_bytes(ctx.h, n_s, p.n_grid, 16) for n_s in (1, 17, 600)])
        finally:
            ctx.close()
    assert sizes[0] == sizes[1]

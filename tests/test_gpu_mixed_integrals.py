"""The mixed path's projector integrals at FP32 level, alone: one s projector or s and p
projectors strong enough that the nonlocal term is all of H X, columns of random sign (the
integrals cancel, so that an error of the products shows in full).  Tolerances: the
table, the coefficients and the scatter's products and sums are FP32, a few 2^-24
each (5e-7 together, rms); products of two bf16 pieces are off by about 2^-18 (4e-6)."""

import math
from types import SimpleNamespace

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

H0 = 0.32


def _apply(n, reps, channels, n_s, precision, X, filtered):
    """H X, or by one filter step over [-1, 1] (which is -H X / 2)."""
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context, ProjectorModel
    length = np.array(n) * H0
    cubes = np.stack(np.meshgrid(*(np.arange(r) for r in reps), indexing="ij"), -1)
    pos = (cubes.reshape(-1, 3) + 0.3) * (length / np.array(reps))
    grid = n[0] * n[1] * n[2]
    none = dict(offsets=np.zeros(1, np.int64), indices=np.zeros(0, np.int32), values=np.zeros(0),
                gamma=np.zeros(0), atom=np.zeros(0, np.int32))
    problem = SimpleNamespace(spec=SimpleNamespace(shape=n, cell=tuple(length)), n_grid=grid,
                              veff=np.zeros(grid), proj=none, positions=pos)
    ctx = Context(problem, precision)
    try:
        ctx.move_atoms(pos, ProjectorModel(channels, 1e-8))
        ctx.ensure_workspace(n_s, 16)
        x = X.to(ctx.dtype)
        print(f"integrals {n} {len(pos)} atoms x {n_s} {precision} filter={filtered}", flush=True)
        if filtered:
            y = x.clone()
            L.dk_filter(ctx.h, y, 1, -1.0, 1.0, -2.0)
            y *= -2.0
        else:
            y = torch.zeros_like(x)
            L.dk_apply_h(ctx.h, x, y)
        return y.double()
    finally:
        ctx.close()


def _error(n, reps, channels, n_s, filtered, positive=False):
    X = torch.randn((n_s, n[0] * n[1] * n[2]), device="cuda",
                    generator=torch.Generator("cuda").manual_seed(n_s))
    if positive:
        X.abs_().add_(0.5)
    ref = _apply(n, reps, channels, n_s, "fp64", X, filtered)
    got = _apply(n, reps, channels, n_s, "mixed", X, filtered)
    return math.sqrt(float((got - ref).square().sum() / ref.square().sum()))


S = ((0, 1.2, 1e5),)
SP = ((0, 1.2, 1e5), (1, 1.4, -6e4))


# 1 to 64 projectors: one, a part of a row block of four groups, and all of four
@pytest.mark.parametrize("filtered", [False, True], ids=["apply", "filter"])
@pytest.mark.parametrize("n,reps,channels,n_s", [((16, 16, 16), (1, 1, 1), S, 16),
                                                 ((17, 15, 19), (1, 1, 1), SP, 33),
                                                 ((24, 24, 24), (2, 2, 1), SP, 203),
                                                 ((40, 40, 20), (4, 4, 1), SP, 64)])
def test_fp32_level_up_to_64_projectors(n, reps, channels, n_s, filtered):
    assert _error(n, reps, channels, n_s, filtered) < 1e-6


# Runs of 63 blocks of 64 points.  Rounded once a block, the sums of a run leave 0.4 2^-24
# sqrt(63 / 2) = 1.3e-7, together with the FP32 roundings of the rest (2e-7) 2.4e-7; rounded
# at each of a block's twelve products, 0.4 2^-24 sqrt(12 63 / 2) = 4.6e-7.
def test_long_runs():
    assert _error((40, 40, 40), (4, 4, 2), SP, 2048, False) < 3.5e-7


# Columns of one sign: the s integrals are far larger than the p ones.  Table, coefficient,
# the last step of the sum over projectors, the sum with the local part and the result round
# once each, 0.42 2^-24 sqrt(5) = 5.6e-8; a sum that takes the s projectors first rounds
# three times more per four groups.
def test_positive_columns():
    assert _error((24, 24, 24), (2, 2, 1), SP, 64, False, positive=True) < 8e-8

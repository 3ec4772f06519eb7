"""Loss gradient of the start-density network at the edges of its kernels: one feature,
widths that are no multiple of four (element-wise ends of the layer products' tiles),
the widest, one point, batches around the 64-point tiles, one and several layers; in
FP32 mode against the FP64 oracle, per layer, to 1e-5 of its largest entry."""

import numpy as np
import pytest
import torch

from oracle import mlp as omlp
from workloads import custom_spec, make_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,hidden,layers,P", [(1, 1, 1, 1), (5, 3, 2, 63), (32, 17, 1, 65),
                                                  (64, 63, 3, 700), (7, 64, 2, 128),
                                                  (64, 64, 1, 33000)])
def test_loss_gradient_edges(n_in, hidden, layers, P):
    from paper_2112_08639_amd import _lib as L
    from paper_2112_08639_amd.pipeline import Context
    ctx = Context(make_problem(custom_spec("mlp7", 97, 3.0, 1, 7, 4, 1.0, basis="sc", noise=False)),
                  "fp64")
    try:
        shapes = omlp.layer_shapes(n_in, hidden, layers)
        theta = omlp.init_params(shapes, 41).astype(np.float32).astype(np.float64)
        rng = np.random.default_rng(P)
        u = rng.standard_normal((P, n_in)).astype(np.float32)
        t = rng.uniform(0.2, 3.0, P).astype(np.float32)
        loss_ref, g_ref = omlp.loss_and_grad(theta, shapes, u.astype(np.float64),
                                             t.astype(np.float64))
        shape = L.MlpShape(n_in, hidden, layers)
        dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")
        ws = torch.empty(L.dk_mlp_workspace_bytes(shape, P) // 4 + 64, dtype=torch.float32,
                         device="cuda")
        grad = torch.zeros(len(theta), dtype=torch.float32, device="cuda")
        print(f"loss gradient {n_in}-{hidden}x{layers}, {P} points", flush=True)
        loss = L.dk_mlp_loss_grad(ctx.h, shape, L.DK_MLP_F32, dev(theta), dev(u.reshape(-1)),
                                  dev(t), P, grad, ws)
        g = grad.cpu().numpy().astype(np.float64)
        off = 0
        for n_out, n_i in shapes:
            for size in (n_out * n_i, n_out):
                gl, rl = g[off:off + size], g_ref[off:off + size]
                assert np.abs(gl - rl).max() < 1e-5 * np.abs(rl).max() + 1e-30, (n_out, n_i, size)
                off += size
        assert abs(loss - loss_ref) < 1e-5 * loss_ref
    finally:
        ctx.close()

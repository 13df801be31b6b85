"""The training step's kernels (k_train_pass, k_train_grads) at the edges of
their splits, against the FP64 oracle with bf16 operands."""
import numpy as np
import pytest

from oracle import mlp
from test_gpu_mlp import as_dict, problem, reference, tess  # noqa: F401

pytestmark = pytest.mark.gpu


# 32 samples a block, slices of 64 (weights, biases) and 256 (output layer),
# 64 slices per chunk of sums: a ragged block, one sample past a slice, past a
# chunk of slices, and past a chunk of the output layer's slices.  Every
# operand is rounded to bf16 (2^-9 relative, random sign) on at most eight
# steps between a sample and its gradient, 8^(1/2) 2^-9 = 5.5e-3 when nothing
# averages.
@pytest.mark.parametrize("n", [33, 65, 257, 4097, 16640])
def test_gradients_at_split_edges(tess, n):  # noqa: F811
    import torch
    q, target, B, params = problem(n, 7 * n)
    loss, grad = tess.mlp_loss_grad(params, B, torch.from_numpy(q).cuda(), torch.from_numpy(target).cuda())
    rl, rg, _ = reference(params, B.astype(np.float64), q, target.astype(np.float64))
    assert abs(loss - rl) / rl < 2e-3
    g = as_dict(grad)
    for k in mlp.NAMES:
        a, b = g[k].ravel(), rg[k].ravel()
        rel = np.linalg.norm(a - b) / np.linalg.norm(b)
        print(f"n={n} {k}: rel L2 {rel:.3e}", flush=True)
        assert rel <= 1e-2, k


# The inference deals its 16-sample tiles to the CUs first (256 blocks: 4096
# samples) and to a block's 16 wavefronts next (65536): a sample's output is
# its own, so a call cut into pieces gives the same bits.
@pytest.mark.parametrize("n", [4095, 4097, 65536, 65553])
def test_inference_does_not_depend_on_the_cut(tess, n):  # noqa: F811
    import torch
    q, _, B, params = problem(n, 11 * n)
    qd = torch.from_numpy(q).cuda()
    whole = tess.mlp_forward(params, B, qd)
    parts = [tess.mlp_forward(params, B, qd[a:a + 1013].contiguous()) for a in range(0, n, 1013)]
    assert torch.equal(whole, torch.cat(parts))

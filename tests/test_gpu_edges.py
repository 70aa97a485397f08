"""Edges of the kernels' work splits: the sizes where a split, a remainder or a
rule of a dispatch changes, each against the oracle or against another route
to the same values."""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_proposal import _bf16_bits, _inputs, _offsets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lnr():
    import paper_1504_01441_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(lnr):
    return lnr.Context(0)


# gradient blocks of one sample, of two with a short last one, of four, the
# first size of the four-sample forward workgroup, more than 256 blocks' worth
@pytest.mark.parametrize("n", [1, 64, 65, 256, 257, 1030])
def test_training_step_at_block_edges(lnr, ctx, n):
    P = synth.proposal_params(11, head_scale=4.0)
    lnr.proposal_set(ctx, torch.from_numpy(P))
    x = _inputs(90 + n, n)
    lab = np.random.default_rng(n).integers(-10, 11, (n, 2)).astype(np.int32)
    xb, lb = _bf16_bits(x).cuda(), torch.from_numpy(lab).cuda()
    _, grad = lnr.proposal_train_step(ctx, xb, lb, 1e-3, 1e-4, want_grad=True)
    g = grad.cpu().numpy().astype(np.float64)
    _, g_o = oracle.cnn_loss_grad(P.astype(np.float64), x, lab, rnd=True)
    # bf16 activations that round the other way: 2 % of a tensor's norm (as in
    # test_gpu_proposal)
    for name, o, k in _offsets():
        nb = np.linalg.norm(g_o[o:o + k])
        assert np.linalg.norm(g[o:o + k] - g_o[o:o + k]) <= 2e-2 * nb + 1e-7, name
    # the step's packed weights are those of its parameters
    after = lnr.proposal_forward(ctx, xb)
    lnr.proposal_set(ctx, lnr.proposal_get(ctx))
    assert torch.equal(after, lnr.proposal_forward(ctx, xb))

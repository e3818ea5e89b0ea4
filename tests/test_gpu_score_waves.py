"""Batches of 1024 images on take two waves per image in the backward pass, smaller ones four.

The mean gradient of a batch is the mean of its halves' mean gradients.  The kernel scales dZ by 1/batch
before rounding it to BF16, and rounding commutes with a power-of-two scale, so a batch of 1024 or 2048
(two waves) and its sub-batches of 512 (four waves, pinned to the oracle elsewhere) agree up to the order
of FP32 sums: 1e-5 relative L2 per tensor, the bound that the other splits of a batch are held to.
"""
import numpy as np
import pytest
import torch

import workloads
from test_gpu_score import NAMES, _flat, _net, _rel_l2, _unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1024, 2048])
def test_two_and_four_waves_per_image_agree(batch):
    p = workloads.cnn_params(41)
    x, lab = workloads.cnn_batch(batch, 42)
    xt = torch.from_numpy(x.astype(np.float32)).cuda()
    lt = torch.from_numpy(lab.astype(np.float32)).cuda()
    g = _unflat(_net(_flat(p), batch).grad(xt, lt).cpu().numpy().astype(np.float64))
    subnet = _net(_flat(p), 512)
    ref = 0.0
    for s0 in range(0, batch, 512):
        ref = ref + 512 / batch * subnet.grad(xt[s0:s0 + 512].contiguous(), lt[s0:s0 + 512].contiguous()).cpu().numpy().astype(np.float64)
    ref = _unflat(ref)
    for k in NAMES:
        assert _rel_l2(g[k], ref[k]) <= 1e-5, (k, _rel_l2(g[k], ref[k]))

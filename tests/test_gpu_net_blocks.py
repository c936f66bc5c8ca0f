"""The correction network's convolution at the edges of its blocks.

A workgroup owns 16 x 8 x 4 voxels (16 x 4 x 4 on grids of fewer than 512 such
blocks) with a one-voxel halo: grids that fill a block, miss it by one either
way, hold less than a row of one, or have their last block one voxel deep.
Bound: the stored values are BF16 (relative spacing 2^-8) and both sides take
every rounding and ReLU on the same exact sums up to FP32 summation order, so
only single-spacing flips survive: 5 spacings of the largest entry.
"""
import numpy as np
import pytest
import torch

from oracle import unet
from paper_1212_1397_amd.workloads import init_net_params, random_field

pytestmark = pytest.mark.gpu
KH = 0.31


@pytest.mark.parametrize("dims", [(2, 1, 3), (16, 4, 4), (16, 8, 4), (15, 7, 3), (17, 9, 5), (33, 8, 13), (80, 65, 57)])
def test_forward_at_block_edges(dims):
    from paper_1212_1397_amd import helmholtz6 as h6
    p = init_net_params(h6.NET_LAYERS, 5)
    rng = np.random.default_rng(6)
    p = {n: (w * (100.0 if n == "out" else 1.0), 0.1 * rng.standard_normal(b.shape)) for n, (w, b) in p.items()}
    net = h6.Net(dims)
    net.set_params(h6.pack_net_params(p))
    r = random_field(dims[::-1], 7)
    c = net.forward(torch.from_numpy(r).cuda(), KH).cpu().numpy()
    q = {n: (unet.round_bf16(w), np.asarray(b, dtype=np.float32).astype(np.float64)) for n, (w, b) in p.items()}
    ref = unet.correction(q, r, KH, 1.0, store=unet.round_bf16)
    err = np.abs(c - ref).max() / np.abs(ref).max()
    print(f"{dims}: {err:.2e}", flush=True)
    assert err < 5 * 2.0 ** -8

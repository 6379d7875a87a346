"""The fused loss at the sizes where its workgroups' shares end: one vector, one short of / one past a
workgroup's elements, one past a trip of its threads, samples on both sides of the prepare launch."""
import numpy as np
import pytest

import workloads as wl
from oracle import nft_loss
from helpers import dev_f32, host_f64
from test_gpu_nft import GRAD_REL, LOSS_REL, _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,elems", [
    ("bf16", 1, 8), ("f32", 1, 4), ("bf16", 3, 8200), ("f32", 3, 8196), ("bf16", 2, 16376), ("bf16", 2, 16392),
    ("f32", 2, 16388), ("bf16", 5, 2056), ("f32", 1025, 8), ("bf16", 1024, 8),
    ("f32", 2, 49156), ("bf16", 2, 65544),   # even shares of four and five workgroups, the last one shorter
    ("bf16", 300, 4104), ("f32", 600, 520),  # more masks than threads
    ("bf16", 3, 6136), ("bf16", 3, 6144), ("f32", 3, 9212), ("f32", 3, 9216),  # both sides of the lines for the threads
])
def test_nft_loss_at_the_edges_of_its_shares(dtype, n, elems):
    import torch
    import paper_2603_17051_amd as A
    dev, wide, adv, mask = _case(n, (elems,), dtype, wl.BASE_SEED + 33, range(0, n, 3))
    loss, grad = torch.full((3,), float("nan"), device="cuda:0"), torch.full((n, elems), float("nan"), device="cuda:0")
    A.astro_nft_loss(*dev, dev_f32(adv), torch.from_numpy(mask).to("cuda:0"), 1.2, 0.8, 0.4, loss, grad)
    ref = nft_loss(*wide, adv.astype(np.float64), 1.2, mask, 0.8, 0.4)
    assert host_f64(loss) == pytest.approx(np.array(ref[:3], dtype=np.float64), rel=LOSS_REL)
    g = host_f64(grad)
    assert np.isfinite(g).all() and np.abs(g - ref[3]).max() <= GRAD_REL * np.abs(ref[3]).max()

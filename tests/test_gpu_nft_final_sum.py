"""The fused loss's final sum around the numbers of partial sums at which its waves change, against the fp64 oracle's
formula; fp32 partial sums of at most 16384 terms and an fp64 sum of those: 1e-5 as elsewhere."""
import pytest
import torch

import paper_2603_17051_amd as A

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,elems,dtype", [
    (1, 8, torch.bfloat16), (63, 8, torch.float32), (64, 40, torch.bfloat16), (65, 8, torch.bfloat16),
    (33, 16384 + 8, torch.float32), (1, 64 * 16384 + 8, torch.bfloat16), (512, 16384 + 8, torch.bfloat16), (1025, 16, torch.float32),
])
@pytest.mark.parametrize("masked", [0, 1, 3])
def test_final_sum(n, elems, dtype, masked):
    g = torch.Generator("cuda:0").manual_seed(n + elems)
    x = [torch.randn((n, elems), generator=g, device="cuda:0").to(dtype) for _ in range(4)]
    adv = 1.5 * torch.randn(n, generator=g, device="cuda:0")
    mask = (torch.arange(n, device="cuda:0") % 3 < masked).to(torch.int32)
    loss, grad = A.astro_nft_loss(*x, adv, mask, 1.2, 0.9, 0.1)
    vt, vo, vr, tg = (t.double() for t in x)
    r = (adv.double() / 1.2).clamp(-1, 1)[:, None] * 0.5 + 0.5
    pos, neg, ref, m = 0.1 * vo + 0.9 * vt - tg, 1.9 * vo - 0.9 * vt - tg, vt - vr, (mask != 0).double()[:, None]
    policy = (r * pos.square() + (1 - r) * neg.square()).sum() / n
    kl = (m * ref.square()).sum() / m.sum() if masked else torch.zeros((), device="cuda:0", dtype=torch.float64)
    want = torch.stack([policy + 0.1 * kl, policy, kl])
    assert torch.all((loss.double() - want).abs() <= 1e-5 * want.abs() + 1e-30), (loss, want)
    dwant = 2 * 0.9 / n * (r * pos - (1 - r) * neg) + (2 * 0.1 / m.sum() * m * ref if masked else 0)
    assert float((grad.double() - dwant).norm() / dwant.norm()) <= 1e-5

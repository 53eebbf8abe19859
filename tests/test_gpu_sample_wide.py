"""Draft token of sampling rows where a row's partials are read by eight waves (more than four drafts and 65536 entries, or more than
163840 entries) and at the edges of that range, against the inverse CDF of the 64-bit mixture of the same logits."""
import pytest
import torch

from paper_2601_20357_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("V,n", [(65536, 5), (65537, 5), (128256, 8), (131073, 16), (163841, 3), (196608, 2), (196609, 6)])
@pytest.mark.parametrize("scale", [8.0, 0.2], ids=["peaked", "flat"])
def test_sampled_draft_token(V, n, scale):
    print(f"sampled V={V} n={n} scale={scale}", flush=True)
    B, d = 9, 64
    g = torch.Generator(device=DEV).manual_seed(V + n)
    buf = binding.RoundBuffers(binding.make_cfg(V=V, d=d, n=n, B=B, gamma=1, h=1, w_dtype=1), DEV)
    buf.weights.copy_(torch.softmax(torch.randn((B, n), generator=g, device=DEV), -1))
    W = (torch.randn((V, d), generator=g, device=DEV) * 0.15).bfloat16()
    H = (torch.randn((B, n, d), generator=g, device=DEV) * scale).bfloat16()
    temp = torch.tensor([1.0, 0.7, 0.0] * 3, device=DEV)
    u = torch.rand((B, 1), generator=g, device=DEV)
    u[0], u[1] = 0.0, 1.0 - 2.0 ** -24
    buf.draft_step(0, 0, W, H, temp, u_draft=u)
    torch.cuda.synchronize()
    inv = torch.where(temp > 0, 1 / temp, torch.ones_like(temp)).double()
    s = buf.draft_logits[0].double() * inv[:, None, None]
    # 2e-6 for the fp32 exponentials and their sums over tiles, and a scaled logit is rounded to fp32
    tol = 2e-6 + 2.0 ** -24 * s.abs().amax(-1)
    assert bool(((buf.draft_lse[0] - torch.logsumexp(s, -1)).abs() <= tol).all())
    q = (torch.softmax(s, -1) * buf.weights.double()[:, :, None]).sum(1)
    y = buf.draft_tokens[:, 0].long()
    off = 2 * tol.amax(-1)                               # a probability is off by that much of itself, and so is the CDF
    cdf = torch.nn.functional.pad(q.cumsum(-1), (1, 0))
    below, upto, at = cdf.gather(1, y[:, None])[:, 0], cdf.gather(1, y[:, None] + 1)[:, 0], u[:, 0].double() * cdf[:, -1]
    inside = (below <= at + off) & (at < upto + off)
    assert bool((inside | (temp == 0)).all()), (y, below, at, upto)
    best = q.topk(2, -1)
    near = (best.values[:, 0] - best.values[:, 1]) <= 2 * off * best.values[:, 0]
    assert bool(((y == best.indices[:, 0]) | near | (temp > 0)).all())
    assert bool(((buf.draft_q[:, 0].double() - q.gather(1, y[:, None])[:, 0]).abs() <= (1e-5 + off) * q.max(-1).values).all())

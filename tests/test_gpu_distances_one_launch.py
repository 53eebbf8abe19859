"""Distances that share a launch with the statistics (hard labels) or with the accept chain (total variation): at sizes on both sides
of the lines between their instances, the values are those of 64-bit softmaxes, and the window and weights of the verification that
advances them are those of the separate call."""
import pytest
import torch

from paper_2601_20357_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(V, n, B, gamma, distance, policy, h):
    g = torch.Generator(device=DEV).manual_seed(V + 16 * n + B)
    r = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa: E731
    cfg = binding.make_cfg(V=V, d=8, n=n, B=B, gamma=gamma, h=h, w_dtype=1, distance=distance, policy=policy, seed=3)
    temp = torch.ones(B, device=DEV)
    temp[1::3] = 0.0
    temp[2::3] = 0.7
    inv = torch.where(temp > 0, 1 / temp, torch.ones_like(temp))
    logits, target = 2.5 * r(gamma, B, n, V), 2.5 * r(B, gamma + 1, V)
    logits[:, :, 0] += target[:, :gamma].transpose(0, 1)             # one draft agrees, so that some positions are accepted
    target[0, 0, V // 2:] = -float("inf")                            # masked entries, whole chunks of them where V allows
    weights = torch.softmax(r(B, n), -1)
    lse = torch.logsumexp(logits.double() * inv[None, :, None, None], -1)
    tokens = logits[:, :, 0].argmax(-1).int().t().contiguous()
    ring = torch.rand((B, max(h, 1), binding.load().tabed_dev_width(cfg)), generator=g, device=DEV) + 0.1
    return cfg, temp, inv, logits, target, weights, lse, tokens, ring


@pytest.mark.parametrize("V,n,B,gamma,policy,h", [
    (3, 3, 2, 2, 0, 4), (4097, 1, 3, 3, 0, 4), (8003, 4, 7, 3, 0, 0),
    (40001, 4, 20, 3, 0, 4), (40001, 4, 20, 2, 0, 4),               # four drafts: 1020 workgroups (up front), 820
    (50261, 4, 12, 5, 0, 4),                                         # 1092 (in turn)
    (30001, 5, 16, 4, 0, 4), (30001, 5, 19, 4, 0, 4),                # five drafts: 768 (up front), 912
    (20001, 8, 16, 4, 0, 4), (20001, 8, 18, 4, 0, 4), (20001, 6, 9, 3, 0, 4),   # eight: 496, 558; six: rows in turn
    (5, 2, 60001, 10, 0, 4), (5, 2, 60001, 10, 2, 4),                # labels: 1260021 workgroups, in two rows of the grid
    (70001, 2, 15, 6, 2, 4), (33, 2, 3, 2, 2, 0)])
@pytest.mark.parametrize("distance", [1, 2], ids=["tv", "labels"])
def test_distances_and_window(V, n, B, gamma, policy, h, distance):
    print(f"distances V={V} n={n} B={B} gamma={gamma} policy={policy} h={h} distance={distance}", flush=True)
    cfg, temp, inv, logits, target, weights, lse, tokens, ring = _inputs(V, n, B, gamma, distance, policy, h)
    q = (weights[None, :, :, None] * torch.softmax(logits * inv[None, :, None, None], -1)).sum(2)
    bufs = []
    for fused in (False, True):
        buf = binding.RoundBuffers(cfg, DEV)
        buf.draft_logits.view(logits.shape).copy_(logits)
        buf.draft_lse.view(lse.shape).copy_(lse)
        buf.draft_tokens.copy_(tokens)
        buf.draft_q.copy_(q.gather(2, tokens.t().long()[:, :, None])[:, :, 0].t())
        buf.weights.copy_(weights)
        buf.ring.view(ring.shape).copy_(ring)
        buf.ring_count.fill_(min(h, 3) if h else 5)
        for _ in range(2 if fused else 1):                           # the counters are reset: a second call finds them so
            if fused:
                buf.weights.copy_(weights); buf.ring.view(ring.shape).copy_(ring); buf.ring_count.fill_(min(h, 3) if h else 5)
                buf.ring_head.zero_()
            buf.verify(4, target, temp, fused_update=fused)
        if not fused:
            buf.update_weights(False, 5)
        torch.cuda.synchronize()
        bufs.append(buf)
    for name in ("accept_len", "out_tokens", "dev", "n_valid", "verify_flags", "ring", "ring_head", "ring_count", "weights"):
        assert torch.equal(getattr(bufs[0], name), getattr(bufs[1], name)), name
    dev = bufs[1].dev.view(B, gamma, -1)
    if policy == 2:
        w1 = torch.arange(11, device=DEV, dtype=torch.float64) / 10
    for i in range(gamma):
        p = torch.softmax(target[:, i].double() * inv[:, None].double(), -1)
        qs = torch.softmax(logits[i].double() * inv[:, None, None].double(), -1)
        if policy == 2:
            qs = (1 - w1)[None, :, None] * qs[:, :1] + w1[None, :, None] * qs[:, 1:]
        if distance == 1:
            want = 0.5 * (p[:, None] - qs).abs().sum(-1)
            assert bool(((dev[:, i].double() - want).abs() <= 1e-5 * want + 1e-6).all())
        else:
            label = bufs[1].out_tokens[:, i].long()
            emitted = i <= bufs[1].accept_len
            top, at = qs.topk(min(2, V), -1)
            clear = (top[..., 0] - top[..., 1]) > 1e-5 * top[..., 0]
            want = (at[..., 0] != label[:, None]).float()
            assert bool(((dev[:, i] == want) | ~clear)[emitted].all())
            assert bool((dev[:, i][~emitted] == 1).all())


def _timed(calls, ids):
    binding.tabed_prof_reset()
    binding.tabed_prof_enable(True)
    for call in calls:
        call()
    binding.tabed_prof_enable(False)
    return [binding.tabed_prof_read(i) for i in ids]


@pytest.mark.parametrize("distance", [0, 1, 2], ids=["kl", "tv", "labels"])
def test_distances_are_timed_under_their_own_id(distance):
    """K_DIST reports the launch that holds the distances, which counts under the id of what it shares it with as well; the
    divergence, which rides in the statistics' records, has none."""
    cfg, temp, _, logits, target, weights, lse, tokens, _ = _inputs(8003, 4, 3, 3, distance, 0, 4)
    buf = binding.RoundBuffers(cfg, DEV)
    buf.draft_logits.view(logits.shape).copy_(logits)
    buf.draft_lse.view(lse.shape).copy_(lse)
    buf.draft_tokens.copy_(tokens)
    buf.draft_q.fill_(0.1)
    buf.weights.copy_(weights)
    stats, resid, dist = _timed([lambda: buf.verify(4, target, temp)] * 3, (binding.K_STATS, binding.K_RESID, binding.K_DIST))
    assert stats[1] == 3 and resid[1] == 3
    assert dist == {0: (0.0, 0), 1: resid, 2: stats}[distance]
    binding.tabed_prof_reset()

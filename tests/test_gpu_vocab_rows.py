"""Passes over the vocabulary at row lengths that are not a multiple of four and draft counts known / not known at compile time."""
import pytest

from paper_2601_20357_amd import synth

import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,n,policy,distance", [(1001, 1, 0, 0), (1002, 3, 0, 1), (1003, 5, 0, 0), (4099, 6, 0, 1), (2, 3, 0, 0), (3, 5, 0, 1),
                                                 (1025, 2, 2, 0), (4102, 2, 2, 1)])
def test_rounds_on_unaligned_rows(oracle, V, n, policy, distance):
    print(f"unaligned rows V={V} n={n} policy={policy} distance={distance}", flush=True)
    wl = synth.scaled(synth.WORKLOADS["serving"], V=V, d=64, n=n, B=5, gamma=3, h=4, cfg_id=160 + V % 9)
    tally = harness.run_rounds(oracle, wl, 4, synth.make_temperature(wl, "mixed07"), policy=policy, distance=distance)
    assert tally.flagged_divergences <= max(2, tally.decisions // 50)


@pytest.mark.parametrize("V,n", [(33, 1), (1003, 3), (8200, 8), (33000, 4), (70004, 4), (128256, 8), (200003, 2), (40001, 6)])
@pytest.mark.parametrize("scale", [8.0, 0.2, 0.0], ids=["peaked", "flat", "ties"])
def test_greedy_draft_token(V, n, scale):
    """Arg-max of the mixture whether a few tiles of the vocabulary can hold it (peaked), many (flat) or all (ties)."""
    import torch
    from paper_2601_20357_amd import binding
    print(f"greedy V={V} n={n} scale={scale}", flush=True)
    B, d = 3, 64
    g = torch.Generator(device="cuda:0").manual_seed(V + n)
    cfg = binding.make_cfg(V=V, d=d, n=n, B=B, gamma=1, h=1, w_dtype=1)
    buf = binding.RoundBuffers(cfg)
    buf.weights.copy_(torch.softmax(torch.randn((B, n), generator=g, device="cuda:0"), -1))
    W = (torch.randn((V, d), generator=g, device="cuda:0") * 0.15).bfloat16()
    H = (torch.randn((B, n, d), generator=g, device="cuda:0") * scale).bfloat16()
    buf.draft_step(0, 0, W, H, torch.zeros(B, device="cuda:0"))
    torch.cuda.synchronize()
    q = (torch.softmax(buf.draft_logits[0].double(), -1) * buf.weights.double()[:, :, None]).sum(1)      # [B,V]
    top, at = q.topk(2, -1)
    near = (top[:, 0] - top[:, 1]) < 1e-6 * top[:, 0]
    y = buf.draft_tokens[:, 0].long()
    assert bool(((y == at[:, 0]) | near).all())
    # a probability is off by at most the fp32 exponentials' and sums' few units in the last place
    assert bool(((buf.draft_q[:, 0].double() - q.gather(1, y[:, None])[:, 0]).abs() <= 1e-5 * top[:, 0]).all())
    flagged = (buf.draft_flags[:, 0] & binding.FLAG_SAMPLE_MARGIN) != 0
    assert bool((flagged | ~((top[:, 0] - top[:, 1]) < 5e-7 * top[:, 0])).all())     # a clear near-tie is flagged,
    assert bool((~flagged | ((top[:, 0] - top[:, 1]) < 2e-6 * top[:, 0])).all())     # a clear winner is not
    if scale == 0.0:
        assert bool((y == 0).all())


@pytest.mark.parametrize("V,n", [(3, 2), (40, 1), (2050, 3), (33000, 4), (128256, 8), (200003, 2)])
@pytest.mark.parametrize("scale", [8.0, 0.2, 0.0], ids=["peaked", "flat", "ties"])
def test_greedy_siblings(V, n, scale):
    """Both siblings of a greedy row: the two largest entries besides the trunk's token, lowest index on ties."""
    import torch
    from paper_2601_20357_amd import binding
    print(f"siblings V={V} n={n} scale={scale}", flush=True)
    B, d = 3, 64
    g = torch.Generator(device="cuda:0").manual_seed(V + n)
    cfg = binding.make_cfg(V=V, d=d, n=n, B=B, gamma=1, h=1, w_dtype=1)
    buf = binding.RoundBuffers(cfg)
    buf.enable_tree(3)
    buf.weights.fill_(1.0 / n)
    W = (torch.randn((V, d), generator=g, device="cuda:0") * 0.15).bfloat16()
    H = (torch.randn((B, n, d), generator=g, device="cuda:0") * scale).bfloat16()
    temp = torch.zeros(B, device="cuda:0")
    sib = buf.prepare_draft_siblings(0, 0, temp)
    for _ in range(2):                                    # the second pass finds the counters re-armed
        buf.draft_step(0, 0, W, H, temp)
        sib()
        torch.cuda.synchronize()
        q = (torch.softmax(buf.draft_logits[0].double(), -1) * buf.weights.double()[:, :, None]).sum(1)
        order = torch.sort(q, stable=True, dim=-1, descending=True)
        got = torch.cat([buf.draft_tokens, buf.sib_tokens[:, 0]], 1).long()
        if scale == 0.0:
            assert bool((got == torch.arange(3, device="cuda:0")).all())
        gap = (order.values[:, :3] - torch.nn.functional.pad(order.values, (0, 1))[:, 1:4]).abs() < 1e-6 * order.values[:, :3]
        clear = ~(gap.any(-1))
        assert bool((got[clear] == order.indices[clear, :3]).all())
        assert bool(((buf.sib_q[:, 0].double() - q.gather(1, got[:, 1:])).abs() <= 1e-5 * order.values[:, :1]).all())


@pytest.mark.parametrize("V", [8200, 8201])
@pytest.mark.parametrize("policy,distance", [(2, 0), (2, 1), (2, 2), (0, 0), (0, 1), (0, 2)])
def test_verify_with_masked_target_logits(oracle, V, policy, distance):
    """Target rows with long runs of -inf (constrained decoding): whole chunks of the passes without a term, at the end, at the
    start, on both sides of one allowed run; a term with p = 0 counts nothing."""
    import numpy as np
    import torch
    print(f"masked target V={V} policy={policy} distance={distance}", flush=True)
    n, B, gamma, h = (2 if policy == 2 else 3), 6, 2, 3
    wl = synth.scaled(synth.WORKLOADS["serving"], V=V, d=64, n=n, B=B, gamma=gamma, h=h, cfg_id=170 + V % 2)
    side = harness.GpuSide(wl, seed=4, policy=policy, distance=distance)
    buf = side.buf
    W = synth.make_lm_head(wl)
    H, target = synth.make_round(wl, W, 1)
    target = np.array(target, np.float32)
    for b, (lo, hi) in enumerate([(0, 1500), (5000, V), (3000, 3600), (V - 2, V), (0, V), (1024, 2048)]):     # allowed entries
        target[b, :, :lo] = -np.inf
        target[b, :, hi:] = -np.inf
    temp = np.array([1.0, 0.7, 1.0, 0.7, 0.0, 0.0], np.float32)
    buf.update_weights(True, rnd=0)
    w = buf.weights.cpu().numpy()
    W_t, temp_t, target_t = harness.to_dev_store(W, 1), torch.from_numpy(temp).cuda(), torch.from_numpy(target).cuda()
    for pos in range(gamma):
        buf.draft_step(0, pos, W_t, harness.to_dev_store(H[pos], 1), temp_t)
    buf.verify(0, target_t, temp_t, fused_update=True)
    torch.cuda.synchronize()
    c = lambda t: t.cpu().numpy()  # noqa: E731
    want = oracle.verify(V=V, n=n, B=B, gamma=gamma, distance=distance, seed=4, rnd=0, target_logits=target, draft_logits=c(buf.draft_logits),
                         draft_tokens=c(buf.draft_tokens), draft_q=c(buf.draft_q), weights=w, temperature=temp,
                         n_cand=oracle.GRID_CANDIDATES if policy == 2 else 0)
    dev, flags = c(buf.dev), c(buf.verify_flags) | want["flags"]
    assert np.isfinite(dev).all() and np.isfinite(c(buf.ring)).all() and np.isfinite(c(buf.weights)).all()
    for b in range(B):
        if flags[b].any():                            # a decision within its margin may differ
            continue
        assert c(buf.accept_len)[b] == want["accept_len"][b] and np.array_equal(c(buf.out_tokens)[b], want["out_tokens"][b])
        valid = slice(0, want["n_valid"][b])          # the parity harness' tolerance of distances; hard labels are exact
        err, bound = np.abs(dev[b, valid] - want["dev"][b, valid]), 1e-5 * np.abs(want["dev"][b, valid]) + 1e-6
        assert (err <= (0.0 if distance == 2 else bound)).all(), (b, dev[b], want["dev"][b])
    assert (flags == 0).all(axis=1).sum() >= 3
    ring = np.zeros((B, h, oracle.dev_width(n, policy)), np.float32)
    nxt = oracle.update_weights(n=n, B=B, gamma=gamma, h=h, policy=policy, tau_w=1.0, eps=1e-6, dev=dev, n_valid=c(buf.n_valid), ring=ring,
                                ring_head=np.zeros(B, np.int32), ring_count=np.zeros(B, np.int32), seed=4, rnd=1)
    np.testing.assert_allclose(c(buf.weights), nxt, rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("V,n", [(8192, 3), (8192, 5), (8191, 4), (8191, 1), (8192, 4), (8192, 6), (8190, 8)])
def test_log_sum_exp_adds_the_tiles_in_64_bits(V, n):
    """One entry of probability ~1 and 252 of 4e-8, each in a tile and a lane that the first one is not in: added in 32 bits, each
    is less than half a unit in the last place of the sum and the log-sum-exp loses up to 6e-8; the exponentials' own error is
    1e-6 of 1e-5."""
    import torch
    from paper_2601_20357_amd import binding
    print(f"tile sums V={V} n={n}", flush=True)
    B = 2
    cfg = binding.make_cfg(V=V, d=8, n=n, B=B, gamma=1, h=1, w_dtype=1)
    buf = binding.RoundBuffers(cfg)
    buf.weights.fill_(1.0 / n)
    W = torch.zeros((V, 8), dtype=torch.bfloat16, device="cuda:0")
    W[:, 0] = -1000.0
    W[5::32, 0] = -17.0
    W[5::64 * 32, 0] = -1000.0
    W[0, 0] = 0.0
    H = torch.zeros((B, n, 8), dtype=torch.bfloat16, device="cuda:0")
    H[..., 0] = 1.0
    buf.draft_step(0, 0, W, H, torch.ones(B, device="cuda:0"))
    torch.cuda.synchronize()
    lse = torch.logsumexp(buf.draft_logits[0].double(), -1)
    assert float((buf.draft_lse[0] - lse).abs().max()) <= 1e-10


def test_arrival_counters_packed_to_fit_the_built_in_scratch():
    """Where a line for every sequence's counters would lift a configuration over the built-in scratch, the counters are packed:
    the same sequences give the same results there as in a smaller batch, whose counters are not (two rounds: re-armed counters)."""
    import torch
    from paper_2601_20357_amd import binding
    V, n, d, gamma, width = 32000, 4, 64, 1, 3
    cfg_of = lambda B: binding.make_cfg(V=V, d=d, n=n, B=B, gamma=gamma, h=3, w_dtype=1, seed=5)  # noqa: E731
    size = lambda B: binding.tabed_workspace_bytes(cfg_of(B))  # noqa: E731
    B = next(B for B in range(20, 2000) if size(B) < size(B - 1))
    assert size(B) <= binding.STATIC_SCRATCH_BYTES < size(B - 1) + (size(B - 1) - size(B - 2))
    few = B // 2
    print(f"packed counters B={B}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(9)
    W = (torch.randn((V, d), generator=g, device="cuda:0") * 0.15).bfloat16()
    H = torch.randn((B, n, d), generator=g, device="cuda:0") * 4.0
    H[::5] = 0.0                                          # rows of equal logits: every workgroup of the row arrives
    H = H.bfloat16()
    target = torch.randn((B, gamma + 1, V), generator=g, device="cuda:0") * 2.0
    leaves = torch.randn((B, gamma, width - 1, V), generator=g, device="cuda:0") * 2.0
    temp = torch.ones(B, device="cuda:0")
    temp[::2] = 0.0

    def run(b):
        buf = binding.RoundBuffers(cfg_of(b))
        buf.enable_tree(width)
        out = []
        sib = buf.prepare_draft_siblings(0, 0, temp[:b])
        tree = buf.prepare_verify_tree(0, target[:b].contiguous(), leaves[:b].contiguous(), temp[:b])
        for rnd in range(2):
            buf.update_weights(rnd == 0, rnd=rnd)
            buf.draft_step(rnd, 0, W, H[:b].contiguous(), temp[:b])
            sib()
            tree()
            first = [buf.out_tokens, buf.leaf, buf.n_out]
            out += [t[:few].clone() for t in first]
            buf.verify(rnd, target[:b].contiguous(), temp[:b], fused_update=True)
            out += [t[:few].clone() for t in (buf.draft_lse[0], buf.draft_tokens, buf.draft_q, buf.draft_flags, buf.sib_tokens, buf.sib_q, buf.accept_len,
                                              buf.out_tokens, buf.dev, buf.n_valid, buf.verify_flags, buf.ring, buf.weights)]
        torch.cuda.synchronize()
        return out

    for x, y in zip(run(B), run(few)):
        assert torch.equal(x, y)

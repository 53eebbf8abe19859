"""LM head on the GPU against a 64-bit product of the same stored values, at the sizes where its kernels and tiles change."""
import pytest
import torch

from paper_2601_20357_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [
    # V,     d,    n,  B    rows = n * B
    # W-streaming kernel, 16 rows: four waves a tile, two, K in chunks, one vocabulary tile, several groups per workgroup
    (8003, 72, 1, 1), (33, 8, 16, 1), (32003, 1160, 3, 5), (5000, 2056, 1, 7), (31001, 2056, 1, 3), (140001, 256, 1, 5),
    # 32 rows
    (6000, 648, 1, 17), (32777, 1032, 4, 8), (31000, 1088, 1, 32), (70001, 1096, 2, 16),
    # runs of more than one k-block a wave (2 x 128, 512, 768 or 896 columns in turn), K whole and in two, three, four chunks of H
    (20000, 1024, 1, 4), (33000, 1024, 1, 32), (33000, 2048, 1, 9), (40000, 3072, 1, 5), (33000, 1536, 4, 4), (33000, 2048, 1, 20),
    (33000, 3072, 1, 24), (70003, 1792, 1, 13), (66000, 2048, 4, 8),
    # kernels with a compile-time hidden size, one block of up to 32 rows: whole rows of H and chunks
    (33000, 512, 1, 5), (20001, 512, 4, 8), (20000, 768, 1, 17), (32001, 896, 4, 8), (20000, 1536, 4, 6), (40000, 2560, 1, 18),
    (20002, 1792, 2, 10), (20000, 2048, 1, 32),
    # tiles of 64 rows, and W streamed with four waves a tile and H in chunks
    (20000, 776, 1, 33), (32768, 1000, 1, 64), (40001, 1920, 1, 48), (3001, 64, 1, 40), (33000, 72, 1, 64), (16384, 3200, 1, 64),
    (129, 648, 1, 35),
    # 64 rows (hidden sizes that the kernels with a compile-time size do not take), K whole and in chunks
    (3001, 640, 1, 33), (32767, 640, 8, 8), (33001, 640, 1, 64), (33001, 1096, 1, 20), (9000, 1160, 1, 50), (32768, 776, 1, 64),
    # tiles of 128 x 128, 128 x 256, 256 x 256 rows x vocabulary; one k-block, a ragged last one, a last row block of one row
    (4099, 72, 1, 65), (33000, 1160, 1, 50), (8200, 2048, 1, 128), (2000, 8, 1, 129),
    (49153, 264, 1, 66), (24600, 136, 1, 257), (49161, 264, 1, 129), (25000, 64, 1, 511),
    (84712, 1328, 1, 120),                                           # W of the last-level cache's size: logits past L2
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"V{s[0]}d{s[1]}M{s[2] * s[3]}")
def test_logits_and_log_sum_exp(shape):
    V, d, n, B = shape
    M = n * B
    print(f"lm head {shape}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(V + d)
    cfg = binding.make_cfg(V=V, d=d, n=n, B=B, gamma=2, h=1, w_dtype=1, seed=1)
    buf = binding.RoundBuffers(cfg, DEV)
    buf.weights.fill_(1.0 / n)
    W = (torch.randn((V, d), generator=g, device=DEV) * 0.05).bfloat16()
    H = torch.randn((B, n, d), generator=g, device=DEV).bfloat16()
    temp = torch.ones(B, device=DEV)
    temp[1::3], temp[2::3] = 0.7, 0.0
    buf.draft_logits.fill_(7.0)
    buf.draft_step(0, 1, W, H, temp)
    torch.cuda.synchronize()
    Hd, Wd = H.view(M, d).double(), W.double()
    exact = Hd @ Wd.t()
    # products of bf16 are exact in fp32; a sum of d of them in any order is off by at most d 2^-24 times the sum of their sizes
    bound = d * 2.0 ** -24 * (Hd.abs() @ Wd.abs().t())
    err = (buf.draft_logits[1].view(M, V).double() - exact).abs()
    assert bool((err <= bound + 1e-30).all()), float((err - bound).max())
    assert bool((buf.draft_logits[0] == 7.0).all())                # the other slot is untouched
    inv = torch.where(temp > 0, 1 / temp, torch.ones_like(temp)).double().repeat_interleave(n)
    lse = torch.logsumexp(exact * inv[:, None], -1)
    # the log-sum-exp moves by at most the largest error of a scaled logit; 2e-6 for the fp32 exponentials and their sums
    tol = (bound.max(-1).values * inv) + 2e-6
    assert bool(((buf.draft_lse[1].view(M) - lse).abs() <= tol).all())


@pytest.mark.parametrize("V,d,n,B", [(8003, 72, 1, 3), (32000, 768, 4, 4), (33000, 768, 4, 16), (5003, 1024, 4, 16), (33000, 640, 2, 32),
                                     (32000, 768, 4, 32), (70001, 264, 4, 64)])
def test_entries_without_mass(V, d, n, B):
    """A logit that is NaN and a whole softmax tile of -inf count nothing: the rest of their tiles keeps its mass, and a greedy row
    takes the largest of the other entries."""
    M = n * B
    print(f"entries without mass V={V} d={d} M={M}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(V)
    cfg = binding.make_cfg(V=V, d=d, n=n, B=B, gamma=1, h=1, w_dtype=1, seed=1)
    buf = binding.RoundBuffers(cfg, DEV)
    buf.weights.fill_(1.0 / n)
    W = (torch.randn((V, d), generator=g, device=DEV) * 0.05).bfloat16()
    H = torch.randn((B, n, d), generator=g, device=DEV).bfloat16()
    H[..., 0] = 1.0
    W[64:96] = 0.0
    W[64:96, 0] = float("-inf")
    W[[17, 5000, V - 1], 0] = float("nan")
    buf.draft_step(0, 0, W, H, torch.ones(B, device=DEV))
    torch.cuda.synchronize()
    L = buf.draft_logits[0].view(M, V)
    assert bool(L[:, [17, 5000, V - 1]].isnan().all()) and bool((L[:, 64:96] == float("-inf")).all())
    rest = torch.ones(V, dtype=torch.bool, device=DEV)
    rest[[17, 5000, V - 1]] = False
    lse = torch.logsumexp(L[:, rest].double(), -1)
    assert bool(((buf.draft_lse[0].view(M) - lse).abs() <= 2e-6).all())      # fp32 exponentials and their sums, as above
    buf.draft_step(0, 0, W, H, torch.zeros(B, device=DEV))
    torch.cuda.synchronize()
    q = (buf.draft_logits[0].double() - lse.view(B, n, 1)).exp().mean(1).nan_to_num(nan=-1.0)
    top, at = q.topk(2, -1)
    y = buf.draft_tokens[:, 0].long()
    assert bool(((y == at[:, 0]) | ((top[:, 0] - top[:, 1]) < 1e-6 * top[:, 0])).all())


@pytest.mark.parametrize("V,d", [(8003, 8), (8003, 72), (8003, 136), (8003, 200), (8003, 264), (8003, 328), (16384, 504), (16384, 640), (12001, 1000), (16385, 64),
                                 (16385, 136), (32768, 200), (20000, 640), (32001, 1160), (32769, 200), (50261, 1160)])
def test_order_of_a_logits_products_up_to_64_rows(V, d):
    """Hidden sizes outside the 512 / 768 / 896 families: a row's logits are the same bits with 32 rows and with 33 to 64, where
    tiles take the place of the kernel that streams W: one, two or four partial sums over the k-blocks, none to all of them filled."""
    g = torch.Generator(device=DEV).manual_seed(V + d)
    W = (torch.randn((V, d), generator=g, device=DEV) * 0.05).bfloat16()
    H = torch.randn((64, 1, d), generator=g, device=DEV).bfloat16()
    out = {}
    for B in (32, 33, 64):
        print(f"lm head order V={V} d={d} rows={B}", flush=True)
        buf = binding.RoundBuffers(binding.make_cfg(V=V, d=d, n=1, B=B, gamma=1, h=1, w_dtype=1, seed=1), DEV)
        buf.weights.fill_(1.0)
        buf.draft_step(0, 0, W, H[:B].contiguous(), torch.ones(B, device=DEV))
        torch.cuda.synchronize()
        out[B] = buf.draft_logits[0].view(B, V)
    assert torch.equal(out[32], out[33][:32]) and torch.equal(out[33], out[64][:33])

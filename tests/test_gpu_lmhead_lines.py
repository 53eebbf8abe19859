"""LM head of more than 64 rows, hidden sizes that are multiples of 64: the kernel whose operands go straight to LDS adds a logit's
products in the order of the kernel that stages them through registers, which takes the same rows with eight columns of zeros
appended (a last k-block that adds zeros).  Same bits, and those within the bound of a 64-bit product."""
import pytest
import torch

from paper_2601_20357_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (through L2: the logits of rows that share 64-byte sectors, from 2^22 logits on; of the staged tiles as well)
@pytest.mark.parametrize("V,d,M", [(4099, 512, 65), (8200, 576, 128), (20000, 896, 192), (13001, 640, 129),      # 128 x 128, one and two a compute unit
                                   (33000, 768, 128),                                                            # through L2
                                   (49153, 512, 66), (24577, 1152, 129),                                         # 128 x 256
                                   (50001, 512, 100), (60004, 640, 128),                                         # through L2
                                   (58600, 2176, 72),                                                            # W of 255 MB: past L2 all the same
                                   (49168, 704, 129), (128256, 512, 500),                                        # 256 x 256
                                   (24600, 512, 257), (49161, 704, 129), (100003, 2048, 512)])                   # through L2
def test_logits_are_those_of_the_staged_tiles(V, d, M):
    print(f"lm head lines V={V} d={d} rows={M}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(V + d)
    W = (torch.randn((V, d), generator=g, device=DEV) * 0.05).bfloat16()
    H = torch.randn((M, 1, d), generator=g, device=DEV).bfloat16()
    temp = torch.ones(M, device=DEV)
    temp[1::3] = 0.7
    out = []
    for pad in (0, 8):
        buf = binding.RoundBuffers(binding.make_cfg(V=V, d=d + pad, n=1, B=M, gamma=1, h=1, w_dtype=1, seed=1), DEV)
        buf.weights.fill_(1.0)
        buf.draft_logits.fill_(7.0)
        Wp, Hp = (torch.cat([t, torch.zeros(t.shape[:-1] + (pad,), dtype=t.dtype, device=DEV)], -1).contiguous() for t in (W, H))
        buf.draft_step(0, 0, Wp, Hp, temp)
        torch.cuda.synchronize()
        out.append((buf.draft_logits[0].view(M, V), buf.draft_lse[0].clone(), buf.draft_tokens[:, 0].clone()))
    assert all(torch.equal(a, b) for a, b in zip(*out))
    for v0 in range(0, V, 16384):
        Wd, Hd = W[v0:v0 + 16384].double(), H[:, 0].double()
        # products of bf16 are exact in fp32; a sum of d of them in any order is off by at most d 2^-24 times the sum of their sizes
        bound = d * 2.0 ** -24 * (Hd.abs() @ Wd.abs().t())
        assert bool(((out[0][0][:, v0:v0 + 16384].double() - Hd @ Wd.t()).abs() <= bound + 1e-30).all())

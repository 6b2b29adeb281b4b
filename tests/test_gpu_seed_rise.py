"""Prompt replay where the logits that weigh lie far above those a pass over the keys meets first: weights as exact as where they do
not, against 64 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# a block of heavy entries behind many light ones: the last of a run of two to six blocks, whichever of these a wavefront takes
@pytest.mark.parametrize("rise", [0, 10, 25, 40, 55])
@pytest.mark.parametrize("G", [1, 4, 7])
def test_weights_above_the_first_block(G, rise):
    import torch
    from paper_2601_16986_amd import ckv
    batch, hkv, P, W, heavy = 16, 8, 2080, 2, 59
    scale = 1.0 / np.sqrt(128.0)
    g = ckv.CrystalKV(1, batch, hkv * G, hkv, 128, 2112, np.full((1, batch, hkv), P, np.int32), t0=P, lam=0.5, softmax_scale=scale,
                      reward_mode=ckv.REWARD_ATTN_WEIGHTED, budget_min=1, budget_max=P + 1)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(10 * rise + G)
    # logits in base 2, of two terms on the bf16 grid whose products and sum are exact: -rise .. 1 - rise, the heavy block's 0 .. 1
    x = torch.rand((batch, hkv, P), generator=gen, device=g.device) - rise
    x[..., 32 * heavy:32 * heavy + 32] += rise
    x = x / float(scale * np.log2(np.e))
    hi = (x / 8.0).to(torch.bfloat16)
    k = torch.zeros((batch, hkv, P, 128), dtype=torch.bfloat16, device=g.device)
    k[..., 0], k[..., 1] = hi, ((x / 8.0 - hi.float()) * 256.0).to(torch.bfloat16)
    q = torch.zeros((W, batch, hkv * G, 128), dtype=torch.bfloat16, device=g.device)
    q[..., 0], q[..., 1] = 8.0, 8.0 / 256.0
    g.load_prompt(0, k, k)
    g.seed_prompt(0, q)
    s = (k[..., 0].double() * 8.0 + k[..., 1].double() * 8.0 / 256.0) * scale
    w = torch.softmax(s, dim=-1)
    seg = g.pool_slots // (batch * hkv)
    crf = g.crf[:batch * hkv * seg].view(batch, hkv, seg)[:, :, :P].double()
    # scores of the heavy block: the last query's weight and half of the one's before, which saw one (light) entry less
    at = slice(32 * heavy, 32 * heavy + 32)
    want = w[..., at] + 0.5 * torch.softmax(s[..., :P - 1], dim=-1)[..., at]
    assert g.status() == 0
    g.close()
    # Roundings of 2^-24 each, at most: the exponent (below 1: half of one), the exponential (two), the column's sum (two), its inverse, the
    # product, the mean over the heads (two), and half as much again for the query before: within 14 of them. An exponent of 40 carries 32 by itself.
    err = float((crf[..., at] / want - 1.0).abs().max())
    assert err < 14 * 2.0 ** -24

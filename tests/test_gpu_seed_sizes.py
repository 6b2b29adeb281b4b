"""Prompt replay at every group size (four heads of a query, or one head of sixteen, per tile) and at the row lengths
where the threshold search changes its width, against weights in 64 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _context(L, batch, hkv, G, P, W, weighted, shape_qk=None):
    import torch
    from paper_2601_16986_amd import ckv
    g = ckv.CrystalKV(L, batch, hkv * G, hkv, 128, (P + 33) // 32 * 32, np.full((L, batch, hkv), P, np.int32), t0=P, lam=0.5,
                      reward_mode=ckv.REWARD_ATTN_WEIGHTED if weighted else ckv.REWARD_TOPP_HIT, budget_min=1, budget_max=P + 1)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(P + G)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device)
    k = rnd(batch, hkv, P, 128).to(torch.bfloat16)
    q = (1.5 * rnd(W, batch, hkv * G, 128)).to(torch.bfloat16)
    if shape_qk:
        q, k = shape_qk(torch, q, k)
    g.load_prompt(0, k, k)
    g.seed_prompt(0, q)
    assert g.status() == 0
    seg = g.pool_slots // (L * batch * hkv)
    live = lambda x: x[:batch * hkv * seg].view(batch, hkv, seg)[:, :, :P]
    crf, tau = live(g.crf).double(), live(g.tau).long()
    kt = k.double().transpose(2, 3).contiguous()
    weights = []                                              # [W] of [batch][hkv][entries seen]
    for j in range(W):
        s = torch.matmul(q[j].view(batch, hkv, G, 128).double(), kt[..., :P - W + j + 1].contiguous()) / np.sqrt(128.0)
        weights.append(torch.softmax(s, dim=-1).mean(2))
    g.close()
    return torch, crf, tau, weights


@pytest.mark.parametrize("L", [1, 24])                        # one group of queries at a time, and several
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 6, 7, 8])
def test_weights_of_every_group_size(G, L):
    _check_weights(L, G, 395, 37)


@pytest.mark.parametrize("W", [1, 2, 5, 18])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 6, 7, 8])
def test_weights_of_few_queries(G, W):
    """Batches that leave tiles of the second pass without queries, and columns of the first."""
    _check_weights(24, G, 130, W)


def _check_weights(L, G, P, W):
    torch, crf, tau, weights = _context(L, 2, 3, G, P, W, True)
    pos = torch.arange(P, device=crf.device)
    want, last = (pos < P - W).double().expand_as(crf).clone(), pos.clone()
    for j, a in enumerate(weights):
        t = P - W + j
        want[..., :t + 1] = want[..., :t + 1] * 0.5 ** (t - last[:t + 1]).double() + a
        last[:t + 1] = t
    # a weight carries a few rounding errors of 2^-24, a score the last few weights'
    assert float(((crf - want).abs() / want.clamp(min=1e-30)).max()) < 4e-6
    assert torch.equal(tau, last.expand_as(tau))


@pytest.mark.parametrize("P", [33, 4096, 4097, 6144, 6145, 8192, 8193, 10240, 10241, 12288, 12289, 14336, 14337, 16384, 16385])
def test_hits_of_every_row_length(P):
    torch, crf, tau, weights = _context(1, 2, 2, 5, P, 1, False)
    a = weights[0]
    hit = tau == P - 1
    assert bool(hit[..., P - 1].all())                        # the query's own entry
    srt, order = torch.sort(a, dim=-1, descending=True)
    inside = torch.cumsum(srt, -1) - srt <= 0.9               # the smallest set that exceeds p
    want = torch.zeros_like(hit).scatter(-1, order, inside)
    want[..., P - 1] = True
    edge = torch.where(inside, srt, torch.inf).amin(-1, keepdim=True)
    # fp32 sums of P weights may put the cut a few entries to either side of the edge, never elsewhere
    wrong = (hit != want)
    assert float(torch.where(wrong, (a / edge - 1).abs(), 0.0).max()) < 1e-3 and int(wrong.sum(-1).max()) <= 2


@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("G", [3, 8])
@pytest.mark.parametrize("q_exp,k_exp", [(9, 9), (14, 14), (18, 18), (40, 36)])
def test_logits_far_beyond_the_exponential(q_exp, k_exp, G, weighted):
    """Logits of about 2^21, 2^31, 2^39 and 2^79 in base 2: every head's weight is all on its largest logit, or shared by what lies
    within a unit of it; nothing overflows, however far the logits are from 1."""
    P, W = 395, 37
    scale = lambda torch, q, k: ((q.float() * 2.0 ** q_exp).to(torch.bfloat16), (k.float() * 2.0 ** k_exp).to(torch.bfloat16))
    torch, crf, tau, weights = _context(1, 2, 3, G, P, W, weighted, scale)
    _check_far(torch, crf, tau, weights, P, W, weighted)


def _check_far(torch, crf, tau, weights, P, W, weighted):
    pos = torch.arange(P, device=crf.device)
    want, last = (pos < P - W).double().expand_as(crf).clone(), pos.expand(crf.shape).clone()
    for j, a in enumerate(weights):
        t = P - W + j
        # G heads of weight 1 / G each: all of them are needed to exceed 0.9 of the whole; and the query's own entry
        reward = a if weighted else ((a > 1e-3) | (pos[:t + 1] == t)).double()
        new = want[..., :t + 1] * 0.5 ** (t - last[..., :t + 1]).double() + reward
        take = torch.ones_like(new, dtype=torch.bool) if weighted else reward > 0
        want[..., :t + 1] = torch.where(take, new, want[..., :t + 1])
        last[..., :t + 1] = torch.where(take, t, last[..., :t + 1])
    assert bool(torch.isfinite(crf).all())
    # a logit of 128 products carries an error of a few 2^-24 of their sum's size: two logits that close share a head's weight
    # in another ratio.  Two of 395 logits are that close in about one head of 10^4.
    off = (crf - want).abs() > 4e-6
    assert int(off.sum()) <= 4, int(off.sum())
    assert int((tau != last).sum()) <= 4


@pytest.mark.parametrize("weighted", [True, False])
@pytest.mark.parametrize("G", [3, 8])
def test_logits_all_far_below_zero(G, weighted):
    """Every logit about -1e32: finite, and the largest of them takes its head's weight like any other."""
    P, W = 395, 37
    scale = lambda torch, q, k: ((q.float().abs() * 2.0 ** 52).to(torch.bfloat16), (-k.float().abs() * 2.0 ** 52).to(torch.bfloat16))
    torch, crf, tau, weights = _context(1, 2, 3, G, P, W, weighted, scale)
    _check_far(torch, crf, tau, weights, P, W, weighted)


def test_a_head_whose_logits_are_all_minus_infinity():
    """Products that overflow to -inf: that head weighs nothing, the others' weights stand."""
    P, W, G = 395, 5, 4
    kept = []

    def scale(torch, q, k):
        q, k = q.float(), k.float()
        k[..., 0] = -2.0 ** 10
        q[..., 0] = 0.0
        q[:, :, 1::G] = 0.0
        q[:, :, 1::G, 0] = 2.0 ** 126
        kept.append((q.to(torch.bfloat16), k.to(torch.bfloat16)))
        return kept[0]

    torch, crf, tau, weights = _context(1, 2, 3, G, P, W, True, scale)
    q, k = kept[0]
    kt = k.double().transpose(2, 3).contiguous()
    pos = torch.arange(P, device=crf.device)
    want, last = (pos < P - W).double().expand_as(crf).clone(), pos.clone()
    for j in range(W):
        t = P - W + j
        s = torch.matmul(q[j].view(2, 3, G, 128).double(), kt[..., :t + 1].contiguous()) / np.sqrt(128.0)
        a = torch.softmax(s, dim=-1)
        a[:, :, 1] = 0.0
        want[..., :t + 1] = want[..., :t + 1] * 0.5 ** (t - last[:t + 1]).double() + a.mean(2)
        last[:t + 1] = t
    assert float(((crf - want).abs() / want.clamp(min=1e-30)).max()) < 4e-6

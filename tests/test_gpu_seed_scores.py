"""Scores of a replayed prompt, bit for bit: queries whose hits are known beforehand (equal weights on a set of entries that the
query's number decides, nothing elsewhere), through decay tables that LDS holds whole and longer ones, at the edges of what a
wavefront (256 entries), a workgroup (1024) and a register of hits (8 queries, 32 asked for at a time) hold."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SETS = 8


def _decay_table(lam):
    """lambda^delta as float32, 0 below the smallest normal number, up to its first 0."""
    out = []
    while len(out) < 1 << 20:
        v = np.float32(float(np.float32(lam)) ** len(out))
        out.append(v if v >= np.finfo(np.float32).tiny else np.float32(0))
        if out[-1] == 0 or lam == 1:
            break
    return np.array(out, np.float32)


def _known_hits(P, lam, L, G, W):
    """A context, which entries of each unit belong to which sets, and keys and queries under which query j finds set j % SETS."""
    import torch
    from paper_2601_16986_amd import ckv
    Bz, Hkv = 2, 2
    g = ckv.CrystalKV(L, Bz, Hkv * G, Hkv, 128, (P + 33) // 32 * 32, np.full((L, Bz, Hkv), P, np.int32), t0=P, lam=lam, top_p=0.99,
                      budget_min=1, budget_max=P + 1)
    rng = np.random.default_rng(P + W)
    # entry i belongs to SETS sets at random, an eighth of the entries each
    member = rng.random((Bz, Hkv, P, SETS)) < 0.125
    member[:, :, 0] = True                                   # no query finds nothing
    k = torch.zeros((Bz, Hkv, P, 128))
    k[..., :SETS] = torch.from_numpy(member.astype(np.float32)) * 32
    q = torch.zeros((W, Bz, Hkv * G, 128))
    q[torch.arange(W), :, :, torch.arange(W) % SETS] = 32.0   # logits 90.5 inside a set, 0 outside
    return g, member, k, q


def _check(g, member, k, q, lam, every=lambda t: None):
    """Replays the queries and compares scores and times; of the unit that `every` names at time t all entries seen are hit, whatever the sets say."""
    import torch
    Bz, Hkv, P = member.shape[:3]
    W = q.shape[0]
    k, q = k.to(torch.bfloat16).to(g.device), q.to(torch.bfloat16).to(g.device)
    g.load_prompt(0, k, k)
    g.seed_prompt(0, q)
    assert g.status() == 0
    seg = g.pool_slots // g.units
    live = lambda x: x[:Bz * Hkv * seg].view(Bz, Hkv, seg)[:, :, :P].cpu().numpy()
    tab = _decay_table(lam)
    pos = np.arange(P)
    crf = np.broadcast_to(np.where(pos < P - W, 1, 0).astype(np.float32), (Bz, Hkv, P)).copy()
    tau = np.broadcast_to(pos, (Bz, Hkv, P)).copy()
    for j in range(W):
        t = P - W + j
        # m equal weights of a set seen by the query: m - 1 of them stay below 0.99 while m < 100, so all are needed
        hit = member[..., j % SETS] & (pos <= t)
        need = hit.sum(-1)
        # of a larger set the first by position whose sum passes 0.99
        most = np.floor(0.99 * need + 1e-4).astype(int) + 1
        hit &= np.cumsum(hit, -1) <= np.minimum(most, need)[..., None]
        if every(t) is not None:
            hit[every(t)] = pos <= t
        hit[..., t] = True
        dec = tab[np.minimum(np.maximum(t - tau, 0), len(tab) - 1)]
        new = (dec * crf).astype(np.float32) + np.float32(1)
        crf, tau = np.where(hit, new, crf), np.where(hit, t, tau)
    assert np.array_equal(live(g.tau), tau)
    assert np.array_equal(live(g.crf), crf)
    g.close()


def _last_place(last):
    """A lambda whose table ends with its first 0 at place `last`: lambda^(last - 1) >= 2^-126 > lambda^last."""
    lam = 2.0 ** (-126.0 / (last - 0.5))
    assert len(_decay_table(lam)) - 1 == last
    return lam


# one layer: batches of 16 queries; 48 layers of one head each: of 48.  LDS holds tables of up to 256 places.
@pytest.mark.parametrize("L,G,W", [(1, 2, 1), (1, 2, 16), (1, 5, 33), (48, 1, 31), (48, 1, 47), (48, 1, 57)])
@pytest.mark.parametrize("lam", [0.5, 0.7, _last_place(255), _last_place(256), 0.9, 1.0])
@pytest.mark.parametrize("P", [64, 255, 257, 1025])
def test_scores_of_known_hits(P, lam, L, G, W):
    g, member, k, q = _known_hits(P, lam, L, G, W)
    _check(g, member, k, q, lam)


@pytest.mark.parametrize("L,G,W", [(1, 2, 16), (1, 5, 33), (48, 1, 31)])
@pytest.mark.parametrize("lam", [0.7, 0.9])
@pytest.mark.parametrize("P,back", [(64, 8), (257, 5), (1025, 700), (2100, 12)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
def test_keys_that_are_no_numbers(bad, P, back, lam, L, G, W):
    """A logit of NaN or +inf makes every weight a NaN of a query that sees the key: no sum exceeds p, so all that the query sees is hit. One of
    -inf has no weight. Queries before it and other units do not notice."""
    g, member, k, q = _known_hits(P, lam, L, G, W)
    at = P - back
    q[..., 100] = 1.0
    k[0, 1, at, 100] = bad
    if bad < 0:
        member[0, 1, at] = False
    _check(g, member, k, q, lam, lambda t: (0, 1) if t >= at and not bad < 0 else None)

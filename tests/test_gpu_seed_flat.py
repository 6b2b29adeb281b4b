"""Hits of replayed prompts whose weights lie so close together that a bin of the threshold's histogram holds more than its list: even
weights, all within one bin, within a few, at a few levels, against the rule in 64 bits; with rows of every kind of length."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = ["even", "bin", "narrow", "close", "levels", "part"]


def _logits(shape, n, rng):
    if shape == "even":
        return np.zeros(n)
    if shape == "bin":                                       # within 1/32 octave
        return rng.random(n) / 40.0
    if shape == "narrow":
        return 0.2 * rng.standard_normal(n)
    if shape == "close":                                     # within 1/256 of a bin: ties but for the last bits
        return rng.random(n) * 2.0 ** -14
    if shape == "levels":
        return np.floor(2.0 * rng.standard_normal(n)) / 2.0
    return rng.random(n) / 32.0 / 256.0 * 3.0                # a few parts of a bin


@pytest.mark.parametrize("P", [520, 4090, 9350, 12300, 16384])
@pytest.mark.parametrize("p", [0.03, 0.5, 0.9])
def test_hits_of_flat_rows(p, P):
    import torch
    from paper_2601_16986_amd import ckv
    rng = np.random.default_rng(P)
    B = len(SHAPES)
    k = torch.zeros((B, 1, P, 128), dtype=torch.bfloat16)
    for b, s in enumerate(SHAPES):
        # a base-2 logit in two terms on the bf16 grid: 8 q . (hi, lo / 256) in units of log2, exactly what the key says
        x = _logits(s, P, rng)
        hi = torch.from_numpy(x / 8.0).to(torch.bfloat16)
        k[b, 0, :, 0], k[b, 0, :, 1] = hi, torch.from_numpy((x / 8.0 - hi.double().numpy()) * 256.0).to(torch.bfloat16)
    q = torch.zeros((1, B, 1, 128), dtype=torch.bfloat16)
    q[..., 0], q[..., 1] = 8.0, 8.0 / 256.0
    g = ckv.CrystalKV(1, B, 1, 1, 128, (P + 33) // 32 * 32, np.full((1, B, 1), P, np.int32), t0=P, top_p=p, softmax_scale=float(np.float32(np.log(2.0))))
    g.load_prompt(0, k.to(g.device), k.to(g.device))
    g.seed_prompt(0, q.to(g.device))
    pf = float(np.float32(p))
    for b, s in enumerate(SHAPES):
        x = (k[b, 0].double() @ q[0, b, 0].double()).numpy()
        w = np.exp2(x - x.max())
        w /= w.sum()
        e = g.export_unit(0, b, 0, with_kv=False)
        at = e["pos"].astype(np.int64)
        order = np.lexsort((at, -w[at]))
        cum = np.cumsum(w[at][order])
        m = int(np.nonzero(cum > pf)[0][0]) + 1
        want = np.zeros(P, bool)
        want[order[:m]] = True
        want[at == P - 1] = True
        # the query's own entry starts as arrived at its position, so its time does not tell; every other hit's time is the query's
        hit = e["tau"] == P - 1
        wrong = np.nonzero(hit != want)[0]
        # fp32 weights (a few units of 2^-24 each, and the logits' share of it) may move the sum at the cut past p, by entries that together
        # weigh no more than that error, or (weights that differ by less than it) exchange places; among equal weights positions decide
        cut = w[at][order[m - 1]]
        near = np.abs(w[at][wrong] / cut - 1.0) < 1e-5 if s != "even" else np.zeros(len(wrong), bool)
        margin = min(abs(cum[m - 1] - pf), abs(pf - cum[m - 2]))
        assert w[at][wrong[~near]].sum() <= 4e-6 or (len(wrong) == 1 and margin < 2e-6), (s, len(wrong), m)
        assert abs(w[at][hit].sum() - w[at][want].sum()) <= 4e-6 + cut, s
    assert g.status() == 0
    g.close()

"""The top-p threshold where its search changes its way (bins of the histogram, the list behind them, rounds over all entries):
weights that are all equal, too many for the list in one bin, spread over more octaves than there are bins, nearly all of one
entry, against the rule in 64 bits; in the step's two implementations and with every number of entries per thread."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = ["flat", "bin", "wide", "heavy", "pair", "normal", "steps"]


def _logits(shape, n, rng):
    """Base-2 logits of n entries, the last of which arrives in the step."""
    if shape == "flat":
        return np.zeros(n)
    if shape == "bin":                                       # within 1/32 octave
        return rng.random(n) / 40.0
    if shape == "wide":
        return -60.0 * rng.random(n)
    x = rng.standard_normal(n)
    if shape in ("heavy", "pair"):
        x[n // 3] = np.log2(20.0 * n)
    if shape == "pair":
        x[n // 2] = x[n // 3]
    if shape == "steps":                                     # many ties at a few levels
        x = np.floor(x)
    return x


@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("n", [3, 250, 700, 2049, 3000, 6000, 8200, 9000])
@pytest.mark.parametrize("p", [0.03, 0.9, 0.9999999, 1.0])
def test_threshold(p, n, path):
    import torch
    from paper_2601_16986_amd import ckv
    rng = np.random.default_rng(n)
    B, t = len(SHAPES), 20000
    # a logit in two terms on the bf16 grid: 8 q . (hi, lo / 256) in units of log2, exactly what the key says
    scale = float(np.float32(np.log(2.0)))
    hi_lo = []
    for s in SHAPES:
        x = _logits(s, n, rng)
        hi = torch.from_numpy(x / 8.0).to(torch.bfloat16)
        hi_lo.append((hi, torch.from_numpy((x / 8.0 - hi.double().numpy()) * 256.0).to(torch.bfloat16)))
    k = torch.zeros((B, 1, n, 128), dtype=torch.bfloat16)
    for b, (hi, lo) in enumerate(hi_lo):
        k[b, 0, :, 0], k[b, 0, :, 1] = hi, lo
    q = torch.zeros((B, 1, 128), dtype=torch.bfloat16)
    q[..., 0], q[..., 1] = 8.0, 8.0 / 256.0
    cap = (n + 32) // 32 * 32
    g = ckv.CrystalKV(1, B, 1, 1, 128, cap, np.full((1, B, 1), cap - 1, np.int32), t0=t, top_p=p, softmax_scale=scale)
    g.set_path(path)
    dev = g.device
    pos = torch.from_numpy(rng.permutation(n - 1).astype(np.int32)).expand(B, 1, n - 1).contiguous().to(dev)
    g.load_cache(0, k[:, :, :n - 1].contiguous().to(dev), k[:, :, :n - 1].contiguous().to(dev), torch.full((B, 1), n - 1, dtype=torch.int32, device=dev),
                 torch.ones((B, 1, n - 1), device=dev), pos, pos)
    new = k[:, :, n - 1].contiguous().to(dev)
    g.decode_step(q[None].to(dev), new[None], new[None], evict=False)
    pf = float(np.float32(p))
    for b, s in enumerate(SHAPES):
        x = (k[b, 0].double() @ q[b, 0].double()).numpy()
        w = np.exp2(x - x.max())
        w /= w.sum()
        e = g.export_unit(0, b, 0, with_kv=False)
        at = e["pos"].astype(np.int64)
        assert e["n"] == n and at[-1] == t
        order = np.lexsort((at, -w))
        cum = np.cumsum(w[order])
        over = np.nonzero(cum > pf)[0]
        m = int(over[0]) + 1 if over.size else n
        want = np.zeros(n, bool)
        want[order[:m]] = True
        want[-1] = True
        hit = e["tau"] == t
        wrong = np.nonzero(hit != want)[0]
        # fp32 weights (a few units of 2^-24, and the logits' share of it) may move the sum at the cut past p, by entries that
        # together weigh no more than that error; among equal weights the positions still decide
        # (a cut that lies closer to p than that itself, 21 of 700 equal weights at p = 0.03, may fall one entry to either side)
        margin = min(abs(cum[m - 1] - pf), abs(pf - cum[m - 2]) if m > 1 else 1.0)
        assert w[wrong].sum() <= 4e-6 or (len(wrong) == 1 and margin < 2e-6), (s, wrong[:5], w[wrong][:5], m)
        if s in ("flat", "steps") and len(wrong) == 0 and m < n:
            assert hit[order[m - 1]] and (not hit[order[m]] or order[m] == n - 1)
    assert g.status() == 0
    g.close()


@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_weights_that_are_no_numbers(bad, path):
    """A logit of +inf or NaN makes every weight of its head a NaN: no sum exceeds p, so every entry is hit."""
    import torch
    from paper_2601_16986_amd import ckv
    n = 300
    g = ckv.CrystalKV(1, 1, 1, 1, 128, 320, np.full((1, 1, 1), 319, np.int32), t0=n)
    g.set_path(path)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(1)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device).to(torch.bfloat16)
    k, q = rnd(1, 1, n, 128), rnd(1, 1, 1, 128).abs()
    k[0, 0, 77, 5] = bad
    g.load_prompt(0, k, rnd(1, 1, n, 128))
    g.decode_step(q, rnd(1, 1, 1, 128), rnd(1, 1, 1, 128), evict=False)
    assert np.all(g.export_unit(0, 0, 0, with_kv=False)["tau"] == n)
    g.close()

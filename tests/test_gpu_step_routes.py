"""Whole steps on either side of the line from which their bookkeeping has a kernel of its own although units are short (many workgroups
without work) or long (few units): against the kernel that takes whole units, entry by entry, and captured."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _steps(path, units, length, cap, extra, G, weighted, graph=False, steps=3):
    import torch
    from paper_2601_16986_amd import ckv
    t = 9000
    rng = np.random.default_rng(units)
    n = rng.integers(max(1, length - 60), length + 61, (units, 1)).astype(np.int32)
    n[0], n[1], n[2] = 1, 31, min(256, length)
    budget = np.clip(n + extra, 1, cap - 1)
    g = ckv.CrystalKV(1, units, G, 1, 128, cap, budget[None], t0=t, budget_min=1, budget_max=cap - 1, headroom=8,
                      reward_mode=ckv.REWARD_ATTN_WEIGHTED if weighted else ckv.REWARD_TOPP_HIT)
    g.set_path(path)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(9)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device).to(torch.bfloat16)
    P = int(n.max())
    pos = torch.arange(P, device=g.device, dtype=torch.int32).expand(units, 1, P).contiguous()
    crf = torch.rand((units, 1, P), generator=gen, device=g.device) + 0.25
    g.load_cache(0, rnd(units, 1, P, 128), rnd(units, 1, P, 128), torch.from_numpy(n).to(g.device), crf, pos, pos)
    q, kn, vn = rnd(steps, units, G, 128), rnd(steps, units, 1, 128), rnd(steps, units, 1, 128)
    out = torch.empty((units, G, 128), device=g.device)
    now = [x[0].clone() for x in (q, kn, vn)]
    step = lambda: g.decode_step(*now, layer=0, out=out)
    if graph:
        torch.cuda.synchronize()
        cg = torch.cuda.CUDAGraph()
        with torch.cuda.graph(cg):
            step()
    outs = []
    for s in range(steps):
        for x, y in zip(now, (q, kn, vn)):
            x.copy_(y[s])
        cg.replay() if graph else step()
        outs.append(out.clone())
    state = [g.export_unit(0, u, 0) for u in range(0, units, 1 if units < 20 else 5)]
    got = torch.stack(outs).double().cpu().numpy(), state, g.lengths(), g.time(), g.status()
    g.close()
    return got


def _same(a, b, exact):
    assert np.array_equal(a[2], b[2]) and a[3:] == b[3:] and a[4] == 0
    # fp32 accumulation and probabilities to 16 bits, in another split of the unit
    assert np.all(np.abs(a[0] - b[0]) <= (0.0 if exact else 4e-5) * np.abs(b[0]).max(-1, keepdims=True))
    for x, y in zip(a[1], b[1]):
        i, j = np.argsort(x["pos"]), np.argsort(y["pos"])
        assert x["n"] == y["n"] and x["n_evicted"] == y["n_evicted"]
        for f in ("pos", "tau", "K", "V"):
            assert np.array_equal(x[f][i], y[f][j]), f
        assert np.allclose(x["crf"][i], y["crf"][j], rtol=0 if exact else 1e-5, atol=0)
        assert np.array_equal(np.sort(x["evicted_pos"]), np.sort(y["evicted_pos"]))


# units, their length and the capacity: in one kernel, and apart
@pytest.mark.parametrize("units,length,cap", [(52, 150, 6144), (64, 150, 6144), (190, 150, 2048), (40, 3500, 3712), (56, 3500, 3712)])
@pytest.mark.parametrize("extra", [3, 0, -6])
@pytest.mark.parametrize("weighted", [False, True])
def test_against_whole_units(weighted, extra, units, length, cap):
    _same(*(_steps(path, units, length, cap, extra, 4, weighted) for path in (1, 2)), exact=False)


@pytest.mark.parametrize("units,length,cap", [(64, 150, 6144), (56, 3500, 3712)])
def test_captured(units, length, cap):
    _same(*(_steps(1, units, length, cap, 0, 2, False, graph=graph) for graph in (True, False)), exact=True)

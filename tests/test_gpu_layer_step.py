"""A step of few units in one kernel, in both of its shapes (by the entries the budgets allow) and widths (by the capacity): lengths at
the edges of blocks, workgroups and entries per thread; units that grow, evict one entry, several, and units that are full; against the
kernel that takes whole units, entry by entry.  Repeated, in other orders of arrival, and captured: the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 31, 32, 255, 256, 257, 511, 700, 1023, 1500, 2016, 2047]
LONG = [2048, 2049, 3000, 4094, 4095, 4096, 4097, 6000, 6110]


def _steps(path, lengths, copies, extra, cap, G, bf16, steps=3, graph=False, weighted=False):
    import torch
    from paper_2601_16986_amd import ckv
    B, H, t = copies * len(lengths), 2, 9000
    n = np.repeat(np.tile(np.asarray(lengths, np.int32), copies), H).reshape(B, H)
    # a budget above the length: grows; equal: evicts one; below: several; the capacity itself: full
    budget = np.clip(n + extra, 1, cap - 1)
    budget[(n == 0) | (np.arange(B * H).reshape(B, H) % 5 == 1)] = cap - 1
    n = np.where(n == max(lengths), cap - 1, n).astype(np.int32)      # one entry short of full: full from the second step on
    g = ckv.CrystalKV(1, B, H * G, H, 128, cap, budget[None], t0=t, budget_min=1, budget_max=cap - 1, out_dtype=ckv.BF16 if bf16 else ckv.F32,
                      reward_mode=ckv.REWARD_ATTN_WEIGHTED if weighted else ckv.REWARD_TOPP_HIT)
    g.set_path(path)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device).to(torch.bfloat16)
    P = cap - 1
    k, v = rnd(B, H, P, 128), rnd(B, H, P, 128)
    pos = torch.arange(P, device=g.device, dtype=torch.int32).expand(B, H, P).contiguous()
    crf = torch.rand((B, H, P), generator=gen, device=g.device) + 0.25
    g.load_cache(0, k, v, torch.from_numpy(n).to(g.device), crf, pos, pos)
    q, kn, vn = rnd(steps, B, H * G, 128), rnd(steps, B, H, 128), rnd(steps, B, H, 128)
    outs = []
    if graph:
        sq, sk, sv = q[0].clone(), kn[0].clone(), vn[0].clone()
        out = torch.empty((B, H * G, 128), dtype=torch.bfloat16 if bf16 else torch.float32, device=g.device)
        torch.cuda.synchronize()
        cg = torch.cuda.CUDAGraph()
        with torch.cuda.graph(cg):
            g.decode_step(sq, sk, sv, layer=0, out=out)
        for s in range(steps):
            sq.copy_(q[s]); sk.copy_(kn[s]); sv.copy_(vn[s])
            cg.replay()
            outs.append(out.clone())
    else:
        outs = [g.decode_step(q[s], kn[s], vn[s], layer=0).clone() for s in range(steps)]
    state = [g.export_unit(0, b, h) for b in range(len(lengths)) for h in range(H)]
    g.status()
    got = torch.stack(outs).double().cpu().numpy(), state, g.lengths(), g.time()
    g.close()
    return got


def _same_state(a, b, exact_scores=True):
    assert np.array_equal(a[2], b[2]) and a[3] == b[3]
    for x, y in zip(a[1], b[1]):
        i, j = np.argsort(x["pos"]), np.argsort(y["pos"])
        assert x["n"] == y["n"] and x["n_evicted"] == y["n_evicted"]
        for f in ("pos", "tau", "K", "V"):
            assert np.array_equal(x[f][i], y[f][j]), f
        if exact_scores:
            assert np.array_equal(x["crf"][i], y["crf"][j])
        else:
            assert np.allclose(x["crf"][i], y["crf"][j], rtol=1e-5, atol=0)
        assert np.array_equal(np.sort(x["evicted_pos"]), np.sort(y["evicted_pos"]))


# 13 lengths below 2048, nine more up to 6111, or those alone; a block per wavefront while the budgets come to no more than 131072 entries (the
# first and the third), else eight
@pytest.mark.parametrize("lengths,cap,copies", [(LENGTHS, 2048, 1), (LENGTHS, 2048, 8), (LONG, 6112, 1), (LENGTHS + LONG, 6112, 1), (LENGTHS + LONG, 6112, 2)])
@pytest.mark.parametrize("extra", [3, 0, -6])
@pytest.mark.parametrize("G", [1, 5, 8])
def test_against_whole_units(G, extra, lengths, cap, copies):
    one, ref = (_steps(path, lengths, copies, extra, cap, G, False) for path in (1, 2))
    # fp32 accumulation and probabilities to 16 bits, in another split of the unit
    assert np.all(np.abs(one[0] - ref[0]) <= 4e-5 * np.abs(ref[0]).max(-1, keepdims=True))
    _same_state(one, ref)


@pytest.mark.parametrize("copies", [1, 2])
def test_weighted_reward(copies):
    one, ref = (_steps(path, LENGTHS + LONG, copies, 0, 6112, 4, True, weighted=True) for path in (1, 2))
    assert np.all(np.abs(one[0] - ref[0]) <= 2.0 ** -7 * np.abs(ref[0]).max(-1, keepdims=True))
    _same_state(one, ref, exact_scores=False)


# work lists that run at once, or queue
@pytest.mark.parametrize("lengths,cap,copies", [(LONG, 6112, 1), (LENGTHS + [3000], 3072, 2), (LENGTHS + [3070], 3104, 1), (LENGTHS + [3070], 3104, 2)])
@pytest.mark.parametrize("extra", [3, -6])
def test_weighted_reward_of_uneven_work_lists(lengths, cap, copies, extra):
    one, ref = (_steps(path, lengths, copies, extra, cap, 5, False, weighted=True) for path in (1, 2))
    assert np.all(np.abs(one[0] - ref[0]) <= 4e-5 * np.abs(ref[0]).max(-1, keepdims=True))
    _same_state(one, ref, exact_scores=False)


@pytest.mark.parametrize("lengths", [LONG, LENGTHS + LONG])
@pytest.mark.parametrize("extra", [0, -6])
def test_repeats_and_replays(extra, lengths):
    a, b, c = (_steps(1, lengths, 1, extra, 6112, 5, False, graph=graph) for graph in (False, False, True))
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[0], c[0])
    _same_state(a, b)
    _same_state(a, c)

"""Evictions of any number of entries at the sizes where the selection changes its width (entries per thread, threads
per unit) and the moves their distribution, against a plain sort by (score descending, position ascending)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LAM = 0.5


def _decay(delta):
    x = np.power(LAM, np.minimum(delta, 200).astype(np.float64)).astype(np.float32)
    x[x < np.finfo(np.float32).tiny] = 0.0
    return x


def _keep(crf, tau, pos, B, t, n_sink):
    """Indices that stay: highest score (or the window policy's key) first, then lower position."""
    if n_sink is None:
        tmp = _decay(t - tau) * crf
        tmp[tmp < np.finfo(np.float32).tiny] = 0.0
        order = np.lexsort((pos, -tmp.astype(np.float64)))
    else:
        sink = pos < n_sink
        order = np.lexsort((np.where(sink, pos, -pos), ~sink))
    return np.sort(order[:B])


def _check(units, cap, lengths, budgets, n_sink, sample, ties):
    import torch
    from paper_2601_16986_amd import ckv
    rng = np.random.default_rng(5)
    n_max = int(max(lengths))
    t = 40000
    budgets = np.asarray(budgets, np.int32).reshape(1, units, 1)
    g = ckv.CrystalKV(1, units, 1, 1, 128, cap, budgets, lam=LAM, t0=t + 1, budget_min=1, budget_max=cap - 1)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(1)
    k = torch.randn((units, 1, n_max, 128), generator=gen, device=g.device).to(torch.bfloat16)
    v = torch.randn((units, 1, n_max, 128), generator=gen, device=g.device).to(torch.bfloat16)
    pos = np.stack([rng.permutation(t - 1)[:n_max] for _ in range(units)]).astype(np.int32)
    tau = np.maximum(pos, (t - rng.geometric(0.05 if ties else 0.3, pos.shape)).astype(np.int32))
    if ties:                                     # few distinct scores, most of them long decayed to zero
        crf = rng.integers(1, 3, pos.shape).astype(np.float32)
        tau = np.where(rng.random(pos.shape) < 0.7, pos, tau).astype(np.int32)
    else:
        crf = (1 + rng.random(pos.shape)).astype(np.float32)
    dev = lambda x: torch.from_numpy(x.reshape(units, 1, n_max)).to(g.device).contiguous()
    g.load_cache(0, k, v, torch.tensor(np.asarray(lengths, np.int32).reshape(units, 1), device=g.device), dev(crf), dev(tau), dev(pos))
    if n_sink is None:
        g.evict(0)
    else:
        g.evict_window(n_sink, 0)
    assert g.status() == 0
    for u in sample:
        n, B = int(lengths[u]), int(budgets[0, u, 0])
        keep = _keep(crf[u, :n], tau[u, :n], pos[u, :n], B, t, n_sink) if n > B else np.arange(n)
        e = g.export_unit(0, u, 0)
        assert e["n"] == len(keep) and e["n_evicted"] == n - len(keep)
        order, want = np.argsort(e["pos"]), keep[np.argsort(pos[u, keep])]
        assert np.array_equal(e["pos"][order], pos[u, want]), (u, n, B)
        assert np.array_equal(e["crf"][order], crf[u, want]) and np.array_equal(e["tau"][order], tau[u, want])
        assert np.array_equal(e["K"][order], k[u, 0].float().cpu().numpy()[want])
        assert np.array_equal(e["V"][order], v[u, 0].float().cpu().numpy()[want])
        gone = np.setdiff1d(np.arange(n), keep)
        assert np.array_equal(e["evicted_pos"], np.sort(pos[u, gone])) and np.all(e["evicted_flags"] == 2)
    g.close()


@pytest.mark.parametrize("ties,n_sink", [(False, None), (True, None), (False, 3000)])
@pytest.mark.parametrize("cap,lengths,budgets", [
    (64, [33, 34, 40, 5], [32, 32, 1, 7]),
    (4128, [4095, 4096, 4097, 1025], [2048, 4094, 4096, 1024]),
    (8224, [8191, 8192, 8193, 300], [100, 8191, 4097, 299]),
    (32768, [16384, 16385, 32767, 9350], [257, 16000, 16384, 2049]),
])
def test_wide_selection(cap, lengths, budgets, ties, n_sink):
    _check(4, cap, lengths, budgets, n_sink, range(4), ties)


@pytest.mark.parametrize("ties", [False, True])
def test_many_small_units(ties):
    """Enough units for workgroups of 256 threads, with lengths at the edges of 4, 8, 16 and 32 entries per thread."""
    units, edge = 1056, [1, 33, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 4600]
    lengths = [edge[i % len(edge)] for i in range(units)]
    budgets = [max(1, (n * (1 + i % 7)) // 8) for i, n in enumerate(lengths)]
    _check(units, 4608, lengths, budgets, None, range(0, units, 37), ties)


@pytest.mark.parametrize("units,cap", [(4, 4096), (300, 2048), (300, 4096)])
def test_widths_by_capacity(units, cap):
    """Kernels for four entries per thread of 1024, and for eight and sixteen per thread of 256, up to the last entry they hold."""
    edge = [cap - 1, cap // 2, cap // 2 + 1, 1024, 1025, 3]
    lengths = [edge[i % len(edge)] for i in range(units)]
    budgets = [max(1, n - 1 - (i * 37) % n // 2) for i, n in enumerate(lengths)]
    _check(units, cap, lengths, budgets, None if cap == 4096 else 40, range(0, units, 1 + units // 24), False)


def test_more_units_than_the_moves_have_workgroups_for():
    """Thousands of units with moves: one workgroup per unit, and workgroups that take several units."""
    units, edge = 4500, [1, 40, 300, 511, 700]
    lengths = [edge[i % len(edge)] for i in range(units)]
    budgets = [max(1, (n * (1 + i % 7)) // 8) for i, n in enumerate(lengths)]
    _check(units, 704, lengths, budgets, None, range(0, units, 101), False)


@pytest.mark.parametrize("path,defer", [(1, False), (1, True), (3, False)])
def test_step_after_a_budget_cut_eager_and_captured(path, defer):
    """A step after budgets were cut evicts many entries per unit: eagerly in kernels behind it, inside a captured graph
    by itself.  Same outputs, same survivors with their scores; the step after it evicts one entry per unit again."""
    import torch
    from paper_2601_16986_amd import ckv
    lengths = [40, 300, 1025, 2049, 4100, 8193, 9001, 64]
    cuts = [40, 100, 1024, 300, 4099, 2000, 8999, 63]           # none, some, one or two entries too many after the append
    units, cap, t, n_max = len(lengths), 9024, 20000, max(lengths)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(2)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda:0").to(torch.bfloat16)
    k, v = rnd(units, 1, n_max, 128), rnd(units, 1, n_max, 128)
    q, kn, vn = rnd(2, 1, units, 4, 128), rnd(2, 1, units, 1, 128), rnd(2, 1, units, 1, 128)
    pos = torch.stack([torch.randperm(t, generator=gen, device="cuda:0")[:n_max] for _ in range(units)]).reshape(units, 1, n_max).int()
    tau = torch.maximum(pos, t - 1 - (torch.rand(pos.shape, generator=gen, device="cuda:0") * 300).int())
    states = []
    for captured in (False, True):
        g = ckv.CrystalKV(1, units, 4, 1, 128, cap, np.asarray(lengths, np.int32).reshape(1, units, 1), t0=t, budget_min=1, budget_max=cap - 1,
                          headroom=1)
        g.set_path(path)
        g.load_cache(0, k, v, torch.tensor(lengths, dtype=torch.int32, device=g.device).reshape(units, 1), torch.ones_like(pos, dtype=torch.float32),
                     tau, pos)
        g.set_budgets(np.asarray(cuts, np.int32).reshape(1, units, 1))
        outs = torch.empty((2, 1, units, 4, 128), device=g.device)

        def step(s):
            if path == 3:
                g.decode_step(q[s], kn[s], vn[s], out=outs[s])
            else:
                g.decode_step(q[s, 0], kn[s, 0], vn[s, 0], layer=0, out=outs[s, 0], defer=defer)
            g.join()

        if captured:
            graph = torch.cuda.CUDAGraph()
            torch.cuda.synchronize()
            with torch.cuda.graph(graph):
                step(0)
            graph.replay()
        else:
            step(0)
        first = [g.export_unit(0, u, 0) for u in range(units)]
        step(1)
        states.append((outs.clone(), first, [g.export_unit(0, u, 0) for u in range(units)]))
        assert g.status() == 0 and g.time() == t + 2
        g.close()
    (o1, a1, b1), (o2, a2, b2) = states
    # the second step's cache is the same set of rows in another order of slots: fp32 sums of the same terms
    assert torch.equal(o1[0], o2[0]) and torch.allclose(o1[1], o2[1], rtol=1e-5, atol=1e-6)
    for x, y in ((a1, a2), (b1, b2)):
        for u, (e, f) in enumerate(zip(x, y)):
            assert e["n"] == f["n"] == min(cuts[u], lengths[u] + 1) and e["n_evicted"] == f["n_evicted"]
            assert np.array_equal(e["evicted_pos"], f["evicted_pos"]) and np.all(e["evicted_flags"] == 2)
            i, j = np.argsort(e["pos"]), np.argsort(f["pos"])
            for key in ("pos", "crf", "tau", "K", "V"):
                assert np.array_equal(e[key][i], f[key][j]), (u, key)


def test_replayed_steps_leave_more_than_the_host_has_seen():
    """A graph of steps without eviction is replayed: the units then hold more entries above their budgets than the host
    has counted, and a window eviction still brings them down to the newest ones."""
    import torch
    from paper_2601_16986_amd import ckv
    P, cap, extra = 60, 128, 9
    g = ckv.CrystalKV(1, 2, 8, 2, 128, cap, np.full((1, 2, 2), P, np.int32), t0=P, budget_min=1, budget_max=cap - 1)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(7)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device).to(torch.bfloat16)
    k, v = rnd(2, 2, P, 128), rnd(2, 2, P, 128)
    g.load_prompt(0, k, v)
    g.evict_window(0)
    q, kn, vn = rnd(1, 2, 8, 128), rnd(1, 2, 2, 128), rnd(1, 2, 2, 128)
    out = torch.empty((1, 2, 8, 128), device=g.device)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.decode_step(q, kn, vn, out=out, attention_only=True)
    for _ in range(extra):
        graph.replay()
    g.evict_window(0)
    assert g.status() == 0
    for b in range(2):
        for h in range(2):
            e = g.export_unit(0, b, h)
            assert sorted(e["pos"].tolist()) == list(range(extra, P + extra)) and e["n_evicted"] == extra
            rows = {int(p): r for p, r in zip(e["pos"], e["K"])}
            assert all(np.array_equal(rows[p], k[b, h, p].float().cpu().numpy()) for p in range(extra, P))
            assert all(np.array_equal(rows[p], kn[0, b, h].float().cpu().numpy()) for p in range(P, P + extra))
    g.close()


@pytest.mark.parametrize("cap,n,B", [(96, 70, 69), (96, 70, 3), (2080, 2000, 1999), (2080, 2000, 200), (9408, 9350, 9349), (9408, 9350, 2048)])
def test_scores_of_any_pattern(cap, n, B):
    """Loaded scores are not checked: infinities and NaNs, one of all bits set among them, are patterns like others (the
    larger, the longer they stay).  More entries to evict than there are finite scores; one entry; all scores the same NaN."""
    import torch
    from paper_2601_16986_amd import ckv
    units, t = 3, 20000
    rng = np.random.default_rng(9)
    g = ckv.CrystalKV(1, units, 1, 1, 128, cap, np.full((1, units, 1), B, np.int32), lam=LAM, t0=t + 1, budget_min=1, budget_max=cap - 1)
    pos = np.stack([rng.permutation(t - 1)[:n] for _ in range(units)]).astype(np.int32)
    bits = np.full((units, n), 0xFFFFFFFF, np.uint32)
    bits[1:, rng.random(n) < 0.1] = np.float32(1.5).view(np.uint32)
    bits[2, rng.random(n) < 0.2] = 0x7FC00000
    bits[2, rng.random(n) < 0.2] = 0x7F800000
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).reshape(units, 1, n)).to(g.device)
    k = torch.randn((units, 1, n, 128), device=g.device).to(torch.bfloat16)
    g.load_cache(0, k, k, torch.full((units, 1), n, dtype=torch.int32, device=g.device), dev(bits.view(np.int32)).view(torch.float32), dev(np.full_like(pos, t)), dev(pos))
    g.evict(0)
    for u in range(units):
        order = np.lexsort((-pos[u], bits[u]))                       # the first go
        e = g.export_unit(0, u, 0)
        assert e["n"] == B and e["n_evicted"] == n - B
        assert np.array_equal(np.sort(e["pos"]), np.sort(pos[u, order[n - B:]])), u
        assert np.array_equal(np.sort(e["evicted_pos"]), np.sort(pos[u, order[:n - B]])), u
    g.close()
